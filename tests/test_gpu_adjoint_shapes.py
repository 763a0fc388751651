"""The adjoint at the edges of its matrix-core tiles: inner dimensions that fill a
few, most and all of the register steps, row and column counts around the tiles'
edges and down to one, each scheme (terms that are absent, accumulated passes) and
the FP32 tensor.  J^T gbar and the loss gradient against the oracle's FP64 autograd
at the parity tolerances of the other adjoint tests."""
import pytest

import inputs
import test_gpu_adjoint as TA

from gpu_common import say

pytestmark = pytest.mark.gpu


def _instance(n, rank, ell, dtype, middle, scheme):
    name = "adjoint_shapes"
    w = inputs.Workload(name, 152, tuple(n), dtype, "tt", tt_rank=rank, noise=1e-4, ell=ell, rank=rank)
    inputs.WORKLOADS[name] = w
    try:
        return TA._instance(name, None, middle, scheme)
    finally:
        del inputs.WORKLOADS[name]


@pytest.mark.parametrize("n,rank,ell,middle,scheme", [
    ((9, 8, 7), 1, 1, "onepass", "nested"),
    ((9, 8, 7), 2, 4, "onepass", "nested"),
    ((13, 5, 13, 5), 5, 9, "onepass", "nested"),            # 65 rows, 65 columns
    ((8, 16, 16, 8), 8, 12, "onepass", "nested"),           # 128 rows, 128 columns
    ((43, 3, 3, 43), 7, 13, "twosided", "nested"),          # 129 rows, 129 columns
    ((33, 4, 31), 16, 24, "onepass", "nested"),
    ((34, 35, 36), 28, 32, "onepass", "nested"),            # all register steps
    ((34, 5, 7, 33), 20, 32, "twosided", "independent"),
    ((12, 11, 10, 12), 10, 17, "onepass", "independent"),
])
def test_adjoint_fp64_tiles(n, rank, ell, middle, scheme):
    say(f"[gpu] adjoint f64 n={n} rank={rank} ell={ell} middle={middle} drm={scheme}")
    w, x, fac, drm, ref = _instance(n, rank, ell, "f64", middle, scheme)
    TA._check(w, x, fac, drm, ref, "f64", 1e-9)


@pytest.mark.parametrize("n,rank,ell,middle,scheme", [
    ((13, 5, 13, 5), 5, 9, "onepass", "nested"),
    ((34, 35, 36), 8, 32, "onepass", "nested"),
    ((43, 3, 3, 43), 7, 13, "onepass", "independent"),
])
def test_adjoint_fp32_tiles(n, rank, ell, middle, scheme):
    say(f"[gpu] adjoint f32 n={n} rank={rank} ell={ell} middle={middle} drm={scheme}")
    w, x, fac, drm, ref = _instance(n, rank, ell, "f32", middle, scheme)
    TA._check(w, x, fac, drm, ref, "f32", 2e-5)
