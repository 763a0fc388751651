"""Gaussian bumps at the edges of the evaluation's tiles: bump counts that are not
multiples of four, rows and columns that fill a tile partly, several row blocks,
a column range; sketches against their definition on the stored tensor and the
error pass against entrywise differences.  FP64 contexts: each sketch entry is a
sum of at most 1e6 rounded terms, 1e-13 of the sum of their absolute values; FP32
contexts hold each entry rounded to FP32 (2^-24 of it, twice for the two sides)."""
import numpy as np
import pytest

import inputs
from oracle import tt_sketch as O

from gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,terms,dtype,drm", [
    ((5, 3), 1, "f64", "nested"),
    ((17, 16, 65), 3, "f64", "nested"),          # 272 rows, 65 columns
    ((17, 16, 65), 3, "f32", "nested"),
    ((33, 31, 130), 6, "f64", "independent"),
    ((16, 16, 8, 8), 101, "f64", "nested"),      # exact tiles
    ((16, 16, 8, 8), 101, "f32", "independent"),
    ((9, 7, 5, 6, 11), 10, "f64", "independent"),
])
def test_gauss_tiles(n, terms, dtype, drm):
    import torch
    import paper_2111_10448_amd as P
    say(f"[gpu] Gaussian tiles n={n} terms={terms} {dtype} {drm}")
    d, ell, rng = len(n), 7, np.random.default_rng(5)
    ctr = rng.uniform(-1, 1, (terms, d))
    x = inputs.gauss_tensor(n, ctr, 4.0)
    fn = P.GaussBumps(ctr, 4.0)
    w = inputs.Workload("tiles", 140 + d, tuple(n), dtype, "gauss", ell=ell, rank=2)
    if drm == "nested":
        psi, om = inputs.drm_factors(w)
        fac, kr = inputs.pack_factors(psi, om, d), O.NestedKR(psi, om)
    else:
        psi, om = inputs.drm_factors_independent(w)
        fac, kr = inputs.pack_factors_independent(psi, om, d), O.IndependentKR(psi, om)
    m = O.middle_index(d)
    R = int(np.prod(n[:m]))
    C = x.size // R
    with P.PSTT2(n, ell, fac, dtype=dtype, prec="f64", ranks=w.ranks(), drm=drm) as ctx:
        cut = (C // 3) * R
        ctx.sketch_fn(fn, cut)                     # the columns in two ranges, the later first
        ctx.sketch_fn(fn, 0, cut)
        tt = ctx.recover()
        unit = 1e-13 if dtype == "f64" else 2.0 ** -23
        for which, ks in ((0, range(1, m + 1)), (1, range(m, d))):
            for k in ks:
                xk = O.unfold(x, n, k)
                if which == 0:
                    a, f = xk, kr.omega_dense(k, d)
                else:
                    a, f = xk.T, kr.psi_dense(k)
                assert np.all(np.abs(ctx.get_sketch(which, k) - a @ f) <= unit * (np.abs(a) @ np.abs(f))), (which, k)
        err = tt.error_fn(fn)
        xt = O.tt_full([g for g in tt.cores_numpy()])
        ref = np.linalg.norm(x - xt) / np.linalg.norm(x)
        say(f"    error {err:.6e} ({ref:.6e})")
        assert abs(err - ref) <= 1e-12 * ref + 1e-13
        tt.free()
