"""The sketch kernels' row operands: first modes below, at and above the length from
which a workgroup tabulates the other modes' products, matrices that end inside a
workgroup's rows, odd row counts (vector loads at the alignment of one entry, the
last row of a column alone), one mode of rows and several, each precision and both
edges of a sketch-size tile.  Against the oracle at the parity tolerances."""
import numpy as np
import pytest

import inputs

from gpu_common import compare, gpu_run, oracle_run, say, setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16x3", "bf16", "f16"])
@pytest.mark.parametrize("n,ell", [
    ((2, 3, 5, 40), 8), ((7, 9, 11, 12), 12), ((8, 9, 11, 12), 13), ((9, 7, 5, 21), 16),
    ((13, 21, 19, 10), 17), ((257, 31), 20), ((5, 5, 5, 5, 5, 5), 24), ((8, 8, 9, 8, 8), 28),
    ((15, 3, 23, 33), 29), ((33, 17, 29), 32),
])
def test_rows(n, ell, prec):
    say(f"[gpu] rows n={n} ell={ell} {prec}")
    dt = "f64" if prec == "f64" else "f32"
    w = inputs.Workload("rows", 154, tuple(n), dt, "tt", tt_rank=2, noise=1e-3, ell=ell, rank=2)
    x, psi, omega, fac = setup(w)
    ref = oracle_run(x, w, psi, omega)
    ctx, tt, xg = gpu_run(x, w, fac, prec)
    out = compare(ctx, tt, xg, x, w, ref, prec)
    say(f"    {out}")
    tt.free()
    ctx.close()


@pytest.mark.parametrize("n,ell", [((7, 9, 11, 12), 12), ((13, 21, 19, 10), 17), ((33, 17, 29), 32)])
def test_rows_partial_columns(n, ell):
    """Slabs that cut columns, of the same row counts."""
    say(f"[gpu] rows, cut columns n={n} ell={ell}")
    w = inputs.Workload("rows", 155, tuple(n), "f64", "tt", tt_rank=2, noise=1e-3, ell=ell, rank=2)
    x, psi, omega, fac = setup(w)
    ref = oracle_run(x, w, psi, omega)
    slabs = inputs.slab_bounds(x.size, n[0], 7)
    ctx, tt, xg = gpu_run(x, w, fac, "f64", slabs=slabs)
    compare(ctx, tt, xg, x, w, ref, "f64")
    tt.free()
    ctx.close()
