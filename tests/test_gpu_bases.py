"""Bases at the edges of the small factorisations: sketch sizes around every register
slot, ranks around the slots of the Q formation, matrices of one partly filled row
block and of several tree levels, and tolerance mode (ranks from the singular
values).  Sketches, pivots, ranks, X~ and the error against the oracle at the FP64
parity tolerances of the other tests."""
import dataclasses

import pytest

import inputs
from oracle import tt_sketch as O

from gpu_common import compare, gpu_run, oracle_run, say, setup

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rank,ell", [
    ((9, 10, 11, 8), 1, 1),
    ((9, 10, 11, 8), 2, 2),
    ((9, 10, 11, 8), 5, 7),
    ((9, 10, 11, 8), 6, 8),
    ((9, 10, 11, 8), 7, 9),
    ((20, 17, 23, 19), 9, 15),
    ((20, 17, 23, 19), 12, 17),
    ((20, 17, 23, 19), 17, 24),
    ((20, 17, 23, 19), 16, 25),
    ((20, 17, 23, 19), 15, 31),
    ((33, 34, 35, 37), 24, 32),          # over one leaf
    ((140, 260, 7), 6, 20),              # 36400 rows: three tree levels
    ((140, 260, 7), 5, 32),
    ((127, 40), 5, 9), ((129, 40), 8, 16),   # one and two waves
    ((512, 40), 9, 12), ((513, 40), 9, 17),  # half a block of eight waves
    ((1024, 33), 20, 24), ((1025, 33), 20, 24), ((1025, 35), 27, 32),   # one block, two levels
    ((900, 640, 4), 3, 6),               # over a thousand blocks: a workgroup a block forms Q
    ((300, 600, 6), 4, 8), ((700, 515, 5), 4, 20),   # many products of one row slice, of two
])
def test_bases_fixed_rank(n, rank, ell):
    say(f"[gpu] bases n={n} rank={rank} ell={ell}")
    w = inputs.Workload("bases", 150, tuple(n), "f64", "tt", tt_rank=rank, noise=1e-6, ell=ell, rank=rank)
    x, psi, omega, fac = setup(w)
    ref = oracle_run(x, w, psi, omega)
    ctx, tt, xg = gpu_run(x, w, fac, "f64")
    out = compare(ctx, tt, xg, x, w, ref, "f64")
    say(f"    {out}")
    tt.free()
    ctx.close()


@pytest.mark.parametrize("n,ell,eps", [
    ((15, 14, 13, 12), 5, 1e-2), ((15, 14, 13, 12), 8, 1e-4), ((15, 14, 13, 12), 16, 1e-6),
    ((15, 14, 13, 12), 23, 1e-8), ((31, 29, 30), 32, 1e-10), ((6, 5, 6, 5, 6), 32, 1e-7),
])
def test_bases_tolerance(n, ell, eps):
    """Smooth samples: singular values fall over many orders, the ranks are read off them."""
    say(f"[gpu] bases n={n} ell={ell} eps={eps:g}")
    w = inputs.Workload("bases_tol", 151, tuple(n), "f64", "invsum", ell=ell, eps=eps, rmax=32)
    x, psi, omega, fac = setup(w)
    ref = O.pstt2(x, w.n, O.NestedKR(psi, omega), eps=eps, rmax=min(32, max(1, ell - 2)))
    ref["drm"] = O.NestedKR(psi, omega)
    w = dataclasses.replace(w, rmax=min(32, max(1, ell - 2)))
    ctx, tt, xg = gpu_run(x, w, fac, "f64")
    out = compare(ctx, tt, xg, x, w, ref, "f64")
    say(f"    {tt.ranks} {out}")
    tt.free()
    ctx.close()
