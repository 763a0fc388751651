"""Slab edges that cut columns of the pass's unfolding: the batched partial-column
kernel against the oracle's sketches, at the edges of its tiles: sketch sizes of
every 16 + 4 mix, one ragged row block and several, a step over more row blocks
than workgroups, more pieces than one launch holds, and several pieces of one
column in one launch.  FP64 sketches (FP64 and FP32 tensors): each entry is a sum
of at most 1e7 products, so 1e-12 of the largest entry bounds its rounding."""
import numpy as np
import pytest

import inputs
from oracle import tt_sketch as O

from gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,ell,cuts,dtype,algo", [
    ((5, 7, 6, 5), 3, 2, "f64", "pstt2"),          # one partly filled row block
    ((9, 29, 6, 7), 6, 60, "f32", "pstt2"),        # 261 rows, 60 slabs: more pieces than a launch holds
    ((16, 16, 4, 6), 16, 383, "f64", "pstt2"),     # one fibre per slab: 16 pieces of every column, 384 in all
    ((13, 11, 9, 10, 3), 20, 7, "f64", "pstt2"),
    ((13, 11, 9, 10, 3), 24, 7, "f32", "pstt2"),
    ((13, 11, 9, 10, 3), 28, 7, "f64", "pstt2"),
    ((13, 11, 9, 10, 3), 32, 7, "f64", "pstt2"),
    ((61, 83, 59, 2), 8, 5, "f64", "pstt"),        # 298717 rows: the row blocks outnumber the workgroups
])
def test_partial_columns_match_oracle(n, ell, cuts, dtype, algo):
    import torch
    import paper_2111_10448_amd as P
    say(f"[gpu] partial columns n={n} ell={ell} cuts={cuts} {dtype} {algo}")
    d, rng = len(n), np.random.default_rng(7)
    x = rng.standard_normal(int(np.prod(n)))
    if dtype == "f32":
        x = x.astype(np.float32)
    psi = {q: rng.standard_normal((n[q - 1], ell)) for q in range(1, d)}
    om = {q: rng.standard_normal((n[q - 1], ell)) for q in range(2, d + 1)}
    fibres = x.size // n[0]
    at = np.sort(rng.choice(np.arange(1, fibres), size=cuts, replace=False))
    at = [0] + [int(v) * n[0] for v in at] + [x.size]
    order = rng.permutation(len(at) - 1)
    xg = torch.from_numpy(x).cuda()
    ctx = P.PSTT2(n, ell, inputs.pack_factors(psi, om, d), dtype=dtype, prec="f64", ranks=[2] * (d - 1), algo=algo)
    ctx.sketch_slabs([xg[at[i]:at[i + 1]] for i in order], [at[i] for i in order])
    ctx.recover().free()
    m = d - 1 if algo == "pstt" else O.middle_index(d)
    xm = O.unfold(x.astype(np.float64), n, m)
    drm = O.NestedKR(psi, om)
    for which, got in ((0, ctx.get_sketch(0, m)), (1, ctx.get_sketch(1, m))):
        ref = xm @ drm.omega_dense(m, d) if which == 0 else xm.T @ drm.psi_dense(m)
        off = float(np.max(np.abs(got - ref)) / np.max(np.abs(ref)))
        say(f"    sketch {which}: {off:.2e}")
        assert off < 1e-12
    ctx.close()
