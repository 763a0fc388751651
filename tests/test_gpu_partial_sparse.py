"""Cut columns of a tall unfolding that touch few of its rows: single fibres, by
themselves and many in one call, values against the oracle's sketches, and a fibre's
cost, which goes with the rows it brings and not with the height of the unfolding."""
import time

import numpy as np
import pytest

import inputs
from oracle import tt_sketch as O

from gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,ell,alone,batched", [
    ((16, 61, 7, 3), 20, 6, 0),         # one call each
    ((16, 61, 7, 3), 4, 0, 60),         # more pieces than a launch holds, in scattered row blocks
    ((256, 9, 31, 2), 12, 4, 9),        # fibres that fill a row block each
    ((250, 9, 1300, 2), 28, 3, 40),     # 2.9 M rows
])
def test_single_fibres_match_oracle(n, ell, alone, batched):
    import torch
    import paper_2111_10448_amd as P
    say(f"[gpu] single fibres n={n} ell={ell} alone={alone} batched={batched}")
    d, rng = len(n), np.random.default_rng(21)
    x = rng.standard_normal(int(np.prod(n)))
    psi = {q: rng.standard_normal((n[q - 1], ell)) for q in range(1, d)}
    om = {q: rng.standard_normal((n[q - 1], ell)) for q in range(2, d + 1)}
    fibres = x.size // n[0]
    pick = np.sort(rng.choice(fibres, size=alone + batched, replace=False))
    xg = torch.from_numpy(x).cuda()
    ctx = P.PSTT2(n, ell, inputs.pack_factors(psi, om, d), ranks=[2] * (d - 1), algo="pstt")
    single = [int(f) * n[0] for f in pick]
    order = rng.permutation(len(single))
    for i in order[:alone]:
        ctx.sketch(xg[single[i]:single[i] + n[0]], single[i])
    if batched:
        ctx.sketch_slabs([xg[single[i]:single[i] + n[0]] for i in order[alone:]], [single[i] for i in order[alone:]])
    edges = [0] + [v for s in single for v in (s, s + n[0])] + [x.size]
    rest = [(edges[i], edges[i + 1]) for i in range(0, len(edges), 2) if edges[i + 1] > edges[i]]
    ctx.sketch_slabs([xg[a:b] for a, b in rest], [a for a, _ in rest])
    ctx.recover().free()
    m = d - 1
    xm = O.unfold(x, n, m)
    drm = O.NestedKR(psi, om)
    for which, got in ((0, ctx.get_sketch(0, m)), (1, ctx.get_sketch(1, m))):
        ref = xm @ drm.omega_dense(m, d) if which == 0 else xm.T @ drm.psi_dense(m)
        off = float(np.max(np.abs(got - ref)) / np.max(np.abs(ref)))
        say(f"    sketch {which}: {off:.2e}")
        assert off < 1e-12   # sums of at most 6e6 products
    ctx.close()


def test_fibre_cost_does_not_grow_with_the_rows():
    """64 single-fibre calls at 2^24 rows: 2.7 GB of sketch, of which each touches 64 rows.
    Reading and writing all of it would take 0.7 ms a call at 8 TB/s."""
    import torch
    import paper_2111_10448_amd as P
    say("[gpu] cost of a fibre at 2^24 rows")
    n, ell = (64, 64, 64, 64, 2), 20
    ctx = P.PSTT2(n, ell, ranks=[2] * 4, algo="pstt", seed=3)
    x = torch.randn(64, dtype=torch.float64, device="cuda")
    took = []
    for rep in range(3):
        ctx.sketch(x, 64 * (7 + 4001 * rep))
        torch.cuda.synchronize()
        t = time.perf_counter()
        for i in range(64):
            ctx.sketch(x, 64 * (1009 + 4001 * rep + 37 * i))
        torch.cuda.synchronize()
        took.append((time.perf_counter() - t) / 64)
    say(f"    {min(took) * 1e6:.1f} us a call")
    assert min(took) < 0.35e-3
    ctx.close()
