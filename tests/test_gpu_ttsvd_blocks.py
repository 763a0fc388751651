"""Parallel-TTSVD at the edges of its column blocks (short sides of 1, 2, 8, 9, 16,
17, 33), with rows in one and in several workgroups, and with spectra where the
rank rule cuts inside a continuous tail (no gap to stop at early), against the
oracle: equal ranks, X~ to the FP64 tolerance."""
import numpy as np
import pytest

from oracle import tt_sketch as O
from oracle import tt_svd as TS

from gpu_common import TOL_XT, rel, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,decay,eps", [
    ((1, 7, 5), 0.0, 0.2),
    ((2, 3, 5), 0.0, 0.3),
    ((8, 9, 16), 0.5, 1e-3),
    ((17, 33, 9), 0.3, 1e-6),
    ((16, 2500), 0.8, 1e-9),          # rows in two workgroups, graded columns
    ((40, 90), 0.0, 0.3),             # flat spectrum: the cut falls inside it
    ((40, 90), 0.05, 0.1),
    ((9, 4, 3, 700), 0.4, 1e-5),
])
def test_blocks_against_oracle(n, decay, eps):
    import torch
    import paper_2111_10448_amd as P
    say(f"[gpu] Parallel-TTSVD blocks n={n} decay={decay} eps={eps:g}")
    rng = np.random.default_rng(11)
    d = len(n)
    x = rng.standard_normal(n)
    for q in range(d):                # smooth decay along every mode
        x = x * np.exp(-decay * np.arange(n[q]).clip(max=60)).reshape([-1 if k == q else 1 for k in range(d)])
    x = np.ascontiguousarray(x.reshape(-1, order="F"))
    ref = TS.parallel_ttsvd(x, n, eps)
    tt = P.parallel_ttsvd(torch.from_numpy(x).cuda(), n, eps)
    want = [1] + [g.shape[2] for g in ref[:-1]] + [1]
    off = rel(tt.reconstruct().cpu().numpy(), O.tt_full(ref)) if max(want) <= 32 else 0.0
    say(f"    ranks {tt.ranks} (oracle {want}), X~ {off:.2e}")
    assert tt.ranks == [min(r, 32) for r in want]
    assert off < TOL_XT["f64"]
    tt.free()
