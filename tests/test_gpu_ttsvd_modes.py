"""Parallel-TTSVD of four and five modes whose oracle ranks all fit the cores' limit of
32, up to that limit: equal ranks, X~ to the FP64 tolerance."""
import numpy as np
import pytest

from oracle import tt_sketch as O
from oracle import tt_svd as TS

from gpu_common import TOL_XT, rel, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,decay,eps", [
    ((9, 4, 3, 700), 0.4, 1e-3),      # ranks 9, 32, 18
    ((9, 4, 3, 700), 0.4, 1e-2),
    ((9, 4, 3, 700), 0.4, 1e-1),
    ((700, 3, 4, 9), 0.4, 1e-2),
    ((6, 7, 5, 8, 9), 0.9, 1e-3),
])
def test_modes_against_oracle(n, decay, eps):
    import torch
    import paper_2111_10448_amd as P
    rng = np.random.default_rng(11)
    d = len(n)
    x = rng.standard_normal(n)
    for q in range(d):                # smooth decay along every mode
        x = x * np.exp(-decay * np.arange(n[q]).clip(max=60)).reshape([-1 if k == q else 1 for k in range(d)])
    x = np.ascontiguousarray(x.reshape(-1, order="F"))
    ref = TS.parallel_ttsvd(x, n, eps)
    want = [1] + [g.shape[2] for g in ref[:-1]] + [1]
    assert max(want) <= 32
    tt = P.parallel_ttsvd(torch.from_numpy(x).cuda(), n, eps)
    off = rel(tt.reconstruct().cpu().numpy(), O.tt_full(ref))
    say(f"[gpu] Parallel-TTSVD modes n={n} eps={eps:g}: ranks {tt.ranks}, X~ {off:.2e}")
    assert tt.ranks == want and off < TOL_XT["f64"]
    tt.free()
