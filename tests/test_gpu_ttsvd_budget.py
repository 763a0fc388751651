"""Parallel-TTSVD under a budget that holds its work matrix and results, but not the
workspace of the leading columns' steps beside them: it goes without."""
import numpy as np
import pytest

from oracle import tt_sketch as O
from oracle import tt_svd as TS

from gpu_common import TOL_XT, rel, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("taken", [False, True])     # no room for it; room, but not for the results beside it
@pytest.mark.parametrize("n", [(17, 100000), (100000, 18)])
def test_without_room_for_the_leading_columns(n, taken):
    import torch
    import paper_2111_10448_amd as P
    say(f"[gpu] Parallel-TTSVD n={n} under a budget")
    rng = np.random.default_rng(61)
    rank, long, s = 3, max(n), min(n)
    x = rng.standard_normal((n[0], rank)) @ rng.standard_normal((rank, n[1]))
    x = np.ascontiguousarray((x + 1e-4 * rng.standard_normal(n)).reshape(-1, order="F"))
    xg = torch.from_numpy(x).cuda()
    ref = O.tt_full(TS.parallel_ttsvd(x, n, 1e-2))
    live = P.memory_stats()["live"]
    work = 8 * long * (s + s % 2)
    result, steps = 2 * 8 * rank * (long + s), 8 * 16 * long      # 4.8 and 12.8 MB
    P.set_memory_limit(live + work + (steps + (1 << 20) if taken else result + (1 << 21)))
    try:
        tt = P.parallel_ttsvd(xg, n, 1e-2)
    finally:
        P.set_memory_limit(0)
    off = rel(tt.reconstruct().cpu().numpy(), ref)
    say(f"    ranks {tt.ranks}, X~ {off:.2e}")
    assert tt.ranks == [1, rank, 1] and off < TOL_XT["f64"]
    tt.free()
