"""Sizes whose natural launch would have 2^32 threads or more, which a launch may not:
a mode of 2^24 in the middle of a tensor (one small product for each index), and
TT-SVD work matrices of 2^28 rows."""
import math

import numpy as np
import pytest

from gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [(2, 2, 1 << 24, 2), (2, 1 << 24, 2)])
def test_wide_middle_mode(n):
    """core_right over n_3 and the middle core's product over n_2."""
    import torch
    import paper_2111_10448_amd as P
    say(f"[gpu] wide mode n={n}")
    d, ell, r = len(n), 4, 2
    gen = torch.Generator(device="cuda").manual_seed(71)
    u = torch.randn(int(np.prod(n[:-1])), r, generator=gen, dtype=torch.float64, device="cuda")
    v = torch.randn(r, n[-1], generator=gen, dtype=torch.float64, device="cuda")
    x = torch.matmul(u, v).t().contiguous().reshape(-1)       # last unfolding of rank 2
    ranks = [2, 4, 2][:d - 1] if d == 4 else [2, 2]
    ctx = P.PSTT2(n, ell, ranks=ranks, seed=7)
    ctx.sketch(x)
    tt = ctx.recover()
    err = tt.error(x)
    say(f"    ranks {tt.ranks}, error {err:.1e}")
    assert err < 1e-10      # every unfolding's rank is kept
    tt.free()
    ctx.close()


def test_ttsvd_2_28_rows():
    import torch
    import paper_2111_10448_amd as P
    free, _ = torch.cuda.mem_get_info()
    if free < 170 << 30:
        pytest.skip("needs 170 GB")
    say("[gpu] Parallel-TTSVD 2^28 x 17")
    rows, s, r = 1 << 28, 17, 2
    gen = torch.Generator(device="cuda").manual_seed(72)
    u = [torch.randn(rows, generator=gen, dtype=torch.float64, device="cuda") for _ in range(r)]
    v = np.random.default_rng(72).standard_normal((r, s))
    x = torch.empty(rows * s, dtype=torch.float64, device="cuda")
    for c in range(s):
        torch.mul(u[0], v[0, c], out=x[c * rows:(c + 1) * rows])
        x[c * rows:(c + 1) * rows].add_(u[1], alpha=v[1, c])
    del u
    torch.cuda.empty_cache()
    torch.cuda.synchronize()
    say("    made")
    tt = P.parallel_ttsvd(x, (rows, s), 1e-6)
    say(f"    ranks {tt.ranks}")
    assert tt.ranks == [1, r, 1]
    for first in (0, rows * s // 2 + 1, rows * s - 4096):
        got = tt.reconstruct(first, 4096)
        assert float(torch.linalg.vector_norm(got - x[first:first + 4096])) < 1e-10 * math.sqrt(4096 * r)
    tt.free()
    del x
    torch.cuda.empty_cache()
