"""Parallel-TTSVD of a tensor times a power of two: the same ranks and bases, the last
core times it, bit for bit, wherever no product of the result leaves FP64's range; with
short sides over and under the number of leading columns, with and without a gap."""
import numpy as np
import pytest

from gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rank,eps", [
    ((40, 90), 4, 1e-2),
    ((90, 40), 4, 1e-2),
    ((24, 60), 60, 0.3),            # no gap: sweeps
    ((12, 30), 3, 1e-2),            # short side under the leading columns
    ((9, 8, 7, 10), 3, 1e-2),
])
@pytest.mark.parametrize("power", [-400, -262, -150, 150, 250, 400])
def test_power_of_two(n, rank, eps, power):
    import torch
    import paper_2111_10448_amd as P
    say(f"[gpu] Parallel-TTSVD n={n} rank={rank} times 2^{power}")
    rng = np.random.default_rng(41)
    t = rng.standard_normal((1, n[0], rank))
    for q in range(1, len(n)):
        g = rng.standard_normal((rank, n[q], 1 if q == len(n) - 1 else rank))
        t = np.tensordot(t, g, axes=([t.ndim - 1], [0]))
    x = np.ascontiguousarray(t.reshape(n).reshape(-1, order="F"))
    x += 1e-5 * np.abs(x).max() * rng.standard_normal(x.size)
    plain = P.parallel_ttsvd(torch.from_numpy(x).cuda(), n, eps)
    scaled = P.parallel_ttsvd(torch.from_numpy(np.ldexp(x, power)).cuda(), n, eps)
    assert scaled.ranks == plain.ranks
    a, b = plain.cores_numpy(), scaled.cores_numpy()
    for k in range(len(n)):
        want = np.ldexp(a[k], power) if k == len(n) - 1 else a[k]
        assert np.array_equal(b[k], want), k
    plain.free()
    scaled.free()
