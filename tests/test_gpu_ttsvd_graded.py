"""Relative accuracy of small singular values in Parallel-TTSVD: a matrix with graded
columns, increasing and in no order, short sides over and under the number of leading
columns.  The rows of G_2 of X = U G_2 have the singular values as norms; against
one-sided Jacobi in extended precision.  The columns are well conditioned but for their
norms (condition number under 20 at these shapes), so one-sided Jacobi in FP64 loses no
more than some 100 rows x 2.2e-16 x 20 = 5e-13 of each."""
import numpy as np
import pytest

from gpu_common import say

pytestmark = pytest.mark.gpu


def _singular_values(a):
    """One-sided Jacobi in extended precision, a: tall."""
    w = a.astype(np.longdouble).copy()
    s = w.shape[1]
    for _ in range(60):
        moved = False
        for p in range(s - 1):
            for q in range(p + 1, s):
                x, y, g = w[:, p] @ w[:, p], w[:, q] @ w[:, q], w[:, p] @ w[:, q]
                if g != 0 and abs(g) > 1e-18 * np.sqrt(x) * np.sqrt(y):
                    moved = True
                    z = (y - x) / (2 * g)
                    t = (1 if z >= 0 else -1) / (abs(z) + np.sqrt(1 + z * z))
                    c = 1 / np.sqrt(1 + t * t)
                    u, v = w[:, p].copy(), w[:, q].copy()
                    w[:, p], w[:, q] = c * u - c * t * v, c * t * u + c * v
        if not moved:
            break
    return np.sort(np.sqrt((w * w).sum(axis=0)))[::-1]


def _graded(rows, s, order):
    rng = np.random.default_rng(31)
    g = 10.0 ** -np.arange(s)
    g = {"increasing": g[::-1], "decreasing": g, "mixed": g[rng.permutation(s)]}[order]
    return rng.standard_normal((rows, s)) * g


@pytest.mark.parametrize("s", [12, 17, 24])
@pytest.mark.parametrize("order", ["increasing", "mixed", "decreasing"])
def test_short_side_first(s, order):
    """n = (s, rows): the graded side is the first mode, G_2 = (X^T U)^T."""
    import torch
    import paper_2111_10448_amd as P
    say(f"[gpu] Parallel-TTSVD graded ({s}, 90) {order}")
    a = _graded(90, s, order)
    ref = _singular_values(a)
    tt = P.parallel_ttsvd(torch.from_numpy(np.ascontiguousarray(a.T.reshape(-1, order="F"))).cuda(), (s, 90), 1e-11)
    g = tt.cores_numpy()[1].reshape(tt.ranks[1], 90, order="F").astype(np.longdouble)
    off = np.abs(np.sqrt((g * g).sum(axis=1)) / ref[:tt.ranks[1]] - 1).astype(float)
    say(f"    rank {tt.ranks[1]}, worst singular value {off.max():.1e}")
    assert tt.ranks[1] >= 11 and off.max() < 5e-13
    tt.free()


@pytest.mark.parametrize("s", [12, 24])
@pytest.mark.parametrize("order", ["increasing", "mixed", "decreasing"])
def test_short_side_last(s, order):
    """n = (rows, s): the graded side is the last mode, small rows of G_2 = Sigma V^T."""
    import torch
    import paper_2111_10448_amd as P
    say(f"[gpu] Parallel-TTSVD graded (90, {s}) {order}")
    a = _graded(90, s, order)
    ref = _singular_values(a)
    tt = P.parallel_ttsvd(torch.from_numpy(np.ascontiguousarray(a.reshape(-1, order="F"))).cuda(), (90, s), 1e-11)
    u = tt.cores_numpy()[0].reshape(90, tt.ranks[1], order="F")
    g = tt.cores_numpy()[1].reshape(tt.ranks[1], s, order="F").astype(np.longdouble)
    off = np.abs(np.sqrt((g * g).sum(axis=1)) / ref[:tt.ranks[1]] - 1).astype(float)
    res = np.linalg.norm(a - u @ g.astype(np.float64)) / np.linalg.norm(a)
    say(f"    rank {tt.ranks[1]}, worst singular value {off.max():.1e}, U^T U - I "
        f"{np.linalg.norm(u.T @ u - np.eye(tt.ranks[1])):.1e}, X~ {res:.1e}")
    assert tt.ranks[1] >= 11 and off.max() < 5e-13
    assert np.linalg.norm(u.T @ u - np.eye(tt.ranks[1])) < 1e-14 and res < 1e-11 + 1e-14
    tt.free()
