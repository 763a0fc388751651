"""Parallel-TTSVD where a gap follows the kept singular values (the leading columns
are turned out by power steps): kept ranks below, at and above their number, short
sides just over it, rows in one and several workgroups, tails from large to none at
all, and structured tensors whose first columns say nothing.  Against the oracle:
equal ranks, X~ to the FP64 tolerance."""
import numpy as np
import pytest

from oracle import tt_sketch as O
from oracle import tt_svd as TS

from gpu_common import TOL_XT, rel, say

pytestmark = pytest.mark.gpu


def _check(x, n, eps):
    import torch
    import paper_2111_10448_amd as P
    ref = TS.parallel_ttsvd(x, n, eps)
    tt = P.parallel_ttsvd(torch.from_numpy(x).cuda(), n, eps)
    want = [1] + [g.shape[2] for g in ref[:-1]] + [1]
    off = rel(tt.reconstruct().cpu().numpy(), O.tt_full(ref)) if max(want) <= 32 else 0.0
    say(f"    ranks {tt.ranks} (oracle {want}), X~ {off:.2e}")
    assert tt.ranks == [min(r, 32) for r in want]
    assert off < TOL_XT["f64"]
    tt.free()


@pytest.mark.parametrize("n,rank,noise,eps", [
    ((17, 40), 3, 1e-3, 1e-1),
    ((40, 17), 15, 1e-4, 1e-2),
    ((40, 90), 16, 1e-4, 1e-2),
    ((40, 90), 17, 1e-4, 1e-2),            # one more than the leading columns
    ((64, 65), 1, 1e-2, 2e-1),
    ((33, 3000), 5, 1e-6, 1e-4),           # rows in two workgroups
    ((1000, 700), 4, 1e-3, 1e-1),          # several waves of rows in the reflectors
    ((300, 301), 6, 0.0, 1e-6),            # no tail but rounding
    ((20, 17, 19, 21), 6, 1e-3, 1e-2),
    ((12, 11, 13, 9, 10), 4, 1e-8, 1e-6),
])
def test_lead_against_oracle(n, rank, noise, eps):
    say(f"[gpu] Parallel-TTSVD lead n={n} rank={rank} noise={noise:g} eps={eps:g}")
    rng = np.random.default_rng(12)
    d = len(n)
    t = rng.standard_normal((1, n[0], rank))
    for q in range(1, d):
        g = rng.standard_normal((rank, n[q], 1 if q == d - 1 else rank))
        t = np.tensordot(t, g, axes=([t.ndim - 1], [0]))
    x = np.ascontiguousarray(t.reshape(n).reshape(-1, order="F"))
    x = x / np.linalg.norm(x) * np.sqrt(x.size)
    _check(x + noise * rng.standard_normal(x.size), n, eps)


@pytest.mark.parametrize("kind", ["zero", "last_columns", "one_entry", "equal"])
def test_lead_structured(kind):
    """Zero leading columns, one nonzero entry, equal singular values, X = 0."""
    n = (24, 60)
    say(f"[gpu] Parallel-TTSVD lead {kind}")
    x = np.zeros(n)
    if kind == "last_columns":
        x[20:, 50:] = np.random.default_rng(13).standard_normal((4, 10))
    elif kind == "one_entry":
        x[23, 59] = 2.0
    elif kind == "equal":
        x[:8, :8] = np.eye(8)
    _check(np.ascontiguousarray(x.reshape(-1, order="F")), n, 1e-3)
