"""tt_reconstruct over ranges of entries against the entry formula (Section 2.2) in
FP64: every register slot of the rank, row counts that do and do not allow the
wide stores, ranges that start and end inside a column, both types.  An entry is
a sum of products of at most d r^(d-1) roundings, so 1e-13 of the same sum over
absolute values bounds it, plus half a unit of the output type."""
import numpy as np
import pytest

import inputs

from gpu_common import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,r,dtype", [
    ((7, 5), (3,), "f64"),                       # d = 2: both interfaces are cores
    ((12, 10, 9), (4, 5), "f64"),
    ((12, 10, 9), (4, 5), "f32"),
    ((11, 13, 7, 5), (6, 12, 5), "f32"),         # odd row count
    ((16, 12, 6, 10), (9, 16, 8), "f32"),
    ((16, 12, 6, 10), (9, 17, 8), "f64"),
    ((18, 11, 8, 9), (18, 24, 9), "f32"),        # R % 4 == 2
    ((40, 34, 36, 35), (32, 32, 32), "f32"),     # more than one row block
    ((40, 34, 36, 35), (32, 27, 32), "f64"),
    ((3, 5, 4, 3, 6, 5), (3, 8, 13, 20, 5), "f64"),
])
def test_reconstruct_ranges(n, r, dtype):
    import torch
    import paper_2111_10448_amd as P
    say(f"[gpu] reconstruct n={n} r={r} {dtype}")
    rng = np.random.default_rng(3)
    d, rk = len(n), (1,) + r + (1,)
    cores = [rng.standard_normal((rk[k], n[k], rk[k + 1])) for k in range(d)]
    ref = inputs.dense_from_cores(cores)
    size = inputs.dense_from_cores([np.abs(g) for g in cores])
    gpu = [torch.from_numpy(np.ascontiguousarray(g.reshape(-1, order="F"))).cuda() for g in cores]
    cs = P.cores_struct(gpu, n, rk)
    N, half = ref.size, 0.0 if dtype == "f64" else 2.0 ** -24
    R = int(np.prod(n[:(d + 1) // 2]))
    for first, count in ((0, N), (4, N - 8), (1, N - 1), (R + 3, min(R, N - R - 3)), (N - 5, 5), (6, 1), (8, 0)):
        got = P.tt_reconstruct(cs, first, count, torch.float64 if dtype == "f64" else torch.float32).cpu().numpy()
        assert got.shape == (count,)
        part = slice(first, first + count)
        assert np.all(np.abs(got - ref[part]) <= 1e-13 * size[part] + half * np.abs(ref[part])), (first, count)
