"""Very tall sketches and short first modes (the one-sided algorithm, whose splits
reach every mode): two-level sums of the left sketch, Q formed by a workgroup a
block, several slices a workgroup of the two-sided products with each width of
their tiles, first modes of four and five that wrap many times in a slice and ones
longer than a slice.  Against the oracle at the tolerances of the one-sided tests."""
import pytest

import inputs
import test_gpu_pstt as TP

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,rank,ell", [
    ((1030, 1024, 3), 3, 6),           # 1.05 M rows, first mode over a slice
    ((31, 33, 32, 33, 3), 3, 20),      # 1.08 M rows, first-mode rows in LDS
    ((4, 9, 8, 9, 4), 3, 16),
    ((4, 9, 8, 9, 4), 4, 17),
    ((5, 9, 8, 9, 5), 5, 20),
    ((5, 9, 8, 9, 5), 4, 21),
    ((4, 5, 41, 9, 5), 4, 32),
    ((130, 9, 8, 5), 4, 20),
    ((65, 9, 8, 5), 5, 16),
])
def test_one_sided_tall(n, rank, ell):
    name = "tall"
    inputs.WORKLOADS[name] = inputs.Workload(name, 153, tuple(n), "f64", "tt", tt_rank=rank, noise=1e-6, ell=ell,
                                             rank=rank)
    try:
        TP._run(name, None, "f64", "onepass", "nested")
    finally:
        del inputs.WORKLOADS[name]
