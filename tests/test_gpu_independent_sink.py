"""The independent scheme forms a right sketch for each split k <= m but a left one only
for k >= m: with d = 3 or 5 (and PSTT, m = d - 1) a pass has a left side that no split
reads.  What stands there must not decide whether the tensor counts as finite."""
import numpy as np
import pytest

from gpu_common import TOL_XT, rel, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,algo", [((7, 5, 6), "pstt2"), ((4, 3, 5, 3, 4), "pstt2"), ((5, 4, 3, 4), "pstt")])
@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_reset_after_a_refused_tensor(n, algo, bad):
    import torch
    import paper_2111_10448_amd as P
    say(f"[gpu] independent scheme, n={n} {algo}: {bad} in X, then a reset")
    rng = np.random.default_rng(len(n))
    x = rng.standard_normal(int(np.prod(n)))
    ell, d = 8, len(n)
    fac = rng.standard_normal((d - 1) * sum(n) * ell)
    kw = dict(ranks=[3] * (d - 1), drm="independent", algo=algo)
    xg = torch.from_numpy(x).cuda()
    xb = xg.clone()
    xb[x.size // 2] = bad
    ctx = P.PSTT2(n, ell, fac, **kw)
    ctx.sketch(xb)
    with pytest.raises(P.PSTT2Error) as e:
        ctx.recover()
    assert e.value.status == -5
    ctx.reset()
    ctx.sketch(xg)
    tt = ctx.recover()
    got = tt.reconstruct().cpu().numpy()
    tt.free()
    ctx.close()
    other = P.PSTT2(n, ell, fac, **kw)
    other.sketch(xg)
    tt = other.recover()
    assert rel(got, tt.reconstruct().cpu().numpy()) <= TOL_XT["f64"]
    tt.free()
    other.close()
