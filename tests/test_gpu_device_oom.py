"""The device's own out-of-memory (not the library's budget): refused with ENOMEM at
once, and no later call sees anything of it."""
import numpy as np
import pytest

import inputs

from gpu_common import compare, oracle_run, say, setup

pytestmark = pytest.mark.gpu


def test_refused_create_leaves_later_calls_alone():
    import torch
    import paper_2111_10448_amd as P
    from paper_2111_10448_amd import _lib as L
    say("[gpu] device out of memory in create, then a whole step")
    w = inputs.WORKLOADS["c1"]
    x, psi, omega, fac = setup(w)
    ref = oracle_run(x, w, psi, omega)
    xg = torch.from_numpy(x).cuda()
    ctx = P.PSTT2(w.n, w.ell, fac, ranks=w.ranks())
    ctx.sketch(xg)
    tt = ctx.recover()
    for again in range(2):
        with pytest.raises(P.PSTT2Error) as e:   # 2^35 rows x 32: 8.8 TB of sketch
            P.PSTT2((128,) * 5 + (2,), 32, ranks=[2] * 5, algo="pstt", seed=1)
        assert e.value.status == L.ENOMEM
        if again == 0:
            assert np.isfinite(tt.reconstruct().sum().item()) and np.isfinite(tt.error(xg))
            tt.free()
            ctx.reset()
    ctx.sketch(xg)
    tt = ctx.recover()
    say(f"    {compare(ctx, tt, xg, x, w, ref, 'f64')}")
    assert float(torch.ones(4, device='cuda').sum()) == 4.0
    tt.free()
    ctx.close()
