"""The FP64 Gaussian-bump sketch with a launch of it failing (tables, moments, Y, T in
this order): nothing added before Y ran, so a retry completes; from then on the context
is poisoned until it is reset."""
import numpy as np
import pytest

import inputs

from gpu_common import compare, oracle_run, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("launch,added", [(0, False), (1, False), (2, False), (3, True)])
def test_each_launch(launch, added):
    import torch
    import paper_2111_10448_amd as P
    from paper_2111_10448_amd import _lib as L
    say(f"[gpu] Gaussian-bump sketch, launch {launch} fails")
    w = inputs.WORKLOADS["gb_small3"]
    x = inputs.make_tensor(w)
    psi, omega = inputs.drm_factors(w)
    ref = oracle_run(x, w, psi, omega)
    xg = torch.from_numpy(x).cuda()
    fn = P.GaussBumps(inputs.gauss_centers(w), w.gamma)
    ctx = P.PSTT2(w.n, w.ell, inputs.pack_factors(psi, omega, w.d), ranks=w.ranks())
    P.inject_launch_failure(launch)
    try:
        with pytest.raises(P.PSTT2Error) as e:
            ctx.sketch_fn(fn)
    finally:
        P.inject_launch_failure(-1)
    assert e.value.status == L.EDEVICE
    if added:
        for call in (lambda: ctx.sketch_fn(fn), ctx.recover):
            with pytest.raises(P.PSTT2Error) as e:
                call()
            assert e.value.status == L.ESTATE
        ctx.reset()
    ctx.sketch_fn(fn)
    tt = ctx.recover()
    say(f"    {compare(ctx, tt, xg, x, w, ref, 'f64')}")
    tt.free()
    ctx.close()
