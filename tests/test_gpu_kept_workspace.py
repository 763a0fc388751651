"""Workspaces that stay allocated between calls: idle they count neither as live nor
against the budget, several threads and streams at once get one each, and a full
device gets them back."""
import threading

import numpy as np
import pytest

import inputs
from oracle import tt_sketch as O

from gpu_common import rel, say

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _clean_limit():
    import paper_2111_10448_amd as P
    P.set_memory_limit(0)
    yield
    P.set_memory_limit(0)


def _gauss(n, terms=20):
    import paper_2111_10448_amd as P
    return P.GaussBumps(np.random.default_rng(51).uniform(-1, 1, (terms, len(n))), 1.0)


@pytest.mark.parametrize("dtype,mid", [("f32", "onepass"), ("f64", "onepass"), ("f64", "twopass")])
def test_function_workspace_is_not_live_between_calls(dtype, mid):
    import torch
    import paper_2111_10448_amd as P
    from paper_2111_10448_amd import _lib as L
    n = (120, 100, 90)
    say(f"[gpu] kept function workspace {dtype} {mid}")
    ctx = P.PSTT2(n, 16, dtype=dtype, mid=mid, ranks=[4, 4], seed=2)
    fn = _gauss(n)
    torch.cuda.synchronize()
    live = P.memory_stats()["live"]
    err = []
    for _ in range(3):
        ctx.reset()
        ctx.sketch_fn(fn)
        assert P.memory_stats()["live"] == live
        tt = ctx.recover()
        if mid == "twopass":
            before = P.memory_stats()["live"]
            ctx.middle_pass_fn(tt, fn)
            assert P.memory_stats()["live"] == before
        err.append(tt.error_fn(fn))
        tt.free()
        live = P.memory_stats()["live"]   # the recovery's and the error pass's own
        torch.cuda.synchronize()
    assert err[0] == err[1] == err[2]
    # the kept block is no way round the budget, and its refusal loses nothing
    ctx.reset()
    P.set_memory_limit(P.memory_stats()["live"] + 256)
    with pytest.raises(P.PSTT2Error) as e:
        ctx.sketch_fn(fn)
    assert e.value.status == L.ENOMEM
    P.set_memory_limit(0)
    ctx.sketch_fn(fn)
    tt = ctx.recover()
    if mid == "twopass":
        ctx.middle_pass_fn(tt, fn)
    assert tt.error_fn(fn) == err[0]
    tt.free()
    ctx.close()


def test_expansion_then_error_under_a_budget():
    """The expansion's workspace does not raise what the error pass asks for."""
    import torch
    import paper_2111_10448_amd as P
    say("[gpu] budget: expansion, then error")
    rng = np.random.default_rng(52)
    n, r = (300, 310, 4), [1, 8, 4, 1]
    cores = [torch.from_numpy(rng.standard_normal(r[k] * n[k] * r[k + 1])).cuda() for k in range(3)]
    tt = P.cores_struct(cores, n, r)
    x = P.tt_reconstruct(tt)
    live = P.memory_stats()["live"]
    for _ in range(3):
        P.tt_reconstruct(tt)
        assert P.memory_stats()["live"] == live
    assert P.tt_error(tt, x) < 1e-15
    P.set_memory_limit(P.memory_stats()["live"] + (8 << 20))   # either takes 3.1 MB, a quarter more to keep
    for _ in range(3):
        P.tt_reconstruct(tt, 0, 600)
        assert P.tt_error(tt, x) < 1e-15


def test_threads_and_streams():
    import torch
    import paper_2111_10448_amd as P
    say("[gpu] kept workspaces: eight threads, a stream each")
    rng = np.random.default_rng(53)
    jobs = []
    for i in range(8):
        n, r = (31 + i, 23, 17, 11 + i), [1, 3 + i % 3, 5, 4, 1]
        cores = [rng.standard_normal((r[k], n[k], r[k + 1])) for k in range(4)]
        dev = [torch.from_numpy(np.ascontiguousarray(c.reshape(-1, order="F"))).cuda() for c in cores]
        jobs.append((n, r, dev, O.tt_full(cores)))
    torch.cuda.synchronize()
    bad = []

    def work(i):
        n, r, dev, ref = jobs[i]
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            tt = P.cores_struct(dev, n, r)
            for _ in range(25):
                x = P.tt_reconstruct(tt, stream=s)
                s.synchronize()
                if not rel(x.cpu().numpy(), ref) < 1e-14:   # ranks of at most 5
                    bad.append(i)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(8)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


def test_full_device_gets_the_block_back():
    """A 4.1 GB block kept by one context serves the allocation of another when nothing
    else is left."""
    import torch
    import paper_2111_10448_amd as P
    say("[gpu] full device: kept block given back")
    n = (1024, 1024, 1024)
    ctx = P.PSTT2(n, 8, dtype="f32", ranks=[3, 3], seed=4)
    fn = _gauss(n, 4)
    for _ in range(2):
        ctx.reset()
        ctx.sketch_fn(fn)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free, _ = torch.cuda.mem_get_info()
    fill = torch.empty(max(free - (2 << 30), 1), dtype=torch.uint8, device="cuda")
    # 2^25 rows x 6: 1.6 GB of sketch and as much of partials
    other = P.PSTT2((2048, 128, 128, 2), 6, ranks=[2, 2, 2], algo="pstt", seed=5)
    other.close()
    del fill
    torch.cuda.empty_cache()
    ctx.reset()
    ctx.sketch_fn(fn)
    tt = ctx.recover()
    assert np.isfinite(tt.error_fn(fn))
    tt.free()
    ctx.close()
