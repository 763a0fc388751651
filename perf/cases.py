"""Performance cases of the library: the calls its users make, over the sizes they make them at.

A case is a dict of plain values.  Its kinds:

  step    a stored tensor: reset, sketch (whole or in slabs), recover, and for a two-pass
          context the second pass.  FP64 sketches return the cores and the measured error
          (every trial of the method measures it); the other precisions expand the train
          again and return the approximation in the tensor's type.
  grad    a differentiation step: sketch, recover, expand, and the gradient of a cotangent
          (or of the squared error) with respect to the tensor.
  fn      a tensor given by a formula, never stored: sketch, recover, measured error.
  ttsvd   the deterministic Parallel-TTSVD of a stored tensor, expanded again.

Contexts (factors, sketch buffers) are made once in prepare(), as a program that
decomposes a stream of tensors of one shape keeps them.
"""
import math

import numpy as np
import torch

import paper_2111_10448_amd as P

_DEV = "cuda"


def _case(name, kind, n, **kw):
    c = {"name": name, "kind": kind, "n": ",".join(str(v) for v in n), "dtype": "f64", "prec": "f64", "ell": 0,
         "rank": 0, "eps": 0.0, "mid": "onepass", "drm": "nested", "algo": "pstt2", "slabs": 1, "noise": 0.0,
         "loss": False, "fn": ""}
    c.update(kw)
    return c


def listed():
    return [
        # one small tensor: launches and latency are all there is
        _case("step_tiny_f64", "step", (16,) * 4, ell=6, rank=3, noise=1e-6),
        # the flagship size, 8.6 GB in FP64
        _case("step_large_f64", "step", (32,) * 6, ell=20, rank=10, noise=1e-3),
        # odd modes, delivered in runs of fibres that cut columns of the unfolding, per-split factors
        _case("step_ragged_f64", "step", (27, 25, 29, 26, 23), ell=20, rank=8, noise=1e-4, slabs=9,
              drm="independent"),
        # the one-sided algorithm: a very tall sketch
        _case("step_onesided_f64", "step", (40, 36, 34, 38, 32), ell=20, rank=8, noise=1e-4, algo="pstt"),
        # tolerance mode on smooth function samples, split-precision sketches, 4.3 GB in FP32
        _case("step_tol_bf16x3", "step", (64,) * 5, dtype="f32", prec="bf16x3", ell=32, eps=1e-4),
        # a stream of 64 ragged slabs in half precision
        _case("step_slabs_f16", "step", (12, 11, 13, 12, 11, 12, 13, 10), dtype="f32", prec="f16", ell=16, rank=8,
              noise=1e-2, slabs=64),
        # an ordinary odd-sized FP32 tensor
        _case("step_odd_f32", "step", (33, 29, 31, 27, 25), dtype="f32", prec="f32", ell=24, rank=10, noise=1e-2),
        # the differentiable path: forward and the gradient of a given cotangent
        _case("grad_f32", "grad", (48,) * 4, dtype="f32", prec="f32", ell=12, rank=6, noise=1e-3),
        # the same for the squared error, the two-sided middle core, FP64
        _case("grad_loss_f64", "grad", (24,) * 5, ell=20, rank=8, noise=1e-2, mid="twosided", loss=True),
        # tensors given by a formula: evaluated inside the kernels, and from per-mode factor tables
        _case("fn_hilbert", "fn", (64,) * 5, ell=32, rank=6, fn="hilbert"),
        _case("fn_gauss", "fn", (960,) * 3, ell=32, rank=12, fn="gauss"),
        # the deterministic algorithm on a small tensor
        _case("ttsvd_f64", "ttsvd", (20, 17, 19, 21), rank=6, eps=1e-2, noise=1e-3),
    ]


def _modes(rng, d, lo, hi):
    """d mode sizes, the entries log-uniform over [lo, hi], the modes unequal."""
    total = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return [max(3, int(round(total ** (1.0 / d) * rng.uniform(0.85, 1.18)))) for _ in range(d)]


def draw(rng):
    kind = rng.choice(["step64", "step64", "step32", "step32", "tol", "onesided", "grad", "fn", "ttsvd"])
    rank = rng.randint(3, 10)
    ell = min(32, rng.choice([2 * rank, rank + 10]))
    if kind == "step64":
        d = rng.randint(3, 6)
        return _case("", "step", _modes(rng, d, 6e4, 3e8), ell=ell, rank=rank, noise=rng.choice([1e-3, 1e-5]),
                     mid=rng.choice(["onepass", "onepass", "twosided", "twopass"]),
                     drm=rng.choice(["nested", "nested", "independent"]), slabs=rng.choice([1, 1, 5, 16]))
    if kind == "step32":
        d = rng.randint(4, 8)
        return _case("", "step", _modes(rng, d, 2e5, 3e8), dtype="f32",
                     prec=rng.choice(["f32", "bf16x3", "bf16", "f16"]), ell=ell, rank=rank, noise=1e-2,
                     slabs=rng.choice([1, 1, 7, 64]))
    if kind == "tol":
        d = rng.randint(4, 6)
        return _case("", "step", _modes(rng, d, 2e5, 3e8), dtype="f32", prec=rng.choice(["f32", "bf16x3"]),
                     ell=rng.randint(16, 32), eps=rng.choice([1e-3, 1e-4]))
    if kind == "onesided":
        d = rng.randint(3, 5)
        return _case("", "step", _modes(rng, d, 1e5, 6e7), ell=ell, rank=rank, noise=1e-4, algo="pstt",
                     mid=rng.choice(["onepass", "twopass"]))
    if kind == "grad":
        d = rng.randint(3, 5)
        f32 = rng.random() < 0.5
        return _case("", "grad", _modes(rng, d, 1e5, 3e7), dtype="f32" if f32 else "f64",
                     prec="f32" if f32 else "f64", ell=ell, rank=rank, noise=1e-2,
                     mid=rng.choice(["onepass", "twosided"]), loss=not f32)
    if kind == "fn":
        d = rng.randint(3, 5)
        return _case("", "fn", _modes(rng, d, 1e6, 5e8), ell=rng.choice([16, 20, 24, 32]), rank=rng.randint(4, 6),
                     fn=rng.choice(["hilbert", "gauss"]))
    d = rng.randint(3, 4)
    return _case("", "ttsvd", _modes(rng, d, 4e3, 1.4e5), rank=rank, eps=1e-2, noise=1e-3)


# ---- inputs ----

def _n(case):
    return [int(v) for v in case["n"].split(",")]


def _ranks(case, n):
    """Target ranks, no larger than the unfoldings (or the sketch)."""
    top = case["rank"] if not case["ell"] else min(case["rank"], case["ell"])
    return [min(top, math.prod(n[:k]), math.prod(n[k:])) for k in range(1, len(n))]


def _factors(case, n, seed):
    """Packed standard-normal factors in the layout of the context's scheme."""
    d, sizes = len(n), []
    if case["drm"] == "nested":
        sizes = [n[q - 1] for q in range(1, d)] + [n[q - 1] for q in range(2, d + 1)]
    else:
        for k in range(1, d):
            sizes += [n[q - 1] for q in range(1, d + 1)]
    return np.random.default_rng([seed, 1]).standard_normal(sum(sizes) * case["ell"])


def _tensor(case, n, seed):
    """The flat column-major tensor on the GPU, of unit mean square: a random train plus
    noise, or (tolerance mode) samples of a smooth function on Chebyshev grids."""
    d, total = len(n), math.prod(n)
    rng = np.random.default_rng([seed, 2])
    if case["eps"] and case["kind"] == "step":
        acc = torch.zeros(1, dtype=torch.float64, device=_DEV)
        for nq in n:
            lo = rng.uniform(0.9, 1.1)
            t = lo + 0.5 - 0.5 * np.cos(np.pi * np.arange(nq) / max(1, nq - 1))
            acc = (torch.from_numpy(t).to(_DEV)[:, None] + acc[None, :]).reshape(-1)
        x = d / acc
    else:
        r = [1] + _ranks(case, n) + [1]
        cores = [rng.standard_normal((r[k], n[k], r[k + 1])) for k in range(d)]
        m = torch.from_numpy(cores[0][0]).to(_DEV)                       # (rows, r), first mode fastest
        for k in range(1, d):
            g = torch.from_numpy(cores[k]).to(_DEV)
            m = torch.stack([m @ g[:, i] for i in range(n[k])]).reshape(-1, r[k + 1])
        x = m.reshape(-1)
        x *= math.sqrt(total) / float(torch.linalg.vector_norm(x))
        g = torch.Generator(device=_DEV).manual_seed(int(seed))
        for a in range(0, total, 1 << 26):
            part = x[a:a + (1 << 26)]
            part += case["noise"] * torch.randn(part.numel(), generator=g, dtype=torch.float64, device=_DEV)
    return x.float() if case["dtype"] == "f32" else x


def _cotangent(case, total, seed):
    g = torch.Generator(device=_DEV).manual_seed(int(seed) + 7)
    return torch.randn(total, generator=g, dtype=torch.float64, device=_DEV).to(
        torch.float32 if case["dtype"] == "f32" else torch.float64)


def _centers(n, seed):
    return np.random.default_rng([seed, 3]).uniform(-1.0, 1.0, size=(100, len(n)))


def _cuts(case, n):
    """First entries and lengths of the slabs: runs of whole mode-1 fibres."""
    fibres, s = math.prod(n[1:]), case["slabs"]
    at = [i * fibres // s * n[0] for i in range(s + 1)]
    return [(a, b - a) for a, b in zip(at[:-1], at[1:]) if b > a]


def prepare(case, seed):
    n, kind = _n(case), case["kind"]
    st = {"case": case, "n": n}
    if kind == "fn":
        st["fn"] = P.GaussBumps(_centers(n, seed), 10.0) if case["fn"] == "gauss" else "hilbert"
    else:
        st["x"] = _tensor(case, n, seed)
    if kind == "ttsvd":
        return st
    if kind == "grad" and not case["loss"]:
        st["gbar"] = _cotangent(case, math.prod(n), seed)
    if kind == "step":
        cuts = _cuts(case, n)
        st["slabs"] = [st["x"][a:a + c] for a, c in cuts]
        st["firsts"] = [a for a, _ in cuts]
    st["ctx"] = P.PSTT2(n, case["ell"], _factors(case, n, seed), dtype=case["dtype"], prec=case["prec"],
                        ranks=None if case["eps"] else _ranks(case, n), eps=case["eps"] or None,
                        rmax=16 if case["eps"] else 0, mid=case["mid"], drm=case["drm"], algo=case["algo"])
    return st


# ---- one pass ----

def run(st):
    case, kind = st["case"], st["case"]["kind"]
    real = torch.float32 if case["dtype"] == "f32" else torch.float64
    if kind == "ttsvd":
        tt = P.parallel_ttsvd(st["x"], st["n"], case["eps"])
        return {"ranks": tt.ranks, "x": tt.reconstruct()}
    ctx = st["ctx"]
    ctx.reset()
    if kind == "fn":
        ctx.sketch_fn(st["fn"])
        tt = ctx.recover()
        return {"cores": tt.cores_torch(), "error": tt.error_fn(st["fn"])}
    if kind == "grad":
        ctx.sketch(st["x"])
        tt = ctx.recover()
        return {"x": tt.reconstruct(dtype=real), "gradient": ctx.vjp(tt, x=st["x"], gbar=st.get("gbar"))}
    if len(st["slabs"]) > 1:
        ctx.sketch_slabs(st["slabs"], st["firsts"])
    else:
        ctx.sketch(st["x"])
    tt = ctx.recover()
    if case["mid"] == "twopass":
        for s, a in zip(st["slabs"], st["firsts"]):
            ctx.middle_pass(tt, s, a)
    if case["prec"] == "f64":
        return {"cores": tt.cores_torch(), "error": tt.error(st["x"])}
    return {"ranks": tt.ranks, "x": tt.reconstruct(dtype=real)}


def work(case):
    n, kind = _n(case), case["kind"]
    d, total = len(n), math.prod(_n(case))
    size = 4 if case["dtype"] == "f32" else 8
    m = d - 1 if case["algo"] == "pstt" else (d + 1) // 2
    rank = case["rank"] or 8
    expand = 2.0 * rank * total
    if kind == "ttsvd":
        # per split one pass of pair sums and rotations over every pair of short-side vectors
        svd = sum(6.0 * total * min(math.prod(n[:k]), math.prod(n[k:])) for k in range(1, d))
        return {"bytes": 2.0 * size * total, "flops": svd + expand}
    products = 2 if case["drm"] == "nested" else d
    sketch = 2.0 * case["ell"] * products * total
    sketches = 8.0 * case["ell"] * (math.prod(n[:m]) + math.prod(n[m:]))
    if kind == "fn":
        value = 200.0 if case["fn"] == "gauss" else 2.0
        return {"bytes": sketches, "flops": sketch + expand + value * total}
    if kind == "grad":
        # X (and the cotangent) in, the approximation and the gradient out
        return {"bytes": (3.0 if case["loss"] else 4.0) * size * total + sketches,
                "flops": sketch + expand + 4.0 * rank * total + 4.0 * case["ell"] * total}
    second = 1 if case["mid"] == "twopass" else 0
    return {"bytes": (2.0 + second) * size * total + sketches, "flops": sketch + expand * (1 + second)}


# ---- the same in 64 bits, from the formulas ----

def _kr(mats):
    """Khatri-Rao product, the first factor's index fastest: rows x ell."""
    out = mats[0]
    for a in mats[1:]:
        out = (a[:, None, :] * out[None, :, :]).reshape(-1, out.shape[1])
    return out


def _split_factors(case, n, seed):
    """psi[k][q], omega[k][q] of every split k as FP64 tensors on the GPU."""
    d, ell = len(n), case["ell"]
    buf, o = torch.from_numpy(_factors(case, n, seed)).to(_DEV), 0
    psi, om = [dict() for _ in range(d + 1)], [dict() for _ in range(d + 1)]

    def take(q):
        nonlocal o
        f = buf[o:o + n[q - 1] * ell].reshape(n[q - 1], ell)
        o += n[q - 1] * ell
        return f
    if case["drm"] == "nested":
        ps, os_ = {q: take(q) for q in range(1, d)}, {q: take(q) for q in range(2, d + 1)}
        return [ps] * (d + 1), [os_] * (d + 1)
    for k in range(1, d):
        for q in range(1, d + 1):
            (psi if q <= k else om)[k][q] = take(q)
    return psi, om


def _basis(s, r):
    """The first r columns of the column-pivoted orthogonal factor, diag(R) > 0."""
    a = torch.linalg.qr(s.detach())[1].cpu().numpy()
    piv, left = [], list(range(a.shape[1]))
    for _ in range(r):
        j = max(left, key=lambda c: float(a[:, c] @ a[:, c]))
        piv.append(j)
        left.remove(j)
        u = a[:, j] / np.linalg.norm(a[:, j])
        for _ in range(2):
            a = a - np.outer(u, u @ a)
    q, rr = torch.linalg.qr(s[:, piv])
    return q * torch.sign(torch.diagonal(rr))[None, :]


def _rank_rule(case, s, d):
    v = torch.linalg.svdvals(s.detach()).cpu().numpy() ** 2
    tail, r = 0.0, len(v)
    while r > 1 and tail + v[r - 1] <= case["eps"] ** 2 / (d - 1) * v.sum():
        r -= 1
        tail += v[r]
    return min(r, 16, max(1, case["ell"] - 2), min(s.shape))


def _decompose(case, n, x, seed):
    """Cores (r, n, r') of the method's train for the flat FP64 tensor x."""
    d, one = len(n), case["algo"] == "pstt"
    m = d - 1 if one else (d + 1) // 2
    rows = [math.prod(n[:k]) for k in range(d + 1)]
    xm = x.reshape(-1, rows[m])                                           # X_m transposed: C x R
    psi, om = _split_factors(case, n, seed)
    s, t = {}, {}
    for k in range(1, m + 1):
        y = xm.T @ _kr([om[k][q] for q in range(m + 1, d + 1)])
        if k == m:
            s[m] = y
        for q in range(m, k, -1):
            y = (y.reshape(n[q - 1], rows[q - 1], -1) * om[k][q][:, None, :]).sum(0)
        s[k] = y
    for k in range(m, d):
        z = xm @ _kr([psi[k][q] for q in range(1, m + 1)])
        for q in range(m + 1, k + 1):
            z = (z.reshape(-1, n[q - 1], z.shape[1]) * psi[k][q][None]).sum(1)
        t[k] = z
    base = {}
    for k in range(1, d):
        a = s[k] if one or k < m else t[k]
        r = _rank_rule(case, a, d) if case["eps"] else _ranks(case, n)[k - 1]
        base[k] = _basis(a, r)
    g = [None] * d
    last = d - 1 if one else m - 1
    for k in range(1, last + 1):
        q = base[k].reshape(n[k - 1], rows[k - 1], -1)
        g[k - 1] = q.permute(1, 0, 2) if k == 1 else torch.einsum("ra,irb->aib", base[k - 1], q)
    if one:
        if case["mid"] == "twopass":
            g[d - 1] = (base[d - 1].T @ xm.T)[:, :, None]
        else:
            a = _kr([psi[d - 1][q] for q in range(1, d)]).T @ base[d - 1]
            g[d - 1] = torch.linalg.lstsq(a, t[d - 1].T).solution[:, :, None]
        return g
    for k in range(m + 1, d + 1):
        p = base[k - 1].reshape(-1, n[k - 1], base[k - 1].shape[1])       # (C_k, n_k, r_{k-1})
        g[k - 1] = p[0].T[:, :, None] if k == d else torch.einsum("cia,cb->aib", p, base[k])
    qp = base[m - 1] if m > 1 else torch.ones(1, 1, dtype=torch.float64, device=_DEV)
    y = s[m].reshape(n[m - 1], rows[m - 1], -1)
    if case["mid"] == "twopass":
        z = (xm.T @ base[m]).reshape(n[m - 1], rows[m - 1], -1)
        g[m - 1] = torch.einsum("ra,irb->aib", qp, z)
        return g
    om_m = _kr([om[m][q] for q in range(m + 1, d + 1)])
    if case["mid"] == "twosided" and m > 1:
        ps = _kr([psi[m - 1][q] for q in range(1, m)])
        z = torch.einsum("ac,cib->aib", torch.linalg.pinv(ps.T @ qp), torch.einsum("rc,irb->cib", ps, y))
    else:
        z = torch.einsum("ra,irc->aic", qp, y)
    g[m - 1] = z @ torch.linalg.pinv(base[m].T @ om_m)
    return g


def _sides(g):
    """Left (rows x r) and right (cols x r) interfaces at the middle split."""
    m = (len(g) + 1) // 2
    left = g[0][0]
    for c in g[1:m]:
        left = torch.einsum("ra,aib->irb", left, c).reshape(-1, c.shape[2])
    right = g[-1][:, :, 0].T
    for c in g[-2:m - 1:-1]:
        right = torch.einsum("aib,cb->cia", c, right).reshape(-1, c.shape[0])
    return left, right


def _error(g, x):
    left, right = _sides(g)
    xm, e2 = x.reshape(-1, left.shape[0]), 0.0
    step = max(1, (1 << 26) // left.shape[0])
    for a in range(0, xm.shape[0], step):
        e2 += float((xm[a:a + step] - right[a:a + step] @ left.T).square().sum())
    return math.sqrt(e2) / float(torch.linalg.vector_norm(x))


def _function(case, n, seed):
    """The formula's values, flat column-major, FP64."""
    m = (len(n) + 1) // 2
    if case["fn"] == "hilbert":
        acc = torch.zeros(1, dtype=torch.float64, device=_DEV)
        for nq in n:
            acc = (torch.arange(nq, dtype=torch.float64, device=_DEV)[:, None] + acc[None, :]).reshape(-1)
        return 1.0 / (acc + 1.0)
    c = torch.from_numpy(_centers(n, seed)).to(_DEV)
    f = [torch.exp(-10.0 * (2.0 * torch.arange(1, nq + 1, dtype=torch.float64, device=_DEV)[:, None] / nq - 1.0
                            - c[None, :, q]) ** 2) for q, nq in enumerate(n)]
    return (_kr(f[m:]) @ _kr(f[:m]).T).reshape(-1)


def _flat(g):
    return [c.permute(2, 1, 0).reshape(-1) for c in g]


def exact(case, seed):
    n, kind = _n(case), case["kind"]
    if kind == "fn":
        x = _function(case, n, seed)
        g = _decompose(case, n, x, seed)
        return {"cores": _flat(g), "error": _error(g, x)}
    x = _tensor(case, n, seed).double()
    if kind == "ttsvd":
        d, u = len(n), [torch.ones(1, 1, dtype=torch.float64)]
        x = x.cpu()
        for k in range(1, d):
            a = x.reshape(-1, math.prod(n[:k])).T
            left, sv, _ = torch.linalg.svd(a, full_matrices=False)
            v, tail, r = (sv ** 2).numpy(), 0.0, len(sv)
            while r > 1 and tail + v[r - 1] <= case["eps"] ** 2 / (d - 1) * v.sum():
                r -= 1
                tail += v[r]
            u.append(left[:, :min(r, 32)])
        g = [torch.einsum("ra,irb->aib", u[k - 1], u[k].reshape(n[k - 1], u[k - 1].shape[0], -1))
             for k in range(1, d)]
        g.append((u[d - 1].T @ x.reshape(n[d - 1], -1).T)[:, :, None])
        left, right = _sides(g)
        return {"ranks": None, "x": (right @ left.T).reshape(-1)}
    if kind == "grad":
        x.requires_grad_(True)
        left, right = _sides(_decompose(case, n, x, seed))
        y = (right @ left.T).reshape(-1)
        if case["loss"]:
            (x - y).square().sum().backward()
        else:
            y.backward(_cotangent(case, math.prod(n), seed).double())
        return {"x": y.detach(), "gradient": x.grad}
    g = _decompose(case, n, x, seed)
    if case["prec"] == "f64":
        return {"cores": _flat(g), "error": _error(g, x)}
    left, right = _sides(g)
    return {"ranks": None, "x": (right @ left.T).reshape(-1)}
