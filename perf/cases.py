"""The decoding work this library is timed on.

Every case is a whole call of a decode a receiver makes: the dictionary is
set up once (``prepare``: a context, as a program keeps for all its signals),
and one pass decodes one measurement vector, one batch that shares the
dictionary, or one set of independent problems, to its stopping rule.  The
listed cases are the sizes the repository's generator, tests and benchmark
name; ``draw`` gives other sizes of the same ranges, ragged ones among them.

A case is a dict of plain values:
  form   f32 | bf16 | fp8 | f64   single signal, by storage of the dictionary
         sign                     single signal, Bernoulli signs in one bit each
         omp                      single signal, Orthogonal Matching Pursuit
         batched                  signals sharing one dictionary
         ragged                   independent problems, each its own dictionary
  n, m, k      rows, columns, nonzeros (batched: k is the largest K)
  eps, cap     stopping rule: relative tolerance, and at most cap steps
               (0: 20 K, the batched and ragged forms per signal)
  dist         nonzeros: normal | loguniform (log-uniform magnitudes in
               [1e-3, 1], random signs) | uniform (U[-1, 1])
  noise        standard deviation of additive measurement noise relative to
               the signal's root mean square (0: none)
  psi          gaussian (unit-norm columns) | bernoulli (+-1/sqrt(N))
  b            batched: signals; kmin: the smallest K
  count        ragged: problems, with sizes drawn from n/8 .. n
  storage      ragged: f32 | bf16
"""
import math
import random

import numpy as np
import torch

from paper_0809_1833_amd.mp import Decoder, RaggedDecoder

STOPS = {"converged": 0, "max_iters": 1, "stalled": 2, "zero_input": 3}


def _case(name, form, n, m, k, **kw):
    c = dict(name=name, form=form, n=n, m=m, k=k, eps=1e-5, cap=0, dist="normal", noise=0.0,
             psi="gaussian", b=1, kmin=0, count=1, storage="f32")
    c.update(kw)
    if name is None:  # a drawn case has no name
        del c["name"]
    return c


def listed():
    return [
        # a short signal block, decoded one at a time: latency is all there is
        _case("small", "f32", 256, 1024, 10, eps=1e-6, cap=2000),
        # an ordinary block, dictionary of 64 MiB
        _case("ordinary", "f32", 2048, 8192, 128),
        # an odd size with measurement noise, stopped at the noise level
        _case("odd-noisy", "f32", 1000, 3001, 50, noise=0.01, eps=0.012),
        # the benchmark's decode: a dictionary of 1 GiB
        _case("large", "f32", 8192, 32768, 512),
        # the same decode in double precision
        _case("large-f64", "f64", 8192, 32768, 512),
        # reduced-precision storage of the large dictionary
        _case("large-bf16", "bf16", 8192, 32768, 256),
        _case("large-fp8", "fp8", 8192, 32768, 256, dist="loguniform"),
        # the paper's own +-1 dictionary held as sign bits
        _case("large-sign", "sign", 8192, 32768, 512),
        # least-squares re-fit of all selected atoms every step
        _case("large-omp", "omp", 8192, 32768, 512),
        # a server's batch against one dictionary
        _case("batch", "batched", 2048, 8192, 256, b=256, kmin=16),
        # one dictionary draw of the recovery diagram: short columns, Bernoulli
        # entries, every sparsity from easy to hopeless
        _case("batch-diagram", "batched", 500, 1000, 500, b=500, kmin=50, psi="bernoulli",
              dist="uniform", eps=1e-7, cap=500),
        # many independent problems of uneven size
        _case("ragged", "ragged", 1024, 4096, 64, count=512),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    form = rng.choice(["f32", "f32", "bf16", "fp8", "f64", "sign", "omp", "batched", "ragged"])
    psi, dist = "gaussian", rng.choice(["normal", "normal", "loguniform", "uniform"])
    eps, noise = rng.choice([1e-6, 1e-5, 1e-5, 1e-4]), 0.0
    if rng.random() < 0.25:
        noise = rng.choice([0.003, 0.01, 0.03])
        eps = 1.2 * noise
    if form == "batched":
        n = _log(rng, 64, 2048)
        m = min(8192, int(n * rng.uniform(1.0, 5.0)))
        b = _log(rng, 2, 256)
        k = max(2, int(n * rng.uniform(0.02, 0.12)))
        if rng.random() < 0.3:
            psi = "bernoulli"
        return _case(None, form, n, m, k, b=b, kmin=max(1, k // 8), psi=psi, dist=dist,
                     eps=eps, noise=noise)
    if form == "ragged":
        n = _log(rng, 128, 1024)
        m = 4 * n
        return _case(None, form, n, m, max(2, n // 16), count=_log(rng, 8, 128), eps=eps,
                     noise=noise, dist=dist, storage=rng.choice(["f32", "bf16"]))
    n = _log(rng, 48, 8192)
    m = min(32768, int(n * rng.uniform(1.0, 6.0)))
    k = max(2, int(n * rng.uniform(0.01, 0.06)))
    if form == "f32" and rng.random() < 0.3:
        psi = "bernoulli"
    return _case(None, form, n, m, k, psi=psi, dist=dist, eps=eps, noise=noise)


# ---- inputs -------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 2654435761 % (1 << 62))
    return g


def _dictionary(g, n, m, kind, dtype):
    """(M, N) rows = columns of Psi, contiguous."""
    if kind == "bernoulli":
        s = torch.randint(0, 2, (m, n), generator=g, device="cuda", dtype=torch.int8)
        return (s.to(dtype) * 2 - 1) * (1.0 / math.sqrt(n))
    p = torch.empty((m, n), dtype=dtype, device="cuda")
    step = max(1, (1 << 26) // n)
    for j in range(0, m, step):
        q = torch.randn((min(step, m - j), n), generator=g, device="cuda", dtype=dtype)
        p[j:j + step] = q / torch.linalg.vector_norm(q.double(), dim=1, keepdim=True).to(dtype)
    return p


def _signal(g, m, k, dist):
    """K-sparse x (double): support, values."""
    sup = torch.randperm(m, generator=g, device="cuda")[:k]
    if dist == "normal":
        v = torch.randn(k, generator=g, device="cuda", dtype=torch.float64)
    else:
        u = torch.rand(k, generator=g, device="cuda", dtype=torch.float64)
        s = torch.randint(0, 2, (k,), generator=g, device="cuda").double() * 2 - 1
        v = s * (10.0 ** (-3.0 * u) if dist == "loguniform" else u)
    return sup, v


def _encode(g, rows, sup, v, noise, dtype):
    """y = Psi x in FP64 (+ noise), rounded to the decoder's type."""
    y = rows[sup].double().T @ v
    if noise:
        y = y + noise * y.square().mean().sqrt() * torch.randn(y.shape, generator=g, device="cuda",
                                                               dtype=torch.float64)
    return y.to(dtype)


def _single(case, seed):
    """Rows of Psi (of +-1 signs for the one-bit form) and y."""
    g = _gen(seed)
    dt = torch.float64 if case["form"] == "f64" else torch.float32
    if case["form"] == "sign":
        neg = torch.randint(0, 2, (case["m"], case["n"]), generator=g, device="cuda",
                            dtype=torch.int8)
        sup, v = _signal(g, case["m"], case["k"], case["dist"])
        y = _encode(g, 1 - 2 * neg[sup].to(torch.float64), torch.arange(case["k"], device="cuda"),
                    v / math.sqrt(case["n"]), case["noise"], dt)
        return neg, y
    rows = _dictionary(g, case["n"], case["m"], case["psi"], dt)
    sup, v = _signal(g, case["m"], case["k"], case["dist"])
    return rows, _encode(g, rows, sup, v, case["noise"], dt)


def _batch(case, seed):
    g = _gen(seed)
    rows = _dictionary(g, case["n"], case["m"], case["psi"], torch.float32)
    b, lo, hi = case["b"], case["kmin"], case["k"]
    if case["cap"]:  # the diagram: every sparsity of a grid, as often
        ks = [lo + (hi - lo) * i // max(b - 1, 1) for i in range(b)]
    else:
        ks = torch.randint(lo, hi + 1, (b,), generator=g, device="cuda").tolist()
    y = torch.empty((b, case["n"]), dtype=torch.float32, device="cuda")
    for j in range(b):
        sup, v = _signal(g, case["m"], ks[j], case["dist"])
        y[j] = _encode(g, rows, sup, v, case["noise"], torch.float32)
    return rows, y.t(), (case["cap"] or [20 * k for k in ks])


def _ragged(case, seed):
    """Problems of N in {n/8, n/4, n/2, n}, M = 4 N, K = N / 16."""
    g = _gen(seed)
    sizes = random.Random(case["count"] * 7919 + case["n"])  # the case's own, whatever the seed
    probs = []
    for _ in range(case["count"]):
        i = sizes.randrange(4)
        n = case["n"] >> i
        k = max(1, n // 16)
        rows = _dictionary(g, n, 4 * n, "gaussian", torch.float32)
        sup, v = _signal(g, 4 * n, k, case["dist"])
        probs.append((rows, _encode(g, rows, sup, v, case["noise"], torch.float32), 20 * k))
    return probs


def _pack(neg):
    """Sign bits, bit q of word w of a column: row 32 w + q."""
    m, n = neg.shape
    pad = torch.zeros((m, (n + 31) // 32 * 32), dtype=torch.uint8, device=neg.device)
    pad[:, :n] = neg.to(torch.uint8)
    w = (pad.view(m, -1, 8) << torch.arange(8, device=neg.device, dtype=torch.uint8)).sum(
        2, dtype=torch.uint8)
    return w.view(torch.int32)


def prepare(case, seed):
    form = case["form"]
    if form == "batched":
        rows, y, cap = _batch(case, seed)
        return dict(case=case, dec=Decoder(rows.t()), y=y, cap=cap)
    if form == "ragged":
        probs = _ragged(case, seed)
        dec = RaggedDecoder([p[0].t() for p in probs], storage=case["storage"])
        return dict(case=case, dec=dec, y=dec.pack([p[1] for p in probs]),
                    cap=[p[2] for p in probs])
    rows, y = _single(case, seed)
    if form == "sign":
        dec = Decoder(_pack(rows), storage="sign", n=case["n"])
    else:
        dec = Decoder(rows.t(), storage="f32" if form == "omp" else form)
    return dict(case=case, dec=dec, y=y, cap=case["cap"] or 20 * case["k"])


def run(state):
    case, dec = state["case"], state["dec"]
    if case["form"] == "batched":
        out = dec.solve_batched(state["y"], case["eps"], state["cap"])
    elif case["form"] == "ragged":
        out = dec.solve(state["y"], case["eps"], state["cap"])
    else:
        out = dec.solve(state["y"], case["eps"], state["cap"], omp=case["form"] == "omp")
        return dict(x=out["x"], r=out["r"], iters=out["iters"], yy=out["yy"], rr=out["rr"],
                    stop=STOPS[out["stop"]])
    return dict(x=out["x"], r=out["r"], iters=np.array(out["iters"]), yy=np.array(out["yy"]),
                rr=np.array(out["rr"]), stop=np.array([STOPS[s] for s in out["stop"]]))


# ---- what a pass cannot do without ---------------------------------------------

def work(case):
    """The dictionary and the measurements read once, x~ and r written once;
    every signal correlated with every column once, and each of its K atoms
    taken off the residual once."""
    form, n, m, k = case["form"], case["n"], case["m"], case["k"]
    if form == "batched":
        b, kb = case["b"], (case["kmin"] + k) / 2
        return {"bytes": 4.0 * n * m + 4.0 * b * (2 * n + m), "flops": b * (2.0 * n * m + 4 * n * kb)}
    if form == "ragged":
        e = 2 if case["storage"] == "bf16" else 4
        sizes = [n >> i for i in range(4)]
        each = case["count"] / 4.0
        return {"bytes": sum(each * (e * 4.0 * s * s + 4.0 * 6 * s) for s in sizes),
                "flops": sum(each * (8.0 * s * s + 4.0 * s * s / 16) for s in sizes)}
    size = {"f32": 4, "omp": 4, "f64": 8, "bf16": 2, "fp8": 1, "sign": 0.125}[form]
    v = 8 if form == "f64" else 4
    return {"bytes": size * n * m + v * (2.0 * n + m), "flops": 2.0 * n * m + 4.0 * n * k}


# ---- the same decodes in 64 bits -------------------------------------------------

def _mp64(rows, y, eps, cap):
    """Section 3's loop: rows (M, N) double, y double."""
    r, x, t = y.clone(), torch.zeros(rows.shape[0], dtype=torch.float64, device=y.device), 0
    yy = rr = float(y @ y)
    while rr > eps * eps * yy and t < cap:
        c = rows @ r
        i = torch.argmax(c.abs())
        x[i] += c[i]
        r -= c[i] * rows[i]
        t += 1
        rr = float(r @ r)
    return x, r, yy, rr


def _omp64(rows, y, eps, cap):
    """r orthogonal to every selected atom: a QR of them, one column a step."""
    m, n = rows.shape
    r, t = y.clone(), 0
    cap = min(cap, n)
    q = torch.zeros((cap, n), dtype=torch.float64, device=y.device)
    tri = torch.zeros((cap, cap), dtype=torch.float64, device=y.device)
    z = torch.zeros(cap, dtype=torch.float64, device=y.device)
    sel = []
    yy = rr = float(y @ y)
    while rr > eps * eps * yy and t < cap:
        i = int(torch.argmax((rows @ r).abs()))
        if i in sel:
            break
        w = rows[i].clone()
        for _ in range(2):
            h = q[:t] @ w
            w -= h @ q[:t]
            tri[:t, t] += h
        rho = float(w @ w) ** 0.5
        if rho * rho <= 1e-10:
            break
        tri[t, t] = rho
        q[t] = w / rho
        z[t] = q[t] @ r
        r -= z[t] * q[t]
        sel.append(i)
        t += 1
        rr = float(r @ r)
    x = torch.zeros(m, dtype=torch.float64, device=y.device)
    if t:
        x[torch.tensor(sel, device=y.device)] = torch.linalg.solve_triangular(
            tri[:t, :t], z[:t, None], upper=True)[:, 0]
    return x, r, yy, rr


def _batch64(rows, y, eps, caps):
    """Every column of y by itself, the correlations of all taken together."""
    b = y.shape[1]
    r, x = y.clone(), torch.zeros((rows.shape[0], b), dtype=torch.float64, device=y.device)
    yy = r.square().sum(0)
    rr, j, t = yy.clone(), torch.arange(b, device=y.device), 0
    caps = torch.tensor(caps if isinstance(caps, list) else [caps] * b, device=y.device)
    while True:
        go = ((rr > eps * eps * yy) & (caps > t)).nonzero()[:, 0]
        if not go.numel():
            return x, r, yy, rr
        rg = r[:, go]
        c = rows @ rg
        i = c.abs().argmax(0)
        ci = c.gather(0, i[None])[0]
        x[i, go] += ci
        rg -= rows[i].T * ci
        r[:, go] = rg
        rr[go] = rg.square().sum(0)
        t += 1


def exact(case, seed):
    """x~ and the norms; the final r where it is carried in 64 bits (the FP64
    and one-bit forms).  An FP32 decode's r after a fall of 1e5 is what its
    own roundings leave, and has no 64-bit counterpart to that many digits."""
    form = case["form"]
    if form == "batched":
        rows, y, caps = _batch(case, seed)
        x, _, yy, _ = _batch64(rows.double(), y.double(), case["eps"], caps)
        # a cap of N steps ends signals that nothing can recover anywhere in
        # their wandering: no value to hold them to
        x = None if case["cap"] else x
        return dict(x=x, r=None, iters=None, yy=yy.cpu().numpy(), rr=None, stop=None)
    if form == "ragged":
        probs = _ragged(case, seed)
        got = [_mp64(p[0].double(), p[1].double(), case["eps"], p[2]) for p in probs]
        return dict(x=torch.cat([g[0] for g in got]), r=None, iters=None,
                    yy=np.array([g[2] for g in got]), rr=None, stop=None)
    rows, y = _single(case, seed)
    if form == "sign":
        rows = (1 - 2 * rows.to(torch.float64)) / math.sqrt(case["n"])
    solve = _omp64 if form == "omp" else _mp64
    x, r, yy, rr = solve(rows.double(), y.double(), case["eps"], case["cap"] or 20 * case["k"])
    wide = form in ("f64", "sign")
    return dict(x=x, r=r if wide else None, iters=None, yy=yy, rr=rr if wide else None, stop=None)
