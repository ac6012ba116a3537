"""Which form a decode takes, and what it may not depend on: caps of any size,
inputs on which a form makes slow progress or hands a decode on, and the
decode forms that are chosen only by size, cap or on request."""
from __future__ import annotations

import math

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0809_1833_amd import mp
    mp.library()


def _rows(n, m, seed=0, dtype=torch.float32):
    g = torch.Generator(device="cuda").manual_seed(100 * seed + n * 7 + m)
    rows = torch.randn((m, n), generator=g, device="cuda", dtype=torch.float64)
    return (rows / rows.norm(dim=1, keepdim=True)).to(dtype)


def _signal(rows, k, noise=0.0, seed=0):
    m, n = rows.shape
    g = torch.Generator(device="cuda").manual_seed(seed + 11)
    sup = torch.randperm(m, generator=g, device="cuda")[:k]
    v = torch.randn(k, generator=g, device="cuda", dtype=torch.float64)
    y = v @ rows[sup].double()
    if noise:
        y = y + noise * y.norm() / math.sqrt(n) * torch.randn(n, generator=g, device="cuda",
                                                               dtype=torch.float64)
    return y.to(rows.dtype)


def _pack(neg):
    """Sign bits (M, N) int8 to the packed words of mp_create_signs."""
    m, n = neg.shape
    pad = torch.zeros((m, (n + 31) // 32 * 32), dtype=torch.uint8, device="cuda")
    pad[:, :n] = neg.to(torch.uint8)
    w = (pad.view(m, -1, 8) << torch.arange(8, device="cuda", dtype=torch.uint8)).sum(
        2, dtype=torch.uint8)
    return w.view(torch.int32)


def _equal(a, b, keys=("x", "r")):
    for key in ("iters", "stop", "yy", "rr"):
        assert a[key] == b[key], (key, a[key], b[key])
    for key in keys:
        assert torch.equal(a[key], b[key]), key


@pytest.mark.parametrize("form", ["f32", "small", "bf16", "fp8", "f64", "sign"])
def test_caps_near_the_largest_integer(form):
    """A cap no decode reaches decodes as any other, up to 2^63 - 1."""
    from paper_0809_1833_amd.mp import Decoder
    n, m = (100, 400) if form == "small" else (500, 3000)
    rows = _rows(n, m, dtype=torch.float64 if form == "f64" else torch.float32)
    if form == "sign":
        g = torch.Generator(device="cuda").manual_seed(5)
        neg = torch.randint(0, 2, (m, n), generator=g, device="cuda", dtype=torch.int8)
        y = _signal((1 - 2 * neg.float()) / math.sqrt(n), 8)
        dec = Decoder(_pack(neg), storage="sign", n=n)
    else:
        y = _signal(rows, 8)
        dec = Decoder(rows.t(), storage="f32" if form == "small" else form)
    with dec:
        want = dec.solve(y, 1e-5, 5000)
        assert want["stop"] == "converged" and want["iters"] >= 8
        for cap in (2**60, 2**61, 2**62 - 2, 2**62 - 1, 2**62, 2**63 - 2, 2**63 - 1):
            print(f"[cap {form} {cap}]", flush=True)
            _equal(dec.solve(y, 1e-5, cap), want)
            if form != "small":
                _equal(dec.solve(y, 1e-5, cap, step_launches=True), want)


# ---- one-bit dictionaries -------------------------------------------------------

def _sign_same(neg, y, eps, cap):
    from paper_0809_1833_amd.mp import Decoder
    kw = dict(trace_cap=max(cap, 1), trace_r=True)
    with Decoder(_pack(neg), storage="sign", n=neg.shape[1]) as dec:
        a = dec.solve(y, eps, cap, **kw)
        b = dec.solve(y, eps, cap, step_launches=True, **kw)
    _equal(a, b, ("x", "r", "idx", "coef", "rr_trace", "r_trace"))
    return a


@pytest.mark.parametrize("n,m,noise", [(2048, 8192, 0.2), (9000, 16384, 0.05)])
def test_signs_with_most_atoms_near_the_largest(n, m, noise):
    """Nested columns, the last ones next to y: thousands of atoms within a few
    percent of the largest |c|, in an order that fills the active atoms with
    the smallest of them.  The batches hand the decode on, in the middle or
    before its first step, and the results are one launch per step's."""
    most = n // 32 - torch.arange(m, device="cuda") * (n // 32 + 1) // m
    neg = (torch.arange(n, device="cuda")[None, :] < most[:, None]).to(torch.int8)
    g = torch.Generator(device="cuda").manual_seed(4)
    y = 1 + noise * torch.randn(n, generator=g, device="cuda")
    print(f"[signs nested {n}x{m}]", flush=True)
    a = _sign_same(neg, y, 1e-6, 200)
    assert a["iters"] > 20
    # nested columns beside independent ones: quick steps first
    neg[: m // 2] = torch.randint(0, 2, (m // 2, n), generator=g, device="cuda", dtype=torch.int8)
    a = _sign_same(neg, y + 3 * (1 - 2 * neg[:40].float()).sum(0), 1e-6, 400)
    assert a["iters"] > 40


@pytest.mark.parametrize("m", [40, 3000])
@pytest.mark.parametrize("cap", [10, 100])
def test_signs_stall(m, cap):
    """No column correlates with y, at once or after one step: with caps that
    take the persistent launch and the batches, and with every atom active and
    only some of them (those that are not have c = 0 as well)."""
    h = torch.zeros((1, 1), dtype=torch.int8, device="cuda")
    for _ in range(6):
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, 1 - h], 1)], 0)
    cols = [j % 40 for j in range(m)]
    for extra in (0.0, 2.0):
        y = (1 - 2 * h[50].float()) + extra * (1 - 2 * h[7].float())
        print(f"[signs stall {m} cap {cap} {extra}]", flush=True)
        a = _sign_same(h[cols].contiguous(), y, 1e-6, cap)
        assert a["stop"] == "stalled" and a["iters"] == (1 if extra else 0)
        assert a["iters"] == 0 or int(a["idx"][0]) == 7


def test_signs_small_with_a_large_cap():
    g = torch.Generator(device="cuda").manual_seed(2)
    neg = torch.randint(0, 2, (65, 33), generator=g, device="cuda", dtype=torch.int8)
    a = _sign_same(neg, _signal((1 - 2 * neg.float()) / math.sqrt(33), 2), 1e-6, 100)
    assert a["iters"] >= 2


@pytest.mark.parametrize("n,clusters", [(2048, 16), (9000, 17)])
def test_signs_handed_on(n, clusters):
    """Clusters of 1000 nested columns of about equal |c|: the atom after the
    first is in a cluster of which no atom is active, and its best come last.
    Too few steps a round: the persistent launch (17 x 1000 columns of 9000 do not
    fit it: one launch per step) goes on from where the batches stopped."""
    from paper_0809_1833_amd.mp import Decoder
    g = torch.Generator(device="cuda").manual_seed(3)
    u = torch.randint(0, 2, (clusters, n), generator=g, device="cuda", dtype=torch.int8)
    flips = n // 32 - torch.arange(1000, device="cuda") * (n // 32 + 1) // 1000
    flip = (torch.arange(n, device="cuda")[None, :] < flips[:, None]).to(torch.int8)
    neg = (u[:, None, :] ^ flip[None]).reshape(1000 * clusters, n)
    a = 1 - 0.003 * torch.arange(clusters, device="cuda")
    y = (a[:, None] * (1 - 2 * u.float())).sum(0)
    print(f"[signs clusters {n}]", flush=True)
    out = _sign_same(neg, y, 1e-6, 300)
    with Decoder(_pack(neg), storage="sign", n=n) as dec:
        _equal(dec.solve(y, 1e-6, 300), out)
        assert 0 < dec.carried_steps() < out["iters"]


# ---- decodes that carried correlations hand on ------------------------------------

@pytest.mark.parametrize("form,n,m", [("f32", 4096, 200), ("small", 300, 40),
                                      ("f64", 2048, 100)])
def test_handed_on_in_the_middle(form, n, m):
    """Noise outside the span of fewer atoms than rows: the correlations fall
    far below ||r||, no shortlist is narrow enough any more, and one launch per
    step (the one launch, for a small dictionary) goes on from there."""
    from paper_0809_1833_amd.mp import Decoder
    rows = _rows(n, m, dtype=torch.float64 if form == "f64" else torch.float32)
    kw = dict(trace_cap=900, trace_r=True)
    with Decoder(rows.t(), storage="f64" if form == "f64" else "f32") as dec:
        for seed in range(4):
            y = _signal(rows, 5, noise=0.3, seed=seed)
            print(f"[handed on {form} {seed}]", flush=True)
            a = dec.solve(y, 1e-7, 900, **kw)
            assert 0 < dec.carried_steps() < a["iters"] == 900 and a["rr"] > 0.01 * a["yy"]
            b = dec.solve(y, 1e-7, 900, step_launches=True, **kw)
            assert dec.carried_steps() == 0
            _equal(a, b, ("x", "r", "idx", "coef", "rr_trace", "r_trace"))


@pytest.mark.parametrize("storage", ["bf16", "fp8"])
def test_reduced_precision_handed_on(storage):
    from paper_0809_1833_amd.mp import Decoder
    rows = _rows(4096, 200)
    with Decoder(rows.t(), storage=storage) as dec:
        for seed in range(2):
            y = _signal(rows, 5, noise=0.3, seed=seed)
            a = dec.solve(y, 1e-7, 901, trace_cap=901, trace_r=True)
            assert 0 < dec.carried_steps() < a["iters"] == 901
            assert float(a["rr_trace"][-1]) == a["rr"]
            back = y.double() - a["x"].double() @ rows.double()
            assert float((back - a["r"].double()).norm()) < 1e-4 * float(y.double().norm())
            # every step takes its own coefficient off the step before's residual
            r = torch.cat([y[None], a["r_trace"][:-1]])
            want = torch.addcmul(r, -a["coef"][:, None], rows[a["idx"].long()])
            assert float((want - a["r_trace"]).abs().max()) < 1e-6 * float(y.abs().max())


def _tied(rows, extra=0.0):
    """100 copies of one atom, and a y that reaches them at its third step."""
    rows[300:400] = rows[300]
    return 3 * rows[10] + 2 * rows[20] + rows[300] + extra


def test_omp_handed_on():
    from paper_0809_1833_amd.mp import Decoder
    rows = _rows(640, 40000)
    y = _tied(rows, 0.4 * rows[41] + 0.3 * rows[17])
    kw = dict(trace_cap=40, trace_r=True, omp=True)
    print("[omp handed on]", flush=True)
    with Decoder(rows.t()) as dec:
        a = dec.solve(y, 1e-5, 40, **kw)
        assert dec.carried_steps() == 2
        b = dec.solve(y, 1e-5, 40, step_launches=True, **kw)
    _equal(a, b, ("x", "r", "idx", "coef", "rr_trace", "r_trace"))
    assert a["idx"][:3].tolist() == [10, 20, 300] and a["stop"] == "converged"


def test_batched_hands_on_the_signals_that_need_it():
    """One signal with more ties than a step scores, one with noise outside the
    span, among ordinary ones, which keep the single decode's results."""
    from paper_0809_1833_amd.mp import Decoder
    rows = _rows(3000, 410)
    tied = _tied(rows)
    ys = [_signal(rows[:300], 6, seed=j) for j in range(5)]
    ys += [tied, torch.zeros(3000, device="cuda"), _signal(rows[:300], 6, noise=0.3, seed=9)]
    Y, caps = torch.stack(ys), [400] * 4 + [3] + [400] * 2 + [733]
    print("[batched handed on]", flush=True)
    with Decoder(rows.t()) as dec:
        a = dec.solve_batched(Y.t(), 1e-6, caps, trace_cap=733, trace_r=True)
        assert 0 < dec.carried_steps() < 733
        for j in range(7):
            b = dec.solve(ys[j].contiguous(), 1e-6, caps[j], step_launches=True, trace_cap=400)
            assert a["iters"][j] == b["iters"] and a["stop"][j] == b["stop"], j
            assert abs(a["rr"][j] - b["rr"]) <= 1e-12 * b["rr"]
            assert torch.equal(a["x"][:, j], b["x"]) and torch.equal(a["r"][:, j], b["r"])
            assert torch.equal(a["idx"][j][: b["iters"]], b["idx"])
            assert torch.equal(a["coef"][j][: b["iters"]], b["coef"])
    assert a["idx"][5][:3].tolist() == [10, 20, 300]
    assert a["iters"][7] == 733 and a["stop"][7] == "max_iters"
    assert float(a["rr_trace"][7][732]) == a["rr"][7]
    r = torch.cat([ys[7][None], a["r_trace"][7][:732]])
    want = torch.addcmul(r, -a["coef"][7][:733, None], rows[a["idx"][7][:733].long()])
    assert float((want - a["r_trace"][7][:733]).abs().max()) < 1e-6 * float(ys[7].abs().max())


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_ragged_hands_on_the_problems_that_need_it(storage, monkeypatch):
    """As the persistent launch alone decodes them (BF16: where that finds the
    FP32 argmax, so without noise outside the span)."""
    from paper_0809_1833_amd.mp import RaggedDecoder
    sizes = [(200, 800), (700, 500), (64, 256), (300, 40), (512, 1500)]
    probs = [_rows(n, m, seed=j) for j, (n, m) in enumerate(sizes)]
    ys = [_signal(p, 4, seed=j) for j, p in enumerate(probs)]
    ys[1] = _tied(probs[1])
    if storage == "f32":
        ys[3] = _signal(probs[3], 4, noise=0.3)
    caps = [300, 200, 100, 501, 0]
    print(f"[ragged handed on {storage}]", flush=True)
    with RaggedDecoder([p.t() for p in probs], storage=storage) as dec:
        y = dec.pack(ys)
        for _ in range(2):  # a second decode replays the launch
            a = dec.solve(y, 1e-6, caps, trace_cap=501, trace_r=True)
            assert 0 < dec.carried_steps() < 501
        monkeypatch.setenv("MP_RAGGED_SPIN_LIMIT", "4194304")
        b = dec.solve(y, 1e-6, caps, trace_cap=501, trace_r=True)
    assert a["iters"] == b["iters"] and a["stop"] == b["stop"]
    assert all(abs(p - q) <= 1e-12 * q for p, q in zip(a["rr"], b["rr"]))
    assert all(abs(p - q) <= 1e-12 * q for p, q in zip(a["yy"], b["yy"]))
    for key in ("x", "r", "idx", "coef", "r_trace"):
        assert torch.equal(a[key], b[key]), key
    assert a["idx"][1][:3].tolist() == [10, 20, 300]


@pytest.mark.parametrize("cap", [1, 2, 3, 4, 7, 15, 16, 31, 33])
def test_omp_short_decodes(cap):
    """Stops inside the first chunks and blocks, by the cap and by convergence:
    an atom outside the block is fitted before the next block's pass."""
    from paper_0809_1833_amd.mp import Decoder
    rows = _rows(700, 36033, seed=2)
    kw = dict(trace_cap=40, trace_r=True, omp=True)
    print(f"[omp short {cap}]", flush=True)
    with Decoder(rows.t()) as dec:
        for k, noise in ((cap, 0.0), (40, 0.05)):
            y = _signal(rows, k, noise=noise, seed=cap)
            a = dec.solve(y, 1e-5, cap if noise else 40, **kw)
            b = dec.solve(y, 1e-5, cap if noise else 40, step_launches=True, **kw)
            _equal(a, b, ("x", "r", "idx", "coef", "rr_trace", "r_trace"))
            assert a["iters"] == (cap if noise else a["iters"]) >= min(cap, 5)


@pytest.mark.parametrize("form", ["f32", "bf16", "fp8", "f64", "omp"])
def test_low_caps(form):
    """Around the caps below which a launch per step is taken: those steps."""
    from paper_0809_1833_amd.mp import Decoder
    n, m = (640, 40000) if form == "omp" else (900, 3000)
    rows = _rows(n, m, dtype=torch.float64 if form == "f64" else torch.float32)
    y = _signal(rows, 12)
    kw = dict(omp=True) if form == "omp" else {}
    few = {"f64": 2, "bf16": 4, "fp8": 6}.get(form, 3)
    with Decoder(rows.t(), storage="f32" if form == "omp" else form) as dec:
        for cap in range(1, 9):
            a = dec.solve(y, 0.0, cap, trace_cap=cap, **kw)
            assert dec.carried_steps() == (cap if cap > few else 0)
            b = dec.solve(y, 0.0, cap, trace_cap=cap, step_launches=True, **kw)
            _equal(a, b, ("x", "r", "idx", "coef", "rr_trace"))
            assert a["iters"] == cap


def test_ragged_sets_of_quick_problems(monkeypatch):
    """Around the line below which an FP32 set takes the persistent launch."""
    from paper_0809_1833_amd.mp import RaggedDecoder
    for sizes in ([(64, 2048), (40, 100), (128, 512)], [(64, 2049), (40, 100)], [(128, 513)],
                  [(129, 300), (17, 33)]):
        probs = [_rows(n, m, seed=j) for j, (n, m) in enumerate(sizes)]
        ys = [_signal(p, 3, seed=j) for j, p in enumerate(probs)]
        with RaggedDecoder([p.t() for p in probs]) as dec:
            y = dec.pack(ys)
            a = dec.solve(y, 1e-5, 60, trace_cap=60)
            assert (dec.carried_steps() == 0) == (len(sizes) == 3)
            monkeypatch.setenv("MP_RAGGED_SPIN_LIMIT", "4194304")
            b = dec.solve(y, 1e-5, 60, trace_cap=60)
            monkeypatch.delenv("MP_RAGGED_SPIN_LIMIT")
        assert a["iters"] == b["iters"] and a["stop"] == b["stop"]
        for key in ("x", "r", "idx", "coef"):
            assert torch.equal(a[key], b[key]), (sizes, key)


@pytest.mark.parametrize("n,m", [(1, 64), (33, 16384), (64, 16384), (64, 16400), (65, 8192)])
def test_rounds_on_short_columns(n, m):
    """The rounds of products on columns of at most 64 rows, which two of the
    product's four waves have no part of (a BF16 dictionary of exactly 2 MiB at
    M = 16384), and on the next longer ones."""
    from paper_0809_1833_amd.mp import Decoder
    rows = _rows(n, m)
    ys = [_signal(rows, 1 + j % 2, seed=j) for j in range(5)]
    print(f"[rounds {n}x{m}]", flush=True)
    with Decoder(rows.t()) as dec:
        a = dec.solve_batched(torch.stack(ys).t(), 1e-3, 30, trace_cap=30, trace_r=True,
                              rescore_k=7)
    for j, y in enumerate(ys):
        k = a["iters"][j]
        assert 0 < k <= 30
        r = torch.cat([y[None], a["r_trace"][j][:k]])
        want = torch.addcmul(r[:-1], -a["coef"][j][:k, None], rows[a["idx"][j][:k].long()])
        assert float((want - r[1:]).abs().max()) <= 1e-6 * float(y.abs().max())
        c = (r[:-1].double() @ rows.double().t()).abs()
        best = c.gather(1, a["idx"][j][:k, None].long())[:, 0]
        # BF16 products are off by at most 2^-8 ||r||: 7 candidates are no further behind
        assert bool((best >= c.max(1).values - r[:-1].double().norm(dim=1) / 128).all())


def test_gram_columns_in_proportion_and_when_they_pay():
    """The Gram columns of all atoms are not made for a dictionary far smaller
    than they are, nor for a few short batches; then for the next long one."""
    from paper_0809_1833_amd.mp import Decoder

    def grown(fn):
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        fn()
        torch.cuda.synchronize()
        return (before - torch.cuda.mem_get_info()[0]) >> 20

    rows = _rows(64, 8192)  # 2 MiB; its columns would be 256
    y = _signal(rows, 4)
    Y = torch.stack([_signal(rows, 3, seed=j) for j in range(8)])
    with Decoder(rows.t()) as dec:
        a = dec.solve(y, 1e-5, 2000)
        _equal(dec.solve(y, 1e-5, 2000, step_launches=True), a)
        assert grown(lambda: dec.solve(y, 1e-5, 2000)) < 64
        assert grown(lambda: dec.solve_batched(Y.t(), 1e-5, 2000)) < 64
    rows = _rows(1024, 8192)  # 32 MiB and 256
    Y = torch.stack([_signal(rows, 3, seed=j) for j in range(2)])
    with Decoder(rows.t()) as dec:
        first = {}
        assert grown(lambda: first.update(dec.solve_batched(Y.t(), 1e-5, 10000))) < 128
        for _ in range(100):
            a = dec.solve_batched(Y.t(), 1e-5, 10000)
            assert a["iters"] == first["iters"] and torch.equal(a["x"], first["x"])
        b = dec.solve(Y[0].contiguous(), 1e-5, 10000)
        assert torch.equal(a["x"][:, 0], b["x"])
        assert grown(lambda: dec.close()) <= -256  # the columns were made on the way


def test_declined_batches_do_not_pay_for_gram_columns():
    """Batches decoded while carried correlations are off are the caller's
    choice, not rounds that Gram columns would have saved."""
    from paper_0809_1833_amd.mp import Decoder
    rows = _rows(1024, 8192)
    Y = torch.stack([_signal(rows, 3, seed=j) for j in range(2)])
    with Decoder(rows.t()) as dec:
        dec.set_carried(False)
        for _ in range(100):
            dec.solve_batched(Y.t(), 1e-5, 10000)
        dec.set_carried(True)
        dec.solve_batched(Y.t(), 1e-5, 10000)
        assert dec.carried_steps() == 0


@pytest.mark.parametrize("apart", [1e-7, 1e-9, 1e-12])
def test_f64_selects_beyond_fp32(apart):
    """Pairs of columns that FP32 cannot tell apart: the shortlist is made in
    FP32, the selection in FP64, so the atoms are one launch per step's and, for
    the first step, the FP64 argmax."""
    from paper_0809_1833_amd.mp import Decoder
    rows = _rows(900, 3000, dtype=torch.float64)
    g = torch.Generator(device="cuda").manual_seed(8)
    rows[1500:] = rows[:1500] + apart * torch.randn((1500, 900), generator=g, device="cuda",
                                                    dtype=torch.float64) / 30
    rows /= rows.norm(dim=1, keepdim=True)
    pick = torch.tensor([7, 1600, 30, 1802, 200, 1999, 2500], device="cuda")
    y = (rows[pick] * torch.linspace(1, 0.4, 7, device="cuda", dtype=torch.float64)[:, None]).sum(0)
    with Decoder(rows.t(), storage="f64") as dec:
        a = dec.solve(y, 1e-12, 400, trace_cap=400, trace_r=True)
        assert dec.carried_steps() > 7
        b = dec.solve(y, 1e-12, 400, step_launches=True, trace_cap=400, trace_r=True)
    _equal(a, b, ("x", "r", "idx", "coef", "rr_trace", "r_trace"))
    assert int(a["idx"][0]) == int((rows @ y).abs().argmax())
