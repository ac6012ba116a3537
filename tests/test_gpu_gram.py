"""The decode on carried correlations against one launch per step.

Larger FP32 dictionaries decode on correlations carried from step to step by
Gram columns, which shortlist the atoms that are then scored with the stepping
form's FP32 inner product.  Every output (x~, r, iterations, stop reason, the
traced atoms, coefficients, norms and residuals) must therefore equal the
stepping form's (MP_SOLVE_STEP_LAUNCHES) bit for bit: at the edges of the
product's 16-atom tiles and of the steps kernel's shares, with exact ties,
when the cache of Gram columns starts over, and where the device hands the
decode back to the stepping form.  Parity of the stepping form with the FP64
oracle is covered by the FP32 tests.
"""
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


def _draw(n, m, k, noise=0.0, seed=0, dtype=torch.float32):
    g = torch.Generator(device="cuda").manual_seed(1000 * seed + n * 7 + m)
    rows = torch.randn((m, n), generator=g, device="cuda", dtype=torch.float64)
    rows = (rows / rows.norm(dim=1, keepdim=True)).to(dtype)
    sup = torch.randperm(m, generator=g, device="cuda")[:k]
    v = torch.randn(k, generator=g, device="cuda", dtype=torch.float64)
    y = v @ rows[sup].double()
    if noise:
        y = y + noise * y.norm() / math.sqrt(n) * torch.randn(n, generator=g, device="cuda",
                                                               dtype=torch.float64)
    return rows.to(dtype), y.to(dtype)


def _same(rows, y, eps, cap, trace=True, storage="f32"):
    from paper_0809_1833_amd.mp import Decoder
    kw = dict(trace_cap=max(cap, 1), trace_r=True) if trace else {}
    with Decoder(rows.t(), storage=storage) as dec:
        a = dec.solve(y, eps, cap, **kw)
        b = dec.solve(y, eps, cap, step_launches=True, **kw)
        torch.cuda.synchronize()
    for key in ("iters", "stop", "yy", "rr"):
        assert a[key] == b[key], (key, a[key], b[key])
    for key in ("x", "r", "idx", "coef", "rr_trace", "r_trace"):
        if key in a:
            assert torch.equal(a[key], b[key]), key
    return a


@pytest.mark.parametrize("n,m", [
    (1536, 1024), (1200, 1025),          # 256 threads x 4 and x 16 correlations
    (350, 4096), (300, 4097),            # 256 x 16 | 512 x 16
    (200, 8192), (190, 8193),            # 512 x 16 | 512 x 32
    (100, 16384), (97, 16385),           # 512 x 32 | 512 x 64
    (40, 32768), (39, 32769),            # 512 x 64 | one launch per step
    (4097, 401), (8192, 200), (16384, 150),  # the longest columns
    (1000, 1999), (65, 20001),
])
def test_equals_step_launches(n, m):
    print(f"[gram {n}x{m}]", flush=True)
    rows, y = _draw(n, m, max(2, min(n, m) // 20), noise=0.01)
    a = _same(rows, y, 0.005, 120)
    assert a["iters"] > 0


@pytest.mark.parametrize("n,m", [
    (700, 1024), (600, 1025), (2048, 300), (2049, 300), (150, 8193), (40, 32768), (39, 32769),
    (8192, 100), (9600, 90), (9601, 90), (63, 4097), (1000, 1999),
])
def test_f64_equals_step_launches(n, m):
    """The FP64 form (its products shortlisted in FP32, scored in FP64), at the
    edges of its shares and of the longest column it takes."""
    print(f"[gram f64 {n}x{m}]", flush=True)
    rows, y = _draw(n, m, max(2, min(n, m) // 20), noise=0.01, dtype=torch.float64)
    a = _same(rows, y, 0.005, 120, storage="f64")
    assert a["iters"] > 0


def test_f64_full_decay_and_handing_back():
    rows, y = _draw(512, 3000, 40, dtype=torch.float64)
    a = _same(rows, y, 1e-10, 2000, storage="f64")
    assert a["stop"] == "converged" and a["iters"] > 100
    _same(rows, y * 1e-60, 1e-4, 50, storage="f64")


@pytest.mark.parametrize("storage", ["bf16", "fp8"])
@pytest.mark.parametrize("n,m,eps", [(600, 3000, 1e-6), (1000, 8193, 1e-5), (250, 900, 1e-6)])
def test_reduced_precision_equals_step_launches(storage, n, m, eps):
    """With all 8 candidates re-scored the reduced-precision forms select the
    FP32 form's atom, on carried correlations as with a pass per step."""
    rows, y = _draw(n, m, max(2, n // 20))
    a = _same(rows, y, eps, 400, storage=storage)
    assert a["stop"] == "converged"


@pytest.mark.parametrize("cap", [0, 1, 2, 5])
def test_short_caps(cap):
    rows, y = _draw(600, 3000, 20)
    a = _same(rows, y, 1e-6, cap)
    assert a["iters"] == cap and a["stop"] == "max_iters"


def test_full_decay():
    """To 1e-6 of ||y||: the carried error is renewed several times."""
    rows, y = _draw(512, 3000, 40)
    a = _same(rows, y, 1e-6, 2000)
    assert a["stop"] == "converged" and a["iters"] > 60


def test_cache_starts_over():
    """Noise with eps = 0: more atoms than the cache holds Gram columns
    (max(256, N / 4) and a few) are selected."""
    rows, y = _draw(512, 8192, 2, noise=30.0)
    a = _same(rows, y, 0.0, 700, trace=True)
    assert torch.unique(a["idx"]).numel() > 280


def test_ties_take_the_smallest_index():
    """Duplicated and negated columns tie exactly; the smallest index wins."""
    rows, y = _draw(640, 2400, 24, seed=3)
    rows[1200:1800] = rows[:600]
    rows[1800:] = -rows[600:1200]
    a = _same(rows, y, 1e-5, 300)
    assert int(a["idx"].max()) < 1200


def test_hands_back_to_step_launches():
    """More atoms tie than a step can score; a norm far outside the error
    bounds' range; no atom correlates with y."""
    rows, y = _draw(640, 2400, 8, seed=4)
    many = rows.clone()
    many[300:400] = many[300]
    _same(many, many[300].contiguous(), 1e-6, 50)
    _same(rows, y * 1e-28, 1e-4, 50)
    half = rows.clone()
    half[:, 320:] = 0
    half /= half.norm(dim=1, keepdim=True)
    z = torch.zeros(640, device="cuda")
    z[400:] = 1.0
    a = _same(half, z, 1e-4, 50)
    assert a["stop"] == "stalled" and a["iters"] == 0


def test_zero_and_non_finite_input():
    from paper_0809_1833_amd import mp
    from paper_0809_1833_amd.mp import Decoder
    rows, y = _draw(600, 3000, 20)
    _same(rows, torch.zeros_like(y), 1e-5, 50)
    with Decoder(rows.t()) as dec:
        y[5] = float("inf")
        with pytest.raises(mp.MPError) as e:
            dec.solve(y, 1e-5, 50)
        assert e.value.status == mp.MP_ENONFINITE


def test_two_streams_and_repeats():
    """Two contexts decode at once from two threads on their own streams, each
    repeatedly; every result is the one of a decode alone."""
    import threading

    from paper_0809_1833_amd.mp import Decoder
    probs = [_draw(800, 2000, 30, seed=s) for s in (1, 2)]
    decs = [Decoder(rows.t()) for rows, _ in probs]
    alone = [d.solve(y, 1e-5, 600) for d, (_, y) in zip(decs, probs)]
    torch.cuda.synchronize()
    got = [[], []]

    def work(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(5):
                got[i].append(decs[i].solve(probs[i][1], 1e-5, 600, stream=s))
        s.synchronize()

    th = [threading.Thread(target=work, args=(i,)) for i in (0, 1)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for i in (0, 1):
        assert len(got[i]) == 5
        for o in got[i]:
            assert o["iters"] == alone[i]["iters"] and torch.equal(o["x"], alone[i]["x"])
            assert torch.equal(o["r"], alone[i]["r"])
        decs[i].close()


# ---- the batched decode (all Gram columns at once) ---------------------------

def _batched_same(rows, ys, eps, caps, storage="f32", solo=None):
    """Every signal of the batch as mp_solve decodes it alone, one launch per
    step: the same atoms, coefficients, x~ and r (||r||^2 to the last digits:
    it is summed in the batched form's order)."""
    from paper_0809_1833_amd.mp import Decoder
    b = ys.shape[1]
    per = caps if isinstance(caps, list) else [caps] * b
    cap = max(max(per), 1)
    with Decoder(rows.t(), storage=storage) as dec, Decoder(rows.t()) as one:
        out = dec.solve_batched(ys, eps, caps, trace_cap=cap, trace_r=True)
        again = dec.solve_batched(ys, eps, caps)
        torch.cuda.synchronize()
        assert torch.equal(out["x"], again["x"]) and torch.equal(out["r"], again["r"])
        assert out["iters"] == again["iters"] and out["rr"] == again["rr"]
        for j in (range(b) if solo is None else solo):
            a = one.solve(ys[:, j].contiguous(), eps, per[j], trace_cap=cap, trace_r=True,
                          step_launches=True)
            t = a["iters"]
            assert out["iters"][j] == t and out["stop"][j] == a["stop"], j
            assert torch.equal(out["x"][:, j].contiguous(), a["x"]), j
            assert torch.equal(out["r"][:, j].contiguous(), a["r"]), j
            assert torch.equal(out["idx"][j, :t], a["idx"]) and torch.equal(out["coef"][j, :t],
                                                                            a["coef"]), j
            assert torch.equal(out["r_trace"][j, :t], a["r_trace"]), j
            assert abs(out["rr"][j] - a["rr"]) <= 1e-13 * a["rr"], j
    return out


def _signals(rows, ks, seed=0, noise=0.01):
    g = torch.Generator(device="cuda").manual_seed(seed + len(ks))
    m, n = rows.shape
    ys = torch.empty((len(ks), n), device="cuda")
    for j, k in enumerate(ks):
        sup = torch.randperm(m, generator=g, device="cuda")[:k]
        v = torch.randn(k, generator=g, device="cuda", dtype=torch.float64)
        y = v @ rows[sup].double()
        y += noise * y.norm() / math.sqrt(n) * torch.randn(n, generator=g, device="cuda",
                                                            dtype=torch.float64)
        ys[j] = y.float()
    return ys.t()


@pytest.mark.parametrize("n,m,b", [
    (300, 1024, 3), (300, 1025, 2), (128, 4096, 65), (129, 4097, 64), (500, 63, 5),
    (64, 8192, 2), (60, 8193, 2), (40, 16384, 2), (40, 16385, 2),
    (513, 129, 130), (1, 7, 3), (2049, 600, 2),
])
def test_batched_equals_single(n, m, b):
    print(f"[gram batched {n}x{m} b{b}]", flush=True)
    rows, _ = _draw(n, m, 1)
    # (columns that do not span the rows would leave noise no atom can take)
    ys = _signals(rows, [1 + (j * 7) % max(1, min(n, m) // 15) for j in range(b)],
                  noise=0.01 if m > n else 0.0)
    _batched_same(rows, ys, 0.005, 2000, solo=range(min(b, 6)))


@pytest.mark.parametrize("storage", ["f32", "bf16", "fp8"])
def test_batched_caps_and_odd_signals(storage):
    """Caps per signal (zero among them), a zero signal, and a decay that
    renews the correlations; then a signal with NaN, which fails the call and
    leaves the others decoded."""
    from paper_0809_1833_amd import mp
    from paper_0809_1833_amd.mp import Decoder
    rows, _ = _draw(256, 900, 1, seed=5)
    ys = _signals(rows, [4, 9, 3, 12, 7], noise=0.0).contiguous()
    ys = torch.empty((5, 256), device="cuda").copy_(ys.t()).t()
    ys[:, 2] = 0
    out = _batched_same(rows, ys, 1e-6, [2000, 3, 50, 0, 2000], storage=storage)
    assert out["stop"] == ["converged", "max_iters", "zero_input", "max_iters", "converged"]
    good = _batched_same(rows, ys, 1e-6, 2000, storage=storage, solo=[0])
    ys[17, 3] = float("nan")
    with Decoder(rows.t(), storage=storage) as dec:
        with pytest.raises(mp.MPError) as e:
            dec.solve_batched(ys, 1e-6, 2000)
        assert e.value.status == mp.MP_ENONFINITE
        ys[:, 3] = 0
        again = dec.solve_batched(ys, 1e-6, 2000)
    assert torch.equal(again["x"][:, 0], good["x"][:, 0])


def test_batched_ties_and_handing_back():
    """Exact ties take the smallest index; a signal on which more atoms tie
    than a step can score sends the batch back to the rounds of products."""
    rows, _ = _draw(200, 1200, 1, seed=6)
    rows[600:] = -rows[:600]
    ys = _signals(rows, [5, 8, 3], seed=2)
    out = _batched_same(rows, ys, 0.005, 400)
    assert int(out["idx"].max()) < 600
    rows[300:400] = rows[300]
    ys = torch.stack([rows[300], ys[:, 1]], dim=0).t()
    _batched_same(rows, ys, 0.005, 400)


# ---- many problems of uneven size ---------------------------------------------

def _ragged_probs(sizes, seed=0):
    return [_draw(n, m, max(1, min(n, m) // 16), noise=0.005 if m > n else 0.0, seed=seed + i)
            for i, (n, m) in enumerate(sizes)]


def _ragged_out(dec, y, eps, caps, cap):
    out = dec.solve(y, eps, caps, trace_cap=cap, trace_r=True)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("sizes", [
    [(64, 256), (63, 200), (128, 1024), (129, 1025), (1, 5), (300, 4096), (1000, 3999), (200, 100)],
    [(4096, 900), (70, 4096), (256, 4095)],          # the largest set of 256 threads
    [(4097, 700), (64, 300), (100, 4097)],           # 512 threads
    [(100, 8192), (90, 8193), (300, 1200), (40, 32768)],
])
def test_ragged_equals_persistent_launch(storage, sizes, monkeypatch):
    """Every problem as the persistent launch (which MP_RAGGED_SPIN_LIMIT
    selects) decodes it: the same atoms, coefficients, x~ and r."""
    from paper_0809_1833_amd.mp import RaggedDecoder
    print(f"[gram ragged {storage} {sizes}]", flush=True)
    probs = _ragged_probs(sizes)
    caps = [20 * max(1, min(s) // 16) + i for i, s in enumerate(sizes)]
    cap = max(caps)
    with RaggedDecoder([rows.t() for rows, _ in probs], storage=storage) as dec:
        y = dec.pack([p[1] for p in probs])
        a = _ragged_out(dec, y, 0.003, caps, cap)
        again = dec.solve(y, 0.003, caps)
        monkeypatch.setenv("MP_RAGGED_SPIN_LIMIT", "4194304")
        b = _ragged_out(dec, y, 0.003, caps, cap)
    assert a["iters"] == b["iters"] and a["stop"] == b["stop"] and max(a["iters"]) > 0
    assert torch.equal(a["x"], again["x"]) and torch.equal(a["r"], again["r"])
    for key in ("x", "r", "idx", "coef", "r_trace"):
        assert torch.equal(a[key], b[key]), key
    for key in ("yy", "rr"):
        assert all(abs(u - v) <= 1e-13 * v for u, v in zip(a[key], b[key])), key


@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_ragged_many_problems_share_right_hand_sides(storage, monkeypatch):
    """So many tiles that none is split: the pass reads its right-hand sides
    from LDS.  Columns of one piece and of several, tiles that do not fill
    their workgroup or have no atoms; as the persistent launch decodes them."""
    from paper_0809_1833_amd.mp import RaggedDecoder
    sizes = [([1, 64, 65, 192, 300][i % 5], [897, 929, 961, 1000, 1024, 1025][i % 6])
             for i in range(110)]
    assert sum(-(-m // 32) for _, m in sizes) > 12 * torch.cuda.get_device_properties(
        0).multi_processor_count
    print(f"[gram ragged many {storage}]", flush=True)
    probs = _ragged_probs(sizes, seed=40)
    caps = [8 + i % 5 for i in range(len(sizes))]
    with RaggedDecoder([rows.t() for rows, _ in probs], storage=storage) as dec:
        y = dec.pack([p[1] for p in probs])
        a = _ragged_out(dec, y, 0.003, caps, max(caps))
        monkeypatch.setenv("MP_RAGGED_SPIN_LIMIT", "4194304")
        b = _ragged_out(dec, y, 0.003, caps, max(caps))
    assert a["iters"] == b["iters"] and a["stop"] == b["stop"] and max(a["iters"]) > 5
    for key in ("x", "r", "idx", "coef", "r_trace"):
        assert torch.equal(a[key], b[key]), key


def test_ragged_odd_inputs_and_handing_back():
    """A zero y, a cap of zero, exact ties; a problem on which more atoms tie
    than a step can score sends the set to the persistent launch; NaN fails
    the call and leaves the others decoded."""
    from paper_0809_1833_amd import mp
    from paper_0809_1833_amd.mp import RaggedDecoder
    probs = _ragged_probs([(200, 800), (150, 600), (100, 400)], seed=20)
    rows0 = probs[0][0]
    rows0[400:] = -rows0[:400]
    for many in (False, True):
        if many:
            rows0[100:200] = rows0[100]
            probs[0] = (rows0, rows0[100].clone())
        with RaggedDecoder([rows.t() for rows, _ in probs]) as dec:
            y = dec.pack([probs[0][1], torch.zeros(150, device="cuda"), probs[2][1]])
            a = _ragged_out(dec, y, 0.01, [200, 50, 0], 200)
            assert a["stop"][1:] == ["zero_input", "max_iters"] and a["iters"][1:] == [0, 0]
            assert int(a["idx"][0].max()) < (400 if not many else 101)
            y[3] = float("nan")
            with pytest.raises(mp.MPError) as e:
                dec.solve(y, 0.01, 50)
            assert e.value.status == mp.MP_ENONFINITE


# ---- Orthogonal Matching Pursuit ----------------------------------------------

def _omp_same(rows, y, eps, cap):
    from paper_0809_1833_amd.mp import Decoder
    kw = dict(trace_cap=max(cap, 1), trace_r=True, omp=True)
    with Decoder(rows.t()) as dec:
        a = dec.solve(y, eps, cap, **kw)
        plain = dec.solve(y, eps, cap, omp=True)
        b = dec.solve(y, eps, cap, step_launches=True, **kw)
        torch.cuda.synchronize()
    for key in ("iters", "stop", "yy", "rr"):
        assert a[key] == b[key] == plain[key], (key, a[key], b[key], plain[key])
    for key in ("x", "r", "idx", "coef", "rr_trace", "r_trace"):
        assert torch.equal(a[key], b[key]), key
    assert torch.equal(plain["x"], b["x"]) and torch.equal(plain["r"], b["r"])
    return a


@pytest.mark.parametrize("n,m,k,noise", [
    (2048, 12289, 60, 0.01), (1025, 24575, 40, 0.0), (700, 36033, 30, 0.01),
    (130, 131200, 12, 0.0), (4097, 6145, 17, 0.0), (16384, 1537, 100, 0.0), (1024, 24577, 2, 3.0),
    (512, 4097, 8, 0.01),  # a pass per step
])
def test_omp_equals_a_pass_per_step(n, m, k, noise):
    """OMP's selection on carried correlations: the atoms, coefficients, x~ and
    r of a pass per step, at the edges of the tiles and groups of atoms, over
    one and several blocks, and with more noise than signal."""
    print(f"[gram omp {n}x{m}]", flush=True)
    rows, y = _draw(n, m, k, noise=noise)
    a = _omp_same(rows, y, min(max(1.2 * noise, 1e-5), 0.5), min(3 * k + 20, n))
    assert a["iters"] >= (k if noise < 1 else 20) // 2


def test_omp_ties_caps_and_handing_back():
    """Exact ties take the smallest index; near copies of selected atoms; caps
    of 0 and 1; zero input; more ties than a step can score."""
    rows, y = _draw(640, 40000, 24, seed=3)
    rows[1200:1800] = rows[:600]
    rows[1800:2400] = -rows[600:1200]
    y = (rows[:24] * torch.arange(1, 25, device="cuda")[:, None]).sum(0)
    a = _omp_same(rows, y, 1e-5, 60)
    assert not bool(((a["idx"] >= 1200) & (a["idx"] < 2400)).any())
    for cap in (0, 1):
        assert _omp_same(rows, y, 1e-5, cap)["iters"] == cap
    _omp_same(rows, torch.zeros_like(y), 1e-5, 20)
    near = rows.clone()
    near[1200:1800] += 1e-3 * torch.randn_like(near[1200:1800]) / math.sqrt(640)
    near /= near.norm(dim=1, keepdim=True)
    _omp_same(near, (near[:40] + 0.5 * near[1200:1240]).sum(0), 1e-6, 120)
    rows[300:400] = rows[300]
    _omp_same(rows, rows[300].contiguous(), 1e-6, 20)


# ---- one-bit dictionaries (batches of steps on the active atoms) -----------------

def _signs(n, m, k, noise, seed=0):
    """+-1 columns (M, N) int8, their packed bits and y."""
    g = torch.Generator(device="cuda").manual_seed(seed * 77 + n * 5 + m)
    neg = torch.randint(0, 2, (m, n), generator=g, device="cuda", dtype=torch.int8)
    sup = torch.randperm(m, generator=g, device="cuda")[:k]
    v = torch.randn(k, generator=g, device="cuda", dtype=torch.float64)
    y = v @ (1 - 2 * neg[sup].double()) / math.sqrt(n)
    y = y + noise * y.norm() / math.sqrt(n) * torch.randn(n, generator=g, device="cuda",
                                                          dtype=torch.float64)
    return neg, y.float()


def _pack_signs(neg):
    m, n = neg.shape
    pad = torch.zeros((m, (n + 31) // 32 * 32), dtype=torch.uint8, device="cuda")
    pad[:, :n] = neg.to(torch.uint8)
    w = (pad.view(m, -1, 8) << torch.arange(8, device="cuda", dtype=torch.uint8)).sum(
        2, dtype=torch.uint8)
    return w.view(torch.int32)


def _sign_same(neg, y, eps, cap):
    from paper_0809_1833_amd.mp import Decoder
    kw = dict(trace_cap=max(cap, 1), trace_r=True)
    with Decoder(_pack_signs(neg), storage="sign", n=neg.shape[1]) as dec:
        a = dec.solve(y, eps, cap, **kw)
        plain = dec.solve(y, eps, cap)
        b = dec.solve(y, eps, cap, step_launches=True, **kw)
        torch.cuda.synchronize()
    for key in ("iters", "stop", "yy", "rr"):
        assert a[key] == b[key] == plain[key], (key, a[key], b[key], plain[key])
    for key in ("x", "r", "idx", "coef", "rr_trace", "r_trace"):
        assert torch.equal(a[key], b[key]), key
    assert torch.equal(plain["x"], b["x"]) and torch.equal(plain["r"], b["r"])
    return a


@pytest.mark.parametrize("n,m,k,noise,cap", [
    (200, 1024, 9, 0.0, 300), (200, 1025, 9, 0.0, 300),   # every atom active | some
    (512, 4097, 20, 0.01, 127), (512, 4097, 20, 0.01, 129),  # a round's most steps, and around
    (2048, 8192, 4, 20.0, 1500),                          # more atoms than can be active
    (9000, 700, 20, 0.0, 200),                            # several rows of r per lane
    (33, 65, 2, 0.0, 40),
])
def test_signs_equal_step_launches(n, m, k, noise, cap):
    print(f"[gram signs {n}x{m}]", flush=True)
    neg, y = _signs(n, m, k, noise)
    a = _sign_same(neg, y, 0.0 if noise > 1 else 1e-6, cap)
    assert a["iters"] >= min(cap, k)
    if noise > 1:
        assert torch.unique(a["idx"]).numel() > 1024


def test_signs_ties_and_stall():
    """Equal and opposite columns tie exactly and the smallest index wins; no
    column correlates with y, at once and after one step."""
    neg, y = _signs(96, 3000, 5, 0.0, seed=3)
    neg[1500:2250] = neg[:750]
    neg[2250:] = 1 - neg[750:1500]
    a = _sign_same(neg, y, 1e-6, 100)
    assert int(a["idx"].max()) < 1500
    h = torch.zeros((1, 1), dtype=torch.int8, device="cuda")
    for _ in range(6):
        h = torch.cat([torch.cat([h, h], 1), torch.cat([h, 1 - h], 1)], 0)
    for extra in (0.0, 2.0):
        y = (1 - 2 * h[50].float()) + extra * (1 - 2 * h[7].float())
        a = _sign_same(h[:40].contiguous(), y, 1e-6, 10)
        assert a["stop"] == "stalled" and a["iters"] == (1 if extra else 0)


# ---- small dictionaries (every atom's Gram column) --------------------------------

@pytest.mark.parametrize("n,m,cap", [
    (256, 1024, 95), (256, 1024, 96),     # the caps below which the one launch stays
    (100, 512, 63), (100, 512, 64),
    (256, 1025, 900), (64, 65, 400), (2048, 512, 900), (33, 17, 64), (700, 900, 2000),
])
def test_small_equals_step_launches(n, m, cap):
    print(f"[gram small {n}x{m}]", flush=True)
    rows, y = _draw(n, m, max(2, min(n, m) // 20))
    a = _same(rows, y, 1e-6, cap)
    assert a["persistent"] and a["iters"] > 3


@pytest.mark.parametrize("eps", [1e-3, 9e-4, 0.04])
def test_small_loose_stop(eps):
    """One round first from eps = 1e-3 on, two below."""
    rows, y = _draw(256, 1024, 12, seed=4)
    a = _same(rows, y, eps, 240)
    assert a["persistent"] and a["stop"] == "converged"


def test_small_ties_and_handing_back():
    """Exact ties take the smallest index; more ties than a step can score go
    back to the launch that holds the dictionary."""
    rows, y = _draw(200, 900, 8, seed=9)
    rows[450:] = -rows[:450]
    a = _same(rows, y, 1e-5, 200)
    assert int(a["idx"].max()) < 450 and a["persistent"]
    rows[300:400] = rows[300]
    a = _same(rows, rows[300].contiguous(), 1e-6, 100)
    assert a["persistent"]
