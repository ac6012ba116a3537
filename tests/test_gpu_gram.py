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
