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
