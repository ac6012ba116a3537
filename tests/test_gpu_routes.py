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
