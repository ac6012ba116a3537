"""The forms without carried correlations, by their own tests.

Decodes that carried correlations now take first were tested in the other
forms: the rounds of products with every tile, the ragged launch in every
shape with its graph, the one-bit and the small persistent launches, and the
reduced-precision passes.  These forms still decode what carried correlations
are not taken for or hand on, so the same tests run here on contexts that have
them switched off, and every decode is checked to have taken no step on them.
"""
from __future__ import annotations

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_batched import (  # noqa: E402,F401
    test_batched_shapes, test_batched_tile_rules, test_hadamard_ties_batched,
    test_mixed_stops_and_caps)
from test_gpu_precision import (  # noqa: E402,F401
    test_hadamard_ties_exact, test_parity_2048x8192, test_parity_8192x32768_whole_run,
    test_parity_small_workload, test_ragged_shapes)
from test_gpu_ragged import (  # noqa: E402,F401
    test_graph_replay_and_recapture, test_launch_shape_does_not_change_selections)
from test_gpu_sign import test_persistent_matches_step_launches  # noqa: E402,F401
from test_gpu_small import test_one_launch_matches_step_launches  # noqa: E402,F401


@pytest.fixture(autouse=True)
def _other_forms(monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_0809_1833_amd import mp
    taken = []
    for cls, calls in ((mp.Decoder, ("solve", "solve_batched")), (mp.RaggedDecoder, ("solve",))):
        def init(self, *a, _was=cls.__init__, **k):
            _was(self, *a, **k)
            self.set_carried(False)
        monkeypatch.setattr(cls, "__init__", init)
        for name in calls:
            def call(self, *a, _was=getattr(cls, name), **k):
                out = _was(self, *a, **k)
                taken.append(self.carried_steps())
                return out
            monkeypatch.setattr(cls, name, call)
    yield
    assert taken and not any(taken)


def test_carried_off_and_on():
    """The switch frees and makes the buffers; its own argument checks."""
    from paper_0809_1833_amd import mp
    g = torch.Generator(device="cuda").manual_seed(1)
    rows = torch.randn((3000, 600), generator=g, device="cuda")
    rows /= rows.norm(dim=1, keepdim=True)
    y = (rows[:8] * torch.arange(1, 9, device="cuda")[:, None]).sum(0)
    with mp.Decoder(rows.t()) as dec:
        a = dec.solve(y, 1e-5, 200)
        for on in (1, 0, 0, 1):
            dec.set_carried(on)
            b = mp.mp_solve(dec.handle, y.data_ptr(), a["x"].data_ptr(), a["r"].data_ptr(),
                            mp.Opts(1e-5, 200, 0, 0))
            assert b.iters == a["iters"] and b.rr == a["rr"]
            assert dec.carried_steps() == (a["iters"] if on else 0)
        with pytest.raises(mp.MPError) as e:
            dec.set_carried(2)
        assert e.value.status == mp.MP_EINVAL
    with mp.RaggedDecoder([rows.t(), rows[:500].t()]) as dec:
        yy = dec.pack([y, y])
        a = dec.solve(yy, 1e-5, 200)
        dec.set_carried(True)
        x, r = torch.empty_like(a["x"]), torch.empty_like(a["r"])
        b = mp.mp_solve_ragged(dec.handle, yy.data_ptr(), x.data_ptr(), r.data_ptr(),
                               mp.Opts(1e-5, 200, 0, 0), 2)
        assert dec.carried_steps() == max(a["iters"]) and torch.equal(x, a["x"])
        assert [q.iters for q in b] == a["iters"] and torch.equal(r, a["r"])
    assert mp.library().mp_set_carried(None, 1) == mp.MP_EINVAL
    assert mp.library().mp_carried_steps(None, None) == mp.MP_EINVAL
