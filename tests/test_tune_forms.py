"""The autotuners time the forms that read what they set: they switch carried
correlations off while they time, and on again, also when a decode fails."""
from __future__ import annotations

import pytest

torch = pytest.importorskip("torch")


class Switched:
    """Counts the decodes it is asked for with carried correlations on."""

    def __init__(self, fail_at=None):
        self.carried, self.on, self.calls, self.fail_at = True, 0, 0, fail_at
        self.n, self.m, self.storage, self.count = 64, 512, "f32", 2
        self.ns, self.ms, self.x_off = [64, 64], [256, 256], [0, 256, 512]

    def set_carried(self, on):
        self.carried = on

    def set_config(self, *a, **k):
        pass

    set_batched_config = set_config

    def solve(self, *a, **k):
        self.calls += 1
        self.on += self.carried
        if self.calls == self.fail_at:
            raise RuntimeError("decode failed")

    solve_batched = solve


def _ragged(tune, dec):
    return tune.tune_ragged(dec, torch.zeros(4), 1e-5, [5, 5], reps=1, shapes=[(256, 1, 1)])


def _batched(tune, dec):
    return tune.tune_batched(dec, torch.zeros(64, 3), 1e-5, [5] * 3, reps=1,
                             rules=[(64, 32, 0), (64, 64, 0)])


@pytest.mark.parametrize("run", [_ragged, _batched])
def test_tuners_time_the_forms_that_read_the_settings(run, tmp_path, monkeypatch):
    from paper_0809_1833_amd import tune
    path = tmp_path / "tune.json"
    monkeypatch.setenv("MP_TUNE_CACHE", str(path))
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a, **k: None)
    monkeypatch.setattr(torch.cuda, "get_device_properties",
                        lambda *a: type("P", (), {"gcnArchName": "gfx950:x"}))
    monkeypatch.setattr(torch, "empty", lambda *a, **k: None)
    dec = Switched()
    assert not run(tune, dec)["cached"]
    assert dec.calls > 3 and dec.on == 0 and dec.carried
    assert tune.VERSION + "|" in path.read_text()
    again = Switched()
    assert run(tune, again)["cached"] and again.calls == 0
    path.write_text(path.read_text().replace(tune.VERSION + "|", ""))  # entries without one
    failing = Switched(fail_at=3)
    with pytest.raises(RuntimeError):
        run(tune, failing)
    assert failing.calls == 3 and failing.carried


@pytest.mark.parametrize("run", [_ragged, _batched])
def test_tuners_leave_a_declined_form_off(run, tmp_path, monkeypatch):
    from paper_0809_1833_amd import tune
    monkeypatch.setenv("MP_TUNE_CACHE", str(tmp_path / "tune.json"))
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a, **k: None)
    monkeypatch.setattr(torch.cuda, "get_device_properties",
                        lambda *a: type("P", (), {"gcnArchName": "gfx950:x"}))
    monkeypatch.setattr(torch, "empty", lambda *a, **k: None)
    dec = Switched()
    dec.set_carried(False)
    assert not run(tune, dec)["cached"]
    assert dec.calls > 3 and dec.on == 0 and not dec.carried
