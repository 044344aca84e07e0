"""Settings that the autotuner stored before the library's automatic choice could be the
fastest are not applied: they force kernels that the automatic choice has left behind."""
import json

from paper_2601_16169_amd import autotune, sqd


class Ctx:
    def __init__(self):
        self.tune = {}

    def set_tuning(self, key, value):
        self.tune[key] = value


def test_entries_of_an_earlier_generation_are_not_used(tmp_path, monkeypatch):
    cache = tmp_path / "cache.json"
    monkeypatch.setattr(autotune, "CACHE", str(cache))
    monkeypatch.setattr(autotune, "_device_name", lambda: "dev")
    monkeypatch.setattr(autotune, "batch_signature", lambda spaces, mode: "sig")
    monkeypatch.setattr(autotune, "signature", lambda space, precision: "sig")
    forced = {"ss": [[sqd.TUNE_SS_ROWS, 4], 1.0], "ab": [[sqd.TUNE_AB_WAVES, 8], 1.0]}
    cache.write_text(json.dumps({"dev|sig": forced, "dev|g1|sig": forced}))
    searched = []
    automatic = {"ss": [[], 0.5], "ab": [[], 0.5]}
    monkeypatch.setattr(autotune, "_best", lambda *a: searched.append(1) or automatic)
    ctx = Ctx()
    assert autotune.tune_batched(ctx, []) == automatic and len(searched) == 1
    assert not any(ctx.tune.values())
    # the new entry is used, and the old ones are still there
    assert autotune.tune_batched(ctx, []) == automatic and len(searched) == 1
    assert json.loads(cache.read_text())["dev|sig"] == forced

    class Space:
        pass
    space = Space()
    space.ctx = ctx
    assert autotune.tune(space) == automatic      # (an entry is found before anything is measured)
