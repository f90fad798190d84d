"""The tile cache: what an entry of another version means is not applied, and a
tile that left its slices to the library is set that way again."""
import json

import pytest


@pytest.fixture()
def tuned(tmp_path, monkeypatch):
    autotune = pytest.importorskip("paper_2310_06650_amd.autotune")
    path = tmp_path / "tune.json"
    monkeypatch.setenv("QG_AUTOTUNE_CACHE", str(path))

    class Prob:
        dims = dict(Lp=2816, Kp=2432, T=48, lodf_kind=0)

        def __init__(self):
            self.given = None

        def set_tile(self, text):
            self.given = text

        def tile(self):
            return self.given + "x4" if self.given.count("x") == 1 else self.given

    monkeypatch.setattr(autotune, "step_us", lambda prob, *a, **k:
                        1.0 if prob.given == "s4x4" else 2.0)
    return autotune, path, Prob()


def test_entry_without_a_version_is_tuned_again(tuned):
    autotune, path, prob = tuned
    path.write_text(json.dumps({autotune.shape_key(prob): dict(
        tile="s1x4x8", times={"s1x4x8": 1.0}, measure="step")}))
    tile, times = autotune.tune(prob, None)
    assert tile == "s4x4x4" and len(times) > 1


def test_slices_left_to_the_library_stay_so(tuned):
    autotune, path, prob = tuned
    tile, times = autotune.tune(prob, None)
    assert prob.given == "s4x4" and tile == prob.tile() == min(times, key=times.get)
    prob.given = None
    assert autotune.tune(prob, None) == (tile, times) and prob.given == "s4x4"
