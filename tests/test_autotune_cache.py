"""The autotuner's saved choices (host logic, no GPU: the timed frame is a stand-in)."""
import json

import numpy as np
import torch

from paper_2404_14044_amd import autotune, scenes


def _tuner(path, calls, best):
    """A tuner whose frames take 1 ms, or half that at launch shapes `best`."""
    tuner = autotune.Autotuner(str(path))

    def frame(xyz, feat, mlp, cams, params, precision, reps):
        calls.append(params)
        return 0.5 if all(getattr(params, k) == v for k, v in best.items()) else 1.0
    tuner._frame = frame
    return tuner


def test_choices_of_former_launch_shapes_are_measured_again(tmp_path):
    cams = [scenes.pinhole(64, 48, 40.0, np.eye(3), np.zeros(3))]
    p, xyz = scenes.default_params(0.01, 1.0, 5.0, K=8, S=16), torch.zeros(10, 3)
    path = tmp_path / "tune.json"
    key = autotune.shape_key(cams, p, 10, 1)
    former = {"layout": 0, "search_chunk": 4, "search_blocks": 65536, "search_band": 1600, "window_shape": 0,
              "render_rays": 16, "render_blocks": 0}
    other = {"best": {"search_chunk": 8}, "ms": 1.0, "default_ms": 2.0, "trials": []}
    path.write_text(json.dumps({key: {"best": former, "ms": 1.0, "default_ms": 1.1, "trials": []}, "other": other}))

    calls = []
    tuner = _tuner(path, calls, {"search_band": 3200})
    assert tuner.entry(xyz, cams, p, 1) is None
    q = tuner.tune(xyz, None, None, cams, p, 1)
    assert calls and (q.search_chunk, q.search_blocks, q.render_rays, q.search_band) == (0, 0, 0, 3200)

    # saved beside what the file held, and taken as it is from then on
    assert json.loads(path.read_text())["other"] == other
    again = []
    tuner = _tuner(path, again, {})
    assert tuner.tune(xyz, None, None, cams, p, 1) == q and not again
    assert tuner.entry(xyz, cams, p, 1)["ms"] == 0.5
