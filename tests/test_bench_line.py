"""bench.py's one line of output."""
import json
import os
import sys

import numpy as np

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench  # noqa: E402


def test_line_is_compact_and_keeps_its_values():
    """Every figure within half a unit of the seventh digit and at most 13
    characters long (sign, point and exponent included), nothing else changed."""
    rng = np.random.default_rng(0)
    vals = [float(v) for v in np.exp(rng.uniform(-12, 22, 720))]
    line = {"metric": "m", "n_gpus": 1, "steps": 20, "ok": True, "none": None,
            "text": "x" * 8000, "deep": [{"a": v, "b": (v, 7)} for v in vals[:240]],
            "flat": vals[240:]}
    out = bench.compact(line)
    text = json.dumps(out)
    assert max(len(json.dumps(v)) for v in out["flat"]) <= 13
    back = json.loads(text)
    assert {k: back[k] for k in ("metric", "n_gpus", "steps", "ok", "none", "text")} == {
        k: line[k] for k in ("metric", "n_gpus", "steps", "ok", "none", "text")}
    assert isinstance(back["steps"], int) and isinstance(back["deep"][0]["b"][1], int)
    np.testing.assert_allclose(back["flat"], vals[240:], rtol=5e-7)
    np.testing.assert_allclose([d["a"] for d in back["deep"]], vals[:240], rtol=5e-7)


def test_no_size_in_words_of_numpy():
    """numpy floats are floats to the line too."""
    assert json.dumps(bench.compact({"v": np.float64(1.0 / 3.0)})) == '{"v": 0.3333333}'
