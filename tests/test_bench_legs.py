"""A failing leg beside the benchmark's headline is reported in its place."""
import json
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
import bench  # noqa: E402


def test_a_failing_leg_does_not_take_the_line(monkeypatch, capsys):
    def fails(*a):
        raise RuntimeError("no room")

    monkeypatch.setattr(bench, "serving_leg", fails)
    monkeypatch.setattr(bench, "stress_serving_leg", lambda *a: {"saturated_qps": 1.0})
    out = json.loads(json.dumps(bench.serving_legs(1, None, None, None, None)))
    assert out == {"serving": {"error": "RuntimeError: no room"},
                   "serving_stress": {"saturated_qps": 1.0}}
    assert "no room" in capsys.readouterr().err
