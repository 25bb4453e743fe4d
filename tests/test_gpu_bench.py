"""The bench's timed region runs what a plain call runs."""
import json
import sys

import pytest

pytestmark = pytest.mark.gpu


def test_timed_steps_run_without_profiling(monkeypatch, capsys):
    """No kernel class is timed during the timed steps (timing keeps the two boundary sweeps of
    an evaluation in turn); the class times come from other steps."""
    import torch  # noqa: F401

    import bench
    from paper_1806_03761_amd import peps
    timing, steps = [False], []
    enable, evaluate = peps.profile_enable, peps.evaluate

    def profile_enable(classes=(), device=0):
        timing[0] = bool(classes)
        return enable(classes, device)

    def counted(*a, **k):
        steps.append(timing[0])
        return evaluate(*a, **k)

    monkeypatch.setattr(peps, "profile_enable", profile_enable)
    monkeypatch.setattr(peps, "evaluate", counted)
    monkeypatch.setattr(sys, "argv", ["bench.py", "--workload", "4x4_D2_Dc4", "--steps", "3", "--warmup", "2",
                                      "--no-legs", "--no-cpu-baseline", "--no-tune"])
    bench.main()
    line = json.loads(capsys.readouterr().out.strip().splitlines()[-1])
    assert line["steps"] == 3 and line["value"] > 0 and line["roofline"]["launches"] > 0
    assert steps.count(False) == 3 and steps == [True] * 2 + [False] * 3 + [True]
