"""Looks at the stop flags of a rollout (no GPU: the device is made up by the check)."""
from test_persistent_turn import _run


def test_no_look_outlives_its_call(tmp_path):
    _run(tmp_path, "stop_looks_check")
