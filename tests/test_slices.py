"""The order in which the slices of a split-K product are added (no GPU)."""
from test_persistent_turn import _run


def test_the_bits_of_a_loop(tmp_path):
    _run(tmp_path, "slices_check")
