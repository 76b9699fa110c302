"""Rules of the dispatch that can be asked without a GPU."""
import ctypes as ct

import pytest

from paper_2012_12544_amd import binding as B


def _lstm_seq_supported(n, hidden, compute_units):
    f = getattr(B.load(), "_ZN6bapipe18lstm_seq_supportedEiii")
    f.restype, f.argtypes = ct.c_bool, [ct.c_int] * 3
    return f(n, hidden, compute_units)


@pytest.mark.parametrize("hidden", [128, 256, 512, 640, 1024])
@pytest.mark.parametrize("units", [0, 8, 32, 64, 128, 256])
def test_one_launch_recurrence_needs_room_for_eight_launches(hidden, units):
    """Blocks of a launch wait for each other.  At one block per compute unit, eight launches that each miss the last
    block of a group must leave a unit free; a partition of fewer units takes two launches per step."""
    blocks_per_group = hidden // 32
    assert _lstm_seq_supported(64, hidden, units) == (8 * (blocks_per_group - 1) < units)


def test_one_launch_recurrence_takes_the_hidden_sizes_it_has_kernels_for():
    assert _lstm_seq_supported(1, 128, 256) and _lstm_seq_supported(512, 1024, 256)
    for n, hidden in ((64, 64), (64, 192), (64, 1152), (528, 1024), (0, 128)):
        assert not _lstm_seq_supported(n, hidden, 256)
