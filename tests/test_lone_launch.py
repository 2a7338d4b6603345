"""When a convolution launch takes one wavefront per SIMD by register count (no
GPU needed): not in plans whose launches all fit a round but two of them do not, so
that two streams' launches can share SIMDs."""
import ctypes

import pytest

from paper_2101_10881_amd import mdpe


def _lone(most, waves, simds):
    f = getattr(mdpe.lib(), "_ZN4mdpe11lone_launchElli")  # mdpe::lone_launch(long, long, int)
    f.argtypes, f.restype = [ctypes.c_long, ctypes.c_long, ctypes.c_int], ctypes.c_bool
    return f(most, waves, simds)


@pytest.mark.parametrize("most,waves,want", [
    (990, 990, False),    # every layer fits a round: two streams share SIMDs
    (990, 330, False),
    (513, 513, False),
    (1024, 1024, False),
    (512, 512, True),     # two fit beside each other
    (378, 257, True),
    (378, 256, False),    # a quarter of the SIMDs
    (1025, 1024, True),   # a layer of more than a round
    (6144, 257, True),
    (6144, 1025, False),  # more than a round
])
def test_lone_launch(most, waves, want):
    assert _lone(most, waves, 1024) is want
