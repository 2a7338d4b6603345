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


@pytest.mark.parametrize("chain_waves,want", [(0, False), (1, False), (2, True), (4, True), (16, True)])
def test_lone_launch_behind_chains(chain_waves, want):
    """A layer of up to a round takes it behind chains of two wavefronts or more, whose
    workgroups leave the SIMDs uneven, and not behind chains of one."""
    f = getattr(mdpe.lib(), "_ZN4mdpe17most_after_chainsEli")  # mdpe::most_after_chains(long, int)
    f.argtypes, f.restype = [ctypes.c_long, ctypes.c_int], ctypes.c_long
    assert f(700, 0) == 700
    assert _lone(f(700, chain_waves), 700, 1024) is want
    assert not _lone(f(700, chain_waves), 256, 1024)
    assert not _lone(f(700, chain_waves), 1025, 1024)


@pytest.mark.parametrize("w,want", [(1, False), (4, False), (5, False), (8, True), (10, True), (20, True)])
def test_lone_launch_of_wide_coefficients(w, want):
    """From eight doubles on every launch of a quarter round to a round takes it."""
    f = getattr(mdpe.lib(), "_ZN4mdpe7lone_atEi")  # mdpe::lone_at(int)
    f.argtypes, f.restype = [ctypes.c_int], ctypes.c_bool
    assert f(w) is want
