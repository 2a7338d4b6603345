"""Which workspaces the kernels of 32-bit byte offsets take (no GPU needed), and the
plan flag for the others' kernels."""
import ctypes

import pytest

from paper_2101_10881_amd import mdpe, workloads as W


@pytest.mark.parametrize("n_series,doubles,want", [
    (1, 1, True), ((1 << 28) - 1, 1, True), (1 << 28, 1, True),                # up to 2 GiB
    (0xffff0000 // 8, 1, True), (0xffff0000 // 8 + 1, 1, False),               # the last 64 KiB are left
    (0xffff0000 // 512, 64, True), (0xffff0000 // 512 + 1, 64, False),
    (1 << 29, 1, False), (1 << 40, 8, False),
])
def test_bound(n_series, doubles, want):
    f = getattr(mdpe.lib(), "_ZN4mdpe13small_offsetsEll")  # mdpe::small_offsets(int64_t, int64_t)
    f.argtypes, f.restype = [ctypes.c_int64, ctypes.c_int64], ctypes.c_bool
    assert f(n_series, doubles) is want


def test_wide_offsets_flag_keeps_jobs_and_results():
    w = W.p2(m=2, d=16)
    a = mdpe.Plan.for_workload(w, device=-1, flags=mdpe.MDPE_LAYER_LAUNCHES)
    b = mdpe.Plan.for_workload(w, device=-1, flags=mdpe.MDPE_LAYER_LAUNCHES | mdpe.MDPE_WIDE_OFFSETS)
    assert b.info["flags"] == a.info["flags"] | mdpe.MDPE_WIDE_OFFSETS
    assert a.info["workspace_bytes"] == b.info["workspace_bytes"] and a.info["n_conv"] == b.info["n_conv"]
