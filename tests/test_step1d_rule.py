"""The rules that choose the launch form of a 1D handle's steps (CPU): whole steps in one
workgroup per instance where its rounds are few or well filled, and the tile width of the stage
launches.  The sizes are those the rules were measured at; expected is the faster side where the
two differ by more than a tenth."""
import ctypes

import numpy as np
import pytest

from paper_2002_08816_amd import capi

LIB = ctypes.CDLL(capi.LIB_PATH)
LIB.hw_step1d_pays.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_long]
LIB.hw_tile1d_default.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_long, ctypes.c_int]


def pays(eq, sizes):
    threads = LIB.hw_step1d_threads(int(max(sizes)), 0)
    assert threads >= max(sizes)
    return bool(LIB.hw_step1d_pays(eq, threads, len(sizes), int(np.sum(sizes))))


def spread(lo, hi, n):
    return np.rint(np.exp(np.linspace(np.log(lo), np.log(hi), n))).astype(int)


@pytest.mark.parametrize("sizes,euler,burgers", [
    ([7], True, True), ([400], True, True), ([1024], True, True), ([64] * 4096, True, True), ([128] * 4096, True, True),
    ([256] * 512, True, True), ([512] * 512, True, True), ([500] * 4096, False, True), ([1000] * 1024, True, True),
    (spread(64, 1024, 256), True, True), (spread(64, 1024, 2048), False, False), (spread(64, 1024, 4096), False, False),
    (spread(500, 1000, 512), True, True), (spread(64, 500, 4096), False, False), (spread(64, 256, 1024), True, True),
    ([64] * 4000 + [1000], False, False), ([64] * 1000 + [1000], False, False), ([64] * 40 + [1000], True, True)])
def test_whole_steps_where_they_are_faster(sizes, euler, burgers):
    assert pays(capi.HW_EULER, sizes) == euler
    assert pays(capi.HW_BURGERS, sizes) == burgers
    assert pays(capi.HW_ADVECTION, sizes) == burgers


def test_no_whole_steps_beyond_a_workgroup_or_on_stretched_meshes():
    assert LIB.hw_step1d_threads(1025, 0) == 0 and LIB.hw_step1d_threads(100, 1) == 0


@pytest.mark.parametrize("sizes,euler,burgers", [
    ([256] * 4096 + [1030], 64, 64), ([512] * 512 + [1030], 64, 64), ([1100] * 2000, 64, 256), ([2048] * 512, 128, 256),
    ([4096] * 64, 128, 256), ([16384], 128, 256), ([262144], 256, 256), ([64] * 1000 + [100000], 256, 256)])
def test_tile_width_of_a_handle_that_is_not_tuned(sizes, euler, burgers):
    for eq, want in ((capi.HW_EULER, euler), (capi.HW_BURGERS, burgers)):
        assert LIB.hw_tile1d_default(eq, len(sizes), int(np.sum(sizes)), int(max(sizes))) == want
