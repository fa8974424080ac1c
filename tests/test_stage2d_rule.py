"""The rule that chooses between one launch and four for a 2D stage (CPU): at the sizes where both
were measured, expected is the faster side where they differ by more than one part in fifty (of
steps, and of recorded runs with their adjoint)."""
import ctypes

import pytest

from paper_2002_08816_amd import capi

LIB = ctypes.CDLL(capi.LIB_PATH)


def one(eq, tc, nx, ny, bc=capi.HW_BC_PERIODIC):
    return bool(LIB.hw_one_launch2d(eq, tc, bc, nx, ny))


@pytest.mark.parametrize("nx,ny,expected", [
    (8, 8, True), (9, 9, True), (12, 12, True), (13, 13, False), (16, 16, False), (32, 32, False), (64, 64, False),
    (90, 90, False), (96, 96, False), (97, 97, True), (100, 100, True), (120, 120, True), (128, 128, True), (8, 512, True), (512, 8, True)])
def test_euler_with_every_cell_troubled(nx, ny, expected):
    assert one(capi.HW_EULER, capi.HW_TC_ALL, nx, ny) == expected


@pytest.mark.parametrize("n,euler", [(8, True), (16, True), (64, True), (320, True), (362, False), (512, False)])
def test_detected_cells_and_scalar_laws(n, euler):
    assert one(capi.HW_EULER, capi.HW_TC_KXRCF, n, n) == euler
    for eq in (capi.HW_BURGERS, capi.HW_ADVECTION):
        for tc in (capi.HW_TC_KXRCF, capi.HW_TC_ALL):
            assert one(eq, tc, n, n)


def test_never_without_detection_or_with_the_named_boundaries():
    assert not one(capi.HW_EULER, capi.HW_TC_NONE, 64, 64)
    assert not one(capi.HW_EULER, capi.HW_TC_KXRCF, 64, 64, capi.HW_BC_DMR)
    assert not one(capi.HW_EULER, capi.HW_TC_KXRCF, 64, 64, capi.HW_BC_STEP)
