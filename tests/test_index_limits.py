"""Host-only checks of the predicates that keep the kernels with 32-bit indices
off shapes they cannot index (no GPU needed: the predicates are host functions
of the library)."""
import ctypes

import pytest

HN, HD, P = 0, 1, 2
SINGLE, REGIONS, SEGMENTS, STEPS = range(4)  # ways a batch steps an instance


class Shape(ctypes.Structure):
    _fields_ = [("d", ctypes.c_int), ("bc", ctypes.c_int), ("M0", ctypes.c_int64), ("M1", ctypes.c_int64),
                ("M2", ctypes.c_int64)]


def _shape(M, bc):
    return Shape(len(M), bc, *([1] * (3 - len(M)) + list(M)))


@pytest.fixture(scope="module")
def lib():
    from paper_2312_07010_amd import ace
    return ace.lib()


def _image_is_32_bit(M):
    """The boundary images' period, twice the nodes (and the walls), of every axis in an int."""
    return all(2 * (m + 1) < 2 ** 31 for m in M)


@pytest.mark.parametrize("bc", [HN, HD, P])
@pytest.mark.parametrize("n", [3, 2 ** 20, 2 ** 30 - 2, 2 ** 30 - 1, 2 ** 30, 2 ** 30 + 2, 2 ** 31 - 1, 2 ** 31])
def test_batch_1d_route(lib, n, bc):
    f = lib._ZN3ace11batch_routeERKNS_5ShapeEi
    for region in (0, 32, 64):
        route = f(ctypes.byref(_shape([n], bc)), region)
        assert route in (SEGMENTS, STEPS)
        assert route == STEPS or _image_is_32_bit([n])
        assert route == SEGMENTS or n >= 2 ** 30 - 1  # (what fits stays on the segments)
