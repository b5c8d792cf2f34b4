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


@pytest.mark.parametrize("bc", [HN, HD, P])
@pytest.mark.parametrize("M", [(1, 2 ** 30 - 2), (1, 2 ** 30 - 1), (2 ** 30 - 2, 1), (2 ** 30 - 1, 1), (2 ** 30, 1), (1, 2 ** 30 + 2),
                               (2 ** 31 - 1, 1), (3, 2 ** 29), (46341, 46340), (46340, 46341), (46341, 46341), (5, 7)])
def test_2d_regions(lib, M, bc):
    s = _shape(M, bc)
    regions = bool(lib._ZN3ace13tb2_supportedERKNS_5ShapeE(ctypes.byref(s)) & 0xff)
    small = M[0] * M[1] < 2 ** 31
    assert not regions or (small and _image_is_32_bit(M))
    assert regions or not small or not _image_is_32_bit(M)  # (what fits stays on the regions)
    route = lib._ZN3ace11batch_routeERKNS_5ShapeEi
    for rows in (32, 64):
        assert route(ctypes.byref(s), rows) == (REGIONS if regions else SINGLE)
    assert route(ctypes.byref(s), 0) == SINGLE
