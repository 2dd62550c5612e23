"""The tile scan takes its counts from the packed arrays only: without them it
is refused on the host (no GPU needed), at tile counts of either of its routes."""
import ctypes

import pytest

from paper_1009_0794_amd import _lib

INVALID_VALUE = 1  # hipErrorInvalidValue
NAME = "_ZN4ldni16launch_tile_scanEPKmPKjPjS4_ljPvS4_P12ihipStream_t"


@pytest.mark.parametrize("n", [0, 1, 16384, 16385])
@pytest.mark.parametrize("pack,ovf", [(None, None), (None, 64), (64, None)])
def test_refuses_missing_counts(n, pack, ovf):
    f = getattr(_lib.lib(), NAME)
    vp = ctypes.c_void_p
    f.argtypes = [vp, vp, vp, vp, ctypes.c_int64, ctypes.c_uint32, vp, vp, vp]
    f.restype = ctypes.c_int
    assert f(pack, ovf, 64, 64, n, 1, 64, 64, None) == INVALID_VALUE
