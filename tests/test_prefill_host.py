"""Host-side checks of the long-chunk prefill kernels, no GPU needed: what their
loads and launches are computed from is shared with the host or visible in
the compiler's output."""
import ctypes

import numpy as np
import pytest

from paper_2607_07046_amd import voltron as vt


@pytest.fixture(scope="module")
def lib():
    return vt.load_library()


# tokens, K, first k-tile, k-tiles: whole, ending in a partial k-tile, a middle
# slice, fewer k-tiles than the ring has stages, one that is partial alone
@pytest.mark.parametrize("M,K,kt0,nkt", [(4096, 4096, 0, 128), (777, 10609, 166, 166), (900, 4096, 64, 64),
                                         (300, 96, 0, 3), (129, 40, 0, 2), (2305, 35, 1, 1), (65536, 8192, 0, 256)])
def test_direct_loads_stay_in_their_ranges(lib, M, K, kt0, nkt):
    """Every load of the 256-row tile's ring lies inside its operand, or has an
    empty range and no scalar offset: then it reads nothing whether the range
    check counts the scalar offset or not."""
    words = np.zeros((2 * nkt + 16, 4), np.uint32)
    n = lib.vt_test_prefill_walk(M, K, kt0, nkt, words.ctypes.data_as(ctypes.c_void_p), len(words))
    tail = (kt0 + nkt) * 32 > K  # the partial k-tile goes through registers
    a_bytes, row_bytes = (K + 15) // 16 * M * 32, K * 2
    full = 0
    for a0, a1, b, empty in words[:n].astype(np.int64):
        if empty:
            assert (a0, a1, b) == (0, 0, 0)
            continue
        assert (a0, a1, b) == ((kt0 + full) * 2 * M * 32, ((kt0 + full) * 2 + 1) * M * 32, (kt0 + full) * 64)
        full += 1
        assert a1 + M * 32 <= a_bytes and b + 64 <= row_bytes
    assert full == nkt - tail and n > full
