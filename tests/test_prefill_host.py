"""Host-side checks of the long-chunk prefill kernels, no GPU needed: what their
loads and launches are computed from is shared with the host or visible in
the compiler's output."""
import ctypes
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2607_07046_amd import build
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


def test_direct_loads_keep_their_target(tmp_path):
    """A load into LDS takes its target from m0, which the compiler may write
    too: every inline write of m0 names it as changed, and in the compiler's output
    each load follows a write of its own, an instruction or more ahead, with
    no other use of m0 anywhere."""
    source = os.path.join(build.CSRC, "prefill.hip")
    with open(source) as f:
        writes = [b for b in re.findall(r"asm volatile\((.*?)\);", f.read(), re.S) if re.search(r"\bm0,", b)]
    assert writes and all('"m0"' in b for b in writes)
    out = tmp_path / "prefill.s"
    subprocess.run([build.HIPCC, *build.FLAGS, "-I", os.path.join(build.ROOT, "include"), "-I", build.CSRC,
                    "--cuda-device-only", "-S", source, "-o", str(out)], check=True, capture_output=True)
    loads, since = 0, None  # instructions since the target was set
    for line in out.read_text().split("\n"):
        t = line.split(";")[0].strip()
        if not t or t.startswith(".") or t.endswith(":"):
            continue
        if re.search(r"\bm0\b", t):
            assert re.match(r"s_add_u32 m0, s\d+, \w+$", t) and since is None, t
            since = 0
        elif re.search(r"\blds$", t):
            assert since is not None and since >= 1, t
            loads, since = loads + 1, None
        elif since is not None:
            since += 1
    assert loads and since is None


# tokens, N, K, an epilogue with the residual stream (O, down), traced us on the
# small and the large tile
TILE_TIMES = [(3000, 5120, 2048, 1, 101.8, 138.3), (617, 31360, 4616, 0, 245.4, 280.1), (145, 30848, 5328, 0, 115.3, 123.1),
              (888, 6912, 5120, 0, 101.5, 90.1), (160, 57344, 8192, 0, 368.4, 267.8), (4096, 6144, 4096, 0, 228.0, 204.0),
              (777, 21248, 8192, 0, 366.0, 347.0), (256, 11008, 4096, 0, 48.3, 64.0), (453, 7920, 24295, 1, 284.7, 235.6)]


@pytest.mark.parametrize("M,N,K,residual,small,large", TILE_TIMES)
def test_tile_choice_follows_the_measured_times(lib, M, N, K, residual, small, large):
    """Products whose two times differ by 5% or more take the faster tile."""
    splits = ctypes.c_int()
    tile = lib.vt_test_prefill_tile(M, N, K, residual, ctypes.byref(splits))
    assert 1 <= splits.value <= 4
    assert tile == (128 if small < large else 256)


def test_tile_choice_depends_on_whole_small_tiles(lib):
    """The workspace is laid out once per count of 128-row tiles: within one, the
    choice must not change with the number of tokens."""
    splits = ctypes.c_int()
    for N, K, residual in ((22016, 4096, 0), (5120, 5530, 1), (8192, 10609, 1), (6912, 5120, 0), (31360, 4616, 0)):
        for tiles in range(1, 33):
            seen = {(lib.vt_test_prefill_tile(M, N, K, residual, ctypes.byref(splits)), splits.value)
                    for M in (128 * tiles - 127, 128 * tiles - 60, 128 * tiles)}
            assert len(seen) == 1, (N, K, tiles, seen)


# tokens, heads, head size, first position, window; traced us with 32 queries per
# workgroup and with shared key blocks
ATTENTION_TIMES = [(3585, 8, 64, 0, 0, 53.5, 72.7), (1793, 16, 64, 0, 0, 31.9, 38.5), (2300, 16, 64, 0, 0, 44.7, 51.4),
                   (130, 128, 64, 1000, 0, 24.2, 26.7), (130, 128, 64, 6000, 0, 101.1, 121.6), (3585, 8, 128, 0, 0, 88.1, 97.9),
                   (1147, 11, 128, 285, 0, 38.8, 46.2), (180, 32, 128, 7253, 0, 81.8, 187.7), (1131, 7, 64, 248, 0, 15.2, 31.4),
                   (3876, 8, 64, 2113, 1024, 31.0, 27.1), (450, 128, 64, 6000, 0, 255.6, 171.0), (1055, 64, 64, 16, 0, 56.4, 29.4),
                   (897, 32, 128, 0, 0, 37.9, 30.8), (2035, 18, 128, 3910, 0, 298.4, 218.0),
                   (2300, 16, 128, 6000, 0, 331.6, 291.6), (1793, 16, 128, 3000, 1024, 50.0, 38.6)]


@pytest.mark.parametrize("T,heads,d,pos0,window,separate,shared", ATTENTION_TIMES)
def test_attention_choice_follows_the_measured_times(lib, T, heads, d, pos0, window, separate, shared):
    """Chunks whose two times differ by 10% or more take the faster kernel."""
    assert lib.vt_test_long_attention(T, heads, d, pos0, window) == (shared < separate)


@pytest.mark.parametrize("d", [64, 128])
def test_attention_choice_over_its_range(lib, d):
    """Any chunk the entry point takes has a choice, up to one head and 65536
    tokens, a window longer than the context, and the largest positions."""
    for T in (1, 127, 128, 129, 4097, 65536):
        for heads in (1, 7, 255, 256, 257, 1024):
            for pos0, window in ((0, 0), (0, 1), (5, 100000), (1000000, 0), (1000000, 4096), (2 ** 31 - 1 - T, 0)):
                assert lib.vt_test_long_attention(T, heads, d, pos0, window) in (0, 1)
