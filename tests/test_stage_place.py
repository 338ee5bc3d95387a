"""Where the staged backward draws read their rows: 64-bit places, checked through the library's host
mirror just below and above 2^31 and 2^32 units of 16 bytes, and at the far end of large plans."""
import ctypes

import pytest

from paper_2510_13866_amd import fhmc


def place(first, value_size, N, unit):
    rows = (ctypes.c_int64 * len(first))(*first)
    out = ctypes.c_int64(-1)
    rc = fhmc.lib.fh_debug_stage_place(rows, len(first), value_size, N, unit, ctypes.byref(out))
    return rc, out.value


@pytest.mark.parametrize("value_size", [4, 8])
@pytest.mark.parametrize("N", [64, 100, 1024, 4096])
def test_places_are_exact_at_any_size(value_size, N):
    upr = N * value_size // 16
    # elements of the rows at 2^31 and 2^32 units, of the last row of a half-filled 64 x 64 chain of
    # 1024 slices, and of slot 2047 of 2048 that each hold 640 slices of 64 x 64 in FP64
    edges = [0, N, (1 << 31) * 16 // value_size, (1 << 32) * 16 // value_size,
             (4095 * 1024 + 1023) * 4096, 2047 * 640 * 4096]
    first = sorted({max(0, (e // N + k) * N) for e in edges for k in (-1, 0, 1)})
    for i in range(0, len(first), 8):
        rows = first[i:i + 8]
        for r, f in enumerate(rows):
            for u in (0, upr // 2, upr - 1):
                assert place(rows, value_size, N, r * upr + u) == (0, f * value_size // 16 + u)


def test_bad_input_is_refused():
    assert place([0], 8, 64, 32)[0] == fhmc.FH_ERR_INVALID_ARG   # past the buffer
    assert place([0], 8, 63, 0)[0] == fhmc.FH_ERR_INVALID_ARG    # rows that are not staged
    assert place([0], 2, 64, 0)[0] == fhmc.FH_ERR_INVALID_ARG
    assert place([0] * 65, 8, 64, 0)[0] == fhmc.FH_ERR_INVALID_ARG
    assert fhmc.lib.fh_debug_stage_place(None, 1, 8, 64, 0, None) == fhmc.FH_ERR_INVALID_ARG
