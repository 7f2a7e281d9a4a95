"""The sizes a plan's greedy loop is laid out for: whatever the trace and the limits of g10_plan_limits, the tiles and
chunks together fit the LDS of a compute unit (the host functions of the library, no GPU)."""
import ctypes
import os

import pytest

from paper_2310_09443_amd import binding, build

LDS, UNIT, NT_MAX, NCH_MAX = 160 * 1024, 256, 8192, 512


@pytest.fixture(scope="module")
def rules():
    if not os.path.exists(build.LIB):
        build.build()
    lib = binding.load()
    shift, need = lib._Z15loop_tile_shiftmjj, lib._Z14loop_lds_bytesjj         # loop_tile_shift, loop_lds_bytes (C++ names)
    shift.argtypes, shift.restype = [ctypes.c_uint64, ctypes.c_uint32, ctypes.c_uint32], ctypes.c_uint32
    need.argtypes, need.restype = [ctypes.c_uint32, ctypes.c_uint32], ctypes.c_size_t

    def geometry(n, max_tiles, nch):
        sh = shift(n, max_tiles, nch)
        nt = -(-n // (UNIT << sh))
        return sh, nt, need(nch, nt)

    return geometry


@pytest.mark.parametrize("nch", [1, 2, 64, 257, 391, 497, 498, 499, 511, NCH_MAX])
def test_tiles_and_chunks_fit_the_lds(rules, nch):
    sizes = [0, 1, 255, 256, 257, 1_150_621, (1 << 32) - 1]
    for top in (NT_MAX // 2, 7899, 7900, NT_MAX, 2 * NT_MAX):                 # tiles of 256: around the limits of both
        sizes += [top * UNIT + d for d in (-257, -256, -255, -1, 0, 1, 255, 256, 257)]
    for n in sizes:
        for max_tiles in (1, 7, 4096, NT_MAX):
            sh, nt, lds = rules(n, max_tiles, nch)
            assert nt <= max_tiles and lds <= LDS, (n, max_tiles, nch, sh, nt, lds)


def test_the_smallest_tile_that_fits_is_taken(rules):
    for nch in (1, 391, 497):                                                # (up to 497 chunks every list of tiles fits)
        for n in (1, 256 * 4097, 256 * NT_MAX):
            assert rules(n, NT_MAX, nch)[0] == 0
        assert rules(256 * NT_MAX + 1, NT_MAX, nch)[0] == 1
    assert rules(256 * 7899, NT_MAX, NCH_MAX)[0] == 0 and rules(256 * 7900, NT_MAX, NCH_MAX)[0] == 1
