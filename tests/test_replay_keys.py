"""The sort keys of the replay's events: a plan whose keys would lose bits is refused, none other (a host function of the
library, no GPU)."""
import ctypes
import os

import pytest

from paper_2310_09443_amd import binding, build


@pytest.fixture(scope="module")
def fits():
    if not os.path.exists(build.LIB):
        build.build()
    f = binding.load()._Z15replay_key_fitsjj               # replay_key_fits (C++ name)
    f.argtypes, f.restype = [ctypes.c_uint32, ctypes.c_uint32], ctypes.c_bool
    return f


KINDS, COPIES = 5, 2                                       # kinds of events, iterations


@pytest.mark.parametrize("K", [1, 24, 100_000, (1 << 29) - 1, 1 << 29, (1 << 30) - 1, 1 << 30, (1 << 31) - 1])
def test_every_key_that_is_accepted_fits(fits, K):
    for n in [0, 1, 2, 65_536] + [(1 << b) + d for b in (26, 27, 28, 29) for d in (-1, 0, 1)] + [((1 << 32) - 1) // 6]:
        rbits = max(1, (max(n, 1) - 1).bit_length())
        top = (((2 * K - 1) << 3) | (KINDS - 1)) << (rbits + 1) | ((max(n, 1) - 1) << 1) | (COPIES - 1)
        if fits(K, n):
            assert top < (1 << 64) - 1                     # (the key of an event that does not take place)
        else:
            assert K >= 1 << 29 and n > 1 << 28            # nothing that a GPU's memory holds


def test_limits(fits):
    assert fits((1 << 31) - 1, 1 << 28) and not fits((1 << 31) - 1, (1 << 28) + 1)
    assert fits((1 << 30) - 1, 1 << 29) and not fits(1 << 30, (1 << 28) + 1)
