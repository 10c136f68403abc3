"""The host's plan of an insert by hash bins, checked without a GPU: the two
functions that make it are called in the built library."""
import ctypes
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2110_00511_amd", "libash.so")
U32, P = ctypes.c_uint32, ctypes.c_void_p

INSERT_MIN = 5 << 19      # positions from which an insert goes by bins
MOST = 256 * 65536        # positions up to which it does
BIN_MEAN = 8192           # most positions per bin, on average
MOST_BINS = 4096
MOST_REGION = 65536       # most table slots per bin


class Plan(ctypes.Structure):
    _fields_ = [(f, U32) for f in ("n", "nrange", "per", "nbins", "nbuckets", "shift", "pos_bits")] + [
        (f, P) for f in ("hist", "total", "base", "reps", "entries")]


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        from paper_2110_00511_amd.build import build
        build()
    import torch  # noqa: F401  (the binding loads torch's HIP runtime first)
    return ctypes.CDLL(LIB)


def plan(lib, n, nbuckets, width):
    """The plan of n positions on a table of nbuckets buckets, or None where the general path runs."""
    ranges = getattr(lib, "_ZN3ash11part_rangesEPNS_8PartPlanEj")
    buckets = getattr(lib, "_ZN3ash12part_bucketsEPNS_8PartPlanEjj")
    ranges.restype = buckets.restype = ctypes.c_bool
    ranges.argtypes = [ctypes.POINTER(Plan), U32]
    buckets.argtypes = [ctypes.POINTER(Plan), U32, U32]
    pl = Plan()
    assert ranges(ctypes.byref(pl), n)
    return pl if buckets(ctypes.byref(pl), nbuckets, width) else None


@pytest.mark.parametrize("width", [2, 4, 8, 16, 32, 64])
@pytest.mark.parametrize("n", [INSERT_MIN, INSERT_MIN + 1, 10_000_000, MOST])
def test_bins_stay_within_their_tables(lib, width, n):
    """From a table of 64 slots to one of 8 slots per position: a plan's bins
    hold at most BIN_MEAN positions on average (a bin fuller than its LDS table
    is settled entry by entry, so a batch in a few bins would take hours), and
    a table with too few buckets for that has no plan."""
    slots = 64
    planned = 0
    while slots <= 8 * n:
        nbuckets = slots // width
        pl = plan(lib, n, nbuckets, width)
        if n > BIN_MEAN * nbuckets:
            assert pl is None
        if pl is not None:
            planned += 1
            assert pl.nbuckets == nbuckets
            assert pl.nbins == -(-nbuckets // (1 << pl.shift)) and pl.nbins <= MOST_BINS
            assert n << pl.shift <= BIN_MEAN * nbuckets
            assert width << pl.shift <= MOST_REGION
            assert pl.nrange % 8 == 0 and pl.nrange <= 256 and pl.nrange * pl.per >= n
            assert pl.per % 4096 == 0 and pl.per <= 65536
        slots = max(slots + width, slots * 17 // 16 // width * width)
    assert planned > 0
