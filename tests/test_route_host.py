"""Which of the two profile kernels runs a call (no GPU): the streaming kernel
at the widths and ranks where it is the better one, the tiled kernel past the
lines of `stream_ranks` in launches that fill the chip with its tiles."""
import ctypes

import pytest

from paper_2401_13680_amd import _lib

L = _lib.load()


def streams(w, k, Nm=60_000, nq=500):
    return bool(L.pst_host_streams(ctypes.c_int32(w), ctypes.c_int32(k), ctypes.c_int64(Nm), ctypes.c_int64(nq)))


# the largest rank of a width that the streaming kernel takes, below 2w
LINES = {12: 16, 17: 16, 23: 16, 32: 10, 33: 11, 35: 11, 36: 16, 47: 16, 48: 19, 65: 26, 79: 31, 80: 48, 129: 77,
         143: 85, 265: 132, 289: 144}


@pytest.mark.parametrize("w", sorted(LINES))
def test_ranks_on_both_sides_of_the_line(w):
    assert streams(w, LINES[w]) and not streams(w, LINES[w] + 1)
    # too few tiles to fill the chip: strips at any rank
    assert streams(w, LINES[w] + 1, Nm=7936, nq=100)
    assert streams(w, w, Nm=1_000_000, nq=1)


@pytest.mark.parametrize("w", [24, 31, 144, 178, 179, 264, 290, 513, 552])
def test_every_rank_streams(w):
    assert all(streams(w, k) for k in (1, w // 2, w, 2 * w - 1, 2 * w))


def test_default_ranks_stream():
    """k = ceil(m / 10) of l = m/2 at every length up to w = 552, and the ends."""
    assert all(streams(m - m // 2 + 1, (m + 9) // 10) for m in range(24, 1103))
    assert not any(streams(w, 1) for w in (1, 11, 553, 1025))
    assert [w for w in range(12, 553) if not streams(w, 2 * w)] == list(range(32, 36)) + list(range(265, 290))


def test_resident_workgroups():
    """Four a CU to w = 144, three to 178, two to 264, then one (the widest strips fill a CU's LDS)."""
    got = {w: L.pst_host_stream_resident(ctypes.c_int32(w)) for w in range(12, 553)}
    want = {w: 1024 if w <= 144 else 768 if w <= 178 else 512 if w <= 264 else 256 for w in got}
    assert got == want, {w: (got[w], want[w]) for w in got if got[w] != want[w]}
    assert L.pst_host_stream_resident(ctypes.c_int32(553)) == -1
