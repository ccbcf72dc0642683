"""The rule that says which periodic matrices run as streaming sweeps, on the
host: the number of blocks at either end of the rows in which h^T E^{-1}
counts, from the reach of its values."""
import ctypes

import pytest

from paper_1807_07382_amd import pentbatch as pb

WAVES, ROWS = 16, 32  # of the streaming kernel's workgroup, of a block


class Aux(ctypes.Structure):  # CycAux
    _fields_ = [("nh", ctypes.c_int), ("bad", ctypes.c_int), ("hq", ctypes.c_int * 10),
                ("hcol", ctypes.c_int64 * 10), ("hv", ctypes.c_double * 10), ("minv", ctypes.c_double * 4),
                ("reach", ctypes.c_int64 * 2)]


def ends(top, bottom, n):
    f = pb.lib()["_ZN4pent15cyc_stream_endsERKNS_6CycAuxEl"]
    f.restype, f.argtypes = ctypes.c_int, [ctypes.POINTER(Aux), ctypes.c_int64]
    aux = Aux()
    aux.reach[0], aux.reach[1] = top, bottom
    return f(ctypes.byref(aux), n)


def runs_through(T, nblk):
    """Whether every item of a tile can end, by the kernel's own waits: items
    (T bottom blocks' products, then the blocks) go round the waves in order,
    a wave takes its next item when it has ended the one before; an item is
    swept forward after all items before it, block T - 1 then has x_tail, and
    a block ends once x_tail is there."""
    swept, ended = 0, set()
    while True:
        before = swept, len(ended)
        if swept < T + nblk and (swept < WAVES or swept - WAVES in ended):
            swept += 1
        for i in range(swept):
            if i < T or swept >= 2 * T:
                ended.add(i)
        if (swept, len(ended)) == before:
            return len(ended) == T + nblk


@pytest.mark.parametrize("n", [514, 1537, 4098, 4100, 40000])
def test_streaming_only_where_a_tile_runs_through(n):
    m = n - 2
    nblk = (m + ROWS - 1) // ROWS
    for T in range(1, min(nblk, 60) + 1):
        for top, bottom in ((T * ROWS - 5, 1), (1, m - (nblk - T) * ROWS), (T * ROWS, m - (nblk - T) * ROWS)):
            if not (0 < top <= m and 0 < bottom <= m):
                continue
            got = ends(top, bottom, n)
            assert got in (0, T)
            if got:
                assert runs_through(T, nblk), (n, T)


def test_short_ends_stream():
    assert ends(90, 90, 4098) == 3
    assert ends(16 * ROWS, 1, 4098) == 16
    assert ends(16 * ROWS + 1, 1, 4098) == 0
    assert ends(1, 17 * ROWS, 4098) == 0


def test_the_model_of_the_waits():
    assert runs_through(16, 128) and not runs_through(17, 128)
