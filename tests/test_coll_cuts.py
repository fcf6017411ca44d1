"""How the header cuts the data-movement collectives into tasks: the functions
run on the host, through the user-test library."""
import ctypes
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "devapi", "libvshmem_usertest.so")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        import __graft_entry__ as g
        g.build()
    import paper_2607_08006_amd  # noqa: F401  (torch's runtime first)
    return ctypes.CDLL(LIB)


@pytest.mark.parametrize("wg", [1, 2, 3, 16, 32, 48, 63, 64, 96, 256, 1024])
def test_a_pair_task_fits_its_work_group(lib, wg):
    """A task's lanes exist in the work-group, are a power of two, at most a
    wavefront, a block's tasks cover it, and a unit's step passes over one task
    of every other unit."""
    out = (ctypes.c_uint64 * 6)()
    for deep in (0, 1):
        for n in (1, 16, 1000, 2048, 2049, 4096, 4097, 16383, 16384, 100001, 1 << 20, 300 << 20):
            for P, workers in ((1, 1), (3, 3), (13, 208), (64, 64), (64, 256), (500, 1000)):
                for chunk in (16, 4112, 256 << 10):
                    lib.usertest_pair_split(deep, ctypes.c_uint64(n), P, workers, wg, ctypes.c_uint64(chunk), out)
                    task, nch, g, schunk, sq, sp = out
                    assert 1 <= g <= min(wg, 64) and g & (g - 1) == 0, (n, P, workers, chunk)
                    assert 0 < task <= chunk and (nch - 1) * task < n <= nch * task, (n, P, workers, chunk)
                    assert schunk < nch and sq < P
                    assert schunk + nch * (sq + P * sp) == workers * (wg // g), (n, P, workers, chunk)


@pytest.mark.parametrize("n", [100000, 262144, 300000, 1 << 20])
def test_blocks_stay_whole_where_units_have_many(lib, n):
    """With eight blocks or more per wavefront a block is cut only by the chunk
    size, into equal tasks."""
    out = (ctypes.c_uint64 * 6)()
    for P, workers, wg in ((64, 64, 64), (64, 64, 256), (64, 128, 256), (16, 16, 64)):
        lib.usertest_pair_split(1, ctypes.c_uint64(n), P, workers, wg, ctypes.c_uint64(256 << 10), out)
        parts = -(-n // (256 << 10))
        assert out[1] == parts and out[0] - (n - (parts - 1) * out[0]) < parts * 8192, (P, workers, wg, out[0])


@pytest.mark.parametrize("chunk", [16, 4096, 20000, 65536, 100000, 262144])
def test_multicast_chunks_stay_within_the_callers(lib, chunk):
    """A chunk is no larger than asked for, chunks cover the range, groups the
    members, none of them empty."""
    out = (ctypes.c_uint64 * 4)()
    for n in (1, 15, 4096, 16384, 20000, 100001, 300000, 1 << 20, 5 << 20, 256 << 20):
        for P in (1, 4, 13, 64, 500):
            for Q in (1, P):
                for workers in (1, P, 4 * P, 256, 1024):
                    lib.usertest_mcast_split(ctypes.c_uint64(n), Q, P, workers, ctypes.c_uint64(chunk), out)
                    size, nch, per, groups = out
                    assert 0 < size <= chunk and (nch - 1) * size < n <= nch * size, (n, P, Q, workers, size)
                    assert (groups - 1) * per < P <= groups * per, (n, P, Q, workers)


@pytest.mark.parametrize("P", [8, 9, 17, 24, 25, 31, 32, 33, 40, 64])
def test_a_reduction_step_leaves_no_tile_slot_idle(lib, P):
    """A task of one step holds as many tiles as the work-group's wavefronts
    take at a time, members in blocks of eight."""
    out = (ctypes.c_uint64 * 3)()
    for waves in range((P + 7) // 8, 9):
        lib.usertest_red_waves_split(ctypes.c_uint64(100000), 4, P, waves, out)
        tpt, slots, blocks = out
        assert blocks == (P + 7) // 8 and slots == waves // blocks and tpt == slots, (waves, list(out))
