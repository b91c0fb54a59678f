"""Which kernels a call would launch (dirac_route), on the CPU: the choice depends on
the lattice and the call alone (without a device the estimates take 256 CUs, an
MI355X's)."""
import ctypes

import pytest

from paper_1309_3452_amd import _abi

C64, C128 = _abi.DIRAC_C64, _abi.DIRAC_C128
STEP, REVERSE, STEP_NORM = 0, 1, 2
AUTO, SPLIT, FUSED, FUSED2 = 0, 1, 2, 3


def route(shape, dtype, n, call=STEP, site=False, links=False, zero=False, slab=False, kernel=AUTO, shift=None,
          size=1024):
    """The route of a context whose arrays (fake pointers, 4 TiB apart) are never touched."""
    L, c = _abi.lib(), ctypes.c_void_p()
    flags = (_abi.DIRAC_ZERO_BC if zero else 0) | (_abi.DIRAC_SLAB_Z if slab else 0)
    nz = shape[2] if len(shape) == 3 else 1
    assert L.dirac_create(ctypes.byref(c), len(shape), shape[0], shape[1], nz, dtype, 0.5, 1.0, 1.0, 1.0, flags) == 0
    try:
        a = [(1 << 50) + (q << 42) for q in range(48)]
        second = [p + shift for p in a[:8]] if shift is not None else a[8:16]
        assert L.dirac_bind_state(c, _abi.ptr_array(a[:8]), _abi.ptr_array(second)) == 0
        if site:
            assert L.dirac_set_theta_field(c, _abi.ptr_array(a[16:24])) == 0
        if links:
            assert L.dirac_set_links(c, _abi.ptr_array(a[24:48])) == 0
        assert L.dirac_set_kernel(c, kernel, 0, 0) == 0
        text = ctypes.create_string_buffer(size)
        rc = L.dirac_route(c, n, call, text, size)
        return text.value.decode() if rc == 0 else rc
    finally:
        L.dirac_destroy(c)


def test_explicit_kernels():
    s = (96, 40, 20)
    assert route(s, C64, 5, kernel=SPLIT) == "5 x split"
    assert route(s, C64, 5, kernel=FUSED) == "5 x fused"
    assert route(s, C64, 5, kernel=FUSED2) == "2 x fused2; 1 x fused"
    assert route(s, C64, 5, REVERSE, kernel=FUSED2) == "1 x half; 2 x fused2; 1 x half"
    assert route(s, C128, 3, links=True) == "3 x fused links"
    assert route(s, C128, 3, REVERSE, links=True) == "3 x split"
    assert route((64, 64, 16), C128, 2, slab=True) == "1 x march3r steps=2"
    assert route((64, 64, 16), C64, 2, slab=True) == "1 x fused2"
    assert route(s, C64, 0) == ""


def test_arguments():
    s = (96, 40, 20)
    assert route(s, C64, -1) == -1
    assert route(s, C64, 0, STEP_NORM) == -1
    assert route(s, C64, 1, 3) == -1
    assert route(s, C64, 5, size=8) == -2
    assert _abi.lib().dirac_route(None, 1, 0, ctypes.create_string_buffer(8), 8) == -1


@pytest.mark.parametrize("shape", [(70, 40), (120, 90, 70)])
@pytest.mark.parametrize("dtype,size", [(C64, 8), (C128, 16)])
def test_sets_that_share_memory_step_in_place(shape, dtype, size):
    for shift in (0, size, -size, (2 * shape[0] + 1) * size):
        for call in (STEP, REVERSE):
            assert route(shape, dtype, 6, call, zero=True, shift=shift) == "6 x split", (shift, call)
    n = size
    for q in shape:
        n *= q
    apart = route(shape, dtype, 6, zero=True, shift=n)                       # neighbours, not shared
    assert "tile2" in apart or "march3r" in apart, apart


def test_tables_beyond_32_bit_offsets():
    long = ((1 << 25) + 8)
    assert "march3r" not in route((1, 1, long), C128, 6, zero=True)
    assert "march3r" not in route((1, 1, 2 * long), C64, 6)
    assert "march3r" in route((1, 1, long), C64, 6)


@pytest.mark.parametrize("shape,dtype,n,call,expect", [
    # two one-step launches took longer than two steps in place
    ((128, 128, 128), C64, 2, STEP, "2 x split"), ((33, 40, 50), C64, 2, STEP, "2 x split"),
    ((63, 100, 30), C128, 2, STEP, "2 x split"), ((64, 512, 4), C128, 2, STEP, "2 x split"),
    # so did any launches where tiles are nearly empty
    ((300, 1, 300), C64, 3, STEP, "3 x split"), ((300, 1, 300), C64, 4, REVERSE, "4 x split"),
    ((512, 4, 64), C128, 3, STEP, "3 x split"),
    # an odd step apart from an even number of launches
    ((128, 128, 128), C64, 5, STEP, "1 x split; 2 x march3r steps=2"),
    # larger boxes keep the march
    ((200, 168, 152), C64, 2, STEP, "2 x march3r steps=1"), ((200, 168, 152), C128, 8, STEP, "4 x march3r steps=2"),
    ((224, 192, 256), C64, 10, STEP_NORM, "2 x march3r steps=3")])
def test_zero_boundary_plans(shape, dtype, n, call, expect):
    r = route(shape, dtype, n, call, zero=True)
    assert r == expect or "march3r" in expect and r.startswith(expect), r


def test_narrow_complex128_rows_keep_the_lds_march():
    for shape in ((1, 300, 300), (4, 64, 512), (12, 200, 200), (16, 200, 200)):
        assert route(shape, C128, 9) == "4 x fused2; 1 x fused", shape
        assert route(shape, C128, 9, REVERSE) == "1 x half; 4 x fused2; 1 x half", shape
        assert "march3r" in route(shape, C128, 9, site=True), shape
    for shape in ((1, 7, 600), (20, 200, 200), (64, 200, 200)):
        assert "4 x march3r" in route(shape, C128, 9), shape
    assert route((8, 200, 200), C128, 2, slab=True) == "1 x fused2"


def test_one_step_of_a_single_odd_row():
    assert route((301, 1, 300), C64, 1) == "1 x fused"
    assert "march3r" in route((301, 1, 300), C64, 1, site=True)
    assert "march3r" in route((301, 2, 300), C64, 1)


@pytest.mark.parametrize("shape,dtype,n,call,kw,tiles", [
    # a few very long rows leave the tiles' regions mostly empty
    ((400000, 1), C128, 1, STEP, dict(site=True), False), ((400000, 1), C64, 7, STEP, {}, False),
    ((400000, 4), C128, 1, STEP, dict(site=True), False), ((400000, 4), C128, 1, STEP, dict(links=True), False),
    ((100000, 2), C128, 2, STEP, dict(site=True, zero=True), False),
    ((100000, 2), C128, 3, REVERSE, dict(site=True), False), ((100000, 1), C64, 1, STEP, {}, False),
    ((8, 100000), C128, 2, STEP, dict(site=True, zero=True), False),
    # more steps, more rows or fewer tiles than rounds: tiles
    ((400000, 4), C128, 7, STEP, dict(site=True), True), ((400000, 12), C128, 1, STEP, dict(site=True), True),
    ((100000, 2), C64, 9, STEP, {}, True), ((5000, 1), C64, 1, STEP, {}, True),
    ((8, 100000), C64, 2, STEP, dict(site=True, zero=True), True), ((3000, 3000), C128, 2, STEP, dict(zero=True, site=True), True),
    ((1024, 512), C64, 100, STEP, dict(site=True), True), ((128, 128), C128, 200, STEP, {}, True),
    ((333, 1000), C128, 4, REVERSE, dict(site=True), True), ((64, 64), C64, 2, STEP_NORM, {}, True)])
def test_planes_that_tiles_fit(shape, dtype, n, call, kw, tiles):
    r = route(shape, dtype, n, call, **kw)
    assert ("tile2" in r) == tiles, r


def test_one_step_launches_are_priced_as_what_runs():
    """Periodic complex64 of even width: an odd step runs on the LDS march's one-step
    kernel, whose time and not the register march's decides against threes."""
    assert route((40, 135, 81), C64, 11).startswith("3 x march3r steps=3 ")      # 149 -> 138 us
    assert route((24, 305, 284), C64, 11).startswith("3 x march3r steps=3 ")     # 729 -> 641 us


def batch_route(sizes, dtype, n):
    L, c, count = _abi.lib(), ctypes.c_void_p(), len(sizes)
    nx, ny = ((ctypes.c_int64 * count)(*[s[q] for s in sizes]) for q in (0, 1))
    assert L.dirac_batch_create(ctypes.byref(c), count, nx, ny, dtype, 0.5, 0) == 0
    text = ctypes.create_string_buffer(256)
    assert L.dirac_route(c, n, STEP_NORM, text, 256) == -6
    assert L.dirac_route(c, n, STEP, text, 256) == 0
    L.dirac_destroy(c)
    return text.value.decode()


def test_batches_of_a_few_long_rows_leave_the_tiles():
    for dtype in (C64, C128):
        assert batch_route([(20000, 1)] * 40, dtype, 1) == "1 x march steps=1 width=128 rows=64"
        assert batch_route([(20000, 1)] * 40, dtype, 3).startswith("1 x march steps=2 width=128 rows=64; 1 x march")
        for sizes in ([(512, 512)] * 15, [(20000, 1)] * 40 + [(64, 64)], [(8, 1024)] * 50, [(500, 1)] * 9):
            assert "tile2" in batch_route(sizes, dtype, 10), sizes
    assert "tile2" in batch_route([(1024, 8)] * 50, C64, 1)
