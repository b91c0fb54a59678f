"""dirac_adjoint_vz_work's arrays: the one-launch backward step reads and writes
lam, work and both buffer sets in one launch, so overlaps are refused before any
HIP call (fake pointers, never dereferenced here); and whether it would be used,
which says if work arrays are worth their memory."""
import ctypes

import pytest
import torch

from paper_1309_3452_amd import _abi

N = 8 * 8 * 8
BASE = 1 << 20


@pytest.fixture()
def ctx():
    L = _abi.lib()
    c = ctypes.c_void_p()
    assert L.dirac_create(ctypes.byref(c), 3, 8, 8, 8, _abi.DIRAC_C128, 0.5, 1.0, 1.0, 1.0, 0) == 0
    assert L.dirac_bind_state(c, _abi.ptr_array(arrays(0)), _abi.ptr_array(arrays(1))) == 0
    nb = ctypes.c_size_t()
    assert L.dirac_scratch_bytes(c, ctypes.byref(nb)) == 0
    assert L.dirac_bind_scratch(c, ctypes.c_void_p(1 << 30), nb.value) == 0
    yield c
    L.dirac_destroy(c)


def arrays(group):
    """8 neighbouring arrays of 8^3 complex128; groups do not meet."""
    return [BASE + (8 * group + q) * N * 16 for q in range(8)]


def call(c, lam, work):
    d = ctypes.c_void_p(1 << 29)
    return _abi.lib().dirac_adjoint_vz_work(c, 2, _abi.ptr_array(lam), _abi.ptr_array(work), d, d, None)


@pytest.mark.parametrize("name,lam,work", [
    ("lam in the idle buffer set", arrays(1), arrays(3)),
    ("lam in the current buffer set", arrays(0), arrays(3)),
    ("lam partly in the idle buffer set", [p - 16 for p in arrays(2)], arrays(3)),
    ("a work array twice", arrays(2), arrays(3)[:7] + arrays(3)[:1]),
    ("work arrays that overlap", arrays(2), arrays(3)[:7] + [arrays(3)[6] + 16]),
    ("work in lam", arrays(2), arrays(3)[:7] + [arrays(2)[3]]),
    ("work partly in lam", arrays(2), [p - 16 for p in arrays(3)]),
    ("work in the idle buffer set", arrays(2), arrays(1)),
    ("work partly in a buffer set", arrays(3), [p + 16 for p in arrays(1)]),
])
def test_overlaps_are_refused(ctx, name, lam, work):
    assert call(ctx, lam, work) == -1, name
    assert b"overlaps" in _abi.lib().dirac_last_error(ctx)


def uses(shape, dtype, n, flags=0, site=False):
    L, c, u = _abi.lib(), ctypes.c_void_p(), ctypes.c_int(-1)
    nz = shape[2] if len(shape) == 3 else 1
    assert L.dirac_create(ctypes.byref(c), len(shape), shape[0], shape[1], nz, dtype, 0.5, 1.0, 1.0, 1.0, flags) == 0
    a = [(1 << 50) + (q << 42) for q in range(24)]
    assert L.dirac_adjoint_uses_work(c, n, ctypes.byref(u)) == 0 and u.value == 0      # nothing bound yet
    assert L.dirac_bind_state(c, _abi.ptr_array(a[:8]), _abi.ptr_array(a[8:16])) == 0
    if site:
        assert L.dirac_set_theta_field(c, _abi.ptr_array(a[16:])) == 0
    assert L.dirac_adjoint_uses_work(c, n, ctypes.byref(u)) == 0
    L.dirac_destroy(c)
    return u.value


def test_where_work_arrays_are_used():
    """Lattices large enough to gain, from two steps on; nowhere the adjoint is refused."""
    big = (200, 168, 152)
    for dtype in (_abi.DIRAC_C64, _abi.DIRAC_C128):
        assert uses(big, dtype, 2) == 1 and uses(big, dtype, 1) == 0 and uses(big, dtype, 0) == 0
        assert uses((64, 64, 64), dtype, 40) == 0
        assert uses(big, dtype, 4, site=True) == 0
        assert uses(big, dtype, 4, flags=_abi.DIRAC_ZERO_BC) == 0 and uses(big, dtype, 4, flags=_abi.DIRAC_SLAB_Z) == 0
        assert uses((300, 300), dtype, 4) == 0
    assert uses((128, 128, 128), _abi.DIRAC_C64, 4) == 0 and uses((128, 128, 128), _abi.DIRAC_C128, 4) == 1
    assert _abi.lib().dirac_adjoint_uses_work(None, 1, ctypes.byref(ctypes.c_int())) == -1


@pytest.mark.gpu
@pytest.mark.parametrize("shape,sets", [((64, 64, 64), 1), ((160, 150, 120), 2)])
def test_potential_gradient_allocates_what_it_uses(shape, sets):
    """lam, and a second set of its size only where the backward steps use it."""
    import numpy as np

    import paper_1309_3452_amd as P
    print("gradient memory %s" % (shape,), flush=True)
    lat = P.Lattice(shape, dtype=torch.complex64, dt=0.5)
    state = [torch.full(lat.tshape, 1e-3, dtype=torch.complex64, device="cuda") for _ in range(8)]
    v = np.linspace(0.0, 1.0, shape[2])
    torch.cuda.synchronize()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    P.potential_gradient(lat, state, 0.4, v, v, 4, shape[2] / 2.0)
    torch.cuda.synchronize()
    one = 8 * state[0].numel() * 8
    assert torch.cuda.max_memory_allocated() - before < (sets + 0.5) * one
