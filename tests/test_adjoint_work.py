"""dirac_adjoint_vz_work's arrays: the one-launch backward step reads and writes
lam, work and both buffer sets in one launch, so overlaps are refused before any
HIP call (fake pointers, never dereferenced here)."""
import ctypes

import pytest

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
