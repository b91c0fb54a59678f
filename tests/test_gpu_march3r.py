"""(3+1)D register march (the default for complex128, per-site records, odd
complex64 widths and zero values outside) against the split kernels, bit for bit:
the same helpers in the same order, so equality is exact.  Sizes at the edges of
the tiles (56 to 62 columns, 4 to 30 rows), fewer planes than a launch's reach,
odd widths, and step counts that split unevenly; forward, reversed and with the
functional summed in the last launch (FP64 sums of the same values, 1e-13
relative: against the reduction with zero values outside, else against the
in-step sums of the one-step march, whose differences are in the lattice's
precision).  The buffer set that ends up with the state is the
one the marches before it left it in."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import paper_1309_3452_amd as P
    assert torch.cuda.is_available(), "needs a GPU"
    P.lib()
    return P


def same(a, b):
    return all(torch.equal(torch.view_as_real(x), torch.view_as_real(y)) for x, y in zip(a, b))


CASES = [((1, 1, 1), 5), ((3, 2, 2), 9), ((5, 4, 3), 4), ((57, 13, 5), 7), ((61, 30, 4), 6), ((121, 29, 33), 10),
         ((64, 64, 40), 11), ((113, 57, 130), 5), ((64, 13, 7), 6), ((32, 21, 9), 4), ((16, 16, 16), 5), ((2, 9, 30), 4)]


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("mode", ["vz", "absorb", "site"])
@pytest.mark.parametrize("zero", [False, True])
@pytest.mark.parametrize("shape,steps", CASES)
def test_march_bitwise_equals_split(P, dtype, mode, zero, shape, steps):
    print("march3r %s n=%d %s zero=%s %s" % (shape, steps, mode, zero, dtype), flush=True)
    nx, ny, nz = shape
    g = np.random.default_rng(81)
    f0 = [torch.from_numpy(g.standard_normal((nz, ny, nx)) + 1j * g.standard_normal((nz, ny, nx))) for _ in range(8)]
    V = [torch.from_numpy(g.standard_normal((nz, ny, nx))) for _ in range(8)]
    vi, vh = g.standard_normal(nz), g.standard_normal(nz)
    lats = []
    for kernel in ("split", "auto"):
        lat = P.Lattice3D(nx, ny, nz, dtype=dtype, dt=workloads.DT3, zero_bc=zero)
        lat.set_kernel(kernel)
        if mode == "site":
            lat.set_fields(0.4, V)
        else:
            lat.set_potential_z(0.4, vi, vh)
            if mode == "absorb":
                lat.set_absorber_z(-np.abs(vi), -np.abs(vh))
        lat.load(f0)
        lat.step(steps)
        lats.append(lat)
    s, a = lats
    assert same(s.state(), a.state())
    two = dtype == torch.complex128 or nx % 2 == 0
    assert a.current == (0 if zero else (steps // 2 + steps % 2 if two else steps) % 2)
    if mode != "absorb":        # the reversed step amplifies there
        s.reverse(steps - 1)
        a.reverse(steps - 1)
        assert same(s.state(), a.state())
    if not zero:
        s.set_kernel("fused")
    for n in (1, 2, 3, 6):
        ref = s.step_norm(n).tolist()
        e = a.step_norm(n).tolist()
        assert same(s.state(), a.state()), n
        assert abs(e[0] - ref[0]) <= 1e-13 * max(abs(ref[0]), ref[1]) and abs(e[1] - ref[1]) <= 1e-13 * ref[1], n


def test_shared_buffers_stay_in_place(P):
    """A zero-boundary context whose two buffer sets are one steps in place."""
    from paper_1309_3452_amd import _abi
    g = np.random.default_rng(82)
    f0 = [torch.from_numpy(g.standard_normal((6, 9, 20)) + 1j * g.standard_normal((6, 9, 20))) for _ in range(8)]
    lats = []
    for shared in (False, True):
        lat = P.Lattice3D(20, 9, 6, dtype=torch.complex128, dt=workloads.DT3, zero_bc=True)
        lat.set_kernel("auto" if shared else "split")
        if shared:
            p = _abi.ptr_array([t.data_ptr() for t in lat.bufs[0]])
            assert P.lib().dirac_bind_state(lat._ctx, p, p) == 0
        lat.set_potential_z(0.3)
        lat.load(f0)
        lat.step(6)
        lat.reverse(3)
        lats.append(lat)
    assert lats[1].current == 0 and same(lats[0].state(), lats[1].state())


@pytest.mark.parametrize("nx,ny,nz", [(340, 5, 4), (421, 9, 7)])
def test_wide_rows_of_60_columns(P, nx, ny, nz):
    """complex128 rows that 60-column tiles cover with fewer columns than 56-column ones."""
    print("march3r wide %dx%dx%d" % (nx, ny, nz), flush=True)
    g = np.random.default_rng(83)
    f0 = [torch.from_numpy(g.standard_normal((nz, ny, nx)) + 1j * g.standard_normal((nz, ny, nx))) for _ in range(8)]
    lats = []
    for kernel in ("split", "auto"):
        lat = P.Lattice3D(nx, ny, nz, dtype=torch.complex128, dt=workloads.DT3)
        lat.set_kernel(kernel)
        lat.set_potential_z(0.4, np.full(nz, 0.3), np.linspace(0.1, 0.9, nz))
        lat.load(f0)
        lat.step(5)
        lats.append(lat)
    assert same(lats[0].state(), lats[1].state())


@pytest.mark.parametrize("slabs", [1, 2, 5])
def test_slab_planes_wrap(P, slabs):
    """Slabs of few planes (2 to 10) under the march, whose plane index wraps over the stored planes."""
    print("march3r slabs %d" % slabs, flush=True)
    g = np.random.default_rng(84)
    nx, ny, nz = 61, 14, 10
    f0 = [torch.from_numpy(g.standard_normal((nz, ny, nx)) + 1j * g.standard_normal((nz, ny, nx))) for _ in range(8)]
    vi, vh = g.standard_normal(nz), g.standard_normal(nz)
    whole = P.Lattice3D(nx, ny, nz, dtype=torch.complex128, dt=workloads.DT3)
    parts = P.SlabDecomposition(nx, ny, nz, slabs, dtype=torch.complex128, dt=workloads.DT3)
    whole.set_kernel("split")
    for lat in (whole, parts):
        lat.set_potential_z(0.4, vi, vh)
        lat.load(f0)
        lat.step(6)
    assert same(whole.state(), parts.state())
