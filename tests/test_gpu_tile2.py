"""(2+1)D register tiles (several steps per pass, the default for a lattice and a
batch) against the split kernels, bit for bit: the same helpers in the same
order, so equality is exact.  Sizes at the edges of the tiles (64 - 2 s columns,
16 / 32 / 48 - 2 s rows for s steps per pass), lattices smaller than a region's
ring, odd widths, and step counts that split into uneven passes; the buffer set
that ends up with the state is the one the marches would leave it in."""
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


def rand_state(shape, seed, dtype):
    g = np.random.default_rng(seed)
    return [torch.from_numpy(g.standard_normal(shape) + 1j * g.standard_normal(shape)).to(dtype) for _ in range(4)]


def same(a, b):
    return all(torch.equal(torch.view_as_real(x), torch.view_as_real(y)) for x, y in zip(a, b))


# (nx, ny), steps: tiles of every shape with ragged and single-cell remainders
CASES = [((1, 1), 5), ((3, 2), 9), ((64, 64), 14), ((51, 3), 7), ((50, 2), 8), ((101, 51), 1), ((257, 130), 12),
         ((640, 512), 11), ((1111, 701), 13), ((1537, 1201), 7)]


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("site", [False, True])
@pytest.mark.parametrize("zero", [False, True])
@pytest.mark.parametrize("shape,steps", CASES)
def test_tiles_bitwise_equal_split(P, dtype, site, zero, shape, steps):
    print("tile2 %s n=%d site=%s zero=%s %s" % (shape, steps, site, zero, dtype), flush=True)
    nx, ny = shape
    f0 = rand_state((ny, nx), 71, dtype)
    g = np.random.default_rng(72)
    V = [torch.from_numpy(g.standard_normal((ny, nx))) for _ in range(4)]
    lats = []
    for kernel in ("split", "auto"):
        lat = P.Lattice2D(nx, ny, dtype=dtype, dt=workloads.DT2, zero_bc=zero)
        lat.set_kernel(kernel)
        lat.set_fields(0.4, V) if site else lat.set_potential_z(0.4)
        lat.load(f0)
        lat.step(steps)
        lats.append(lat)
    assert same(lats[0].state(), lats[1].state())
    two = nx * ny >= 1 << 18 and (dtype == torch.complex128 or nx % 2 == 0)
    assert lats[1].current == (0 if zero else (steps // 2 + steps % 2 if two else steps) % 2)
    back = [lat.reverse(steps - 1) or lat for lat in lats]
    assert same(back[0].state(), back[1].state())
    for lat in lats:
        lat.set_kernel("auto")
    a, b = lats[0].step_norm(4), lats[1].step_norm(4)
    assert same(lats[0].state(), lats[1].state()) and torch.equal(a, b)


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("site", [False, True])
@pytest.mark.parametrize("shape,steps", [((1, 1), 4), ((5, 3), 9), ((51, 4), 7), ((129, 77), 6), ((700, 611), 11)])
def test_link_tiles_bitwise_equal_split(P, dtype, site, shape, steps):
    print("tile2 links %s n=%d site=%s %s" % (shape, steps, site, dtype), flush=True)
    nx, ny = shape
    f0 = rand_state((ny, nx), 77, dtype)
    g = np.random.default_rng(78)
    V = [torch.from_numpy(g.standard_normal((ny, nx))) for _ in range(4)]
    U = [torch.from_numpy(np.exp(1j * g.uniform(0, 6.28, (ny, nx)))).to(dtype) for _ in range(8)]
    lats = []
    for kernel in ("split", "auto"):
        lat = P.Lattice2D(nx, ny, dtype=dtype, dt=workloads.DT2)
        lat.set_kernel(kernel)
        lat.set_fields(0.4, V) if site else lat.set_potential_z(0.4)
        lat.set_links(U)
        lat.load(f0)
        lat.step(steps)
        lats.append(lat)
    s, a = lats
    assert same(s.state(), a.state()) and a.current == steps % 2
    assert torch.equal(s.step_norm(3), a.step_norm(3)) and same(s.state(), a.state())


def test_shared_buffers_stay_in_place(P):
    """A zero-boundary context whose two buffer sets are one steps in place."""
    from paper_1309_3452_amd import _abi
    nx, ny = 70, 40
    f0 = rand_state((ny, nx), 73, torch.complex128)
    ref = P.Lattice2D(nx, ny, dtype=torch.complex128, dt=0.6, zero_bc=True)
    ref.set_kernel("split")
    ref.set_potential_z(0.3)
    ref.load(f0)
    ref.step(6)
    lat = P.Lattice2D(nx, ny, dtype=torch.complex128, dt=0.6, zero_bc=True)
    p = _abi.ptr_array([t.data_ptr() for t in lat.bufs[0]])
    assert P.lib().dirac_bind_state(lat._ctx, p, p) == 0
    lat.set_potential_z(0.3)
    lat.load(f0)
    lat.step(6)
    assert lat.current == 0 and same(lat.state(), ref.state())


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("count,steps", [(1, 3), (5, 1), (70, 9), (130, 6)])
def test_batch_tiles_bitwise_equal_split(P, dtype, graph, count, steps):
    """Lattice search over one and two looks, every tile shape's row count."""
    print("batch tiles n=%d steps=%d graph=%s %s" % (count, steps, graph, dtype), flush=True)
    g = np.random.default_rng(74)
    lats = []
    for b in range(count):
        nx, ny = (int(g.integers(1, 90)), int(g.integers(1, 90))) if count > 5 else (900 + 2 * b, 700 + b)
        lats.append(dict(nx=nx, ny=ny, m=0.1 * b, v_site=[torch.from_numpy(g.standard_normal((ny, nx))) for _ in range(4)],
                         state=rand_state((ny, nx), 75 + b, dtype)))
    batch = P.BatchedLattices(lats, dtype=dtype, dt=workloads.DT2)
    # the second run splits its steps differently while the first may still run
    batch.run(steps, mode=1, graph=graph)
    batch.run(steps + 5, mode=1, graph=graph)
    for b, L in enumerate(lats):
        solo = P.Lattice2D(L["nx"], L["ny"], dtype=dtype, dt=workloads.DT2)
        solo.set_kernel("split")
        solo.load(L["state"])
        solo.set_coef_records(batch.theta[b])
        solo.step(2 * steps + 5)
        assert same(solo.state(), batch.state(b)), b


def test_replayed_capture_keeps_its_buffer_set(P):
    """An even number of steps of a small lattice, captured once, replays any
    number of times: the passes leave the state where they found it."""
    lat = P.Lattice2D(96, 80, dtype=torch.complex64, dt=0.6)
    ref = P.Lattice2D(96, 80, dtype=torch.complex64, dt=0.6)
    ref.set_kernel("split")
    f0 = rand_state((80, 96), 76, torch.complex64)
    for q in (lat, ref):
        q.set_potential_z(0.3)
        q.load(f0)
        q.step(10)
    torch.cuda.synchronize()
    cur = lat.current
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lat.step(10)
    assert lat.current == cur
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        ref.step(10)
        assert same(lat.state(), ref.state())
