"""(2+1)D: the functional after steps on register tiles against the split kernels'
(state bit for bit; the same reduction of the same state, so the same value), and
gauge links on a plane that takes the tile of 32 rows."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


def same(a, b):
    return all(torch.equal(torch.view_as_real(x), torch.view_as_real(y)) for x, y in zip(a, b))


def pair(P, shape, dtype, site, zero=False, links=False):
    g = torch.Generator(device="cuda").manual_seed(79)
    tshape = tuple(reversed(shape))
    rnd = lambda dt: torch.randn(tshape, generator=g, device="cuda", dtype=dt)
    f0, V = [rnd(dtype) for _ in range(4)], [rnd(torch.float64) for _ in range(4)]
    U = [torch.polar(torch.ones_like(t), t) for t in (rnd(torch.float64) for _ in range(8))]
    out = []
    for kernel in ("split", "auto"):
        lat = P.Lattice(shape, dtype=dtype, dt=workloads.DT2, zero_bc=zero)
        lat.set_kernel(kernel)
        lat.set_fields(0.4, V) if site else lat.set_potential_z(0.4)
        if links:
            lat.set_links(U)
        lat.load(f0)
        out.append(lat)
    return out


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("site", [False, True])
@pytest.mark.parametrize("zero", [False, True])
@pytest.mark.parametrize("shape", [(50, 33), (333, 257), (1030, 701)])
def test_step_norm_equals_split(dtype, site, zero, shape):
    import paper_1309_3452_amd as P
    print("tile2 step_norm %s site=%s zero=%s %s" % (shape, site, zero, dtype), flush=True)
    s, a = pair(P, shape, dtype, site, zero)
    for n in (1, 2, 3, 4, 9):
        assert n == 1 or "tile2" in a.route(n, "step_norm")
        before = a.current
        flips = 0 if zero else n
        if not zero and shape[0] * shape[1] >= 1 << 18 and (dtype == torch.complex128 or shape[0] % 2 == 0):
            flips = (n - 1) // 2 + (n - 1) % 2 + 1      # as two-step marches and a last single step leave it
        ref, e = s.step_norm(n), a.step_norm(n)
        assert torch.equal(ref, e) and same(s.state(), a.state()), n
        assert a.current == (before + flips) % 2, n


@pytest.mark.parametrize("site", [False, True])
@pytest.mark.parametrize("shape", [(2047, 1531), (1500, 2001)])
def test_link_tile_of_32_rows_equals_split(site, shape):
    import paper_1309_3452_amd as P
    print("tile2 links %s site=%s" % (shape, site), flush=True)
    s, a = pair(P, shape, torch.complex64, site, links=True)
    for n in (5, 3, 1):
        route = a.route(n)
        assert n < 3 or "tile2 links" in route and "rows=32" in route, route
        s.step(n)
        a.step(n)
        assert same(s.state(), a.state()), route
