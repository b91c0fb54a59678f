"""(3+1)D register march: the built shapes that only larger lattices take (16 to 32
rows, several rows per thread), each compared bit for bit with the split kernels,
forward, reversed and with the functional summed in the last launch.  The route
of every call is looked up first, so that a case which no longer reaches its shape
fails.  The functional sums the same FP64 terms in another order: a thread adds
fewer than a thousand of them and trees the rest, so 1000 x 2^-53 = 1e-13 of the
plain norm (the sum of the terms' moduli, up to a factor near one) bounds it."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


def same(a, b):
    return all(torch.equal(torch.view_as_real(x), torch.view_as_real(y)) for x, y in zip(a, b))


# dtype, coefficients, lattice, {steps per launch: (rows per thread, waves)}
CASES = [(torch.complex64, "vz", (57, 626, 74), {2: (2, 16), 3: (3, 8)}),
         (torch.complex64, "vz", (115, 626, 37), {2: (1, 16), 3: (1, 12)}),
         (torch.complex64, "vz", (191, 130, 47), {2: (1, 16)}),
         (torch.complex64, "vz", (96, 96, 96), {2: (1, 16)}),
         (torch.complex64, "site", (113, 130, 64), {2: (2, 8)}),
         (torch.complex64, "site", (96, 96, 96), {2: (2, 8)}),
         (torch.complex128, "vz", (57, 725, 33), {2: (2, 8)}),
         (torch.complex128, "vz", (190, 131, 64), {2: (1, 12)}),
         (torch.complex128, "site", (190, 131, 64), {2: (1, 8)})]


@pytest.mark.parametrize("zero", [False, True])
@pytest.mark.parametrize("dtype,mode,shape,shapes", CASES)
def test_every_shape_bitwise_equals_split(dtype, mode, shape, shapes, zero):
    import paper_1309_3452_amd as P
    print("march3r shapes %s %s zero=%s %s" % (shape, mode, zero, dtype), flush=True)
    nz = shape[2]
    g = torch.Generator(device="cuda").manual_seed(87)
    rnd = lambda *s, **k: torch.randn(*s, generator=g, device="cuda", **k)
    tshape = tuple(reversed(shape))
    f0 = [rnd(tshape, dtype=dtype) for _ in range(8)]
    V = [rnd(tshape) for _ in range(8)] if mode == "site" else None
    vi, vh = rnd(nz).double().cpu().numpy(), rnd(nz).double().cpu().numpy()
    lats = []
    for kernel in ("split", "auto"):
        lat = P.Lattice(shape, dtype=dtype, dt=workloads.DT3, zero_bc=zero)
        lat.set_kernel(kernel)
        lat.set_fields(0.4, V) if V else lat.set_potential_z(0.4, vi, vh)
        lat.load(f0)
        lats.append(lat)
    s, a = lats
    word = {T: "steps=%d rows=%d waves=%d " % ((T,) + rw) for T, rw in shapes.items()}
    routes = []
    for n in (4, 3, 5):
        routes.append(a.route(n))
        for lat in lats:
            lat.step(n)
        assert same(s.state(), a.state()), routes[-1]
    for T, w in word.items():
        assert any(w in r for r in routes), (w, routes)
    route = a.route(5, "reverse")
    assert word[2] in route, route
    for lat in lats:
        lat.reverse(5)
    assert same(s.state(), a.state()), route
    route = a.route(4, "step_norm")
    assert word[2] in route, route
    if not zero:
        s.set_kernel("fused")       # its in-step sums have the differences in the lattice's precision too
    ref, e = s.step_norm(4).tolist(), a.step_norm(4).tolist()
    assert same(s.state(), a.state()), route
    assert abs(e[0] - ref[0]) <= 1e-13 * max(abs(ref[0]), ref[1]) and abs(e[1] - ref[1]) <= 1e-13 * ref[1]
