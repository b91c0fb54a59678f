"""Zero values outside a (3+1)D lattice: plans that mix in-place steps with an even
number of launches, bit for bit the split kernels, forward, reversed and with the
functional (the same FP64 terms in another order, fewer than a thousand additions in
a row: 1e-13 of the plain norm)."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


def same(a, b):
    return all(torch.equal(torch.view_as_real(x), torch.view_as_real(y)) for x, y in zip(a, b))


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("site", [False, True])
@pytest.mark.parametrize("shape", [(57, 29, 9), (100, 41, 31), (128, 30, 41)])
def test_mixed_plans_bitwise_equal_split(dtype, site, shape):
    import paper_1309_3452_amd as P
    print("zero plans %s site=%s %s" % (shape, site, dtype), flush=True)
    g = torch.Generator(device="cuda").manual_seed(88)
    tshape = tuple(reversed(shape))
    f0 = [torch.randn(tshape, generator=g, device="cuda", dtype=dtype) for _ in range(8)]
    V = [torch.randn(tshape, generator=g, device="cuda") for _ in range(8)]
    v = torch.randn(2, shape[2], generator=g, device="cuda").double().cpu().numpy()
    s, a = lats = [P.Lattice(shape, dtype=dtype, dt=workloads.DT3, zero_bc=True) for _ in range(2)]
    s.set_kernel("split")
    for lat in lats:
        lat.set_fields(0.4, V) if site else lat.set_potential_z(0.4, v[0], v[1])
        lat.load(f0)
    mixed = 0
    for n in (1, 2, 3, 5, 7, 10):
        for call in ("step", "reverse", "step_norm"):
            r = a.route(n, call)
            mixed += "split" in r and "march3r" in r
            if call == "step_norm":
                ref, e = s.step_norm(n).tolist(), a.step_norm(n).tolist()
                assert abs(e[0] - ref[0]) <= 1e-13 * max(abs(ref[0]), ref[1]) and abs(e[1] - ref[1]) <= 1e-13 * ref[1], r
            else:
                for lat in lats:
                    getattr(lat, call)(n)
            assert same(s.state(), a.state()) and a.current == 0, r
    assert mixed >= 3
