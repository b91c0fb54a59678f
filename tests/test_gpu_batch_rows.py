"""Batches of a few very long rows: the march that the estimate picks there, graphs and
changing and repeated step counts included (an odd number of launches alternates
between the buffer sets, each with its captured graph), bit for bit the split kernels on each lattice."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("graph", [False, True])
def test_long_rows_bitwise_equal_split(dtype, graph):
    import paper_1309_3452_amd as P
    print("batch rows graph=%s %s" % (graph, dtype), flush=True)
    g = torch.Generator(device="cuda").manual_seed(62)
    rnd = lambda ny, nx, dt: torch.randn((ny, nx), generator=g, device="cuda", dtype=dt)
    lats = [dict(nx=20000 + 2 * b, ny=1 + b % 2, m=0.1, v_site=[rnd(1 + b % 2, 20000 + 2 * b, torch.float64) for _ in range(4)],
                 state=[rnd(1 + b % 2, 20000 + 2 * b, dtype) for _ in range(4)]) for b in range(30)]
    batch = P.BatchedLattices(lats, dtype=dtype, dt=workloads.DT2)
    total, routes = 0, set()
    for n in (1, 3, 3, 3, 3, 12, 2, 1, 1, 1):
        r = batch.route(n)
        routes.add("tile2" if "tile2" in r else "march")
        batch.run(n, mode=1, graph=graph)
        total += n
    assert "march" in routes, routes
    for b, L in enumerate(lats):
        solo = P.Lattice((L["nx"], L["ny"]), dtype=dtype, dt=workloads.DT2)
        solo.set_kernel("split")
        solo.load(L["state"])
        solo.set_coef_records(batch.theta[b])
        solo.step(total)
        for x, y in zip(solo.state(), batch.state(b)):
            assert torch.equal(torch.view_as_real(x), torch.view_as_real(y)), b
