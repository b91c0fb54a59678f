"""The one-launch backward step of the adjoint where it surely runs (the work arrays
come back written) against the in-place sweeps: few planes, single and ragged
tiles, both widths, both precisions.  State and lam bit for bit (the same
expressions).  The gradient of a plane sums the same FP64 terms in another order:
fewer than a thousand additions in a row, so 1000 x 2^-53 = 1e-13 of the sum of their
moduli bounds the difference, and that sum is at most steps x 8 arrays x |lam| |psi|
of a plane (a term is dt times a product of one value of each, coefficients near one)."""
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


def same(a, b):
    return all(torch.equal(torch.view_as_real(x), torch.view_as_real(y)) for x, y in zip(a, b))


C64, C128 = torch.complex64, torch.complex128


@pytest.mark.parametrize("dtype,shape,steps", [
    (C64, (5600, 1400, 1), 2), (C64, (1500, 900, 2), 3), (C64, (1003, 805, 3), 4), (C64, (61, 333, 90), 3),
    (C64, (62, 1301, 33), 2), (C64, (123, 650, 40), 5), (C64, (112, 98, 120), 4), (C64, (620, 141, 50), 2),
    (C128, (2800, 1536, 1), 2), (C128, (1003, 805, 2), 3), (C128, (1003, 805, 3), 4), (C128, (61, 333, 90), 3),
    (C128, (62, 700, 70), 2), (C128, (57, 101, 133), 5), (C128, (112, 98, 120), 4)])
def test_march_runs_and_equals_sweeps(dtype, shape, steps):
    import paper_1309_3452_amd as P
    print("adjoint march %s n=%d %s" % (shape, steps, dtype), flush=True)
    nz, tshape = shape[2], tuple(reversed(shape))
    g = torch.Generator(device="cuda").manual_seed(96)
    f0, l0 = ([torch.randn(tshape, generator=g, device="cuda", dtype=dtype) for _ in range(8)] for _ in range(2))
    vi, vh = (torch.randn(nz, generator=g, device="cuda").double().cpu().numpy() for _ in range(2))
    out = []
    for march in (False, True):
        lat = P.Lattice(shape, dtype=dtype, dt=workloads.DT3)
        lat.set_potential_z(0.4, vi, vh)
        lat.load(f0)
        lam = [t.clone() for t in l0]
        work = [torch.full_like(t, complex("nan")) for t in lam] if march else None
        dvi, dvh = lat.adjoint_vz(steps, lam, work)
        assert lat.current == 0
        if march:
            assert not any(bool(torch.isnan(torch.view_as_real(t)).any()) for t in work), "the sweeps ran"
        out.append((lat.state(), lam, torch.cat([dvi, dvh])))
        del lat, work
    (s0, a0, d0), (s1, a1, d1) = out
    assert same(s0, s1) and same(a0, a1)
    moduli = 8 * steps * max(float(torch.linalg.vector_norm(l)) * float(torch.linalg.vector_norm(f))
                             for l, f in zip(l0, f0)) / nz
    assert float((d0 - d1).abs().max()) <= 1e-13 * moduli
