"""The adjoint's backward steps as one launch each against the in-place sweeps:
state and lam bit for bit (the same expressions), the gradient to the reordering of
its FP64 sums (1e-13 of its largest component: at most ~1e5 terms per plane, whose
random signs keep the sum of their moduli within ~300 of the result).  Odd and even
step counts, ragged tiles, few planes; sizes from where the march is taken up."""
import ctypes

import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


def same(a, b):
    return all(torch.equal(torch.view_as_real(x), torch.view_as_real(y)) for x, y in zip(a, b))


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("shape,steps", [((62, 96, 95), 4), ((57, 101, 133), 5), ((180, 150, 96), 3),
                                         ((260, 130, 141), 2), ((500, 300, 2), 4), ((700, 400, 3), 3)])
def test_march_equals_sweeps(dtype, shape, steps):
    import paper_1309_3452_amd as P
    print("adjoint march %s n=%d %s" % (shape, steps, dtype), flush=True)
    nx, ny, nz = shape
    g = np.random.default_rng(95)
    rnd = lambda: [torch.from_numpy(g.standard_normal((nz, ny, nx)) + 1j * g.standard_normal((nz, ny, nx))) for _ in range(8)]
    f0, l0 = rnd(), rnd()
    vi, vh = g.standard_normal(nz), g.standard_normal(nz)
    out = []
    for march in (False, True):
        lat = P.Lattice3D(nx, ny, nz, dtype=dtype, dt=workloads.DT3)
        lat.set_potential_z(0.4, vi, vh)
        lat.load(f0)
        lam = [t.to(device="cuda", dtype=dtype) for t in l0]
        work = [torch.empty_like(t) for t in lam] if march else None
        dvi, dvh = lat.adjoint_vz(steps, lam, work)
        torch.cuda.synchronize()
        assert lat.current == 0
        out.append((lat.state(), lam, torch.cat([dvi, dvh])))
    (s0, a0, d0), (s1, a1, d1) = out
    assert same(s0, s1) and same(a0, a1)
    assert float((d0 - d1).abs().max()) <= 1e-13 * float(d0.abs().max())


def test_work_arrays_are_checked():
    import paper_1309_3452_amd as P
    lat = P.Lattice3D(8, 8, 8, dtype=torch.complex64, dt=0.5)
    lam = [torch.zeros_like(t) for t in lat.state()]
    p = P._abi.ptr_array([t.data_ptr() for t in lam])
    d = torch.zeros(8, dtype=torch.float64, device="cuda")
    f = lambda w: P.lib().dirac_adjoint_vz_work(lat._ctx, 1, p, w, ctypes.c_void_p(d.data_ptr()),
                                                ctypes.c_void_p(d.data_ptr()), None)
    assert f(p) == -1
    assert f(P._abi.ptr_array([t.data_ptr() for t in lat.bufs[1]])) == -1
