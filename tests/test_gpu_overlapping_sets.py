"""Buffer sets that overlap without being the same arrays: steps with zero values
outside, reversed steps and adjoints run in place then, as they do where the sets
are the same (bit for bit the split kernels' results)."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


def overlapping(P, shape, shift, **kw):
    """A lattice whose second set lies `shift` cells behind the first."""
    lat = P.Lattice(shape, **kw)
    n = lat.bufs[0][0].numel()
    mem = [torch.zeros(n + shift, dtype=lat.dtype, device="cuda") for _ in range(lat.narr)]
    lat.bufs = [[t[o:o + n].view(lat.tshape) for t in mem] for o in (0, shift)]
    p = [P._abi.ptr_array([t.data_ptr() for t in b]) for b in lat.bufs]
    assert P.lib().dirac_bind_state(lat._ctx, p[0], p[1]) == 0
    return lat


@pytest.mark.parametrize("dtype", [torch.complex64, torch.complex128])
@pytest.mark.parametrize("shape", [(70, 40), (20, 9, 12)])
def test_zero_boundary_steps_in_place(dtype, shape):
    import paper_1309_3452_amd as P
    print("overlapping sets %s %s" % (shape, dtype), flush=True)
    g = np.random.default_rng(61)
    kw = dict(dtype=dtype, dt=workloads.DT3, zero_bc=True)
    ref, lat = P.Lattice(shape, **kw), overlapping(P, shape, 2 * shape[0], **kw)
    ref.set_kernel("split")
    f0 = [torch.from_numpy(g.standard_normal(ref.tshape) + 1j * g.standard_normal(ref.tshape)) for _ in range(ref.narr)]
    for q in (ref, lat):
        q.set_potential_z(0.4)
        q.load(f0)
        q.step(6)
        q.reverse(3)
    assert lat.current == 0
    for a, b in zip(ref.state(), lat.state()):
        assert torch.equal(torch.view_as_real(a), torch.view_as_real(b))
