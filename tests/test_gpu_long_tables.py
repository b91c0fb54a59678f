"""V(z) tables of 4 GiB and more (2^25 planes and up in complex128): the default
kernels against the split ones, which index the tables with 64 bits."""
import numpy as np
import pytest
import torch

import workloads

pytestmark = pytest.mark.gpu


def test_default_kernels_read_the_last_planes():
    import paper_1309_3452_amd as P
    nz = (1 << 25) + 8
    print("long tables, 1 x 1 x %d complex128" % nz, flush=True)
    v = np.linspace(0.0, 1.0, nz)
    lat = P.Lattice3D(1, 1, nz, dtype=torch.complex128, dt=workloads.DT3, zero_bc=True)
    lat.set_potential_z(0.4, v, v + 0.1)
    tails = []
    for kernel in ("split", "auto"):
        lat.set_kernel(kernel)
        for t in lat.state():
            t.fill_(1.0 + 0.5j)
        lat.step(2)
        # planes beyond the first 4 GiB of a table's offsets, and what they reach
        tails.append([t[-64:].clone() for t in lat.state()])
        print("  %s done" % kernel, flush=True)
    for a, b in zip(*tails):
        assert torch.equal(torch.view_as_real(a), torch.view_as_real(b))
