"""The complex64 V(z) tables are formed on the device: the bits of the host's
records (dirac_coef_from_theta_host) and, for beta and for a complex theta, of
FP64 evaluated and rounded once.  One plane per (V, W) pair: small, large, zero,
negative and equal to the mass (theta 0)."""
import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nz", [1, 15, 300])
@pytest.mark.parametrize("absorb", [False, True])
def test_tables_bitwise_equal_host_records(nz, absorb):
    import paper_1309_3452_amd as P
    g = np.random.default_rng(91)
    special = np.array([0.0, -0.4, 0.4, 1e-12, -3.0, 40.0, 1e6, -1e-6])
    v = [np.concatenate([special, 2.0 * g.standard_normal(nz)])[:nz].copy() for _ in range(2)]
    w = [(-0.3 * (np.arange(nz) % 3)).astype(np.float64) for _ in range(2)]
    dt, m = 0.5, 0.4
    lat = P.Lattice3D(4, 4, nz, dtype=torch.complex64, dt=dt)
    lat.set_potential_z(m, v[0], v[1])
    if absorb:
        lat.set_absorber_z(w[0], w[1])
    lat.step(1)
    torch.cuda.synchronize()
    # the tables lie behind the partials and the 256-byte result area; the scratch
    # ends with them and the adjoint's partial sums
    nbytes = ctypes.c_size_t()
    P._abi.check(P.lib().dirac_scratch_bytes(lat._ctx, ctypes.byref(nbytes)), lat._ctx)
    base = (lat.scratch.data_ptr() + 255) & ~255
    raw = lat.scratch[base - lat.scratch.data_ptr():].cpu().numpy()
    half = (4 * nz * 16 + 255) & ~255
    gpart = (1 * nz * 16 + 255) & ~255
    off = int(nbytes.value) - gpart - 2 * half
    for direction in (0, 1):
        tab = raw[off + direction * half:][:4 * nz * 16].view(np.float32).reshape(4, nz, 4)
        sg = 1.0 if direction == 0 else -1.0
        for q in range(4):
            cls = 0 if q in (0, 3) else 1
            th = sg * (0.5 * dt * ((m if q < 2 else -m) + v[cls]))
            ti = sg * (0.5 * dt * w[cls]) if absorb else np.zeros(nz)
            rec = (ctypes.c_float * (2 * nz))()
            assert P.lib().dirac_coef_from_theta_host(rec, np.ascontiguousarray(th).ctypes.data_as(ctypes.c_void_p), nz) == 0
            rec = np.array(rec, dtype=np.float32).reshape(nz, 2)
            for k in range(nz):
                if ti[k] == 0.0:
                    d = 1.0 + th[k] * th[k]
                    ref = np.array([rec[k, 0], rec[k, 1], 1.0 / d, -th[k] / d], dtype=np.float32)
                else:
                    d = (1.0 - ti[k]) * (1.0 - ti[k]) + th[k] * th[k]
                    ref = np.array([1.0 - (1.0 - ti[k] * ti[k] - th[k] * th[k]) / d, (2.0 * th[k]) / d,
                                    (1.0 - ti[k]) / d, -(th[k] / d)], dtype=np.float32)
                assert np.array_equal(tab[q, k].view(np.int32), ref.view(np.int32)), (direction, q, k, tab[q, k], ref)
