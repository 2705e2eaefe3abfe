"""Every field row that is read straight from the populations, against sums of the populations themselves.

The library sums in FP64 and rounds a deviation to the population type before adding its offset, so a value
near 1 is off by at most a few units of 2^-53 (FP64, sums of up to 95 terms below 1) or 2^-24 (FP32).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

E2 = np.array([(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (1, 1, 0), (1, -1, 0), (-1, 1, 0), (-1, -1, 0)])
E3 = np.array([(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (1, -1, 0),
               (-1, 1, 0), (-1, -1, 0), (0, 1, 1), (0, 1, -1), (0, -1, 1), (0, -1, -1), (1, 0, 1), (1, 0, -1),
               (-1, 0, 1), (-1, 0, -1)])


@pytest.mark.parametrize("size", [(3, 3, 1), (65, 13, 1), (3, 4, 3), (33, 7, 5)], ids=lambda s: "%dx%dx%d" % s)
@pytest.mark.parametrize("walls", [0, 1])
@pytest.mark.parametrize("nc", [3, 4, 5])
def test_field_rows(size, walls, nc):
    from paper_1511_02155_amd import tlb

    nx, ny, nz = size
    N = nx * ny * nz
    E = E2 if nz == 1 else E3
    rng = np.random.default_rng(N)
    C = 1.0 / nc + rng.uniform(-0.05, 0.05, (nc, N))
    u = rng.uniform(-0.05, 0.05, (2 if nz == 1 else 3, N))
    for prec, tol in ((tlb.TLB_F64, 200 * 2.0 ** -53), (tlb.TLB_F32, 4 * 2.0 ** -24)):
        s = tlb.Sim(tlb.make_params(0 if nz == 1 else 1, nx, ny, nz, prec=prec, walls_y=walls, kappa=[0.01] * nc))
        s.init_equilibrium(C, u)
        s.step(3)
        p = s.all_populations()
        rho, phi, psi = p[0].sum(0), p[1].sum(0), p[2:].sum(1)
        want = dict(C1=0.5 * (rho + phi - psi.sum(0)), C2=0.5 * (rho - phi - psi.sum(0)), rho=rho, phi=phi, psi=psi[0])
        for m in range(2, nc):
            want["C%d" % (m + 1)] = psi[m - 2]
        for a, name in enumerate(("ux", "uy", "uz")):
            want[name] = (E[:, a, None] * p[0]).sum(0) / rho
        for name, w in want.items():
            assert np.abs(s.field(name) - w).max() <= tol, name
