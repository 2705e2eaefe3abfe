"""Every field row that is read straight from the populations, against sums of the populations themselves.

The library sums in FP64 and rounds a deviation to the population type before adding its offset, so a value
near 1 is off by at most a few units of 2^-53 (FP64, sums of up to 95 terms below 1) or 2^-24 (FP32).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def torch_first():
    """torch finds the GPU only where it starts before the library does: later test files need it."""
    import torch

    torch.cuda.init()

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


def test_batch_fields_read_many_times():
    """The first fields of a batch come through device memory, later ones through pinned host memory: both are the
    single lattice's bit for bit (tolerance zero), also after further steps and between domains of unlike size."""
    from paper_1511_02155_amd import tlb

    sizes = [(3, 3), (65, 13), (130, 70)]
    for prec in (tlb.TLB_F64, tlb.TLB_F32):
        ps = [tlb.make_params(0, nx, ny, prec=prec, walls_y=1) for nx, ny in sizes]
        b = tlb.Batch(ps)
        sims = [tlb.Sim(p) for p in ps]
        for d, (nx, ny) in enumerate(sizes):
            C = 1.0 / 3 + np.random.default_rng(d).uniform(-0.05, 0.05, (3, nx * ny))
            b.init_equilibrium(d, C)
            sims[d].init_equilibrium(C)
        for turn in range(3):  # 30 fields a turn
            b.step(2)
            for s in sims:
                s.step(2)
            for name in tlb.FIELDS:
                for d, s in enumerate(sims):
                    assert np.array_equal(b.field(d, name), s.field(name)), (turn, name, d)
