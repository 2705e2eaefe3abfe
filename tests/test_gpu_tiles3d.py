"""D3Q19 tiles of run-time size (lattices the compiled-in 64 x 4 and 32 x 8 tiles fit badly) against those.

The default launch takes the run-time tiles, a shape set by the caller the compiled-in ones; the kernels are
the same but for the tile's size, and the results are the same bit for bit (tolerance zero).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def torch_first():
    """torch finds the GPU only where it starts before the library does: later test files need it."""
    import torch

    torch.cuda.init()


@pytest.mark.parametrize("size", [(70, 50, 45), (47, 154, 9), (100, 12, 20), (18, 30, 60), (13, 3, 40), (124, 5, 6)],
                         ids=lambda s: "%dx%dx%d" % s)
@pytest.mark.parametrize("walls,nc,mrt", [(0, 3, 0), (1, 3, 1), (1, 4, 0), (0, 5, 1)])
def test_run_time_tiles_equal_compiled_in_ones(size, walls, nc, mrt):
    from paper_1511_02155_amd import tlb

    nx, ny, nz = size
    for prec in (tlb.TLB_F32, tlb.TLB_F64):
        rng = np.random.default_rng(nx)
        C = 1.0 / nc + rng.uniform(-0.05, 0.05, (nc, nx * ny * nz))
        u = rng.uniform(-0.02, 0.02, (3, nx * ny * nz))
        h = rng.uniform(-0.002, 0.002, (2, nc, nx * nz))
        sims = []
        for fixed in (False, True):
            s = tlb.Sim(tlb.make_params(1, nx, ny, nz, prec=prec, walls_y=walls, kappa=[0.01 + 0.005 * m for m in range(nc)],
                                        collision=mrt, tau_f=0.8, tau_g=0.9, tau_k=1.1, tau_bulk=0.8, tau_ghost=1.2,
                                        gamma_phi=0.4, gamma_psi=0.13))
            if walls:
                s.set_wetting_both(h)
            s.init_equilibrium(C, u)
            if fixed:
                s.set_launch(**s.launch())
            s.step(3)
            sims.append(s)
        for k in range(nc):
            assert np.array_equal(sims[0].populations(k), sims[1].populations(k))


@pytest.mark.parametrize("size", [(99, 29, 21), (133, 33, 127), (164, 63, 24), (132, 141, 17), (133, 131, 75)],
                         ids=lambda s: "%dx%dx%d" % s)
@pytest.mark.parametrize("walls,nc,mrt", [(0, 3, 0), (1, 3, 1), (1, 4, 0), (0, 4, 1), (0, 5, 0), (1, 5, 1)])
def test_run_time_tiles_side_by_side(size, walls, nc, mrt):
    """Sizes that take several columns of run-time tiles in both types, so that ring nodes come from a neighbouring
    tile and the last tile of a row is narrower; the largest is stored past the caches."""
    from paper_1511_02155_amd import tlb

    N = size[0] * size[1] * size[2]
    rng = np.random.default_rng(N)
    C = 1.0 / nc + rng.uniform(-0.05, 0.05, (nc, N))
    h = rng.uniform(-0.002, 0.002, (2, nc, size[0] * size[2]))
    for prec in (tlb.TLB_F32, tlb.TLB_F64):
        states = []
        for fixed in (False, True):
            s = tlb.Sim(tlb.make_params(1, *size, prec=prec, walls_y=walls, kappa=[0.01 + 0.005 * m for m in range(nc)],
                                        collision=mrt, tau_f=0.8, tau_g=0.9, tau_k=1.1, tau_bulk=0.8, tau_ghost=1.2,
                                        gamma_phi=0.4, gamma_psi=0.13))
            if walls:
                s.set_wetting_both(h)
            s.init_equilibrium(C)
            if fixed:
                s.set_launch(**s.launch())
            s.step(3)
            states.append(s.save_state()[0])
            s.close()
        assert np.array_equal(*states)
