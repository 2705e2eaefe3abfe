"""Two-step launches of the D2Q9 step (tlb_pair2d.hip) against single steps.

With the default launch shape tlb_step advances D2Q9 lattices two steps per launch; with a launch shape
set by the caller every step is a launch of the one-step kernel.  Both form every value by the same
operations in the same order, so the results are the same bit for bit (tolerance zero).  Sizes sit at the
edges of the two-step kernel's strips (58 columns) and chunks, with the smallest lattices and odd ones,
with and without walls, in both directions of the sweep.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _pair(tlb, nx, ny, prec, walls, nc, mrt):
    rng = np.random.default_rng(nx * 1000 + ny)
    C = 1.0 / nc + rng.uniform(-0.05, 0.05, (nc, nx * ny))
    u = rng.uniform(-0.02, 0.02, (2, nx * ny))
    h = rng.uniform(-0.002, 0.002, (2, nc, nx))
    sims = []
    for single in (False, True):
        s = tlb.Sim(tlb.make_params(0, nx, ny, prec=prec, walls_y=walls, kappa=[0.01 + 0.005 * m for m in range(nc)],
                                    collision=mrt, tau_f=0.8, tau_g=0.9, tau_k=1.1, tau_bulk=0.8, tau_ghost=1.2,
                                    gamma_phi=0.4, gamma_psi=0.13))
        if walls:
            s.set_wetting_both(h)
        s.init_equilibrium(C, u)
        if single:
            s.set_launch(**s.launch())
        sims.append(s)
    return sims


@pytest.mark.parametrize("size", [(3, 3), (5, 4), (58, 7), (59, 31), (64, 64), (117, 40), (700, 9), (61, 300)],
                         ids=lambda s: "%dx%d" % s)
@pytest.mark.parametrize("walls", [0, 1])
@pytest.mark.parametrize("nc,mrt", [(3, 0), (3, 1), (4, 0), (4, 1)])
def test_two_step_launches_equal_single_steps(size, walls, nc, mrt):
    from paper_1511_02155_amd import tlb

    for prec in (tlb.TLB_F32, tlb.TLB_F64):
        two, one = _pair(tlb, *size, prec, walls, nc, mrt)
        for n in (2, 4, 3):  # the odd count ends with a single step
            two.step(n)
            one.step(n)
            assert np.array_equal(two.all_populations(), one.all_populations())


def test_many_chunks_and_rounds():
    """More items than the chip holds at once, chunks of several rows, both sweep directions."""
    from paper_1511_02155_amd import tlb

    for prec in (tlb.TLB_F32, tlb.TLB_F64):
        two, one = _pair(tlb, 1500, 1100, prec, 1, 3, 0)
        two.step(5)
        one.step(5)
        assert np.array_equal(two.populations(0), one.populations(0))
        assert np.array_equal(two.populations(2), one.populations(2))


@pytest.mark.parametrize("chain", [2, 6, 8])
def test_captured_chains(chain):
    """Chains whose pairs are odd or even in number, replayed several times with eager work between."""
    from paper_1511_02155_amd import tlb

    two, one = _pair(tlb, 90, 50, tlb.TLB_F64, 1, 3, 0)
    two.set_graph(chain)
    for n in (chain, 3 * chain + 1, chain + 5, 2 * chain):
        two.step(n)
        one.step(n)
        assert np.array_equal(two.all_populations(), one.all_populations())
        assert np.array_equal(two.field("C2"), one.field("C2"))


def test_checks_between_odd_counts():
    from paper_1511_02155_amd import tlb

    two, one = _pair(tlb, 70, 33, tlb.TLB_F32, 0, 3, 0)
    two.set_check_every(3)
    two.step(11)
    one.step(11)
    assert np.array_equal(two.all_populations(), one.all_populations())
