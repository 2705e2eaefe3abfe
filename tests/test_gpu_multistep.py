"""Launches of several D2Q9 steps (tlb_pair2d.hip, tlb_tile2d.hip) against single steps.

With the default launch shape tlb_step advances D2Q9 lattices two to four steps per launch; with a launch
shape set by the caller every step is a launch of the one-step kernel.  All form every value by the same
operations in the same order, so the results are the same bit for bit (tolerance zero).  The small sizes sit
at the edges of the tiles (8 x 4, 16 x 8, 12 x 8 and 32 x 8 nodes, each the default of one of the sizes), the
large ones at those of the sweeps' strips (58 columns for two steps, 50 for four) and chunks.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def torch_first():
    """torch finds the GPU only where it starts before the library does: later test files need it."""
    import torch

    torch.cuda.init()


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


@pytest.mark.parametrize("size", [(3, 3), (5, 4), (8, 4), (64, 64), (117, 40), (161, 153), (239, 241), (333, 217)],
                         ids=lambda s: "%dx%d" % s)
@pytest.mark.parametrize("walls", [0, 1])
@pytest.mark.parametrize("nc,mrt", [(3, 0), (3, 1), (4, 0), (4, 1), (5, 0), (5, 1)])
def test_launches_of_several_steps_equal_single_steps(size, walls, nc, mrt):
    from paper_1511_02155_amd import tlb

    for prec in (tlb.TLB_F32, tlb.TLB_F64):
        two, one = _pair(tlb, *size, prec, walls, nc, mrt)
        for n in (2, 3, 4, 5):  # every remainder of launches of two and three steps
            two.step(n)
            one.step(n)
            assert np.array_equal(two.all_populations(), one.all_populations())


@pytest.mark.parametrize("size", [(1045, 800), (1501, 1100)], ids=lambda s: "%dx%d" % s)
@pytest.mark.parametrize("walls,nc,mrt", [(0, 3, 0), (1, 3, 0), (1, 3, 1), (1, 4, 0), (0, 4, 1), (1, 5, 1), (0, 5, 0)])
def test_sweeps_of_many_chunks_and_rounds(size, walls, nc, mrt):
    """Chunks of several rows, strips of 57 and 58 columns, more items than the chip holds at once, both sweep
    directions."""
    from paper_1511_02155_amd import tlb

    for prec in (tlb.TLB_F32, tlb.TLB_F64):
        two, one = _pair(tlb, *size, prec, walls, nc, mrt)
        for n in (5, 6, 3):  # launches of four and what they leave over
            two.step(n)
            one.step(n)
            for s in (0, nc - 1):
                assert np.array_equal(two.populations(s), one.populations(s))


@pytest.mark.parametrize("size", [(90, 50), (333, 217), (1045, 800)], ids=lambda s: "%dx%d" % s)
@pytest.mark.parametrize("chain", [2, 4, 6, 8, 10])
def test_captured_chains(chain, size):
    """Chains of an odd or even number of launches, replayed several times with eager work between."""
    from paper_1511_02155_amd import tlb

    two, one = _pair(tlb, *size, tlb.TLB_F64, 1, 3, 0)
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


@pytest.mark.parametrize("walls", [0, 1])
@pytest.mark.parametrize("chain", [0, 4, 6])
def test_batch_two_steps_per_launch(walls, chain):
    """A batch in its default (two steps per launch) against single steps of its domains: strips of one and
    several, chunks of one and several, odd counts (a single step between launches of two), captured chains
    of an odd and an even number of launches, and again after the tuner."""
    from paper_1511_02155_amd import tlb

    sizes = [(3, 3), (5, 70), (58, 9), (59, 31), (116, 64), (117, 200), (256, 33), (64, 256)]
    for prec in (tlb.TLB_F32, tlb.TLB_F64):
        rng = np.random.default_rng(chain + walls)
        ps, sims = [], []
        for d, (nx, ny) in enumerate(sizes):
            ps.append(tlb.make_params(0, nx, ny, prec=prec, walls_y=walls, kappa=rng.uniform(0.005, 0.03, 3), tau_f=0.8,
                                      tau_g=0.9, tau_k=1.1, gamma_phi=0.4, gamma_psi=0.13))
        b = tlb.Batch(ps)
        for d, (nx, ny) in enumerate(sizes):
            s = tlb.Sim(ps[d])
            s.set_launch(**s.launch())
            C = 1.0 / 3.0 + rng.uniform(-0.05, 0.05, (3, nx * ny))
            u = rng.uniform(-0.02, 0.02, (2, nx * ny))
            if walls:
                h = rng.uniform(-0.001, 0.001, (2, 3, nx))
                s.set_wetting_both(h)
                for w in (0, 1):
                    b.set_wetting(d, w, h[w])
            s.init_equilibrium(C, u)
            b.init_equilibrium(d, C, u)
            sims.append(s)
        if chain:
            b.set_graph(chain)
        for n in (1, 2, 3, 2 * chain + 5, 4 * chain + 2):
            b.step(n)
            for d, s in enumerate(sims):
                s.step(n)
                assert np.array_equal(b.all_populations(d), s.all_populations())
        b.autotune(2)
        b.step(2 * chain + 3)
        for d, s in enumerate(sims):
            s.step(2 * chain + 3)
            assert np.array_equal(b.all_populations(d), s.all_populations())


def _replays(torch, tlb, stream, step, runs):
    """Record step(n) for each n of runs (an even sum) on the stream; replay the graphs in turn."""
    graphs = []
    for n in runs:
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            step(n)
        graphs.append(g)
    for _ in range(3):
        with torch.cuda.stream(stream):
            for g in graphs:
                g.replay()
        torch.cuda.synchronize()


@pytest.mark.parametrize("runs", [(2,), (4,), (6,), (10,), (1, 3), (5, 3)], ids=str)
@pytest.mark.parametrize("size", [(64, 64), (333, 217), (1045, 800)], ids=lambda s: "%dx%d" % s)
def test_runs_recorded_by_the_caller(size, runs):
    """Steps captured into a caller's graph, replayed several times: a run swaps the state's buffers as often as
    single steps would (modulo two), so that each replay goes on from where the last one ended."""
    import torch

    from paper_1511_02155_amd import tlb

    nx, ny = size
    C = 1.0 / 3.0 + np.random.default_rng(nx).uniform(-0.05, 0.05, (3, nx * ny))
    for prec in (tlb.TLB_F32, tlb.TLB_F64):
        stream = torch.cuda.Stream()
        p = tlb.make_params(0, nx, ny, prec=prec)
        a, b, s = tlb.Sim(p, stream=stream.cuda_stream), tlb.Batch([p, p], stream=stream.cuda_stream), tlb.Sim(p)
        s.set_launch(**s.launch())
        a.init_equilibrium(C)
        s.init_equilibrium(C)
        for d in (0, 1):
            b.init_equilibrium(d, C)
        _replays(torch, tlb, stream, a.step, runs)
        _replays(torch, tlb, stream, b.step, runs)
        s.step(3 * sum(runs))
        want = s.all_populations()
        assert np.array_equal(a.all_populations(), want)
        assert np.array_equal(b.all_populations(1), want)


@pytest.mark.parametrize("sizes", [[(300, 500)], [(700, 300), (40, 40)], [(200, 300)] * 9], ids=["one", "two", "nine"])
def test_batch_of_few_large_domains(sizes):
    """Two-step launches of domains that are dealt out in pieces, against single steps of each (tolerance zero)."""
    from paper_1511_02155_amd import tlb

    ps = [tlb.make_params(0, nx, ny, prec=tlb.TLB_F32, walls_y=1) for nx, ny in sizes]
    b, sims = tlb.Batch(ps), [tlb.Sim(p) for p in ps]
    for d, (nx, ny) in enumerate(sizes):
        C = 1.0 / 3.0 + np.random.default_rng(d).uniform(-0.05, 0.05, (3, nx * ny))
        b.init_equilibrium(d, C)
        sims[d].set_launch(**sims[d].launch())
        sims[d].init_equilibrium(C)
    b.step(4)
    for d, s in enumerate(sims):
        s.step(4)
        assert np.array_equal(b.all_populations(d), s.all_populations())


def test_tuner_cache_keeps_its_choice(tmp_path, monkeypatch):
    """A tuner's file names the single-step shape, and in a last word that two steps per launch were faster; results
    after a lookup are those of the tuned batch, with and without that word (tolerance zero)."""
    from paper_1511_02155_amd import tlb

    path = tmp_path / "tune.txt"
    monkeypatch.setenv("TLB_TUNE_CACHE", str(path))
    ps = [tlb.make_params(0, 64, 64, prec=tlb.TLB_F64) for _ in range(3)]
    C = 1.0 / 3.0 + np.random.default_rng(2).uniform(-0.05, 0.05, (3, 64 * 64))
    out = []
    for turn in range(3):
        if turn == 2:
            path.write_text(path.read_text().replace(" two", ""))
        b = tlb.Batch(ps)
        for d in range(3):
            b.init_equilibrium(d, C)
        shape = b.autotune(2)
        b.step(5)
        out.append((shape, b.all_populations(2)))
    for shape, pop in out[1:]:
        assert shape == out[0][0] and np.array_equal(pop, out[0][1])
