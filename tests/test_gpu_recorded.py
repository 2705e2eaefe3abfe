"""Live runs between replays of work that a caller recorded into a graph of its own.

A recorded launch holds the addresses of the buffers it was recorded with, so a live run of an even number of steps
between two replays has to leave the state in the buffer where it found it, whatever number of steps its launches
take.  Everything is compared with single steps (a launch shape set by the caller) bit for bit (tolerance zero).  The
sizes are stepped in tiles, in sweeps of two steps and (FP64) in sweeps of four.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SIZES = [(64, 64), (512, 512), (1045, 800)]


@pytest.fixture(scope="module")
def torch():
    import torch

    torch.cuda.init()
    return torch


def _sims(torch, tlb, nx, ny, prec):
    """A simulation in its default launch on a stream of torch's, one that takes single steps, and their input."""
    C = 1.0 / 3.0 + np.random.default_rng(nx).uniform(-0.05, 0.05, (3, nx * ny))
    stream = torch.cuda.Stream()
    p = tlb.make_params(0, nx, ny, prec=prec)
    a, s = tlb.Sim(p, stream=stream.cuda_stream), tlb.Sim(p)
    s.set_launch(**s.launch())
    for x in (a, s):
        x.init_equilibrium(C)
    return stream, a, s, C


def _record(torch, stream, work):
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        work()
    return g


def _replay(torch, stream, g):
    with torch.cuda.stream(stream):
        g.replay()
    torch.cuda.synchronize()


@pytest.mark.parametrize("size", SIZES, ids=lambda s: "%dx%d" % s)
@pytest.mark.parametrize("prec", [0, 1], ids=["f32", "f64"])
def test_live_runs_between_replays_of_recorded_steps(torch, size, prec):
    from paper_1511_02155_amd import tlb

    stream, a, s, _ = _sims(torch, tlb, *size, prec)
    graphs = [(n, _record(torch, stream, lambda: a.step(n))) for n in (2, 4)]
    for live in ((), (2,), (4,), (6,), (10,), (1, 3), (5, 1)):
        for n in live:
            a.step(n)
            s.step(n)
        for n, g in graphs:
            _replay(torch, stream, g)
            s.step(n)
        assert np.array_equal(a.field("C2"), s.field("C2")), live
        assert np.array_equal(a.all_populations(), s.all_populations()), live


@pytest.mark.parametrize("chain", [0, 6, 8])
@pytest.mark.parametrize("prec", [0, 1], ids=["f32", "f64"])
def test_live_runs_between_replays_of_recorded_batch_steps(torch, prec, chain):
    """Also odd runs, whose single steps take items from queues that a replay has to find full, and the batch's own
    chains of launches, which start from buffer 0."""
    from paper_1511_02155_amd import tlb

    stream = torch.cuda.Stream()
    ps = [tlb.make_params(0, nx, ny, prec=prec) for nx, ny in ((40, 30), (130, 75), (64, 64))]
    b, sims = tlb.Batch(ps, stream=stream.cuda_stream), [tlb.Sim(p) for p in ps]
    for d, s in enumerate(sims):
        C = 1.0 / 3.0 + np.random.default_rng(d).uniform(-0.05, 0.05, (3, s.N))
        b.init_equilibrium(d, C)
        s.set_launch(**s.launch())
        s.init_equilibrium(C)
    b.set_graph(chain)
    graphs = [(n, _record(torch, stream, lambda: b.step(n))) for n in (2, 4)]
    for live in ((), (2,), (4,), (6,), (3, 1), (10,), (1, 17), (5, 3, 2), (24,)):
        for n in live:
            b.step(n)
        for n, g in graphs:
            _replay(torch, stream, g)
        for d, s in enumerate(sims):
            s.step(sum(live) + 6)
            assert np.array_equal(b.all_populations(d), s.all_populations()), (live, d)


@pytest.mark.parametrize("size", SIZES, ids=lambda s: "%dx%d" % s)
def test_live_runs_between_replays_of_recorded_readouts(torch, size):
    """The state's buffers are also in the graph of a readout, a copy out of or into the state, or an
    initialisation, whether or not any step was recorded."""
    from paper_1511_02155_amd import tlb

    nx, ny = size
    for what in ("field", "populations", "save", "load", "set", "init"):
        stream, a, s, C = _sims(torch, tlb, nx, ny, 1)
        n = dict(field=nx * ny, populations=9 * nx * ny, set=9 * nx * ny, init=3 * nx * ny).get(what, 27 * nx * ny)
        t = torch.empty(n, dtype=torch.float64, device="cuda")
        if what == "init":
            t.copy_(torch.as_tensor(C).reshape(-1))
        else:
            tlb.check(tlb.tlb_save_state_dev(a.handle, t.data_ptr()) if what == "load" else
                      tlb.tlb_get_populations_dev(a.handle, 1, t.data_ptr()) if what != "field" else 0)
            a.synchronize()
        start = t.cpu().numpy().copy()
        call = dict(field=lambda: tlb.tlb_get_field_dev(a.handle, 1, t.data_ptr()),
                    populations=lambda: tlb.tlb_get_populations_dev(a.handle, 1, t.data_ptr()),
                    save=lambda: tlb.tlb_save_state_dev(a.handle, t.data_ptr()),
                    load=lambda: tlb.tlb_load_state_dev(a.handle, t.data_ptr(), 0),
                    set=lambda: tlb.tlb_set_populations_dev(a.handle, 1, t.data_ptr()),
                    init=lambda: tlb.tlb_init_equilibrium_dev(a.handle, t.data_ptr(), None))[what]
        torch.cuda.synchronize()
        g = _record(torch, stream, lambda: tlb.check(call()))
        for n in (2, 4, 10):
            a.step(n)
            s.step(n)
            _replay(torch, stream, g)
            got = t.cpu().numpy()
            if what == "field":
                assert np.array_equal(got, s.field("C2")), n
            elif what == "populations":
                assert np.array_equal(got, s.populations(1).reshape(-1)), n
            elif what == "save":
                assert np.array_equal(got.view(np.uint8), s.save_state()[0]), n
            elif what == "set":
                assert np.array_equal(a.populations(1).reshape(-1), start), n
                s.set_populations(1, start)
            else:  # back at the initial state
                s.init_equilibrium(C)
                assert np.array_equal(a.all_populations(), s.all_populations()), (what, n)
