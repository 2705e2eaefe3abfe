"""Host code of the library over a stand-in HIP runtime (standin.py): which kernels a call launches with which
buffers, and what a call that fails leaves behind.  Nothing is computed."""
import pytest

import standin


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    folder = tmp_path_factory.mktemp("standin")
    return lambda body, **env: standin.run(folder, body, env)


def test_a_failed_launch_leaves_the_state_in_its_buffer(run):
    """Of every kind of launch: the next step reads the buffer that the last successful one wrote."""
    run("""
for size, prec, n in (((64, 64, 1), 1, 3), ((512, 512, 1), 0, 2), ((1045, 800, 1), 1, 4), ((64, 64, 1), 1, 1), ((20, 13, 9), 0, 1)):
    s = tlb.Sim(tlb.make_params(int(size[2] > 1), *size, prec=prec))
    s.init_equilibrium(np.zeros((3, s.N)))
    s.step(n)
    wrote = buffers()[-1][1]
    hip.standin_fail_launch(0)
    assert tlb.tlb_step(s.handle, n) == tlb.TLB_EHIP
    assert buffers() == []
    s.step(n)
    assert buffers()[0][0] == wrote, (size, n)
""")


def test_a_batch_shape_that_cannot_be_set_leaves_the_batch_as_it_was(run):
    """Also in two-step launches, with its own chains of them."""
    run("""
ps = [tlb.make_params(0, nx, ny) for nx, ny in ((40, 30), (130, 75))]
b = tlb.Batch(ps)
for d in (0, 1):
    b.init_equilibrium(d, np.zeros((3, ps[d].nx * ps[d].ny)))
shape = b.launch()
for chain in (0, 6):
    b.set_graph(chain)
    kernels()
    b.step(12)
    before = kernels()
    assert len(before) == 6 and all(k.startswith("k_batch_pair2d") for k in before), before
    for after in (0, 1):
        hip.standin_fail_malloc(after)
        rc = tlb.tlb_batch_set_launch(b.handle, ctypes.byref(tlb.tlb_launch(64, 2, 8, 0)))
        hip.standin_fail_malloc(-1)
        if rc == 0:  # no allocation left to fail
            break
        assert rc == tlb.TLB_ENOMEM and b.launch() == shape
        kernels()
        b.step(12)
        assert kernels() == before
    b.close()
    b = tlb.Batch(ps)
    for d in (0, 1):
        b.init_equilibrium(d, np.zeros((3, ps[d].nx * ps[d].ny)))
""")


def test_tuner_file_says_whether_two_steps_share_a_launch(run, tmp_path):
    """Lines of both words are taken as they are; one without a word (written before two-step launches were timed)
    keeps its shape, has the two ways timed, and is followed by a line that says which was faster."""
    out = run("""
def tuned(text=None):
    if text is not None:
        open(path, "w").write(text)
    b = tlb.Batch([tlb.make_params(0, nx, ny) for nx, ny in ((40, 30), (130, 75))])
    for d in (0, 1):
        b.init_equilibrium(d, np.zeros((3, b._N(d))))
    b.step(1)  # the state is in buffer 1
    kernels()
    shape = b.autotune(2)
    timed = len(kernels())
    b.step(4)
    used = {k.split("<")[0] for k in kernels()}
    return shape, timed, used, open(path).read().splitlines()

import os
path = os.environ["TLB_TUNE_CACHE"]
hip.standin_cost(b"k_batch2d", 1.0)
for pair_ms, word, kernel in ((1.0, "two", "k_batch_pair2d"), (3.0, "one", "k_batch2d")):
    hip.standin_cost(b"k_batch_pair2d", pair_ms)
    shape, timed, used, lines = tuned("")
    assert timed > 0 and used == {kernel} and len(lines) == 1 and lines[0].endswith(" " + word), (used, lines)
    bare = lines[0].rsplit(" ", 1)[0]
    for w, k in (("two", "k_batch_pair2d"), ("one", "k_batch2d")):
        assert tuned(bare + " " + w + chr(10)) == (shape, 0, {k}, [bare + " " + w])
    old = tuned(bare + chr(10))
    assert old[0] == shape and 0 < old[1] < 60 and old[2] == {kernel} and old[3] == [bare, bare + " " + word], old
    assert tuned()[1:] == (0, {kernel}, [bare, bare + " " + word])
""", TLB_TUNE_CACHE=str(tmp_path / "tune.txt"))
    assert out == ""


def test_tiles_of_small_and_narrow_3d_lattices(run):
    """The default tile: 32 x 8 for at most 32 columns, 64 x 4 where the chip holds all its one-plane items at once,
    and of run-time size (0 x 0 in the kernel's name) where these fit badly, in one column of tiles and in several,
    the last of them narrower."""
    run("""
tiles = {(3, 3, 3): (32, 8), (5, 8, 4): (32, 8), (20, 20, 20): (32, 8), (32, 5, 90): (32, 8), (18, 62, 48): (32, 8),
         (236, 4, 3): (64, 4), (98, 14, 11): (64, 4), (33, 9, 4): (64, 4),
         (70, 50, 45): (0, 0), (99, 29, 21): (0, 0), (133, 33, 127): (0, 0), (164, 63, 24): (0, 0), (132, 141, 17): (0, 0)}
for size, tile in tiles.items():
    for prec in (tlb.TLB_F32, tlb.TLB_F64):
        s = tlb.Sim(tlb.make_params(1, *size, prec=prec))
        s.init_equilibrium(np.zeros((3, s.N)))
        kernels()
        s.step(1)
        name, = kernels()
        assert name.startswith("k_step3d<%s, %d, %d, " % (("float", "double")[prec], *tile)), (size, prec, name)
        s.close()
""")


def test_single_steps_of_five_fp32_components(run):
    """Lattices whose one-row items fill the chip once are stepped singly, smaller, larger and very wide ones in tiles."""
    run("""
for size, kernel in (((400, 60), "k_tile2d"), ((1229, 45), "k_step2d"), ((1398, 38), "k_step2d"), ((1496, 41), "k_step2d"),
                     ((2000, 28), "k_step2d"), ((4073, 15), "k_tile2d"), ((1219, 52), "k_tile2d")):
    s = tlb.Sim(tlb.make_params(0, *size, prec=tlb.TLB_F32, kappa=[0.01] * 5))
    s.init_equilibrium(np.zeros((5, s.N)))
    kernels()
    s.step(4)
    assert {k.split("<")[0] for k in kernels()} == {kernel}, size
""")


def test_creation_of_a_large_batch(run):
    """Choosing the items of the two-step launches takes no longer than a few times what laying out the single-step
    ones does (both grow with the batch's nodes), and finds the same items as dealing out every candidate."""
    run("""
import time
n = 256
ps = (tlb.tlb_params * n)(*[tlb.make_params(0, 1024, 1024, prec=tlb.TLB_F32)] * n)
create, shape = [], []
for _ in range(3):
    h = ctypes.c_void_p()
    t0 = time.perf_counter()
    tlb.check(tlb.tlb_batch_create(ps, n, None, ctypes.byref(h)))
    t1 = time.perf_counter()
    tlb.check(tlb.tlb_batch_set_launch(h, ctypes.byref(tlb.tlb_launch(64, 1, 16, 0))))
    t2 = time.perf_counter()
    create.append(t1 - t0)
    shape.append(t2 - t1)
    tlb.tlb_batch_destroy(h)
assert min(create) < 10 * min(shape), (create, shape)

# the choice by its definition: the rows that end first when every queue's items are dealt in order to its slots
import heapq
import random


def grid(sizes):
    best = None
    order = sorted(range(len(sizes)), key=lambda d: -sizes[d][0] * sizes[d][1])
    for target in (2, 4, 6, 8, 12, 16, 20, 24, 28, 32, 36, 40, 48, 56, 64, 80, 96, 128, 192, 256):
        rows = [-(-ny // max(1, (ny + target // 2) // target)) for _, ny in sizes]
        chunks = [-(-ny // r) for (_, ny), r in zip(sizes, rows)]
        work = [-(-nx // 58) * c * (r + 7) for (nx, _), c, r in zip(sizes, chunks, rows)]
        total, load, items = sum(work), [0] * 8, [[] for _ in range(8)]
        for d in order:
            ntx, c = -(-sizes[d][0] // 58), chunks[d]
            pieces = min(c, -(-work[d] * 16 // total))
            for j in range(pieces):
                i0, i1 = c * j // pieces, c * (j + 1) // pieces
                k = load.index(min(load))
                load[k] += ntx * (i1 - i0) * (rows[d] + 7)
                items[k] += [min(rows[d], sizes[d][1] - i * rows[d]) + 7 for i in range(i0, i1) for _ in range(ntx)]
        end = 0
        for q in items:
            free = []
            for t in q:
                at = heapq.heappop(free) if len(free) >= 4 * 256 // 8 else 0
                heapq.heappush(free, at + t)
                end = max(end, at + t)
        if best is None or end < best[0]:
            best = end, 8 * max(map(len, items))
    return best[1]


R = random.Random(3)
for n, lo, hi in ((1, 300, 900), (2, 900, 1100), (5, 3, 700), (40, 20, 60), (120, 30, 300), (300, 3, 100), (60, 100, 400)):
    sizes = [(R.randint(lo, hi), R.randint(lo, hi)) for _ in range(n)]
    b = tlb.Batch([tlb.make_params(0, *s) for s in sizes])
    b.init_equilibrium(0, np.zeros((3, sizes[0][0] * sizes[0][1])))
    hip.standin_clear()
    b.step(2)
    assert hip.standin_grid(0) == grid(sizes), (n, lo, hi)
""")


def test_the_default_launch_can_be_asked_for_again(run):
    """A shape set by the caller is used for every step; the default's width, height and variant without a chunk is the
    default, with several D2Q9 steps to a launch and run-time D3Q19 tiles; a captured chain is dropped each time."""
    run("""
for size, prec in (((1045, 800, 1), 1), ((512, 512, 1), 0), ((64, 64, 1), 1), ((70, 50, 45), 1)):
    s = tlb.Sim(tlb.make_params(int(size[2] > 1), *size, prec=prec))
    s.init_equilibrium(np.zeros((3, s.N)))
    shape = s.launch()
    for graph in (0, 4):
        s.set_graph(graph)
        kernels()
        s.step(4)
        default = kernels()
        s.set_launch(**shape)
        s.step(4)
        fixed = kernels()
        assert len(fixed) == 4 and set(fixed) != set(default), (size, graph, fixed, default)
        s.set_launch(**dict(shape, chunk=0))
        s.step(4)
        assert kernels() == default and s.launch() == shape, (size, graph)
    s.set_launch(**dict(shape, chunk=0, variant=0 if shape["variant"] else 1))
    s.step(4)
    assert len(kernels()) == 4, size
    s.close()
""")


def test_a_default_chunk_leaves_the_reverse_launch_alone(run):
    run("""
s = tlb.Sim(tlb.make_params(0, 300, 190))
s.set_adjoint_launch(width=128, chunk=7, variant=1, rows=2)
mine = s.adjoint_launch()
s.set_launch(width=64, chunk=0, variant=0)
assert s.adjoint_launch() == mine
""")


def test_a_chain_that_cannot_be_recorded_leaves_the_state_in_its_buffer(run):
    run("""
for size, lattice in (((1045, 800, 1), 0), ((20, 13, 9), 1)):
    s = tlb.Sim(tlb.make_params(lattice, *size))
    s.init_equilibrium(np.zeros((3, s.N)))
    s.step(1)
    s.step(1)
    holds = buffers()[-1][1]
    s.set_graph(4)
    hip.standin_fail_launch(1)
    assert tlb.tlb_step(s.handle, 8) == tlb.TLB_EHIP
    assert len(kernels()) == 1  # one of the chain's launches was recorded, none has run
    s.set_graph(0)
    s.step(1)
    assert buffers()[0][0] == holds, size
""")
