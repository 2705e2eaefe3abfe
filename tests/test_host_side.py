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
