"""Captured and directly launched cycles against the oracle: cycles of few and
of many kernels, odd numbers of cycles per call (each cycle starts from the
clock entry the one before wrote), and single LB steps, saved states and set
counters in between.  FP64, 1e-12 as for the other FP64 runs."""
import numpy as np
import pytest

from paper_1610_02733_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_02733_amd import lbmd
    lbmd.lib()
    return lbmd


def compare(g, o, w, N):
    e = np.abs(g.populations().cpu().numpy() + w[:, None] - o.populations()) / w[:, None]
    assert e.max() < 1e-12
    if N:
        x, v, img = o.particles()
        assert np.abs(g.x.cpu().numpy() - x).max() < 1e-11
        assert np.abs(g.v.cpu().numpy() - v).max() < 1e-12


@pytest.mark.parametrize("N,n_sub", [(0, 1), (24, 1), (24, 2), (24, 3), (300, 3)])
def test_cycles_direct_and_captured(lb, orc, N, n_sub):
    _, w, _, _ = orc.tables()
    shape = (12, 10, 9)
    kw = dict(kT=1e-4, seed=9, n_particles=N, friction=0.3, n_sub=n_sub, variant=2)
    g = lb.Lattice(shape, precision=64, **kw)
    o = orc.Oracle(*shape, **kw)
    if N:
        x, v = wl.free_particles(shape, N, 1e-4, 1.0, 4)
        g.bind_particles(x, v)
        o.set_particles(x, v)
    for k in (1, 3, 9, 2, 7):
        g.run_cycles(k)
        g.cycle(1)
    o.cycle(27)
    compare(g, o, w, N)
    assert g.counters()["t_lb"] == 27
    state = g.save_state()
    g.run_cycles(5)
    g.load_state(state)
    g.run_cycles(4)
    o.cycle(4)
    compare(g, o, w, N)
