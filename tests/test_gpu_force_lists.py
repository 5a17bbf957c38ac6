"""Candidate lists of the force kernel against the FP64 oracle: none, fewer
and more candidates than one window of the list holds, cells with more than
the eight slots read at once and with more than their capacity, and
wavefronts whose two particles belong to different replicas.

The potentials are scaled down so that close pairs stay gentle; tolerance
1e-12 as for the other FP64 polymer runs (same sums in another order).
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_02733_amd import lbmd
    lbmd.lib()
    return lbmd


def beads(n, region, seed, min_dist=0.25):
    rng = np.random.default_rng(seed)
    x = np.zeros((0, 3))
    while len(x) < n:
        q = 0.05 + rng.random(3) * (region - 0.05)
        if len(x) == 0 or ((x - q) ** 2).sum(1).min() >= min_dist ** 2:
            x = np.vstack([x, q])
    return np.ascontiguousarray(x.T)


def params(model, n, chain, replica=0):
    return dict(kT=0.0, seed=3, replica=replica, n_particles=n, friction=0.5, n_sub=3, variant=2,
                force_model=model, chain_len=chain, k_bond=1e-4, r0_bond=1.0 if model == 2 else 20.0,
                wca_eps=1e-12, wca_sigma=1.0)


def check(g_x, g_v, o):
    x, v, _ = o.particles()
    assert np.abs(g_x - x).max() < 1e-12 and np.abs(g_v - v).max() < 1e-12


@pytest.mark.parametrize("model,n,box,region,chain", [(3, 1, 9, 2.0, 1), (2, 2, 5, 1.0, 1),
                                                      (3, 150, 12, 5.0, 3),
                                                      (3, 520, 12, 6.6, 2),
                                                      (2, 330, 6, 3.3, 1)])
def test_force_list_lengths(lb, orc, model, n, box, region, chain):
    x = beads(n, region, n)
    kw = params(model, n, chain)
    g = lb.Lattice((box,) * 3, precision=64, **kw)
    g.bind_particles(x, 0 * x)
    g.run_cycles(2)
    o = orc.Oracle(box, box, box, **kw)
    o.set_particles(x, 0 * x)
    o.cycle(2)
    if n > 2:
        assert np.abs(o.particles()[1]).max() > 1e-7  # the forces moved the beads
    check(g.x.cpu().numpy(), g.v.cpu().numpy(), o)


def test_force_lists_across_replicas(lb, orc):
    sizes = [(3, 7, 9), (2, 13, 6), (3, 9, 10), (2, 1, 5)]
    reps = [((b,) * 3, dict(precision=64, **params(m, n, 1, r)))
            for r, (m, n, b) in enumerate(sizes)]
    xs = [beads(n, 2.2, 50 + n) for _, n, _ in sizes]
    B = lb.Batch(reps)
    B.bind_particles(xs, [0 * x for x in xs])
    B.run_cycles(2)
    for r, (shape, kw) in enumerate(reps):
        o = orc.Oracle(*shape, **{k: v for k, v in kw.items() if k != "precision"})
        o.set_particles(xs[r], 0 * xs[r])
        o.cycle(2)
        check(B.particles(r)[0].cpu().numpy(), B.particles(r)[1].cpu().numpy(), o)
