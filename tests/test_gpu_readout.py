"""Moment sums over several 256-site items per reduction and population copies
on both load paths, where a lattice is large enough for chunks of more than
one item, ends inside a chunk, or shares a chunk with its neighbours in a
batch.

Reference: plain torch FP64 sums of the populations that were set.  Tolerance:
each site's momentum is a sum of ten run-precision values, so a component's
total is off by at most ten roundings of the summed magnitudes; the mass is
the run's density sum with nineteen.
"""
import ctypes

import numpy as np
import pytest

from paper_1610_02733_amd import workloads as wl

pytestmark = pytest.mark.gpu

VEL = np.array([(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
                (1, 1, 0), (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1),
                (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)], float)
EPS = {32: 2.0 ** -24, 64: 2.0 ** -53}


@pytest.fixture(scope="module")
def lb():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_02733_amd import lbmd
    lbmd.lib()
    return lbmd


def state(lb, shape, prec, seed):
    import torch
    dt = torch.float32 if prec == 32 else torch.float64
    g = torch.Generator(device="cuda").manual_seed(seed)
    w = torch.tensor(lb.WEIGHTS, dtype=dt, device="cuda").reshape(19, 1)
    return 0.02 * w * torch.randn((19, int(np.prod(shape))), generator=g, dtype=dt, device="cuda")


def check_totals(lb, tot, f, prec):
    import torch
    d = f.double()
    S, mag = d.shape[1], float(d.abs().sum())
    vel = torch.tensor(VEL, dtype=torch.float64, device="cuda")
    assert abs(tot[lb.TOT["mass"]] - (S + float(d.sum()))) < 20 * EPS[prec] * mag
    for k, p in enumerate((vel.T @ d).sum(1).tolist()):
        assert abs(tot[lb.TOT["pfluid"]][k] - p) < 10 * EPS[prec] * mag, k


@pytest.mark.parametrize("shape,prec", [((128, 128, 129), 32), ((129, 131, 127), 32),
                                        ((130, 128, 127), 64), ((7, 5, 3), 64)])
def test_chunked_moments_and_copies(lb, shape, prec):
    import torch
    s = lb.Lattice(shape, precision=prec)
    f = state(lb, shape, prec, 3)
    s.set_populations(f)
    assert torch.equal(s.populations(), f)
    for noalloc in (False, True):
        tot, rho, u = s.moments(fields=True, noalloc=noalloc)
        check_totals(lb, tot, f, prec)
        ref = 1.0 + f.double().sum(0)
        assert float((rho.double() - ref).abs().max()) < 20 * EPS[prec]
        j = torch.tensor(VEL, dtype=torch.float64, device="cuda").T @ f.double()
        assert float((u.double() - j / ref).abs().max()) < 20 * EPS[prec]


def test_chunked_moments_of_a_batch(lb):
    shapes = [(128, 128, 128), (17, 13, 11), (64, 5, 3), (130, 128, 128), (2, 2, 2)]
    B = lb.Batch([(s, dict(precision=32, n_particles=0)) for s in shapes])
    B.x = None
    fs = [state(lb, s, 32, 10 + r) for r, s in enumerate(shapes)]
    for r, f in enumerate(fs):
        assert lb.lib().lbmd_batch_set_populations(B._h, r, ctypes.c_void_p(f.data_ptr())) == 0
    tot = B.moments()
    for r, f in enumerate(fs):
        check_totals(lb, tot[r], f, 32)
        assert bool((B.populations(r) == f).all())


@pytest.mark.parametrize("shape,other", [((128, 128, 64), (5, 4, 3)), ((66, 67, 65), (64, 3, 2)),
                                         ((256, 128, 81), (5, 4, 3))])
def test_kept_and_reversed_steps(lb, shape, other):
    """Steps whose stores stay in the caches, with aligned rows in reverse item
    order every other step, against the same system in a batch with a replica
    of the other load path, where neither applies: same arithmetic per site
    (five roundings a step of deviations up to 0.1 w_i rho0)."""
    import torch
    kw = dict(precision=32, kT=1e-4, seed=5, replica=0, body_force=(1e-4, 0.0, 0.0))
    f = state(lb, shape, 32, 6)
    a = lb.Lattice(shape, **kw)
    a.set_populations(f)
    b = lb.Batch([(shape, dict(kw, n_particles=0)), (other, dict(kw, replica=1, n_particles=0))])
    assert lb.lib().lbmd_batch_set_populations(b._h, 0, ctypes.c_void_p(f.data_ptr())) == 0
    a.run_cycles(5)
    b.run_cycles(5)
    w = torch.tensor(lb.WEIGHTS, dtype=torch.float64, device="cuda").reshape(19, 1)
    d = (a.populations().double() - b.populations(0).double()).abs() / w
    assert float(d.max()) < 25 * 0.1 * EPS[32]
