"""Totals of a large single system, summed over many blocks, against the
one-block sums of the version without workspace scratch (the same values per
site, FP64, in another order) and the particles' own sums: 1e-12 of the sum of
the magnitudes.  Either side of the sizes from which the many blocks are used,
and a non-finite particle, which both must report."""
import numpy as np
import pytest
import torch

from paper_1610_02733_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_02733_amd import lbmd
    lbmd.lib()
    return lbmd


@pytest.mark.parametrize("shape,N,precision", [
    ((128, 128, 128), 1, 32), ((128, 128, 128), 4097, 64), ((131, 127, 129), 0, 32),
    ((131, 127, 129), 9001, 32), ((127, 127, 129), 5000, 64), ((40, 30, 20), 5000, 32)])
def test_sums_over_many_blocks(lb, shape, N, precision):
    sim = lb.Lattice(shape, precision=precision, kT=1e-4, seed=3, n_particles=N, friction=0.5, n_sub=2,
                     variant=2, particle_mass=1.5)
    S = int(np.prod(shape))
    g = torch.Generator(device="cuda").manual_seed(7)
    dev = 0.01 * torch.randn((19, S), generator=g, device="cuda", dtype=torch.float64)
    sim.set_populations(dev.to(torch.float32 if precision == 32 else torch.float64))
    v = None
    if N:
        x, v = wl.free_particles(shape, N, 1e-2, 1.0, 5)
        sim.bind_particles(x, v)
    a = sim.moments()
    b = sim.moments(noalloc=True)
    scale = S + 10.0 * N
    assert np.abs(a - b).max() <= 1e-12 * scale
    if N:
        p = 1.5 * np.asarray(v, np.float64).reshape(3, N)
        at = [i for i in range(len(a) - 2) if np.abs(a[i:i + 3] - p.sum(1)).max() <= 1e-12 * scale]
        assert at  # the particles' momentum is among the totals
        ke = 0.5 / 1.5 * (p ** 2).sum()
        assert np.abs(a - ke).min() <= 1e-12 * scale
        sim.v[1, N - 1] = float("nan")
        sim.run_cycles(1)
        for noalloc in (False, True):
            with pytest.raises(lb.LbmdError):
                sim.moments(noalloc=noalloc)
