"""Reverse MD steps whose corners change from step to step: cycles of one, two
and more MD steps (odd and even numbers of buffer changes), particles that
cross several cells in a cycle and share corners, against torch.autograd
through the FP64 reference.  Same bounds as for slow particles: 1e-10."""
import numpy as np
import pytest
import torch

from paper_1610_02733_amd import workloads as wl  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lb():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_02733_amd import lbmd
    lbmd.lib()
    return lbmd


@pytest.mark.parametrize("variant,n_sub,N", [(2, 1, 9), (2, 2, 9), (2, 3, 1), (2, 4, 33), (2, 5, 70),
                                             (1, 1, 9), (1, 4, 33)])
def test_reverse_steps_over_changing_corners(lb, orc, variant, n_sub, N):
    from oracle.torch_oracle import TorchOracle
    from paper_1610_02733_amd.adjoint import coupled_run
    _, w, _, _ = orc.tables()
    shape, cycles = (6, 5, 4), 4
    rng = np.random.default_rng(31 + n_sub)
    dev = 0.02 * w[:, None] * rng.standard_normal((19, int(np.prod(shape))))
    x0 = rng.random((3, N)) * np.asarray(shape, float)[:, None]
    v0 = 0.7 * rng.standard_normal((3, N))
    ax, av = rng.standard_normal((2, 3, N))
    # (friction low enough that 70 particles on 120 sites stay stable)
    start = [0.2, 0.23, np.array([2e-3, -1e-3, 4e-4]), x0, v0]
    kw = dict(n_sub=n_sub, variant=variant, kT=1e-3, seed=6, particle_mass=1.2)

    def leaves(device):
        return [torch.tensor(a, dtype=torch.float64, device=device, requires_grad=True) for a in start]

    g = leaves("cuda")
    x, v = coupled_run(*g, shape=shape, cycles=cycles, checkpoint=3, precision=64,
                       populations=torch.tensor(dev, device="cuda"), **kw)
    ((torch.tensor(ax, device="cuda") * x).sum() + (torch.tensor(av, device="cuda") * v).sum()).backward()
    o = leaves("cpu")
    T = TorchOracle(shape, n_sub, variant, 1e-3, seed=6, particle_mass=1.2)
    xr, vr, _ = T.run(torch.tensor(w[:, None] + dev), o[3], o[4], o[0], o[1], o[2], cycles)
    ((torch.tensor(ax) * xr).sum() + (torch.tensor(av) * vr).sum()).backward()
    assert np.abs(xr.detach().numpy() - x.detach().cpu().numpy()).max() < 1e-10
    for k, (a, b) in enumerate(zip(g, o)):
        ga, gb = a.grad.cpu().numpy(), b.grad.numpy()
        err = np.abs(ga - gb).max() / max(np.abs(gb).max(), 1e-12)
        assert err < 1e-10, (k, err)


def test_reverse_steps_beside_a_lost_particle(lb):
    """A particle without a finite position takes no part: the others'
    derivatives are those of the run without it."""
    from paper_1610_02733_amd.adjoint import coupled_run
    shape, N = (6, 5, 4), 10
    rng = np.random.default_rng(5)
    x0 = rng.random((3, N)) * np.asarray(shape, float)[:, None]
    v0 = 0.5 * rng.standard_normal((3, N))
    out = []
    for n in (N, N - 1):
        xn, vn = x0[:, :n].copy(), v0[:, :n].copy()
        if n == N:
            xn[:, -1] = np.nan
        ls = [torch.tensor(a, dtype=torch.float64, device="cuda", requires_grad=True)
              for a in (0.5, 0.23, np.array([1e-3, 0.0, 0.0]), xn, vn)]
        x, v = coupled_run(*ls, shape=shape, cycles=3, checkpoint=2, precision=64, n_sub=4, variant=2,
                           kT=1e-3, seed=6)
        (x[:, :N - 1].sum() + (v[:, :N - 1] ** 2).sum()).backward()
        out.append([t.grad.cpu().numpy() for t in ls])
    for a, b in zip(*out):
        a = a[:, :N - 1] if a.ndim == 2 else a
        assert np.abs(a - b).max() <= 1e-10 * max(np.abs(b).max(), 1e-12)
