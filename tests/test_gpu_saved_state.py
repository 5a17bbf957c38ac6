"""Saved states copied to and from any address of a byte tensor: 16-byte
aligned, 8-, 4- and 1-byte aligned ones (wide copies, single words, and the
byte copies of the runtime).  The copies have no arithmetic, so a resumed run
without MD-order atomics repeats bit for bit; a state with negative counters is
refused and changes nothing."""
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


@pytest.mark.parametrize("N", [0, 1, 7])
@pytest.mark.parametrize("offset", [0, 8, 4, 1])
@pytest.mark.parametrize("precision", [32, 64])
def test_saved_state_at_any_address(lb, precision, offset, N):
    import torch
    shape = (7, 6, 5)
    kw = dict(kT=1e-4, seed=9, n_particles=N, friction=0.3, n_sub=2, variant=2,
              precision=precision)

    def system():
        g = lb.Lattice(shape, **kw)
        if N:
            g.bind_particles(*wl.free_particles(shape, N, 1e-4, 1.0, 4))
        return g

    a = system()
    a.run_cycles(3)
    n = a.save_state().numel()
    buf = torch.full((n + 64,), 0xA5, dtype=torch.uint8, device="cuda")
    state = a.save_state(buf[offset:])
    assert bool((buf[:offset] == 0xA5).all()) and bool((buf[offset + n:] == 0xA5).all())
    pop = a.populations().cpu()
    x = a.x.cpu().clone() if N else None

    b = system()
    b.run_cycles(5)
    before = b.populations().cpu()
    was = a.counters()
    assert was["t_lb"] == 3
    bad = state.clone()
    i = bad.cpu().numpy().tobytes().find(np.array([was["t_lb"], was["t_md"]], np.int64).tobytes())
    assert i >= 0
    bad[i:i + 8] = 0xFF
    with pytest.raises(lb.LbmdError):
        b.load_state(bad)
    assert torch.equal(b.populations().cpu(), before)
    assert b.counters()["t_lb"] == 5

    b.load_state(state)
    assert b.counters() == was
    assert torch.equal(b.populations().cpu(), pop)
    if N:
        assert torch.equal(b.x.cpu(), x)
    a.run_cycles(1)
    b.run_cycles(1)
    tol = 1e-5 if precision == 32 else 1e-12  # (order of the transfer's atomic sums)
    assert float((a.populations() - b.populations()).abs().max()) < tol
