"""A molecule's readouts (dipole, norm, yield, the moments of Eq. (8)) do not depend on
the batch it is in: nine random molecules repeated over a batch give each copy the bits
that the nine have alone, with batch sizes on both sides of every rule that the launches
have (no tolerance)."""

import numpy as np
import pytest
import torch

from gpu_helpers import banner, random_state
from workloads import get_config

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [512, 513, 1024, 1025])
@pytest.mark.parametrize("prec, basis, n_r, j_max", [("fp32", "jm", 64, 2), ("fp64", "jm", 128, 4), ("fp32", "jm", 128, 5),
                                                     ("fp32", "jm", 256, 5), ("fp64", "jm", 256, 2), ("mixed", "jm", 256, 1),
                                                     ("fp64", "jm", 512, 1), ("fp32", "jm", 512, 3), ("fp64", "m0", 64, 3),
                                                     ("fp64", "m0", 128, 10), ("mixed", "m0", 256, 10),
                                                     ("fp64", "m0", 256, 4), ("fp32", "m0", 512, 2)])
def test_readouts_do_not_depend_on_the_batch(prec, basis, n_r, j_max, n):
    from paper_2209_04487_amd import msqd
    banner(f"readouts {prec} {basis} n_r={n_r} j_max={j_max} in a batch of {n}")
    few = 9
    psi = torch.as_tensor(random_state(n_r + j_max, few, (j_max + 1) ** (2 if basis == "jm" else 1), n_r, 11.0 / n_r))
    out = []
    for size in (few, n):
        m = msqd.Molecules.from_config(get_config("cfg0", n_r=n_r, j_max=j_max, basis=basis, n_mol=size), prec=prec)
        at = torch.arange(size, device="cuda") % few
        m.psi.copy_(psi.cuda().to(m.psi.dtype)[at])
        m.absorbed.copy_(0.01 * at)
        d, nrm, yld = m.readout()
        num, pop, _ = msqd.excited_r(m)
        out.append([v.cpu().numpy()[:size] for v in (d, nrm, yld, num, pop)])
    at = np.arange(n) % few
    for name, a, b in zip(("dipole", "norm", "yield", "r_num", "pop"), *out):
        assert np.abs(a).max() > 0
        assert np.array_equal(a[at], b), name


@pytest.mark.parametrize("n", [1, 64, 512, 513, 8193])
def test_excited_sums_at_the_edges_of_their_passes(n):
    """The ensemble sums of Eq. (8): one and several passes of their loads, one wavefront
    and sixteen (1e-12: at most 8,193 positive terms, each addition rounded to 1.1e-16)."""
    from paper_2209_04487_amd import msqd
    banner(f"excited-state sums over {n} molecules")
    m = msqd.Molecules.from_config(get_config("cfg0", n_r=64, j_max=0, n_mol=n), prec="fp64")
    g = torch.Generator(device="cuda").manual_seed(n)
    m.psi.copy_(torch.randn(m.psi.shape, generator=g, device="cuda", dtype=m.psi.dtype))
    num, pop, r_e = msqd.excited_r(m)
    num, pop = num.cpu().numpy(), pop.cpu().numpy()
    assert num.min() > 0 and pop.min() > 0
    np.testing.assert_allclose(float(r_e), num.sum() / pop.sum(), rtol=1e-12)


@pytest.mark.parametrize("prec, n_r", [("fp32", 64), ("fp32", 512), ("fp64", 256)])
def test_excited_readout_of_a_wavepacket_buffer_off_16_bytes(prec, n_r):
    """excited_r_readout takes wavepackets on their elements' own alignment (8 bytes off a
    multiple of 16 here) and gives the bits of the aligned buffer."""
    from paper_2209_04487_amd import msqd
    banner(f"excited-state readout off 16 bytes {prec} n_r={n_r}")
    m = msqd.Molecules.from_config(get_config("cfg0", n_r=n_r, j_max=3, n_mol=7), prec=prec)
    psi = torch.as_tensor(random_state(n_r, 7, 4, n_r, 11.0 / n_r)).to(m.psi.dtype).cuda()
    m.psi.copy_(psi)
    want = [v.cpu().numpy() for v in msqd.excited_r(m)]
    real = torch.view_as_real(psi).reshape(-1)
    buf = torch.empty(real.numel() + 2, dtype=real.dtype, device="cuda")
    off = 2 if prec == "fp32" else 1
    buf[off:off + real.numel()] = real
    assert buf.data_ptr() % 16 == 0
    m.psi = buf[off:off + real.numel()]
    assert m.psi.data_ptr() % 16 == 8
    for a, b in zip(want, msqd.excited_r(m)):
        assert np.array_equal(a, b.cpu().numpy())
