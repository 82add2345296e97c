"""The FP32 reverse step of the molecules (adjoint_step) at the edges of its
forms: one and two exchange rounds, half and full contractions, one angular line
and the longest and largest molecules accepted, with the state after the step
given and recomputed, against the transpose of the oracle's step in 64 bits.

Tolerance 8e-6 of the adjoint's 2-norm per molecule: along any path an element
takes at most some 136 roundings (four transforms' 2 log2(n_r) stages, phases, two
contractions of 16 terms each way), each at most 2^-24 relative to the norm, all
of them factors of norm one.  dY/dE the same in units of |dt mu12|_max |psi| |lambda|."""

import numpy as np
import pytest
import torch

from gpu_helpers import banner
from oracle.molecule import model_from_config
from workloads import get_config
from workloads.molecule_inputs import potentials
from workloads.units import EA0

pytestmark = pytest.mark.gpu


def _reverse_step(m, psi, E, lam, labs, ld, nxt):
    """The transpose of m.step and m.dipole in 64 bits: adjoint before the step and dY/dE."""
    chi = m.potential_half(m.kinetic_half(psi))
    pre = nxt / m.mask if nxt is not None else m.kinetic_half(m.potential_half(m.coupling(chi, E)))
    new = pre * m.mask
    c = np.zeros(m.n_j + 1)
    c[1:m.n_j] = m.cj
    other = new[:, ::-1]
    dp = np.zeros_like(new)
    dp[:, :, 1:] += c[1:m.n_j, None] * other[:, :, :-1]
    dp[:, :, :-1] += c[1:m.n_j, None] * other[:, :, 1:]
    per = lambda v: v[:, None, None, None]  # noqa: E731
    lam = m.mask * (lam + 2.0 * m.dr * per(ld) * m.mu12 * dp) + 2.0 * m.dr * per(labs) * (1.0 - m.mask ** 2) * pre

    def transposed(v):
        return np.fft.ifft(np.conj(m.kin_half) * np.fft.fft(v, axis=-1), axis=-1)

    lam = transposed(lam) * np.conj(m.v_half)
    turned = m.to_angle(m.coupling(chi, E))[:, ::-1]
    dphi = m.rotation_angle(np.ones(len(E)))
    lE = (np.conj(m.to_angle(lam)) * (1j * dphi[:, None] * turned)).real.sum((1, 2, 3))
    return transposed(m.coupling(lam, -E) * np.conj(m.v_half)), lE


@pytest.mark.parametrize("next_state", [True, False])
@pytest.mark.parametrize("n_r, j_max", [(64, 0), (64, 7), (64, 15), (128, 0), (128, 6), (128, 7), (128, 8), (128, 15),
                                        (256, 0), (256, 7), (256, 8), (256, 15), (512, 0), (512, 7), (512, 8)])
def test_fp32_reverse_step_against_fp64(n_r, j_max, next_state):
    from paper_2209_04487_amd import msqd
    banner(f"fp32 reverse step n_r {n_r} j_max {j_max} state after the step "
           f"{'given' if next_state else 'recomputed'}")
    n = 5
    cfg = get_config("cfg0", n_r=n_r, j_max=j_max, n_mol=n, r_min=1.0, r_max=12.0)
    # angles up to mu12 dt E = 0.41 (library sine), 0.027 (series), 0
    E = torch.tensor([0.0, 0.02, -3.0, 0.2, -0.2], dtype=torch.float64, device="cuda")
    g = torch.Generator(device="cpu").manual_seed(n_r + j_max)
    shape = (n, 2, j_max + 1, n_r)

    def rnd():
        z = torch.complex(torch.randn(shape, generator=g, dtype=torch.float64),
                          torch.randn(shape, generator=g, dtype=torch.float64))
        z /= torch.linalg.vector_norm(z, dim=(1, 2, 3), keepdim=True)
        return z.to(torch.complex64).to(torch.complex128).cuda()

    psi, lam = rnd(), rnd()
    labs = torch.randn(n, generator=g, dtype=torch.float64).cuda()
    lP = torch.randn(n, generator=g, dtype=torch.float64).cuda() * (cfg.dx ** 3 / (cfg.mol_weight * EA0))
    run = msqd.Coupled(cfg, prec="fp32", cells=np.arange(n, dtype=np.int32) + cfg.block_lo * cfg.nx * cfg.ny, n_freq=0)
    adj, buf = run.adjoint_buffers()
    buf["lpsi"].copy_(lam)
    buf["labs"].copy_(labs)
    buf["lP"].copy_(lP)
    mol = model_from_config(cfg, *potentials(cfg))
    nxt = mol.step(psi.cpu().numpy(), E.cpu().numpy(), np.zeros(n))[0].astype(np.complex64)
    src = torch.zeros(1, dtype=torch.float64, device="cuda")
    msqd.adjoint_step(run.desc, run.state, psi.to(torch.complex64), E, adj, 0, src,
                      psi_np1=torch.as_tensor(nxt).cuda() if next_state else None)
    torch.cuda.synchronize()
    ld = buf["ld"].cpu().numpy()
    assert 0.01 < np.abs(ld).max() < 100.0
    l64, e64 = _reverse_step(mol, psi.cpu().numpy(), E.cpu().numpy(), lam.cpu().numpy(), labs.cpu().numpy(), ld,
                             nxt.astype(np.complex128) if next_state else None)
    l32, e32 = buf["lpsi"].cpu().numpy(), buf["lE"].cpu().numpy()
    norm = np.sqrt((np.abs(l64) ** 2).sum((1, 2, 3)))
    err = np.sqrt((np.abs(l32 - l64) ** 2).sum((1, 2, 3)))
    mu = np.abs(mol.mu12).max() * cfg.dt_au
    print(f"  lpsi {np.max(err / norm):.2e}  lE {np.max(np.abs(e32 - e64) / (mu * norm)):.2e}")
    assert np.all(np.isfinite(l32)) and np.all(err <= 8e-6 * norm)
    assert np.all(np.abs(e32 - e64) <= 8e-6 * mu * norm)
