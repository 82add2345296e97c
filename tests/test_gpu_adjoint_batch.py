"""The FP32 reverse step at n_r = 128 on both sides of the batch sizes up to which it
takes one exchange round: five molecules repeated over the batch, every copy against the
transpose of the oracle's step in 64 bits.

Tolerance 8e-6 of the adjoint's 2-norm per molecule, as for the other FP32 reverse steps
(some 136 roundings of 2^-24 along any path); dY/dE the same in units of |dt mu12|_max
|psi| |lambda|."""

import numpy as np
import pytest
import torch

from gpu_helpers import banner
from oracle.molecule import model_from_config
from test_gpu_adjoint_rounds import _reverse_step
from workloads import get_config
from workloads.molecule_inputs import potentials
from workloads.units import EA0

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("next_state", [True, False])
@pytest.mark.parametrize("j_max, n", [(6, 1024), (6, 1025), (10, 512), (10, 513)])
def test_fp32_reverse_step_at_the_batch_limits(j_max, n, next_state):
    from paper_2209_04487_amd import msqd
    banner(f"fp32 reverse step n_r 128 j_max {j_max} n_mol {n} state after the step "
           f"{'given' if next_state else 'recomputed'}")
    cfg = get_config("cfg0", n_r=128, j_max=j_max, n_mol=n, r_min=1.0, r_max=12.0)
    rng = np.random.default_rng(n)
    E = np.array([0.0, 0.02, -3.0, 0.2, -0.2])       # angles up to 0.41 (library sine), 0.027 (series), 0

    def rnd():
        z = rng.standard_normal((5, 2, j_max + 1, 128)) + 1j * rng.standard_normal((5, 2, j_max + 1, 128))
        return (z / np.sqrt((np.abs(z) ** 2).sum((1, 2, 3), keepdims=True))).astype(np.complex64)

    psi, lam, labs, lP = rnd(), rnd(), rng.standard_normal(5), rng.standard_normal(5)
    mol = model_from_config(cfg, *potentials(cfg))
    nxt = mol.step(psi.astype(np.complex128), E, np.zeros(5))[0].astype(np.complex64)
    at = np.arange(n) % 5
    # a cell of its own for every molecule, so that the deposit's transpose gives each its ld
    run = msqd.Coupled(cfg, prec="fp32", cells=np.arange(n, dtype=np.int32) + cfg.block_lo * cfg.nx * cfg.ny, n_freq=0)
    adj, buf = run.adjoint_buffers()
    dev = lambda v: torch.as_tensor(v[at]).cuda()  # noqa: E731
    buf["lpsi"].copy_(dev(lam))
    buf["labs"].copy_(dev(labs))
    buf["lP"].copy_(dev(lP * (cfg.dx ** 3 / (cfg.mol_weight * EA0))))
    src = torch.zeros(1, dtype=torch.float64, device="cuda")
    msqd.adjoint_step(run.desc, run.state, dev(psi), dev(E), adj, 0, src, psi_np1=dev(nxt) if next_state else None)
    torch.cuda.synchronize()
    ld = buf["ld"].cpu().numpy()
    assert np.array_equal(ld, ld[:5][at]) and np.abs(ld[:5]).min() > 0
    want, lE = _reverse_step(mol, psi.astype(np.complex128), E, lam.astype(np.complex128), labs, ld[:5],
                             nxt.astype(np.complex128) if next_state else None)
    got, e32 = buf["lpsi"].cpu().numpy(), buf["lE"].cpu().numpy()
    norm = np.sqrt((np.abs(want) ** 2).sum((1, 2, 3)))[at]
    err = np.sqrt((np.abs(got - want[at]) ** 2).sum((1, 2, 3)))
    mu = np.abs(mol.mu12).max() * cfg.dt_au
    assert np.all(np.isfinite(got)) and np.all(err <= 8e-6 * norm)
    assert np.all(np.abs(e32 - lE[at]) <= 8e-6 * mu * norm)
