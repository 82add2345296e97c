"""The FP64 reverse step of the molecules at n_r = 512, where molecules on either side
of the coupling angle's series limit take their own path, and at n_r = 256, where there
is one, against the transpose of the oracle's step.

Tolerance 1e-11 of the adjoint's 2-norm per molecule, as for the FP64 step tests; dY/dE
the same in units of |dt mu12|_max |psi| |lambda|."""

import numpy as np
import pytest
import torch

from gpu_helpers import TOL, banner
from oracle.molecule import model_from_config
from test_gpu_adjoint_rounds import _reverse_step
from workloads import get_config
from workloads.molecule_inputs import potentials
from workloads.units import EA0

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("next_state", [True, False])
@pytest.mark.parametrize("n_r, j_max", [(256, 3), (512, 0), (512, 3)])
def test_fp64_reverse_step(n_r, j_max, next_state):
    from paper_2209_04487_amd import msqd
    banner(f"fp64 reverse step n_r {n_r} j_max {j_max} state after the step {'given' if next_state else 'recomputed'}")
    n = 5
    cfg = get_config("cfg0", n_r=n_r, j_max=j_max, n_mol=n, r_min=1.0, r_max=12.0)
    # angles up to mu12 dt E = 0.41 (library sine), 0.027 (series), 0
    E = np.array([0.0, 0.02, -3.0, 0.2, -0.2])
    rng = np.random.default_rng(n_r + j_max)

    def rnd():
        z = rng.standard_normal((n, 2, j_max + 1, n_r)) + 1j * rng.standard_normal((n, 2, j_max + 1, n_r))
        return z / np.sqrt((np.abs(z) ** 2).sum((1, 2, 3), keepdims=True))

    psi, lam, labs = rnd(), rnd(), rng.standard_normal(n)
    mol = model_from_config(cfg, *potentials(cfg))
    nxt = mol.step(psi, E, np.zeros(n))[0]
    run = msqd.Coupled(cfg, prec="fp64", cells=np.arange(n, dtype=np.int32) + cfg.block_lo * cfg.nx * cfg.ny, n_freq=0)
    adj, buf = run.adjoint_buffers()
    dev = lambda v: torch.as_tensor(v).cuda()  # noqa: E731
    buf["lpsi"].copy_(dev(lam))
    buf["labs"].copy_(dev(labs))
    buf["lP"].copy_(dev(rng.standard_normal(n) * cfg.dx ** 3 / (cfg.mol_weight * EA0)))
    src = torch.zeros(1, dtype=torch.float64, device="cuda")
    msqd.adjoint_step(run.desc, run.state, dev(psi), dev(E), adj, 0, src, psi_np1=dev(nxt) if next_state else None)
    torch.cuda.synchronize()
    want, lE = _reverse_step(mol, psi, E, lam, labs, buf["ld"].cpu().numpy(), nxt if next_state else None)
    norm = np.sqrt((np.abs(want) ** 2).sum((1, 2, 3)))
    err = np.sqrt((np.abs(buf["lpsi"].cpu().numpy() - want) ** 2).sum((1, 2, 3)))
    tol = TOL["fp64"]
    assert np.all(err <= tol * norm)
    assert np.all(np.abs(buf["lE"].cpu().numpy() - lE) <= tol * np.abs(mol.mu12).max() * cfg.dt_au * norm)
