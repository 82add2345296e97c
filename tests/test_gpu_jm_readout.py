"""The streaming (j, m) readouts (dipole vector, norm, yield) against the FP64 oracle
on seeded random states: every j_max, the shortest and longest lines, batches that do
not fill a workgroup of four molecules, and single outputs.

Tolerances: the dipole's products and sums are FP64 in every form, 1e-12 of 2 dr sum_r
|mu12| |g(r)| |e(r)| (at most 5e4 terms, rounding 1e-16 each); norm and yield 1e-12 in
FP64, 2e-6 where each |psi|^2 is rounded to float."""

import numpy as np
import pytest
import torch

from gpu_helpers import banner, random_state
from oracle.molecule_jm import jm_model_from_config
from workloads import get_config
from workloads.molecule_inputs import potentials

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec, n_r, j_max, n_mol", [("fp64", 64, 1, 1), ("fp64", 128, 5, 5), ("fp64", 256, 3, 3),
                                                     ("fp64", 512, 2, 4), ("fp32", 64, 5, 3), ("fp32", 256, 5, 2),
                                                     ("fp32", 512, 4, 1), ("mixed", 128, 3, 9), ("mixed", 256, 1, 6),
                                                     ("fp32", 64, 2, 7), ("fp64", 64, 4, 2),
                                                     ("fp32", 256, 5, 1024), ("fp32", 256, 5, 1025)])
def test_jm_streaming_readouts(prec, n_r, j_max, n_mol):
    from paper_2209_04487_amd import msqd
    banner(f"jm readouts {prec} n_r={n_r} j_max={j_max} n_mol={n_mol}")
    cfg = get_config("cfg0", n_r=n_r, j_max=j_max, basis="jm", n_mol=n_mol)
    m = msqd.Molecules.from_config(cfg, prec=prec)
    dr = (cfg.r_max - cfg.r_min) / n_r
    m.psi.copy_(torch.as_tensor(random_state(11 + j_max, n_mol, (j_max + 1) ** 2, n_r, dr)).to(m.psi.dtype))
    psi = m.psi.cpu().numpy().astype(np.complex128)
    ab = np.linspace(0.0, 0.3, n_mol)
    m.absorbed.copy_(torch.as_tensor(ab))
    d, nrm, yld = (t.cpu().numpy()[:n_mol] for t in m.readout())
    om = jm_model_from_config(cfg, *potentials(cfg))
    amp = np.sqrt((np.abs(psi) ** 2).sum(2))                      # [mol, state, r]
    bound = 2.0 * dr * (np.abs(potentials(cfg)[2]) * amp[:, 0] * amp[:, 1]).sum(1)
    assert np.all(np.abs(d - om.dipole(psi)) <= 1e-12 * bound[:, None])
    tol = 1e-12 if prec == "fp64" else 2e-6
    np.testing.assert_allclose(nrm, om.norm(psi), rtol=tol)
    np.testing.assert_allclose(yld, om.dissociated(psi, ab), rtol=tol)
    # one output at a time
    only = torch.zeros(n_mol, dtype=torch.float64, device="cuda")
    msqd.dipole_readout(m.desc, m.ws, m.psi, m.absorbed, None, None, only, None)
    assert np.array_equal(only.cpu().numpy(), yld)
    d2 = torch.zeros((n_mol, 3), dtype=torch.float64, device="cuda")
    msqd.dipole_readout(m.desc, m.ws, m.psi, m.absorbed, d2, None, None, None)
    assert np.array_equal(d2.cpu().numpy(), d)
