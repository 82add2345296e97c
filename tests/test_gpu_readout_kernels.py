"""The streaming readouts (dipole, norm, yield; the moments of Eq. (8)) against
the FP64 oracle on seeded random states: the shortest and longest lines, a
single J, batches that do not fill a workgroup of four molecules.

Tolerances: FP64 1e-12 (sums of at most 1.6e4 terms, rounding 1e-16 each).  The
single-precision forms round each |psi|^2 and each J sum of the dipole to float
(at most 20 roundings of 6e-8): 2e-6 of the same sum over absolute values."""

import numpy as np
import pytest
import torch

from gpu_helpers import banner, model_arrays, random_state
from oracle.molecule import MoleculeModel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec, n_r, j_max, n_mol", [("fp64", 64, 0, 1), ("fp64", 256, 10, 5), ("fp64", 512, 8, 3),
                                                     ("fp32", 64, 1, 3), ("fp32", 512, 15, 2), ("mixed", 128, 4, 9),
                                                     ("mixed", 256, 10, 6)])
def test_streaming_readouts(prec, n_r, j_max, n_mol):
    from paper_2209_04487_amd import msqd
    banner(f"readouts {prec} n_r={n_r} j_max={j_max} n_mol={n_mol}")
    r, ug, ue, mu = model_arrays(n_r)
    m = msqd.Molecules(n_mol, n_r, j_max, 1.0, 12.0, 1.0e4, 0.1, ug, ue, mu, np.ones(n_r), prec=prec, r_diss=8.0)
    psi = random_state(7, n_mol, j_max + 1, n_r, 11.0 / n_r)
    m.psi.copy_(torch.as_tensor(psi, dtype=m.psi.dtype))
    psi = m.psi.cpu().numpy().astype(np.complex128)
    ab = np.linspace(0.0, 0.3, n_mol)
    m.absorbed.copy_(torch.as_tensor(ab))
    d, nrm, yld = (t.cpu().numpy()[:n_mol] for t in m.readout())
    num, pop, r_e = msqd.excited_r(m)
    om = MoleculeModel(n_r, 1.0, 12.0, j_max, 1.0e4, 0.1, ug, ue, mu)
    tol = 1e-12 if prec == "fp64" else 2e-6
    bound = np.abs(om.dipole(np.abs(psi) + 0j)) + 1e-30      # the dipole's sum over absolute values
    assert np.all(np.abs(d - om.dipole(psi)) <= tol * bound)
    np.testing.assert_allclose(nrm, om.norm(psi), rtol=tol)
    np.testing.assert_allclose(yld, om.dissociated(psi, ab), rtol=tol)
    on, op = om.excited_r_moments(psi)
    np.testing.assert_allclose(num.cpu().numpy(), on, rtol=tol)
    np.testing.assert_allclose(pop.cpu().numpy(), op, rtol=tol)
    np.testing.assert_allclose(float(r_e), on.sum() / op.sum(), rtol=tol)
