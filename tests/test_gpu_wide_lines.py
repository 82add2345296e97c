"""The complex64 molecular step at n_r = 256 where its launch changes between 8 and 16
lanes per line: N_J = 8 and 9 (any batch, and up to 512 molecules), 512 and 513
molecules, the smallest and the largest N_J, single steps and step loops, angles on
both sides of the series limit, against the FP64 oracle with the step tests'
tolerances."""

import numpy as np
import pytest

from gpu_helpers import TOL, banner, rel_err
from test_gpu_molecule import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_steps", [1, 2])
@pytest.mark.parametrize("prec", ["fp32", "mixed"])
@pytest.mark.parametrize("j_max, n_mol", [(0, 5), (2, 5), (7, 5), (7, 513), (8, 5), (8, 512), (8, 513), (15, 5),
                                          (15, 513)])
def test_wide_lines(prec, j_max, n_mol, n_steps):
    banner(f"wide lines {prec} j_max={j_max} n_mol={n_mol} steps={n_steps}")
    E = np.resize([0.0, 0.02, -3.0, 0.2, -0.2], n_mol)
    out = _run(prec, 256, j_max, n_mol, n_steps, E, seed=j_max + n_mol)
    tol = TOL[prec]
    assert rel_err(out["psi_gpu"], out["psi"]) < tol
    np.testing.assert_allclose(out["ab_gpu"], out["ab"], rtol=tol, atol=tol * 1e-2)
    scale = max(np.abs(out["d"]).max(), 1e-3)      # J = 0 alone has no dipole
    assert np.abs(out["d_step"] - out["d"]).max() < 10 * tol * scale
    np.testing.assert_allclose(out["n_gpu"], out["n"], rtol=10 * tol)
