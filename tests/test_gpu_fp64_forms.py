"""The FP64 molecular step where its launch changes form: two, three and four K
instructions of the contraction (N_J = 8, 9, 12, 13), the exchange by parts and
in one round, single steps and step loops, and molecules of one batch on either
side of the series limit of the coupling angle (decided per molecule), against
the FP64 oracle.

Tolerance 1e-11 of the largest amplitude, as for the other FP64 step tests."""

import numpy as np
import pytest

from gpu_helpers import TOL, banner, rel_err
from test_gpu_molecule import _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_steps", [1, 2])
@pytest.mark.parametrize("n_r, j_max", [(64, 7), (64, 8), (64, 12), (64, 15), (128, 7), (128, 11), (128, 12),
                                        (256, 0), (256, 7), (256, 8), (256, 11), (256, 12), (512, 0), (512, 1),
                                        (512, 7), (512, 8)])
def test_fp64_step_forms(n_r, j_max, n_steps):
    banner(f"fp64 forms n_r={n_r} j_max={j_max} steps={n_steps}")
    # angles up to mu12 dt E = 0.41 (library path), 0.027 (series), 0
    E = np.array([0.0, 0.02, -3.0, 0.2, -0.2])
    out = _run("fp64", n_r, j_max, len(E), n_steps, E, seed=n_r + j_max)
    tol = TOL["fp64"]
    assert rel_err(out["psi_gpu"], out["psi"]) < tol
    np.testing.assert_allclose(out["ab_gpu"], out["ab"], rtol=tol, atol=tol * 1e-2)
    scale = max(np.abs(out["d"]).max(), 1e-3)      # J = 0 alone has no dipole
    assert np.abs(out["d_step"] - out["d"]).max() < 10 * tol * scale
    np.testing.assert_allclose(out["n_gpu"], out["n"], rtol=10 * tol)
