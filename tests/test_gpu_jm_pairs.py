"""The general (j, m) step in every form it is built in, single steps and step loops:
pair, even-state and odd-state counts with and without a partial row group, a second
set of odd rows (j_max = 5), one and two exchange rounds, and workgroups with a
partial last wavefront (j_max = 2, 4), against the oracle with its tolerances."""

import pytest

from test_gpu_jm import test_jm_general_step_matches_oracle as _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_steps", [1, 2])
@pytest.mark.parametrize("prec,n_r,j_max", [("fp32", n_r, j) for n_r in (64, 128, 256) for j in (2, 3, 4, 5)]
                         + [("fp32", 512, j) for j in (2, 3, 4)]
                         + [("fp64", n_r, j) for n_r in (64, 128) for j in (2, 3, 4, 5)]
                         + [("fp64", 256, 2), ("fp64", 256, 3), ("fp64", 512, 2)])
def test_jm_general_forms(prec, n_r, j_max, n_steps):
    _check(prec, n_r, j_max, 5, n_steps)
