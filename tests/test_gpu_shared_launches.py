"""The H update's shared launches (with the deposit into the held array, with the
emitters' step) and the monitor samples that the E update stages, where the
extra threads take several rows of the launch: a plane of one run of 256 cells,
700 molecules or emitters on ten planes, two detection planes.

The molecules' run equals the one whose deposit is a launch of its own after the
E update (held=False) bit for bit; the emitters' run equals the oracle to 1e-10
of the largest value, as for the other coupled runs."""

import numpy as np
import pytest
import torch

from gpu_helpers import banner
from oracle.bloch import CoupledBlochOracle
from workloads import get_config
from workloads.pulses import source_values

pytestmark = pytest.mark.gpu


def _cfg(**kw):
    return get_config("cfg1", nx=16, ny=16, nz=28, npml=4, src_k=5, mon_k=22, mon_k2=7, n_freq=5, mon_every=2,
                      geom=dict(cell=16, outer=12, arm=3, gap=3, z0=19, z1=21, glass_k=21), n_mol=700, slab_k0=8,
                      slab_nk=10, n_r=64, j_max=2, t0_steps=6.0, t0_fs=None, fwhm_fs=0.2, e0_au=0.02, **kw)


@pytest.mark.parametrize("prec, basis, every", [("fp64", "m0", 1), ("mixed", "m0", 3), ("fp32", "jm", 1)])
def test_shared_deposit_launch_equals_separate(prec, basis, every):
    from paper_2209_04487_amd import msqd
    cfg = _cfg(basis=basis)
    banner(f"shared deposit {prec} {basis} M={every}")
    src = source_values(cfg, 0, 20)
    runs = []
    for held in (True, False):
        s = msqd.Coupled(cfg, prec=prec, mol_every=every, held=held)
        for a, b in ((0, 1), (1, 8), (8, 20)):     # one sample per call, and several
            s.step(src[a:b])
        torch.cuda.synchronize()
        runs.append({**{k: s.fields.t[k] for k in s._STATE if k != "dft"}, "flux": s.fields.flux(), "psi_m": s.mol.psi,
                     "P": s.P_c, "J": s.J_mol, "d": s.mol.d})
    assert float(runs[0]["J"].abs().max()) > 0 and float(runs[0]["flux"].abs().max()) > 0
    assert len(s.occ_cell) > 2 * 256
    for k in runs[0]:
        assert torch.equal(runs[0][k], runs[1][k]), k


def test_shared_bloch_launch_matches_oracle():
    from paper_2209_04487_amd import msqd
    cfg = _cfg()
    banner("shared Bloch launch fp64")
    src = source_values(cfg, 0, 20)
    s = msqd.CoupledBloch(cfg, prec="fp64")
    s.step(src)
    o = CoupledBlochOracle(cfg)
    for n in range(20):
        o.step(n, src[n])
    emax = max(np.abs(e).max() for e in o.yee.E)
    assert np.abs(s.fields.Ex.cpu().numpy() - o.yee.E[0]).max() < 1e-10 * emax
    y = s.em.state.cpu().numpy()
    assert np.abs(y - o.y).max() < 1e-10 * np.abs(o.y).max() and np.abs(o.y).max() > 0
