"""The field update on planes around the sizes where its launch changes: below
and from 16 runs of 256 cells per plane, whole and padded to a multiple of
eight runs, with odd row lengths, against the FP64 oracle.

Tolerance 1e-11 of the largest field value, as for the other field tests: 30
steps of about ten rounded operations each."""

import numpy as np
import pytest

from gpu_helpers import banner
from oracle.fdtd import yee_from_config
from workloads import get_config
from workloads.geometry import eps_table
from workloads.pulses import source_values

pytestmark = pytest.mark.gpu


# runs per plane: 1, 15 (exactly), 16 (ragged), 16 (exactly), 17 -> 24, 33 -> 40
@pytest.mark.parametrize("nx, ny", [(7, 5), (64, 60), (61, 63), (64, 64), (65, 67), (131, 64)])
def test_planes_around_the_strip_rule(nx, ny):
    from paper_2209_04487_amd import msqd
    nz, nsteps = 14, 30
    cfg = get_config("cfg1", nx=nx, ny=ny, nz=nz, npml=3, src_k=4, mon_k=9, n_freq=0, t0_steps=10.0, t0_fs=None,
                     fwhm_fs=0.1)
    banner(f"stencil {nx}x{ny}x{nz}")
    mat = np.random.default_rng(nx * 1000 + ny).integers(0, 3, (3, nz, ny, nx)).astype(np.uint8)
    src = source_values(cfg, 0, nsteps)
    fl = msqd.Fields(msqd.fdtd_desc_from_config(cfg, "fp64"), mat, cfg.freqs)
    yee = yee_from_config(cfg, mat, eps_table(cfg))
    for n in range(nsteps):
        fl.step(n, src[n])
        yee.update_H()
        yee.update_E(src[n], cfg.src_k)
    for names, ref in ((("Ex", "Ey", "Ez"), yee.E), (("Hx", "Hy", "Hz"), yee.H), (("JDx", "JDy", "JDz"), yee.JD)):
        scale = max(np.abs(r).max() for r in ref)
        assert scale > 0
        for nm, r in zip(names, ref):
            assert np.abs(getattr(fl, nm).cpu().numpy() - r).max() < 1e-11 * scale, nm
