"""The guard of the held-current array: at a molecular update, every occupied cell
outside the held planes sets its coupled E components to NaN and nothing else does,
whatever order the caller's CSR lists the cells in.  Expected values are exact (NaN or
finite), so there is no tolerance."""

import numpy as np
import pytest
import torch

from gpu_helpers import banner
from workloads import get_config
from workloads.pulses import source_values

pytestmark = pytest.mark.gpu


def _reorder(sysm, order):
    """List the run's occupied cells in another order (occ_cell, occ_ptr, mol_perm)."""
    occ, ptr, perm = (t.cpu().numpy() for t in (sysm.occ_cell, sysm.occ_ptr, sysm.mol_perm))
    n = len(occ)
    o = np.arange(n)[::-1] if order == "descending" else np.random.default_rng(3).permutation(n)
    new_ptr = np.concatenate([[0], np.cumsum(np.diff(ptr[:n + 1])[o])])
    new_perm = np.concatenate([perm[ptr[c]:ptr[c + 1]] for c in o])
    for t, v in ((sysm.occ_cell, occ[o]), (sysm.occ_ptr[:n + 1], new_ptr), (sysm.mol_perm, new_perm)):
        t.copy_(torch.as_tensor(np.ascontiguousarray(v, np.int32)))


@pytest.mark.parametrize("k0, nk", [(23, 1), (12, 2)])     # none of the cells, and those of planes 12 and 13, held
@pytest.mark.parametrize("prec, basis, order", [("fp64", "m0", "shuffled"), ("fp32", "m0", "descending"),
                                                ("fp64", "jm", "shuffled")])
def test_guard_does_not_depend_on_the_cells_order(prec, basis, order, k0, nk):
    from paper_2209_04487_amd import msqd
    cfg = get_config("cfg0", j_max=2, basis=basis)
    banner(f"held guard {prec} {basis} {order} planes {k0}+{nk}")
    sysm = msqd.Coupled(cfg, prec=prec)
    assert (sysm.desc.held_k0, sysm.desc.held_nk) == (10, 4)
    _reorder(sysm, order)
    sysm.desc.held_k0, sysm.desc.held_nk = k0, nk
    sysm.step(source_values(cfg, 0, 1))
    torch.cuda.synchronize()
    occ = sysm.occ_cell.cpu().numpy()
    k = occ // (cfg.nx * cfg.ny)
    outside = occ[(k < k0) | (k >= k0 + nk)]
    assert 0 < len(outside)
    for nm in ("Ex", "Ey", "Ez"):
        e = getattr(sysm.fields, nm).cpu().numpy().reshape(-1)
        want = np.zeros(e.shape, bool)
        if nm == "Ex" or basis == "jm":
            want[outside] = True
        assert np.array_equal(np.isnan(e), want), nm
        assert np.isfinite(e[~want]).all()


def test_guard_of_runs_that_share_a_field_workspace():
    """Runs on streams of their own with one field workspace: two whose cells lie outside
    their held planes are marked at their update, and one with the right planes keeps the
    bits it has with a workspace of its own, also after the others marked its planes."""
    from paper_2209_04487_amd import msqd
    cfg = get_config("cfg0")
    banner("held guard with a shared field workspace")
    src = source_values(cfg, 0, 12)
    runs = [msqd.Coupled(cfg, prec="fp64") for _ in range(4)]
    alone, good, bad = runs[0], runs[1], runs[2:]
    for r in runs[1:]:
        r.state.fd_ws = good.state.fd_ws
    for r in bad:
        r.desc.held_k0, r.desc.held_nk = cfg.nz - 1, 1
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in runs]
    for r, st in zip(runs, streams):
        with torch.cuda.stream(st):
            r.step(src[:1])
    torch.cuda.synchronize()
    for r in bad:
        ex = r.fields.Ex.cpu().numpy().reshape(-1)
        want = np.zeros(ex.shape, bool)
        want[r.occ_cell.cpu().numpy()] = True
        assert np.array_equal(np.isnan(ex), want)
    for r, st in zip(runs, streams):
        with torch.cuda.stream(st):
            r.step(src[1:])
    torch.cuda.synchronize()
    assert float(alone.J_mol.abs().max()) > 0
    for k in alone._STATE:
        assert torch.equal(alone.fields.t[k], good.fields.t[k]), k
    for a, b in ((alone.mol.psi, good.mol.psi), (alone.P_c, good.P_c), (alone.J_mol, good.J_mol)):
        assert torch.equal(a, b)
