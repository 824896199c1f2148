"""Gridded reciprocal sums of a batch of 1400 small frames on 48^3 meshes: 67 200 x
planes, more blocks than the grid's y and z dimensions take (65 536), forward and
adjoint, against the CPU oracle.

Tolerance: as for the other gridded sums, 1e-12 of each output's largest element."""
import numpy as np
import pytest
import torch

from paper_2408_03273_amd import workloads as wl
from paper_2408_03273_amd.ewald import EwaldConfig, Plan
from tests import _harness as H

pytestmark = pytest.mark.gpu
TOL = 1e-12
FRAMES = 1400


def test_more_planes_than_a_grid_dimension(monkeypatch):
    monkeypatch.setenv("MPEWALD_MESH", "1")
    kinds = [wl.random_system(820 + i, 1 + i % 3, 5 + 7 * i, box=(18.0, 19.0 + i, 20.0), alpha=0.35, rcut=8.0,
                              kmax=(3, 4, 3), neutral=False) for i in range(5)]
    fr = [kinds[i % 5] for i in range(FRAMES)]
    qo, mo = np.cumsum([0] + [f.nq for f in fr]), np.cumsum([0] + [f.nm for f in fr])
    plan = Plan(EwaldConfig(box=tuple(fr[0].box), alpha=0.35, rcut=8.0, kmax=(3, 4, 3), max_qm=int(qo[-1]),
                            max_mm=int(mo[-1]), max_frames=FRAMES))
    assert "mesh=48x48x48" in plan.describe() and FRAMES * 48 > 65536
    cat = lambda k: torch.tensor(np.concatenate([getattr(f, k) for f in fr]), dtype=torch.float64,  # noqa: E731
                                 device="cuda")
    desc = [dict(box=f.box, n_qm=f.nq, n_mm=f.nm, qm_offset=int(qo[i]), mm_offset=int(mo[i]))
            for i, f in enumerate(fr)]
    out = plan.batch(desc, cat("qm_pos"), cat("Q"), cat("mu"), cat("theta"), cat("mm_pos"), cat("q"))
    got = {k: out[k].cpu().numpy() for k in out}
    refs = [H.oracle_outputs(f) for f in kinds]
    worst = 0.0
    for i, f in enumerate(fr):
        q, m = slice(qo[i], qo[i + 1]), slice(mo[i], mo[i + 1])
        one = dict(energy=got["energy"][i], phi=got["phi"][q], efield=got["efield"][q], efgrad=got["efgrad"][q],
                   g_qm_pos=got["g_qm_pos"][q], g_Q=got["g_Q"][q], g_mu=got["g_mu"][q], g_theta=got["g_theta"][q],
                   g_mm_pos=got["g_mm_pos"][m], g_mm_q=got["g_mm_q"][m])
        errs = H.compare(one, refs[i % 5], H.FWD_KEYS + H.BWD_KEYS)
        assert max(errs.values()) <= TOL, (i, errs)
        worst = max(worst, max(errs.values()))
    print(f"[mesh] {FRAMES} frames, worst {worst:.1e}", flush=True)
