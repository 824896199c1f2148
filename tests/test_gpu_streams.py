"""Forward+backward on the caller's stream alone and with the adjoint and real space on
two more streams, forced each way, for the dense and the gridded reciprocal sums, with real
space by pairs, by tiles (from 64 x 1024 atoms on) and for batches: each schedule
against the CPU oracle, several calls in a row on one plan.  A wait that is missing between
two streams would let a kernel read what another has not written yet.

Tolerance: sums of up to 7e4 terms as a random walk, 265 x 1.1e-16, and one digit of
cancellation: 1e-12 of each output's largest element."""
import numpy as np
import pytest
import torch

from paper_2408_03273_amd import workloads as wl
from paper_2408_03273_amd.ewald import EwaldConfig, Plan
from tests import _harness as H

pytestmark = pytest.mark.gpu
TOL = 1e-12
ALL = H.FWD_KEYS + H.BWD_KEYS


@pytest.mark.parametrize("serial", ["0", "1"])
@pytest.mark.parametrize("mesh", ["0", "1"])
@pytest.mark.parametrize("nm", [3000, 65537])
def test_single_frame(nm, mesh, serial, monkeypatch):
    monkeypatch.setenv("MPEWALD_MESH", mesh)
    monkeypatch.setenv("MPEWALD_SERIAL", serial)
    s = wl.random_system(880, 9, nm, box=(40.0, 41.0, 42.0), alpha=0.25, rcut=10.0, kmax=(8, 9, 7), neutral=False)
    plan = H.make_plan(s)
    ref = H.oracle_outputs(s)
    for _ in range(4):
        errs = H.compare(H.gpu_outputs(s, plan=plan), ref, ALL)
        assert max(errs.values()) <= TOL, errs
    assert plan.describe().endswith(" sums=mesh") == (mesh == "1")


@pytest.mark.parametrize("serial", ["0", "1"])
@pytest.mark.parametrize("mesh", ["0", "1"])
def test_batch(mesh, serial, monkeypatch):
    monkeypatch.setenv("MPEWALD_MESH", mesh)
    monkeypatch.setenv("MPEWALD_BATCH_SERIAL", serial)
    fr = [wl.random_system(881 + i, 3 + 5 * i, 900 + 400 * i, box=(22.0, 23.0 + i, 24.0), alpha=0.33, rcut=9.0,
                           kmax=(9, 10, 11), neutral=False) for i in range(3)]
    qo, mo = np.cumsum([0] + [f.nq for f in fr]), np.cumsum([0] + [f.nm for f in fr])
    plan = Plan(EwaldConfig(box=tuple(fr[0].box), alpha=0.33, rcut=9.0, kmax=(9, 10, 11), max_qm=int(qo[-1]),
                            max_mm=int(mo[-1]), max_frames=3))
    cat = lambda k: torch.tensor(np.concatenate([getattr(f, k) for f in fr]), dtype=torch.float64,  # noqa: E731
                                 device="cuda")
    desc = [dict(box=f.box, n_qm=f.nq, n_mm=f.nm, qm_offset=int(qo[i]), mm_offset=int(mo[i]))
            for i, f in enumerate(fr)]
    x = [cat(k) for k in ("qm_pos", "Q", "mu", "theta", "mm_pos", "q")]
    refs, out = [H.oracle_outputs(f) for f in fr], None
    for _ in range(4):
        out = plan.batch(desc, *x, out=out)
        got = {k: v.cpu().numpy() for k, v in out.items()}
        for i in range(3):
            q, m = slice(qo[i], qo[i + 1]), slice(mo[i], mo[i + 1])
            one = {k: got[k][i] if k == "energy" else got[k][m if k.startswith("g_mm") else q] for k in ALL}
            errs = H.compare(one, refs[i], ALL)
            assert max(errs.values()) <= TOL, (i, errs)
    assert plan.describe().endswith(" sums=mesh") == (mesh == "1")
