"""The plan names the reciprocal sums that its last call took: the mesh where it pays
or is forced, the dense sums for small calls, boxes with too little damping and frames that
share MM rows, call by call on one plan."""
import pytest
import torch

from paper_2408_03273_amd import workloads as wl
from paper_2408_03273_amd.ewald import EwaldConfig, Plan
from tests import _harness as H
from tests import test_gpu_mesh as mesh_cases

pytestmark = pytest.mark.gpu


def _plan(s, frames=1, **kw):
    return Plan(EwaldConfig(box=tuple(s.box), alpha=s.alpha, rcut=s.rcut, kmax=s.kmax, max_qm=frames * s.nq,
                            max_mm=s.nm, max_frames=frames, **kw))


def _x(s):
    d = H.to_dev(s)
    return [d[k] for k in ("qm_pos", "Q", "mu", "theta", "mm_pos", "mm_q")]


def test_report_by_call(monkeypatch):
    monkeypatch.setenv("MPEWALD_MESH", "1")
    s = wl.random_system(840, 3, 500, box=(20.0, 20.0, 20.0), alpha=0.3, rcut=9.0, kmax=(14, 14, 14))
    plan, x = _plan(s, frames=2), _x(s)
    assert "mesh=" in plan.describe() and "sums=" not in plan.describe()
    ctx = plan.forward(*x, want_ctx=True)[4]
    assert plan.describe().endswith(" sums=mesh")
    plan.set_box((44.0, 44.0, 44.0))
    plan.forward(*x)
    assert plan.describe().endswith(" sums=dense")
    plan.set_box(s.box)
    plan.backward(ctx, *x, g_phi=torch.ones_like(x[1]))
    assert plan.describe().endswith(" sums=mesh")
    frame = dict(box=s.box, n_qm=1, n_mm=250, qm_offset=0, mm_offset=0)
    for second, sums in ((0, "dense"), (250, "mesh"), (249, "dense")):
        plan.batch([frame, dict(frame, qm_offset=1, mm_offset=second)], *x)
        assert plan.describe().endswith(f" sums={sums}")
    torch.cuda.synchronize()


def test_report_by_size_and_precision():
    s = wl.random_system(841, 3, 60000, box=(60.0, 60.0, 60.0), alpha=0.25, rcut=9.0, kmax=(20, 20, 20), min_qm_mm=0.8)
    for kw, n, sums in ((dict(), s.nm, " sums=mesh"), (dict(), 2000, " sums=dense"),
                        (dict(precision="fp32_recip"), s.nm, ""), (dict(plain=True), 2000, "")):  # plans without a mesh
        plan = _plan(s, **kw)
        before, x = plan.describe(), _x(s)
        plan.forward(*x[:4], x[4][:n].contiguous(), x[5][:n].contiguous())
        assert plan.describe() == before + sums and ("mesh=" in before) == bool(sums), (kw, n, plan.describe())
    torch.cuda.synchronize()


@pytest.mark.parametrize("case", mesh_cases.CASES, ids=lambda c: f"seed{c[0]}")
def test_the_mesh_cases_take_the_mesh(case, monkeypatch):
    monkeypatch.setenv("MPEWALD_MESH", "1")
    s = mesh_cases._system(*case)
    plan = H.make_plan(s)
    H.gpu_outputs(s, plan=plan)
    assert plan.describe().endswith(" sums=mesh")
