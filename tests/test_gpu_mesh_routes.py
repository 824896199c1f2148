"""The routes beside the fused forward+backward step that take the gridded reciprocal
sums: the full adjoint with gradients of the field outputs, the adjoint after a
moments-only update, a forward pass without a context on unwrapped positions, forward-only and
deterministic batches, and non-finite input, against the CPU oracle; each checks that the
call did take the mesh.

Tolerance: as for the other gridded sums, 1e-12 of each output's largest element."""
import numpy as np
import pytest
import torch

from oracle.oracle import oracle_ewald
from paper_2408_03273_amd import workloads as wl
from paper_2408_03273_amd.ewald import EwaldConfig, Plan
from tests import _harness as H

pytestmark = pytest.mark.gpu
TOL = 1e-12


@pytest.fixture(autouse=True)
def _mesh(monkeypatch):
    monkeypatch.setenv("MPEWALD_MESH", "1")


def _system(seed=861, nq=5, nm=1800, box=(22.0, 23.0, 25.0)):
    return wl.random_system(seed, nq, nm, box=box, alpha=0.33, rcut=9.0, kmax=(10, 11, 12), neutral=False)


def _plan(s, nq=None, nm=None, frames=1, **kw):
    return Plan(EwaldConfig(box=tuple(s.box), alpha=s.alpha, rcut=s.rcut, kmax=s.kmax, max_qm=nq or s.nq,
                            max_mm=nm or s.nm, max_frames=frames, **kw))


def _x(s):
    d = H.to_dev(s)
    return [d[k] for k in ("qm_pos", "Q", "mu", "theta", "mm_pos", "mm_q")]


def _took_mesh(plan):
    assert plan.describe().endswith(" sums=mesh"), plan.describe()


def _oracle(s, Q, mu, theta, qmqm):
    return oracle_ewald(s.box, s.alpha, s.rcut, s.kmax, s.qm_pos, Q, mu, theta, s.mm_pos, s.q, qmqm=qmqm)


@pytest.mark.parametrize("deterministic", [False, True])
def test_gradients_of_the_field_outputs(deterministic):
    """By linearity of the QM-MM energy in the moments, the gradient of a E + g_phi.phi +
    g_F.efield + g_G.efgrad is a times the QM-QM part plus the QM-MM part of the moments
    (a Q + g_phi, a mu - g_F, a theta - (2,1,1,2,1,2) g_G)."""
    s = _system()
    plan, x = _plan(s, deterministic=deterministic), _x(s)
    rng = np.random.default_rng(5)
    a, gphi, gF, gG = 0.7, rng.normal(size=s.nq), rng.normal(size=(s.nq, 3)), rng.normal(size=(s.nq, 6))
    up = [torch.tensor(v, dtype=torch.float64, device="cuda") for v in (a, gphi, gF, gG)]
    ctx = plan.forward(*x, want_ctx=True)[4]
    runs = []
    for _ in range(3):
        runs.append([v.cpu().numpy() for v in plan.backward(ctx, *x, *up)])
        _took_mesh(plan)
    full, mm = _oracle(s, s.Q, s.mu, s.theta, True), _oracle(s, s.Q, s.mu, s.theta, False)
    eff = _oracle(s, a * s.Q + gphi, a * s.mu - gF, a * s.theta - np.array([2, 1, 1, 2, 1, 2.0]) * gG, False)
    ref = dict(g_qm_pos=a * (full.g_qm_pos - mm.g_qm_pos) + eff.g_qm_pos, g_Q=a * full.g_Q, g_mu=a * full.g_mu,
               g_theta=a * full.g_theta, g_mm_pos=eff.g_mm_pos, g_mm_q=eff.g_mm_q)
    for r in runs:
        errs = H.compare(dict(zip(H.BWD_KEYS, r)), ref, H.BWD_KEYS)
        assert max(errs.values()) <= TOL, errs
        assert not deterministic or all(np.array_equal(u, v) for u, v in zip(r, runs[0]))


def test_adjoint_after_a_moments_update():
    s = _system(862)
    plan, x = _plan(s), _x(s)
    ctx = plan.forward(*x, want_ctx=True)[4]
    rng = np.random.default_rng(8)
    s.Q, s.mu, s.theta = rng.uniform(-0.9, 0.9, s.nq), rng.normal(0, 0.15, (s.nq, 3)), rng.normal(0, 0.08, (s.nq, 6))
    x[1:4] = _x(s)[1:4]
    E, gQ, gmu, gth = plan.update_moments(ctx, *x[:4], s.nm)
    g = plan.backward(ctx, *x)
    _took_mesh(plan)
    ref = H.oracle_outputs(s)
    errs = H.compare(dict(zip(H.BWD_KEYS, (v.cpu().numpy() for v in g))), ref, H.BWD_KEYS)
    up = dict(energy=E.cpu().numpy(), g_Q=gQ.cpu().numpy(), g_mu=gmu.cpu().numpy(), g_theta=gth.cpu().numpy())
    errs.update({"update " + k: v for k, v in H.compare(up, ref, tuple(up)).items()})
    assert max(errs.values()) <= TOL, errs


@pytest.mark.parametrize("backward", [False, True])
def test_unwrapped_positions(backward):
    """Every MM atom moved by up to two and every QM site by one box length per axis, which
    rounds a coordinate to 8e-15 of 70: forces of alpha 0.33 move by 1e-14 of theirs."""
    s = _system(863)
    rng = np.random.default_rng(9)
    s.mm_pos += rng.integers(-2, 3, size=s.mm_pos.shape) * s.box
    s.qm_pos += rng.integers(-1, 2, size=s.qm_pos.shape) * s.box
    plan = _plan(s)
    got = H.gpu_outputs(s, plan=plan, backward=backward)
    _took_mesh(plan)
    errs = H.compare(got, H.oracle_outputs(s), H.FWD_KEYS + (H.BWD_KEYS if backward else ()))
    assert max(errs.values()) <= TOL, errs


def _pack(fr):
    qo, mo = np.cumsum([0] + [f.nq for f in fr]), np.cumsum([0] + [f.nm for f in fr])
    desc = [dict(box=f.box, n_qm=f.nq, n_mm=f.nm, qm_offset=int(qo[i]), mm_offset=int(mo[i]))
            for i, f in enumerate(fr)]
    return desc, [torch.cat(v) for v in zip(*(_x(f) for f in fr))], qo, mo


def _check_frames(fr, out, qo, mo, keys, skip=()):
    got = {k: v.cpu().numpy() for k, v in out.items()}
    for i, f in enumerate(fr):
        if i in skip:
            continue
        q, m = slice(qo[i], qo[i + 1]), slice(mo[i], mo[i + 1])
        one = {k: got[k][i] if k == "energy" else got[k][m if k.startswith("g_mm") else q] for k in keys}
        errs = H.compare(one, H.oracle_outputs(f), keys)
        assert max(errs.values()) <= TOL, (i, errs)


def _frames():
    return [_system(864, 3, 1300), _system(865, 17, 64, (21.0, 21.0, 24.0)), _system(866, 6, 2049, (20.0, 24.0, 22.0))]


@pytest.mark.parametrize("deterministic", [False, True])
@pytest.mark.parametrize("with_grad", [False, True])
def test_batches(with_grad, deterministic):
    fr = _frames()
    desc, x, qo, mo = _pack(fr)
    plan = _plan(fr[0], int(qo[-1]), int(mo[-1]), 3, deterministic=deterministic)
    keys = H.FWD_KEYS + (H.BWD_KEYS if with_grad else ())
    out, first = None, None
    for _ in range(3):  # capture and replays
        out = plan.batch(desc, *x, with_grad=with_grad, out=out)
        _took_mesh(plan)
        _check_frames(fr, out, qo, mo, keys)
        first = first or {k: v.clone() for k, v in out.items()}
        assert not deterministic or all(torch.equal(out[k], first[k]) for k in out)


@pytest.mark.parametrize("where,bad", [("mm_pos", np.nan), ("mm_pos", np.inf), ("q", np.nan), ("Q", np.nan)])
def test_non_finite_input(where, bad):
    """The bad frame's energy is NaN, a batch's other frames are exact, and the next clean
    call of the same plan is exact."""
    fr = _frames()
    desc, x, qo, mo = _pack(fr)
    plan = _plan(fr[0], int(qo[-1]), int(mo[-1]), 3)
    y = [v.clone() for v in x]
    {"mm_pos": y[4][int(mo[2]) + 17], "q": y[5][int(mo[2]) + 17:], "Q": y[1][int(qo[2]) + 1:]}[where][:1] = bad
    print(f"[mesh] batch with {where} = {bad}", flush=True)
    out = plan.batch(desc, *y)
    _took_mesh(plan)
    assert torch.isnan(out["energy"][2])
    _check_frames(fr, out, qo, mo, H.FWD_KEYS + H.BWD_KEYS, skip=(2,))
    _check_frames(fr, plan.batch(desc, *x), qo, mo, H.FWD_KEYS + H.BWD_KEYS)
    # single frame, fused and full adjoint
    s = fr[2]
    z = [v[int(o[2]):int(o[3])].contiguous() for v, o in zip(y, (qo, qo, qo, qo, mo, mo))]
    E, phi, _, _, ctx = plan.forward(*z, want_ctx=True)
    plan.backward(ctx, *z, g_phi=torch.ones_like(phi))
    assert torch.isnan(E)
    single = _plan(s)
    errs = H.compare(H.gpu_outputs(s, plan=single), H.oracle_outputs(s), H.FWD_KEYS + H.BWD_KEYS)
    assert max(errs.values()) <= TOL, errs
