"""Small meshes with many charges: a frame's few tiles make spreading the slower way, so
forward sums go dense there, in a forward pass alone sooner than with the adjoint, while the
adjoint alone, which spreads nothing, takes the mesh; batches fill the GPU with more
tiles.  Either way the outputs are those of the other sums.

Tolerance: both sides sum up to 1e5 terms in FP64: 1e-12 of each output's largest element."""
import numpy as np
import pytest
import torch

from paper_2408_03273_amd.ewald import EwaldConfig, Plan
from tests import _harness as H

pytestmark = pytest.mark.gpu
TOL = 1e-12


def _inputs(nq, nm, box, seed=7):
    r = np.random.default_rng(seed)
    a = (box / 2 + r.uniform(-2, 2, (nq, 3)), r.uniform(-0.5, 0.5, nq), r.normal(0, 0.2, (nq, 3)),
         r.normal(0, 0.1, (nq, 6)), r.uniform(0, box, (nm, 3)), r.uniform(-0.9, 0.9, nm))
    return [torch.tensor(v, dtype=torch.float64, device="cuda") for v in a]


def _plan(nq, nm, box, m, frames=1):
    # pi m / (alpha L) = 4.5: the smallest meshes
    return Plan(EwaldConfig(box=(box,) * 3, alpha=np.pi * m / (4.5 * box), rcut=9.0, kmax=(m,) * 3, max_qm=nq, max_mm=nm,
                            max_frames=frames))


def _sums(plan):
    return plan.describe().split("sums=")[1]


@pytest.mark.parametrize("nm,m,mesh,forward,both", [(60000, 14, 48, "dense", "dense"), (40000, 16, 64, "dense", "mesh"),
                                                    (30000, 20, 80, "mesh", "mesh")])
def test_single_frame(nm, m, mesh, forward, both, monkeypatch):
    x = _inputs(6, nm, 50.0)
    plan = _plan(6, nm, 50.0, m)
    assert f"mesh={mesh}x{mesh}x{mesh}" in plan.describe()
    got = plan.forward(*x)[:4]
    assert _sums(plan) == forward
    *full, ctx = plan.forward(*x, want_ctx=True)
    assert _sums(plan) == both
    g = plan.backward(ctx, *x, g_phi=torch.ones_like(x[1]))
    assert _sums(plan) == "mesh"
    monkeypatch.setenv("MPEWALD_MESH", "0")
    dense = _plan(6, nm, 50.0, m)
    *ref, ctx = dense.forward(*x, want_ctx=True)
    ref_g = dense.backward(ctx, *x, g_phi=torch.ones_like(x[1]))
    for a, b in zip([*got, *full, *g], [*ref, *ref, *ref_g]):
        assert H.relerr(a.cpu().numpy(), b.cpu().numpy()) <= TOL


@pytest.mark.parametrize("with_grad", [False, True])
def test_batch_of_the_same_mesh(with_grad):
    frames, nm, m = 8, 30000, 14
    x = _inputs(3 * frames, nm * frames, 50.0)
    plan = _plan(3 * frames, nm * frames, 50.0, m, frames)
    desc = [dict(box=(50.0,) * 3, n_qm=3, n_mm=nm, qm_offset=3 * i, mm_offset=nm * i) for i in range(frames)]
    plan.batch(desc, *x, with_grad=with_grad)
    assert _sums(plan) == "mesh"
    torch.cuda.synchronize()
