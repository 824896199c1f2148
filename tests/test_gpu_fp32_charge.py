"""FP32 pair terms in the adjoint with gradients of the field outputs: the MM charge
multiplies the gradient in FP64.  Pair terms, phases and weights do not depend on
the charges, so dL/dR of an atom of charge 1 + 2^-25, which FP32 cannot hold, divided by
it is dL/dR at charge 1, by pairs (minimum image) and per atom (images, deterministic).

Tolerance: FP64 rounding of sums of 2e3 terms as a random walk, 45 x 1.1e-16, and two digits
of cancellation: 1e-12 of the largest element (a charge in FP32 gives 3e-8)."""
import pytest
import torch

from paper_2408_03273_amd import workloads as wl
from paper_2408_03273_amd.ewald import EwaldConfig, Plan
from tests import _harness as H

pytestmark = pytest.mark.gpu
TOL = 1e-12


@pytest.mark.parametrize("rcut,deterministic", [(9.0, False), (9.0, True), (19.0, False)])
def test_gradient_is_linear_in_the_charge(rcut, deterministic):
    s = wl.random_system(890, 6, 500, box=(20.0, 21.0, 22.0), alpha=0.3, rcut=rcut, kmax=(6, 6, 7), neutral=False)
    plan = Plan(EwaldConfig(box=tuple(s.box), alpha=s.alpha, rcut=s.rcut, kmax=s.kmax, max_qm=s.nq, max_mm=s.nm,
                            precision="fp32_real", deterministic=deterministic))
    d = H.to_dev(s)
    x = [d[k] for k in ("qm_pos", "Q", "mu", "theta", "mm_pos")]
    up = dict(g_phi=torch.ones(s.nq, dtype=torch.float64, device="cuda"))
    g = []
    for q in (1.0, 1.0 + 2.0 ** -25):
        charge = torch.full((s.nm,), q, dtype=torch.float64, device="cuda")
        ctx = plan.forward(*x, charge, want_ctx=True)[4]
        g.append(plan.backward(ctx, *x, charge, **up)[4].cpu().numpy() / q)
    assert H.relerr(g[1], g[0]) <= TOL
