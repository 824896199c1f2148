"""QM-site projection (matrix cores, tiles of 16 sites x 16 (nx, ny) columns x 4
values of |nz|) against the CPU oracle at the edges of its tiles: 1, 15, 16, 17
and 33 sites, fewer columns than a tile, |nz| counts of one step, of whole steps
and with remainders, and the split of the |nz| range; with and without the
QM-QM sums, forward only, fused and with upstream field gradients, in both
summation orders.

Tolerance: sums of at most 1e4 terms in FP64, as a random walk 1e2 x 1.1e-16,
and up to two digits of cancellation between them: 1e-12 of each output's
largest element."""
import numpy as np
import pytest
import torch

from paper_2408_03273_amd import workloads as wl
from paper_2408_03273_amd.ewald import EwaldConfig, Plan
from tests import _harness as H

pytestmark = pytest.mark.gpu
TOL = 1e-12

CASES = [
    # nq, kmax, qmqm, deterministic
    (1, (1, 1, 1), True, False),
    (15, (2, 3, 6), True, False),
    (16, (3, 2, 7), True, True),
    (17, (2, 5, 8), True, False),
    (17, (4, 3, 3), False, False),
    (33, (6, 5, 11), True, True),
    (33, (5, 7, 12), True, False),
]


@pytest.mark.parametrize("nq,kmax,qmqm,det", CASES)
def test_projection_tiles(nq, kmax, qmqm, det):
    s = wl.random_system(100 + nq, nq, 150, box=(19.0, 22.0, 20.0), alpha=0.32, rcut=8.5, kmax=kmax, neutral=False)
    plan = Plan(EwaldConfig(box=tuple(s.box), alpha=s.alpha, rcut=s.rcut, kmax=s.kmax, max_qm=nq, max_mm=s.nm,
                            qmqm=qmqm, deterministic=det))
    ref = H.oracle_outputs(s, qmqm=qmqm)
    fused = H.compare(H.gpu_outputs(s, plan=plan), ref, H.FWD_KEYS + H.BWD_KEYS)
    fwd = H.compare(H.gpu_outputs(s, plan=plan, backward=False), ref, H.FWD_KEYS)
    d = H.to_dev(s)
    args = [d[k] for k in ("qm_pos", "Q", "mu", "theta", "mm_pos", "mm_q")]
    _, phi, ef, eg, ctx = plan.forward(*args, want_ctx=True)
    z = torch.zeros_like
    g = plan.backward(ctx, *args, gE=torch.ones((), dtype=torch.float64, device="cuda"), g_phi=z(phi), g_efield=z(ef),
                      g_efgrad=z(eg))
    names = ("g_qm_pos", "g_Q", "g_mu", "g_theta", "g_mm_pos", "g_mm_q")
    adj = H.compare({k: v.cpu().numpy() for k, v in zip(names, g)}, ref, names)
    worst = max(max(e.values()) for e in (fused, fwd, adj))
    print(f"[project] nq {nq} kmax {kmax}: {worst:.1e}", flush=True)
    assert np.isfinite(worst) and worst <= TOL, (fused, fwd, adj)
