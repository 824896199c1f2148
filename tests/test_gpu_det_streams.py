"""Deterministic plans give the same bytes on one stream and on three, whichever the size
rule takes: few and many sites, and lattice images; the counts of partial sums (columns of
the k grid, sites) lie at and around the eight that the fixed-order sums hold in flight."""
import numpy as np
import pytest

from paper_2408_03273_amd import workloads as wl
from paper_2408_03273_amd.ewald import EwaldConfig, Plan
from tests import _harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,nm,kmax,rcut", [(1, 300, (1, 1, 1), 9.0), (8, 1500, (3, 5, 7), 9.0), (16, 900, (6, 4, 4), 9.0),
                                             (101, 700, (8, 8, 8), 9.0), (5, 400, (5, 5, 6), 18.0),
                                             (13, 400, (5, 5, 6), 18.0)])
def test_one_stream_and_three(nq, nm, kmax, rcut, monkeypatch):
    s = wl.random_system(900 + nq, nq, nm, box=(25.0, 26.0, 27.0), alpha=0.25, rcut=rcut, kmax=kmax, neutral=False)
    ref = H.oracle_outputs(s)
    outs = []
    for serial in (None, "0", "1"):
        if serial is not None:
            monkeypatch.setenv("MPEWALD_SERIAL", serial)
        plan = Plan(EwaldConfig(box=tuple(s.box), alpha=s.alpha, rcut=s.rcut, kmax=s.kmax, max_qm=s.nq, max_mm=s.nm,
                                deterministic=True))
        outs += [H.gpu_outputs(s, plan=plan) for _ in range(2)]
    errs = H.compare(outs[0], ref, H.FWD_KEYS + H.BWD_KEYS)
    assert max(errs.values()) <= 1e-10, errs  # the parity bar
    for o in outs[1:]:
        assert all(np.array_equal(o[k], outs[0][k]) for k in o)
