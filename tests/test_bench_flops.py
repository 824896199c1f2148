"""The benchmark charges the flops of the sums that the plan's last call took."""
import bench

KMAX, NM = (24, 24, 24), 35000.0
PLAN = "fwd=mfma-fold ct=2 nt=3 xcd=1 blocks~1024 kgrid=25x49x49 precision=fp64"


def test_flops_of_the_sums_that_ran():
    dense = bench.recip_flops(PLAN, KMAX, NM)
    assert dense[0] == {"sfac_mm": 4.0 * 58824 * NM, "force_mm": 6.0 * 58824 * NM}
    assert bench.recip_flops(PLAN + " mesh=80x80x80 sums=dense", KMAX, NM) == dense  # a mesh that the call did not take
    assert bench.recip_flops(PLAN + " mesh=80x80x80", KMAX, NM) == dense             # no call yet
    mesh = bench.recip_flops(PLAN + " mesh=80x80x80 sums=mesh", KMAX, NM)
    contract = 2.0 * (80 ** 3 * 49 + 80 ** 2 * 49 ** 2 + 80 * 49 ** 3)
    assert mesh[0] == {"mesh_sfac": 8192.0 * NM + contract, "mesh_force": 16384.0 * NM + contract} == mesh[1]
