"""The smoother's executed share of Alg. 3's flops against a count phase by phase."""
import pytest

import bench


def test_sap_executed_share():
    w = bench.WORKLOADS["c3"]
    formed, carried, mr = 1848, 330, bench.sap_flops_per_site(w["block"], 4) - 1848
    done = phases = 0
    for n in (1, 2, 3):  # initial passes on the test vectors, from zero
        for ph in range(2 * n):
            done += w["ntv"] * (mr + (0 if ph == 0 else carried))
            phases += w["ntv"]
    for nrhs, cycles in ((w["ntv"], 3), (w["nrhs"], 6)):  # V-cycles of the setup, of the solve
        for ph in range(6):
            done += nrhs * cycles * (mr + (formed if ph < 2 else carried))
            phases += nrhs * cycles
    assert bench.sap_executed_share(w, 5 * phases, 5) == pytest.approx(done / (phases * (mr + formed)))
    assert bench.sap_executed_share(bench.WORKLOADS["c1"], 100, 1) == 1.0
