"""How the library decides to make a projection (tdp_gemm_plan, a host function): checked against what launches of it measured."""
import pytest

from paper_2506_10470_amd import tdp

WORKSPACE = 64 << 20            # floats: what a stage of these shapes has

# The QKV projection and the rotation behind it inside a stage, microseconds together on an MI355X:
# (M, N, K): {(rows of a tile, weight rows, splits): time}
MEASURED = {
    (256, 15360, 5120): {(128, 128, 1): 91.2, (256, 128, 2): 87.0, (128, 256, 2): 86.8, (256, 256, 4): 90.1},
    (512, 15360, 5120): {(256, 128, 1): 129.0, (256, 256, 2): 122.8, (128, 256, 1): 132.1},
    (256, 12288, 4096): {(128, 128, 1): 82.4, (256, 128, 2): 79.1, (256, 256, 4): 77.4, (128, 256, 2): 77.7},
    (512, 7168, 5120): {(128, 128, 1): 72.9, (256, 128, 2): 63.1, (128, 256, 2): 64.9, (192, 256, 3): 64.2, (256, 256, 4): 64.2},
    (384, 10240, 8192): {(128, 128, 1): 102.9, (192, 256, 3): 85.9, (128, 256, 2): 91.6},
    (512, 10240, 8192): {(256, 256, 3): 98.4, (256, 128, 2): 139.6, (256, 256, 2): 115.6},
}


@pytest.mark.parametrize("shape", MEASURED)
def test_qkv_of_a_stage_is_made_within_3_percent_of_the_fastest_measured_way(shape):
    p = tdp.tdp_gemm_plan(*shape, epilogue=0, deferred=True, workspace_elems=WORKSPACE)
    way = (p["rows"], p["weight_rows"], p["splits"])
    times = MEASURED[shape]
    assert way in times, "%s: a way that was not timed: %s" % (shape, way)
    assert times[way] <= 1.03 * min(times.values()), (shape, way)


def test_plan_entry_rejects_bad_arguments():
    import ctypes as C
    out = (C.c_int32 * 5)()
    P = tdp.lib.tdp_gemm_plan
    for M, N, K, epi, deferred, ws in [(0, 64, 64, 0, 0, 0), (1, 66, 64, 0, 0, 0), (1, 64, 100, 0, 0, 0), (1, 64, 64, 3, 0, 0),
                                       (1, 68, 64, 2, 0, 0), (1, 64, 64, 2, 1, 0), (1, 64, 64, 0, 0, -1)]:
        assert P(M, N, K, epi, deferred, ws, out) == tdp.EINVAL
    assert P(1, 64, 64, 0, 0, 0, None) == tdp.EINVAL
    assert P(1, 64, 64, 0, 0, 0, out) == tdp.OK and out[3] == 1 and out[4] == 0
