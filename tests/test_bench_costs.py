"""The benchmark's cost model counts what the fused call moves: an element per step
(FP64, FP32 up to d = 3) or an element per lane and d + 3 FP64 values per step."""
import pytest

import bench


@pytest.mark.parametrize("chunk", [4, 16, 64])
@pytest.mark.parametrize("d,tsize", [(1, 4), (2, 4), (3, 4), (2, 8), (6, 8), (8, 8)])
def test_element_per_step(d, tsize, chunk):
    assert bench.fused_costs(d, tsize, chunk) == bench.pass_costs(d, tsize, chunk)


@pytest.mark.parametrize("chunk", [4, 16, 64])
@pytest.mark.parametrize("d", [4, 6, 8])
def test_element_per_lane(d, chunk):
    c, e = bench.fused_costs(d, 4, chunk), bench.pass_costs(d, 4, chunk)
    assert set(c) == set(bench.PASSES)
    assert c["filter_fold"] == e["filter_fold"] and c["smoother_fold"] == (0.0, 0.0)
    ns = d * (d + 1) // 2
    # (chunk + 1) (d + 3) FP64 values, the end moments and the element of a lane
    handed = (8 * ((chunk + 1) * (d + 3) + d + ns) + 4 * (d * d + d + ns)) / chunk
    assert c["smoother_finish"][0] == pytest.approx(handed + 8)
    assert c["filter_finish"][0] == pytest.approx(13 * (chunk + 1) / chunk + 4 * (d * d + 2 * d + 2 * ns) / chunk + handed)
    assert all(f >= 0 for _, f in c.values())
