"""Calls whose grid would not fit one launch (2^32 threads in a dimension) are split over several that
cover the same work.  Host code on a recorder, no GPU."""
import pytest

from tests import launches


@pytest.fixture(scope="module")
def record(tmp_path_factory):
    d = tmp_path_factory.mktemp("recorder")
    return lambda *calls: launches.record(calls, d)


@pytest.mark.parametrize("call,kernel,covered", [
    # vector-ALU tiles: (groups of 256 rows, rounded up to 8) x (blocks of 16 queries)
    (("search", 10_000_000, 8, 8192, 1, "f32", "l2"), "search_valu_kernel", 39064 * 512),
    (("search", 20_000_000, 8, 8192, 2, "f32", "ip"), "search_valu_kernel", 78128 * 512),
    (("search", 2_000_000_000, 24, 100, 1, "f16", "l2"), "search_valu_kernel", 7_812_504 * 7),
    # a workgroup of 1,024 threads per query in the second phase
    (("search", 300_000, 64, 5_000_000, 2, "f16", "ip"), "finalize_topk_kernel", 5_000_000),
    # narrow binary32 heads: eight times as many workgroups as (item, layer, head) tiles
    (("apply", 600_000, 1, 4, 4, 512, 4, True, "f32"), "apply_f32_kernel", 2_400_000 * 8),
], ids=lambda x: "-".join(map(str, x)) if isinstance(x, tuple) else None)
def test_a_grid_that_does_not_fit_is_split(record, call, kernel, covered):
    (status, ls), = record(call)
    assert status == 0
    mine = [la for la in ls if la[0].startswith(kernel)]
    assert len(mine) > 1 and sum(la[1] * la[2] for la in mine) >= covered
    assert all(la[1] * la[4] < 2**32 for la in ls)


@pytest.mark.parametrize("B,Lc,Hq", [(3_000_000, 1, 4), (700_001, 3, 6), (600_000_000, 1, 4), (3, 900_000_001, 2)])
def test_launches_of_small_maps_start_where_the_last_one_ended(record, B, Lc, Hq):
    """A workgroup per (query, layer, head), 2^31 and more of them in the last two."""
    (status, ls), = record(("apply", B, Lc, Hq, Hq, 1, 1, True, "f32"))
    assert status == 0 and len(ls) > 1
    done = 0
    for kernel, gx, gy, gz, block, _, b, l, h in ls:
        assert kernel == "apply_f32_small_kernel" and gy == gz == 1 and gx * block < 2**32
        assert 0 <= h < Hq and 0 <= l < Lc and (b * Lc + l) * Hq + h == done
        done += gx
    assert done == B * Lc * Hq
