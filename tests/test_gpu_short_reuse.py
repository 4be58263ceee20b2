"""Reuse of short maps (up to 128 rows): units of 32 rows of several heads and K/V heads in one workgroup."""
import numpy as np
import pytest
import torch

from tests import parity
from tests.test_gpu_parity_small import _build, _gen, _maps, ac  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # B, Lc, Hkv, heads on one K/V head: four, two, one K/V head a workgroup, the last one with fewer; units that leave waves
    # without one; parts of a K/V head's units, and all of them one after the other
    (5, 2, 1, 1), (3, 1, 5, 1), (4, 2, 3, 2), (5, 2, 2, 3), (4, 1, 2, 4), (3, 2, 1, 7), (180, 2, 1, 4), (150, 3, 1, 6), (175, 2, 1, 12),
]
CASES_128 = [(180, 3, 1, 1), (180, 3, 1, 4), (4, 1, 2, 3), (3, 2, 5, 1)]


@pytest.mark.parametrize("layout", ["dense", "packed"])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("case", CASES_128, ids=lambda c: "B%d-L%d-%dx%d" % c)
def test_maps_of_128_rows(ac, oracle_mod, case, D, causal, layout):  # noqa: F811
    # few tiles and more than 512 of them, which packed causal maps of 64 columns have a kernel for
    test_short_maps(ac, oracle_mod, case, 128, D, causal, layout)


@pytest.mark.parametrize("layout", ["dense", "packed"])
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("S,D", [(32, 64), (32, 128), (64, 64), (64, 128), (96, 64), (96, 128)])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "B%d-L%d-%dx%d" % c)
def test_short_maps(ac, oracle_mod, case, S, D, causal, layout):  # noqa: F811
    B, Lc, Hkv, g = case
    M, Hq = 4, Hkv * g
    maps = _maps(M, Lc + 1, Hq, S, torch.bfloat16, causal, S + D)
    V = torch.randn(B, Lc, Hkv, S, D, generator=_gen(B + S)).bfloat16()
    hit = torch.randint(0, M, (B,), generator=_gen(B), dtype=torch.int32)
    hit[1], hit[B - 1] = -1, M   # a miss, no such entry
    db = _build(ac, torch.zeros(M, 16), maps, layout, causal, n_kv_heads=Hkv, head_dim=D)
    O = torch.full((B, Lc, Hq, S, D), 7.0, dtype=torch.bfloat16, device="cuda")
    ac.attncache_apply(db, hit.cuda(), V.cuda(), O, layer_begin=1, layer_count=Lc)
    torch.cuda.synchronize()
    db.close()
    assert (O[1] == 7.0).all() and (O[B - 1] == 7.0).all()
    few = list(range(min(B, 3))) + ([B // 2, B - 2] if B > 5 else [])
    few = [b for b in few if 0 <= hit[b] < M]
    ref = oracle_mod.apply(parity.to_np(maps), hit[few].numpy(), parity.to_np(V[few]), layer_begin=1,
                           out=np.zeros((len(few), Lc, Hq, S, D)))
    got = O[few].double().cpu().numpy()
    # one rounding to eight significant bits, and binary32 sums of at most 128 products of weights that add up to one with |V| < 6
    assert (np.abs(got - ref) <= 2.0 ** -8 * 1.01 * np.abs(ref) + 128 * 2.0 ** -23 * 6).all()
    hits = [b for b in range(B) if 0 <= hit[b] < M]
    want = torch.matmul(maps[hit[hits].long(), 1:].float(), V[hits].float().repeat_interleave(g, 2))
    assert ((O[hits].float().cpu() - want).abs() <= 2.0 ** -8 * 1.01 * want.abs() + 1e-4).all()


# B, Lc, Hkv, heads on one K/V head, S, D, causal, layout: a workgroup has four units of a tile, those of a tile are on one XCD; the
# number of tiles is no multiple of the eight XCDs
LARGE_CASES = [(1639, 5, 1, 8, 32, 64, True, "dense"), (683, 4, 3, 4, 64, 128, False, "packed"), (1639, 5, 1, 2, 128, 128, True, "packed"),
               (1093, 5, 1, 3, 128, 128, True, "dense"), (1639, 5, 1, 3, 128, 64, True, "packed")]


@pytest.mark.parametrize("case", LARGE_CASES, ids=lambda c: "B%d-L%d-%dx%d-S%d-D%d-%s-%s" % c)
def test_large_launches(ac, case):  # noqa: F811
    B, Lc, Hkv, g, S, D, causal, layout = case
    M, Hq, gen = 4, Hkv * g, torch.Generator(device="cuda").manual_seed(B)
    maps = _maps(M, Lc, Hq, S, torch.bfloat16, causal, S + D)
    V = torch.randn(B, Lc, Hkv, S, D, generator=gen, device="cuda").bfloat16()
    hit = torch.randint(-1, M + 1, (B,), generator=gen, device="cuda", dtype=torch.int32)   # -1: a miss, M: no such entry
    db = _build(ac, torch.zeros(M, 16), maps, layout, causal, n_kv_heads=Hkv, head_dim=D)
    O = torch.full((B, Lc, Hq, S, D), 7.0, dtype=torch.bfloat16, device="cuda")
    ac.attncache_apply(db, hit, V, O)
    torch.cuda.synchronize()
    db.close()
    assert (O[(hit < 0) | (hit >= M)] == 7.0).all()
    maps = maps.cuda().float()
    for e in range(M):
        of = torch.nonzero(hit == e).flatten()
        for some in of.split(64):
            want = torch.matmul(maps[e][None], V[some].float().repeat_interleave(g, 2))
            assert ((O[some].float() - want).abs() <= 2.0 ** -8 * 1.01 * want.abs() + 1e-4).all()
