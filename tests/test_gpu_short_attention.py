"""Exact attention and insert of short sequences (up to 128 rows): several K/V heads a workgroup, parts of one, units of 32 rows.
The reference is plain torch in binary32; the bounds are those of the roundings to bfloat16 (weights and result, 2^-8 of the
value each)."""
import pytest
import torch

from tests.test_gpu_parity_small import ac  # noqa: F401

pytestmark = pytest.mark.gpu

# B, Hq, Hkv: one head on a K and V, and two, three, twelve; enough units for the kernel, more K and V than workgroups that fit
EXACT = [(57, 12, 12), (60, 10, 5), (43, 9, 3), (50, 12, 1), (700, 6, 3), (1100, 2, 2)]
EXACT_CASES = [(*c, S, D, causal) for S in (32, 64, 96, 128) for D in (64, 128) for causal in (True, False)
               for c in EXACT if c[0] < 500 or S < 96]
# the last workgroup has fewer K/V heads than the others (four of one row block, two of two), the last one of them a miss or short
EXACT_CASES += [(*c, S, D, causal) for c, S in (((1101, 1, 1), 32), ((701, 6, 3), 32), ((1101, 1, 1), 64), ((577, 3, 3), 64))
                for D in (64, 128) for causal in (True, False)]
INSERT_CASES = [(*c, S, D, causal) for S in (32, 64, 96, 128) for D in (64, 128) for causal in (True, False)
                for c in [(70, 2, 13, 13), (40, 2, 8, 4), (41, 1, 18, 6), (50, 1, 12, 1)]]
INSERT_CASES += [(641, 1, 3, 3, S, D, causal) for S in (32, 64) for D in (64, 128) for causal in (True, False)]   # (as above)
INSERT_CASES += [(50, 1, 3, 3, 64, D, causal) for D in (64, 128) for causal in (True, False)]   # two passes: a few units, one head each


def _data(B, Lc, Hq, Hkv, S, D, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda h: torch.randn(B, Lc, h, S, D, generator=g, device="cuda").bfloat16()  # noqa: E731
    lens = torch.randint(1, S + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    lens[0], lens[1], lens[-1] = S, 1, 3
    return r(Hq), r(Hkv), r(Hkv), lens


def _reference(q, k, v, causal, lens):
    """Weights and result in binary32, and the sum of the terms' magnitudes, of [n, L, H, S, D]."""
    g, S = q.shape[2] // k.shape[2], q.shape[3]
    k, v = (t.float().repeat_interleave(g, 2).contiguous() for t in (k, v))
    s = torch.matmul(q.float(), k.transpose(3, 4).contiguous()) / q.shape[4] ** 0.5
    hide = torch.arange(S, device="cuda") >= lens.view(-1, 1, 1, 1, 1)
    if causal:
        hide = hide | torch.ones(S, S, dtype=torch.bool, device="cuda").triu_(1)
    p = torch.softmax(s.masked_fill(hide, float("-inf")), -1)
    return p, torch.matmul(p, v), torch.matmul(p, v.abs())


def _check_result(O, want, terms):
    assert ((O.float() - want).abs() <= 2.0 ** -8 * 1.05 * (want.abs() + 2 * terms) + 1e-5).all()


# workgroups of four units of a K and V of 32 rows, those of one on an XCD; no multiple of eight K and V
LARGE_CASES = [(547, 120, 15, 32, 64, True), (1367, 24, 2, 32, 128, False), (683, 96, 6, 32, 128, True)]


@pytest.mark.parametrize("case", LARGE_CASES, ids=lambda c: "B%d-%d/%d-S%d-D%d-%s" % c)
def test_large_launches_of_32_rows(ac, case):  # noqa: F811
    B, Hq, Hkv, S, D, causal = case
    Q, K, V, lens = _data(B, 1, Hq, Hkv, S, D, B)
    _, want, terms = _reference(Q, K, V, causal, lens)
    O = torch.full_like(Q, 7.0)
    ac.attention_exact(Q[:, 0], K[:, 0], V[:, 0], O[:, 0], causal=causal, key_len=lens)
    _check_result(O, want, terms)
    M = B + 1
    maps, emb = torch.full((M, 1, Hq, S, S), 7.0, dtype=torch.bfloat16, device="cuda"), torch.zeros(M, 64, device="cuda").half()
    slot = torch.randperm(M, generator=torch.Generator().manual_seed(B)).int()[:B].cuda()
    feat = torch.randn(B, 64, device="cuda").half()
    O2 = torch.full_like(Q, 7.0)
    db = ac.attncache_build_db(emb, maps, n_kv_heads=Hkv, head_dim=D, causal=causal)
    ac.attncache_insert(db, Q, K, V, O2, slot=slot, feat=feat, key_len=lens)
    torch.cuda.synchronize()
    db.close()
    _check_result(O2, want, terms)
    p = _reference(Q, K, V, causal, lens)[0][:, 0]
    got = maps[slot.long(), 0].float()
    assert ((got - p).abs() <= 2.0 ** -8 * 1.05 * p).all() and torch.equal(emb[slot.long()], feat)
    left = torch.ones(M, dtype=torch.bool, device="cuda")
    left[slot.long()] = False
    assert (maps[left] == 7.0).all()


@pytest.mark.parametrize("padded,routed", [(False, False), (True, True)])
@pytest.mark.parametrize("case", EXACT_CASES, ids=lambda c: "B%d-%d/%d-S%d-D%d-%s" % c)
def test_exact(ac, case, padded, routed):  # noqa: F811
    B, Hq, Hkv, S, D, causal = case
    Q, K, V, lens = (t if t.dim() == 1 else t[:, 0].contiguous() for t in _data(B, 1, Hq, Hkv, S, D, S + D + B))
    sel = torch.where(torch.arange(B, device="cuda") % 3 == 1, 5, -1).int() if routed else None
    room = torch.full((B + 1, *Q.shape[1:]), 7.0, dtype=Q.dtype, device="cuda")
    O = room[:B]
    ac.attention_exact(Q, K, V, O, causal=causal, key_len=lens if padded else None, row_sel=sel)
    torch.cuda.synchronize()
    some = torch.tensor(sorted({0, 2, 3, 5, B // 2, B - 3, B - 2, B - 1}), device="cuda")
    for b in some.tolist():
        if sel is not None and sel[b] >= 0:
            assert (O[b] == 7.0).all()
            continue
        n = lens[b:b + 1] if padded else torch.full((1,), S, device="cuda")
        _, want, terms = _reference(Q[b][None, None], K[b][None, None], V[b][None, None], causal, n)
        _check_result(O[b], want[0, 0], terms[0, 0])
    assert (room[B] == 7.0).all()
    done = torch.ones(B, dtype=torch.bool, device="cuda") if sel is None else sel < 0
    assert O[done].isfinite().all() and (O[done] != 7.0).any(-1).all() and (O[~done] == 7.0).all()


@pytest.mark.parametrize("hits", [0.0, 0.5, 0.97, 1.0])
def test_routed_launches_of_many_tiles(ac, hits):  # noqa: F811
    # (kernels of their own: workgroups that look for the tiles they have to do)
    Q, K, V, _ = (t if t.dim() == 1 else t[:, 0].contiguous() for t in _data(300, 1, 60, 60, 32, 64, 1))
    sel = torch.where(torch.rand(300, generator=torch.Generator().manual_seed(2)) < hits, 1, -1).int().cuda()
    O = torch.full_like(Q, 7.0)
    ac.attention_exact(Q, K, V, O, row_sel=sel)
    done = torch.nonzero(sel < 0).flatten()
    assert (O[sel >= 0] == 7.0).all()
    for b in done[:: max(1, len(done) // 9)].tolist():
        _, want, terms = _reference(Q[b][None, None], K[b][None, None], V[b][None, None], True, torch.full((1,), 32, device="cuda"))
        _check_result(O[b], want[0, 0], terms[0, 0])


@pytest.mark.parametrize("case", INSERT_CASES, ids=lambda c: "B%d-L%d-%d/%d-S%d-D%d-%s" % c)
def test_insert(ac, case):  # noqa: F811
    B, Lc, Hq, Hkv, S, D, causal = case
    Q, K, V, lens = _data(B, Lc, Hq, Hkv, S, D, S + D)
    M = B + 3
    slot = torch.randperm(M, generator=torch.Generator().manual_seed(B)).int()[:B].cuda()
    slot[4] = -1                                  # O only
    sel = torch.full((B,), -1, dtype=torch.int32, device="cuda")
    sel[6] = 0                                    # not at all
    feat = torch.randn(B, 64, device="cuda").half()
    maps, emb, out = [], [], []
    for layout in ("dense", "packed"):
        shape = (M, Lc, Hq, S, S) if layout == "dense" else (M, Lc, Hq, ac.packed_tile_elems(S, causal))
        room, e = torch.full((M + 1, *shape[1:]), 7.0, dtype=torch.bfloat16, device="cuda"), torch.full((M, 64), 7.0, device="cuda").half()
        store, O_room = room[:M], torch.full((B + 1, *Q.shape[1:]), 7.0, dtype=Q.dtype, device="cuda")
        db = ac.attncache_build_db(e, store, n_kv_heads=Hkv, head_dim=D, causal=causal, **({} if layout == "dense" else {"seq_len": S}))
        O = O_room[:B]
        ac.attncache_insert(db, Q, K, V, O, slot=slot, feat=feat, key_len=lens, row_sel=sel)
        torch.cuda.synchronize()
        db.close()
        assert (room[M] == 7.0).all() and (O_room[B] == 7.0).all()
        maps, emb, out = maps + [store], emb + [e], out + [O]
    one_kernel = not (causal and S == 128 and D == 64)   # (dense maps take the two passes there)
    assert (torch.equal(out[0], out[1]) or not one_kernel) and torch.equal(emb[0], emb[1])
    packed = torch.empty_like(maps[1])
    ac.attncache_pack_maps(maps[0], packed, causal=causal)
    kept = [b for b in range(B) if b not in (4, 6)]
    slots = slot[kept].long()
    off = (packed[slots].float() - maps[1][slots].float()).abs()
    assert (off == 0).all() if one_kernel else (off <= 2.0 ** -7 * packed[slots].float()).all()   # a last place apart
    left = torch.ones(M, dtype=torch.bool, device="cuda")
    left[slots] = False
    assert all((m[left] == 7.0).all() for m in maps) and (emb[0][left] == 7.0).all() and torch.equal(emb[0][slots], feat[kept])
    assert (out[0][6] == 7.0).all()
    for b in (0, 1, 2, 4, B // 2, B - 1):
        p, want, terms = _reference(Q[b:b + 1], K[b:b + 1], V[b:b + 1], causal, lens[b:b + 1])
        for o in out:
            _check_result(o[b], want[0], terms[0])
        if b != 4:
            got = maps[0][slot[b]].float()
            assert ((got - p[0]).abs() <= 2.0 ** -8 * 1.05 * p[0]).all() and (got[p[0] == 0] == 0).all()
