"""Attention in bfloat16 away from unit Gaussian inputs: scores up to a million, infinite and NaN ones, in every kernel.

Large scores are whole numbers that binary32 holds exactly (a large common part, small differences), so the weights of the
definition are known in 64 bits and what is left are the roundings of the weights and of the result to bfloat16."""
import pytest
import torch

from tests.test_gpu_parity_small import ac  # noqa: F401

pytestmark = pytest.mark.gpu

LOG2E = torch.tensor(1.44269504088896340736, dtype=torch.float32)   # scale 1, in the log2 domain
# B, Lc, Hq, Hkv, S, D, causal
INSERT_CASES = [
    (8, 1, 8, 2, 288, 128, True), (8, 1, 8, 2, 288, 128, False), (12, 1, 8, 4, 288, 64, True), (5, 2, 9, 3, 320, 64, False),   # two passes
    (10, 1, 6, 6, 128, 128, True), (10, 1, 6, 6, 128, 64, True), (10, 1, 6, 6, 96, 128, False), (20, 1, 4, 4, 64, 64, True),
    (44, 1, 6, 6, 128, 128, True), (44, 1, 6, 6, 128, 64, False), (12, 1, 32, 8, 96, 128, True), (41, 1, 18, 6, 64, 64, True),   # one
    (2, 1, 8, 2, 288, 128, True), (2, 1, 8, 2, 160, 64, False), (4, 1, 8, 2, 128, 128, True),   # keys split
]
# B, Hq, Hkv, S, D, causal, routed
EXACT_CASES = [
    (8, 16, 8, 288, 128, True, False), (8, 16, 8, 320, 64, False, False),   # streaming
    (44, 6, 6, 128, 128, True, False), (44, 12, 3, 64, 64, False, False), (44, 6, 6, 96, 64, True, False),   # short
    (35, 60, 60, 128, 64, True, True), (35, 60, 60, 96, 128, False, True),   # resident
    (2, 4, 2, 288, 128, True, False), (2, 4, 2, 128, 64, False, False),   # split
]
_id = lambda c: "-".join(map(str, c))   # noqa: E731


def _whole(shape, large, g, alternate):
    """Whole numbers: a large first column (of either sign by row), a few of -1, 0 and 1, zeros."""
    x = torch.zeros(*shape, device="cuda")
    x[..., 1:9] = torch.randint(-1, 2, (*shape[:-1], 8), generator=g, device="cuda").float()
    x[..., 0] = large
    if alternate:
        x[..., 1::2, 0] *= -1
    return x.bfloat16()


def _weights(q, k, c, causal, length):
    """Weights of [H, S, D] by [H, S, D] in 64 bits, `c` to the log2 domain."""
    S = q.shape[1]
    t = torch.matmul(q.double(), k.double().transpose(1, 2).contiguous()) * c
    hide = torch.arange(S, device="cuda") >= length
    if causal:
        hide = hide | torch.ones(S, S, dtype=torch.bool, device="cuda").triu_(1)
    t = t.masked_fill(hide, float("-inf"))
    w = torch.exp2(t - t.amax(-1, keepdim=True))
    return w / w.sum(-1, keepdim=True)


def _check(O, p, v):
    """Two roundings to eight bits (weights and result), the sum of the rounded weights as divisor or not."""
    want, terms = torch.matmul(p, v.double()), torch.matmul(p, v.double().abs())
    nan = want.isnan()
    assert torch.equal(O.isnan(), nan)
    off = (O.double() - want).abs()
    assert (nan | (off <= 2.0 ** -8 * 1.05 * (want.abs() + 2 * terms) + 1e-5)).all(), off[~nan].max()


def _insert(ac, Q, K, V, layout, causal, lens):  # noqa: F811
    B, Lc, Hq, S, D = Q.shape
    shape = (B, Lc, Hq, S, S) if layout == "dense" else (B, Lc, Hq, ac.packed_tile_elems(S, causal))
    maps, O = torch.zeros(shape, dtype=torch.bfloat16, device="cuda"), torch.full_like(Q, 7.0)
    db = ac.attncache_build_db(torch.zeros(B, 16, device="cuda").half(), maps, n_kv_heads=K.shape[2], head_dim=D, causal=causal,
                               **({} if layout == "dense" else {"seq_len": S}))
    slot = torch.arange(B, dtype=torch.int32, device="cuda")
    return db, maps, O, slot


def _packed(ac, p, causal):  # noqa: F811
    """One item's [H, S, S] in the packed layout (in binary32: the layout is a permutation)."""
    H, S = p.shape[0], p.shape[1]
    t = p.view(H, S // 16, 16, S // 32, 4, 8).permute(0, 1, 3, 4, 2, 5).reshape(H, S // 16, S // 32, 512)
    return torch.cat([t[:, r, :(r + 2) // 2 if causal else S // 32].reshape(H, -1) for r in range(S // 16)], 1)


def _some(B):
    return sorted({0, 1, 2, 3 % B, B // 2, B - 1} & set(range(B)))


@pytest.mark.parametrize("large", [(32.0, 32.0), (256.0, 512.0), (1024.0, 1024.0)], ids=["1e3", "1e5", "1e6"])
@pytest.mark.parametrize("layout", ["dense", "packed"])
@pytest.mark.parametrize("case", INSERT_CASES, ids=_id)
def test_insert_of_large_scores(ac, case, layout, large):  # noqa: F811
    B, Lc, Hq, Hkv, S, D, causal = case
    g = torch.Generator(device="cuda").manual_seed(S + D)
    Q, K = _whole((B, Lc, Hq, S, D), large[0], g, True), _whole((B, Lc, Hkv, S, D), large[1], g, False)
    V = torch.randn(B, Lc, Hkv, S, D, generator=g, device="cuda").bfloat16()
    lens = torch.randint(1, S + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    lens[0], lens[-1] = S, 1
    db, maps, O, slot = _insert(ac, Q, K, V, layout, causal, lens)
    ac.attncache_insert(db, Q, K, V, O, slot=slot, key_len=lens, scale=1.0)
    torch.cuda.synchronize()
    db.close()
    for b in _some(B):
        for l in range(Lc):
            k, v = (t[b, l].repeat_interleave(Hq // Hkv, 0) for t in (K, V))
            p = _weights(Q[b, l], k, float(LOG2E), causal, int(lens[b]))
            want = p if layout == "dense" else _packed(ac, p, causal)
            assert ((maps[b, l].double() - want).abs() <= 2.0 ** -8 * 1.01 * want).all()
            if layout == "dense":
                assert ((maps[b, l].double().sum(-1) - 1).abs() <= 2.0 ** -8 * 1.01).all()
            _check(O[b, l], p, v)


@pytest.mark.parametrize("large", [(32.0, 32.0), (1024.0, 1024.0)], ids=["1e3", "1e6"])
@pytest.mark.parametrize("case", EXACT_CASES, ids=_id)
def test_exact_of_large_scores(ac, case, large):  # noqa: F811
    B, Hq, Hkv, S, D, causal, routed = case
    g = torch.Generator(device="cuda").manual_seed(S + D)
    Q, K = _whole((B, Hq, S, D), large[0], g, True), _whole((B, Hkv, S, D), large[1], g, False)
    V = torch.randn(B, Hkv, S, D, generator=g, device="cuda").bfloat16()
    O, sel = torch.full_like(Q, 7.0), torch.full((B,), -1, dtype=torch.int32, device="cuda") if routed else None
    ac.attention_exact(Q, K, V, O, causal=causal, scale=1.0, row_sel=sel)
    torch.cuda.synchronize()
    for b in _some(B):
        k, v = (t[b].repeat_interleave(Hq // Hkv, 0) for t in (K, V))
        _check(O[b], _weights(Q[b], k, float(LOG2E), causal, S), v)


def _spoil(Q, K, lens):
    """Q and K [B, heads, S, D] with NaN and infinities, some of them in the padding; what they spoil is defined by the sums."""
    S, last = Q.shape[2], Q.shape[0] - 1
    Q[0, 0, 5, 3] = float("nan")
    K[0, -1, S - 2, 1] = float("inf")     # scores of both signs
    K[1, 0, 9, :] = float("nan")
    K[1, -1, 3, 0] = float("-inf")
    lens[last] = S // 2 + 3               # hidden: not one row
    K[last, :, S // 2 + 3:, :] = float("nan")


@pytest.mark.parametrize("layout", ["dense", "packed"])
@pytest.mark.parametrize("case", INSERT_CASES, ids=_id)
def test_insert_of_nan_and_infinities(ac, case, layout):  # noqa: F811
    B, Lc, Hq, Hkv, S, D, causal = case
    g = torch.Generator(device="cuda").manual_seed(S + D)
    Q, K, V = (torch.randn(B, Lc, h, S, D, generator=g, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    lens = torch.full((B,), S, dtype=torch.int32, device="cuda")
    _spoil(Q[:, 0], K[:, 0], lens)
    db, maps, O, slot = _insert(ac, Q, K, V, layout, causal, lens)
    ac.attncache_insert(db, Q, K, V, O, slot=slot, key_len=lens)
    torch.cuda.synchronize()
    db.close()
    for b in _some(B):
        k, v = (t[b, 0].repeat_interleave(Hq // Hkv, 0) for t in (K, V))
        p = _weights(Q[b, 0], k, float(LOG2E) / D ** 0.5, causal, int(lens[b]))
        want = p if layout == "dense" else _packed(ac, p, causal)
        off = (maps[b, 0].double() - want).abs()
        assert (want.isnan() | (off <= 2.0 ** -8 * 1.05 * want)).all()
        _check(O[b, 0], p, v)


@pytest.mark.parametrize("case", EXACT_CASES, ids=_id)
def test_exact_of_nan_and_infinities(ac, case):  # noqa: F811
    B, Hq, Hkv, S, D, causal, routed = case
    g = torch.Generator(device="cuda").manual_seed(S + D)
    Q, K, V = (torch.randn(B, h, S, D, generator=g, device="cuda").bfloat16() for h in (Hq, Hkv, Hkv))
    lens = torch.full((B,), S, dtype=torch.int32, device="cuda")
    _spoil(Q, K, lens)
    O, sel = torch.full_like(Q, 7.0), torch.full((B,), -1, dtype=torch.int32, device="cuda") if routed else None
    ac.attention_exact(Q, K, V, O, causal=causal, row_sel=sel, key_len=lens)
    torch.cuda.synchronize()
    for b in _some(B):
        k, v = (t[b].repeat_interleave(Hq // Hkv, 0) for t in (K, V))
        _check(O[b], _weights(Q[b], k, float(LOG2E) / D ** 0.5, causal, int(lens[b])), v)
