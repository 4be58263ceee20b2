"""Exact attention and insert of a small launch: the waves of a workgroup share the rows of one unit (32 rows in
bf16, 16 in binary32) and split its keys.  Sizes: fewer key blocks than waves, one more than a
multiple of them, lengths that end on and inside a block; each case also as a batch of many copies,
which goes to the kernels of larger launches, and every copy has to agree with the oracle.  Bars:
those of tests/parity.py."""
import pytest
import torch

from tests import parity
from tests.test_gpu_parity_small import _gen, ac  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # Hq, Hkv, S, D, causal, dtype, lengths
    (1, 1, 32, 64, True, torch.bfloat16, [32, 1]),         # one key block, three idle waves
    (2, 1, 96, 128, False, torch.bfloat16, [96, 64, 33]),
    (3, 1, 160, 64, True, torch.bfloat16, [160, 128, 97]),     # five blocks: one wave has two
    (4, 2, 288, 128, True, torch.bfloat16, [288, 31]),
    (2, 2, 1024, 64, False, torch.bfloat16, [1024, 513]),
    (1, 1, 1, 16, True, torch.float32, [1]),
    (3, 1, 33, 64, True, torch.float32, [33, 16, 17]),
    (2, 1, 65, 80, False, torch.float32, [65, 64, 1]),       # five blocks, columns past D
    (2, 2, 94, 128, True, torch.float32, [94, 80, 50]),
    (1, 1, 200, 256, True, torch.float32, [200, 7]),
    (2, 1, 130, 48, False, torch.float32, [130, 129]),
    (2, 1, 40, 144, True, torch.float32, [40, 17]),
]


def copies(case):
    """Copies of the batch that go to the kernels of larger launches."""
    return -(-2400 // (len(case[6]) * case[0] * -(-case[2] // 32)))


@pytest.mark.parametrize("case", CASES, ids=lambda c: "H%d/%d-S%d-D%d-%s-%s" % (
    *c[:4], "causal" if c[4] else "dense", str(c[5])[6:]))
def test_exact_matches_the_oracle(ac, oracle_mod, case):  # noqa: F811
    Hq, Hkv, S, D, causal, dt, lens = case
    B, g = len(lens), _gen(7 * S + D + Hq)
    Q, K, V = (torch.randn(B, h, S, D, generator=g).to(dt) for h in (Hq, Hkv, Hkv))
    key_len = torch.tensor(lens, dtype=torch.int32)
    many = copies(case)
    for kl in (None, key_len):
        want = oracle_mod.attention_exact(*(parity.to_np(t) for t in (Q, K, V)), causal=causal,
                                          key_len=None if kl is None else kl.numpy())
        for n in (1, many):
            q, k, v = (t.cuda().repeat(n, 1, 1, 1) for t in (Q, K, V))
            if kl is not None and dt == torch.float32:        # what a padded batch holds past its sentences
                for b, m in enumerate(lens):
                    k[b::B, :, m:], v[b::B, :, m:] = float("nan"), float("inf")
            sel = torch.full((n * B,), -1, dtype=torch.int32, device="cuda")
            sel[-1] = 0                                       # the last item was served by the reuse branch
            O = torch.full((n * B, Hq, S, D), 7.0, dtype=dt, device="cuda")
            ac.attention_exact(q, k, v, O, causal=causal, row_sel=sel,
                               key_len=None if kl is None else kl.cuda().repeat(n))
            O = O.cpu().view(n, B, Hq, S, D)
            assert (O[-1, -1] == 7.0).all()
            O[-1, -1] = torch.from_numpy(want[-1]).to(dt)
            assert (O == O[0]).all() or n * B == 1 or parity.max_abs_err(O - O[0], 0 * O.float().numpy()) <= parity.TOL[dt]
            assert max(parity.max_abs_err(O[i], want) for i in (0, n - 1)) <= parity.TOL[dt]


@pytest.mark.parametrize("S", [40, 200])
def test_infinite_v_touches_visible_rows_only(ac, S):  # noqa: F811
    """V[j] = inf or NaN: rows before j are what they are without it, in a small and in a large launch."""
    g, j = _gen(S), S - 20
    Q, K, V = (torch.randn(1, 2, S, 64, generator=g).cuda() for _ in range(3))
    want = torch.softmax((Q @ K.transpose(2, 3).contiguous() / 8).masked_fill(
        torch.ones(S, S, dtype=torch.bool, device="cuda").triu_(1), float("-inf")), -1) @ V
    V[:, 0, j], V[:, 1, j] = float("inf"), float("nan")
    for n in (1, 1200):
        O = torch.zeros(n, 2, S, 64, device="cuda")
        ac.attention_exact(*(t.repeat(n, 1, 1, 1) for t in (Q, K, V)), O, causal=True)
        assert (O[:, :, :j] - want[:, :, :j]).abs().max() <= parity.TOL[torch.float32]
        assert (O[:, 0, j:] == float("inf")).all() and O[:, 1, j:].isnan().all()


@pytest.mark.parametrize("packed", [False, True], ids=["dense", "packed"])
@pytest.mark.parametrize("case", [c for c in CASES if c[5] == torch.bfloat16] + [
    (4, 1, 32, 128, True, torch.bfloat16, [32, 5]),           # one block, several heads on one K and V
    (2, 1, 128, 64, False, torch.bfloat16, [128, 70]),
], ids=lambda c: "H%d/%d-S%d-D%d-%s" % (*c[:4], "causal" if c[4] else "dense"))
def test_insert_matches_the_oracle(ac, oracle_mod, case, packed):  # noqa: F811
    """A stored map may differ from the oracle's rounded one by one bf16 step (2^-8 relative), zeros are exact."""
    Hq, Hkv, S, D, causal, dt, lens = case
    B, E, g = len(lens), 32, _gen(3 * S + D + Hq)
    Q, K, V = (torch.randn(B, h, S, D, generator=g).to(dt) for h in (Hq, Hkv, Hkv))
    key_len = torch.tensor(lens, dtype=torch.int32)
    feat = torch.randn(B, E, generator=g).half()
    want, P = oracle_mod.attention_exact(*(parity.to_np(t) for t in (Q, K, V)), causal=causal, key_len=key_len.numpy(),
                                         return_map=True)
    rounded = oracle_mod.round_maps(P)
    for n in (1, -(-1400 // (B * Hq * S // 32))):
        M = n * B
        shape = (M, 1, Hq, ac.packed_tile_elems(S, causal)) if packed else (M, 1, Hq, S, S)
        maps = torch.full(shape, 3.0, dtype=dt, device="cuda")
        emb = torch.zeros(M, E, dtype=torch.float16, device="cuda")
        db = ac.attncache_build_db(emb, maps, n_kv_heads=Hkv, head_dim=D, causal=causal, seq_len=S)
        slot = torch.arange(M - 1, -1, -1, dtype=torch.int32)
        slot[-1] = -1                                         # the last item is computed, not kept
        O = torch.zeros(M, 1, Hq, S, D, dtype=dt, device="cuda")
        ac.attncache_insert(db, *(t[:, None].cuda().repeat(n, 1, 1, 1, 1) for t in (Q, K, V)), O, slot=slot.cuda(),
                            feat=feat.cuda().repeat(n, 1), key_len=key_len.cuda().repeat(n))
        torch.cuda.synchronize()
        db.close()
        assert max(parity.max_abs_err(O[i * B:i * B + B, 0], want) for i in (0, n - 1)) <= parity.TOL[dt]
        assert (maps[0] == 3.0).all() and (emb[0] == 0).all()
        for item in {0, 1, M - 2}:
            s, b = int(slot[item]), item % B
            if s < 0:
                continue
            assert torch.equal(emb[s].cpu(), feat[b])
            for h in range(Hq):
                got = parity.to_np(maps[s, 0, h])
                got = parity.unpack_map(got, S, causal) if packed else got
                assert ((got == 0) == (rounded[b, h] == 0)).all()
                assert abs(got - rounded[b, h]).max() <= 2.0 ** -8 * abs(rounded[b, h]).max()
