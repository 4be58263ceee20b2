"""Sequences longer than 128 deal units of 32 rows of one head to the waves of a workgroup: head
groups and row-block counts that leave units over, and sentence lengths that end inside a block, on
a block and inside the first one.  Bars: the bf16 bar of tests/parity.py; a stored map may differ
from the oracle's rounded one by one bf16 step (2^-8 relative), zeros are exact."""
import numpy as np
import pytest
import torch

from tests import parity
from tests.test_gpu_parity_small import _gen, ac  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # Hq, Hkv, S, D, causal, lengths
    (3, 1, 160, 64, True, [160, 33, 1]),      # 15 units: the lightest workgroup has three
    (5, 1, 192, 128, True, [64, 192, 65]),    # 30 units, rows of two blocks in one workgroup
    (4, 1, 416, 128, True, [300, 128, 416]),  # one row block of four heads
    (2, 2, 288, 64, True, [288, 31, 96]),     # nine units of one head
    (6, 2, 160, 128, False, [160, 32, 97]),
    (7, 1, 160, 64, False, [1, 159, 128]),
]


@pytest.mark.parametrize("packed", [False, True], ids=["dense", "packed"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "H%d/%d-S%d-D%d-%s" % (*c[:4], "causal" if c[4] else "dense"))
def test_exact_and_insert_match_the_oracle(ac, oracle_mod, case, packed):  # noqa: F811
    Hq, Hkv, S, D, causal, lens = case
    B, g = len(lens), _gen(S + D + Hq)
    Q, K, V = (torch.randn(B, h, S, D, generator=g).to(torch.bfloat16) for h in (Hq, Hkv, Hkv))
    key_len = torch.tensor(lens, dtype=torch.int32)
    want, P = oracle_mod.attention_exact(*(parity.to_np(t) for t in (Q, K, V)), causal=causal, key_len=key_len.numpy(),
                                         return_map=True)
    O = torch.zeros(B, Hq, S, D, dtype=torch.bfloat16, device="cuda")
    ac.attention_exact(Q.cuda(), K.cuda(), V.cuda(), O, causal=causal, key_len=key_len.cuda())
    assert parity.max_abs_err(O, want) <= parity.TOL[torch.bfloat16]

    M, E = 5, 32
    shape = (M, 1, Hq, ac.packed_tile_elems(S, causal)) if packed else (M, 1, Hq, S, S)
    maps = torch.full(shape, 3.0, dtype=torch.bfloat16, device="cuda")
    emb = torch.zeros(M, E, dtype=torch.float16, device="cuda")
    feat = torch.randn(B, E, generator=g).half()
    slot = torch.tensor([3, -1, 0], dtype=torch.int32)   # the middle item is computed, not kept
    db = ac.attncache_build_db(emb, maps, n_kv_heads=Hkv, head_dim=D, causal=causal, seq_len=S)
    O2 = torch.zeros(B, 1, Hq, S, D, dtype=torch.bfloat16, device="cuda")
    ac.attncache_insert(db, *(t[:, None].cuda() for t in (Q, K, V)), O2, slot=slot.cuda(), feat=feat.cuda(),
                        key_len=key_len.cuda())
    torch.cuda.synchronize()
    db.close()
    assert parity.max_abs_err(O2[:, 0], want) <= parity.TOL[torch.bfloat16]
    rounded = oracle_mod.round_maps(P)
    for b, s in enumerate(slot.tolist()):
        if s < 0:
            continue
        assert torch.equal(emb[s].cpu(), feat[b])
        for h in range(Hq):
            got = parity.to_np(maps[s, 0, h])
            got = parity.unpack_map(got, S, causal) if packed else got
            ref = rounded[b, h]
            assert ((got == 0) == (ref == 0)).all()
            assert np.abs(got - ref).max() <= 2.0 ** -8 * np.abs(ref).max()
    untouched = [m for m in range(M) if m not in slot.tolist()]
    assert (maps[untouched] == 3.0).all() and (emb[untouched] == 0).all()
