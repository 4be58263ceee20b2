"""Sequences longer than 128 deal units of 32 rows of one head to the waves of a workgroup: head
groups and row-block counts that leave units over, and sentence lengths that end inside a block, on
a block and inside the first one.  Launches of few units go to the kernels that split the keys of a
unit, so every case runs twice: as it is, and as a batch of so many copies that the kernels of large
launches take it; the same copies are made of the bf16 cases of test_gpu_parity_small.py.
Bars: the bf16 bar of tests/parity.py; a stored map may differ
from the oracle's rounded one by one bf16 step (2^-8 relative), zeros are exact."""
import numpy as np
import pytest
import torch

from tests import parity
from tests import test_gpu_parity_small as small
from tests.test_gpu_parity_small import _gen, ac  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # Hq, Hkv, S, D, causal, lengths
    (3, 1, 160, 64, True, [160, 33, 1]),      # 15 units: the heaviest workgroup has three
    (5, 1, 192, 128, True, [64, 192, 65]),    # 30 units, rows of two blocks in one workgroup
    (4, 1, 416, 128, True, [300, 128, 416]),  # one row block of four heads
    (2, 2, 288, 64, True, [288, 31, 96]),     # nine units of one head
    (6, 2, 160, 128, False, [160, 32, 97]),
    (7, 1, 160, 64, False, [1, 159, 128]),
]
BF16 = torch.bfloat16
# the same shapes in a large launch: Hq, Hkv, S, D, causal, lengths (or the number of full sentences)
LARGE_CASES = ([(c[1], c[2], c[3], c[4], c[5], c[0]) for c in small.EXACT_CASES if c[7] == BF16] +
               [(c[1], c[2], c[3], c[4], c[5], c[7]) for c in small.PADDED_CASES if c[6] == BF16] +
               [(c[2], c[3], c[4], c[5], c[6], c[0]) for c in small.INSERT_CASES] +
               [(c[2], c[3], c[4], c[5], c[6], [max(1, c[4] - 27), 33, c[4]] if c[8] else c[0])
                for c in small._random_attention_shapes(24, 20251129)])


def copies(Hq, S, items):
    """Copies of a batch that no rule of the exact or the insert kernel takes for a small launch (at most 1,024 units)."""
    return -(-1100 // (items * Hq * (S // 32)))


def _exact_and_insert(ac, oracle_mod, case, packed, large):  # noqa: F811
    Hq, Hkv, S, D, causal, lens = case
    B, key_len = (lens, None) if isinstance(lens, int) else (len(lens), torch.tensor(lens, dtype=torch.int32))
    n, g = copies(Hq, S, B) if large else 1, _gen(S + D + Hq)
    Q, K, V = (torch.randn(B, h, S, D, generator=g).to(BF16) for h in (Hq, Hkv, Hkv))
    want, P = oracle_mod.attention_exact(*(parity.to_np(t) for t in (Q, K, V)), causal=causal,
                                         key_len=None if key_len is None else key_len.numpy(), return_map=True)
    q, k, v = (t.cuda().repeat(n, 1, 1, 1) for t in (Q, K, V))
    kl = None if key_len is None else key_len.cuda().repeat(n)
    O = torch.zeros(n * B, Hq, S, D, dtype=BF16, device="cuda")
    ac.attention_exact(q, k, v, O, causal=causal, key_len=kl)
    assert parity.max_abs_err(O[:B], want) <= parity.TOL[BF16]
    assert (O.view(n, B, Hq, S, D) == O[:B]).all()

    M, E = n * B + 2, 32
    shape = (M, 1, Hq, ac.packed_tile_elems(S, causal)) if packed else (M, 1, Hq, S, S)
    maps = torch.full(shape, 3.0, dtype=BF16, device="cuda")
    emb = torch.zeros(M, E, dtype=torch.float16, device="cuda")
    feat = torch.randn(B, E, generator=g).half()
    slot = torch.arange(M - 1, 1, -1, dtype=torch.int32)
    if n * B > 1:
        slot[1] = -1                                     # computed, not kept
    db = ac.attncache_build_db(emb, maps, n_kv_heads=Hkv, head_dim=D, causal=causal, seq_len=S)
    O2 = torch.zeros(n * B, 1, Hq, S, D, dtype=BF16, device="cuda")
    ac.attncache_insert(db, q[:, None], k[:, None], v[:, None], O2, slot=slot.cuda(), feat=feat.cuda().repeat(n, 1), key_len=kl)
    torch.cuda.synchronize()
    db.close()
    assert parity.max_abs_err(O2[:B, 0], want) <= parity.TOL[BF16]
    assert (O2.view(n, B, Hq, S, D) == O2[:B, 0]).all()
    rounded = oracle_mod.round_maps(P)
    last = (n - 1) * B
    for item in {*range(B), *range(last, last + B)} - {1 if n * B > 1 else -1}:
        b, s = item % B, int(slot[item])
        assert torch.equal(emb[s].cpu(), feat[b])
        for h in range(Hq):
            got = parity.to_np(maps[s, 0, h])
            got = parity.unpack_map(got, S, causal) if packed else got
            ref = rounded[b, h]
            assert ((got == 0) == (ref == 0)).all()
            assert np.abs(got - ref).max() <= 2.0 ** -8 * np.abs(ref).max()
    untouched = [m for m in range(M) if m not in slot.tolist()]
    assert (maps[untouched] == 3.0).all() and (emb[untouched] == 0).all()


def _id(c):
    return "H%d/%d-S%d-D%d-%s" % (*c[:4], "causal" if c[4] else "dense")


@pytest.mark.parametrize("large", [False, True], ids=["small", "large"])
@pytest.mark.parametrize("packed", [False, True], ids=["dense", "packed"])
@pytest.mark.parametrize("case", CASES, ids=_id)
def test_exact_and_insert_match_the_oracle(ac, oracle_mod, case, packed, large):  # noqa: F811
    _exact_and_insert(ac, oracle_mod, case, packed, large)


@pytest.mark.parametrize("case", list(enumerate(LARGE_CASES)), ids=lambda c: "%d-%s" % (c[0], _id(c[1])))
def test_the_small_cases_in_a_large_launch(ac, oracle_mod, case):  # noqa: F811
    _exact_and_insert(ac, oracle_mod, case[1], case[0] % 2 == 0, True)
