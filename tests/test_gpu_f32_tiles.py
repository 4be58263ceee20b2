"""Binary32 attention on the matrix cores, at the sizes where its tiles end: row blocks of 16,
stages of 32 and 64 keys, output blocks of 64 columns, units of one head and 16 rows dealt to four
waves.  Bars: the fp32 bar of tests/parity.py (a sum of S products is within S * 2^-24 of its
terms, here below 3e-5)."""
import ctypes
import subprocess

import numpy as np
import pytest
import torch

from tests import launches, parity
from tests.test_gpu_parity_small import _gen, _maps, ac  # noqa: F401

pytestmark = pytest.mark.gpu

CASES = [
    # B, Hq, Hkv, S, D, causal
    (1, 1, 1, 1, 1, True),          # the smallest call
    (2, 3, 1, 15, 3, True),         # less than a row block, rows of odd length
    (3, 2, 2, 16, 16, False),
    (2, 4, 2, 17, 64, True),        # one row past a block
    (2, 1, 1, 33, 65, False),       # one key past a stage, one column past an output block
    (2, 6, 2, 94, 128, True),       # three heads on one V, ragged everywhere
    (1, 2, 1, 64, 132, False),
    (1, 5, 5, 65, 80, True),        # one key past the reuse stage
    (1, 2, 1, 129, 256, True),      # the widest rows
    (9, 1, 1, 47, 40, False),       # tiles not a multiple of eight
    (3, 4, 2, 5, 256, True),        # reuse: a thread per output, more outputs than threads
    (5, 3, 1, 16, 12, False),
    (4, 2, 1, 16, 20, True),        # and the first size beyond
    (2, 2, 1, 23, 33, True),        # rows of odd length of one, two and four output blocks
    (2, 2, 1, 34, 99, False),
    (1, 4, 2, 50, 199, True),
    (16, 24, 8, 94, 128, True),     # workgroups for every compute unit two and a half times
    (2, 2, 1, 60, 1, True),         # rows of less than one piece
    (1, 3, 1, 61, 2, False),
    (2, 2, 2, 59, 3, True),
    (2, 2, 1, 50, 5, True),         # rows of one piece and part of another
    (1, 2, 1, 40, 6, False),
    (3, 1, 1, 33, 7, True),
    (1, 2, 2, 31, 66, True),        # and of the second and fourth output block
    (1, 2, 1, 47, 127, False),
    (1, 1, 1, 65, 130, True),
    (1, 2, 1, 33, 253, False),
    (2, 1, 1, 20, 255, True),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "B%d-H%d/%d-S%d-D%d-%s" % (
    *c[:5], "causal" if c[5] else "dense"))
def test_exact_and_reuse_match_the_oracle(ac, oracle_mod, case):  # noqa: F811
    B, Hq, Hkv, S, D, causal = case
    g = _gen(40 + S + D)
    Q, K, V = (torch.randn(B, h, S, D, generator=g) for h in (Hq, Hkv, Hkv))
    key_len = torch.randint(1, S + 1, (B,), generator=g, dtype=torch.int32)
    Kp, Vp = K.clone(), V.clone()
    for b in range(B):                                  # what a padded batch holds past its sentences
        Kp[b, :, key_len[b]:], Vp[b, :, key_len[b]:] = float("nan"), float("inf")
    for kl, k, v in ((None, K, V), (key_len, Kp, Vp)):
        O = torch.zeros(B, Hq, S, D, device="cuda")
        ac.attention_exact(Q.cuda(), k.cuda(), v.cuda(), O, causal=causal,
                           key_len=None if kl is None else kl.cuda())
        want = oracle_mod.attention_exact(parity.to_np(Q), parity.to_np(K), parity.to_np(V), causal=causal,
                                          key_len=None if kl is None else kl.numpy())
        assert parity.max_abs_err(O, want) <= parity.TOL[torch.float32]

    maps = _maps(2, 2, Hq, S, torch.float32, causal, 70 + S)
    clean = parity.to_np(maps).copy()
    if causal:                                          # nothing above the diagonal is ever used
        maps.masked_fill_(torch.ones(S, S, dtype=torch.bool).triu_(1), float("nan"))
    V2 = V[:, None].repeat(1, 2, 1, 1, 1)
    hit = torch.arange(B, dtype=torch.int32) % 3 - 1    # misses, entry 0, entry 1
    db = ac.attncache_build_db(torch.zeros(2, 16).cuda(), maps.cuda(), n_kv_heads=Hkv, head_dim=D, causal=causal)
    O = torch.full((B, 2, Hq, S, D), 7.0, device="cuda")
    ac.attncache_apply(db, hit.cuda(), V2.cuda(), O)
    want = oracle_mod.apply(clean, hit.numpy(), parity.to_np(V2), out=np.full((B, 2, Hq, S, D), 7.0))
    assert parity.max_abs_err(O, want) <= parity.TOL[torch.float32]
    db.close()


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_a_value_that_is_not_finite_reaches_only_the_rows_that_see_its_key(ac, oracle_mod, bad):  # noqa: F811
    Hq, Hkv, S, D, j0 = 3, 1, 40, 24, 21
    g = _gen(9)
    Q, K, V = (torch.randn(1, h, S, D, generator=g) for h in (Hq, Hkv, Hkv))
    clean = V.clone()
    clean[0, 0, j0, 5] = 0.0
    V[0, 0, j0, 5] = bad
    O = torch.zeros(1, Hq, S, D, device="cuda")
    ac.attention_exact(Q.cuda(), K.cuda(), V.cuda(), O, causal=True)
    want, P = oracle_mod.attention_exact(parity.to_np(Q), parity.to_np(K), parity.to_np(clean), causal=True,
                                         return_map=True)
    maps = torch.from_numpy(P.astype(np.float32)).reshape(1, 1, Hq, S, S)
    db = ac.attncache_build_db(torch.zeros(1, 16).cuda(), maps.cuda(), n_kv_heads=Hkv, head_dim=D, causal=True)
    O2 = torch.zeros(1, 1, Hq, S, D, device="cuda")
    ac.attncache_apply(db, torch.zeros(1, dtype=torch.int32).cuda(), V[:, None].cuda(), O2)
    db.close()
    for got in (O.cpu().numpy(), O2[:, 0].cpu().numpy()):
        assert not np.isfinite(got[:, :, j0:, 5]).any()
        got[:, :, j0:, 5] = want[:, :, j0:, 5]
        assert np.abs(got - want).max() <= parity.TOL[torch.float32]


@pytest.mark.parametrize("D", [3, 5, 21, 67, 131, 254])
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_the_end_of_a_row_stays_in_its_column(ac, oracle_mod, D, bad):  # noqa: F811
    """Rows that are no whole pieces are read in pieces that overlap: a value that is not finite shows in its own column only."""
    Hq, Hkv, S, j0 = 2, 1, 61, 37
    g = _gen(13 + D)
    Q, K, V = (torch.randn(1, h, S, D, generator=g) for h in (Hq, Hkv, Hkv))
    for c in {D - 1, max(0, D - 4), max(0, D - 5)}:
        clean, dirty = V.clone(), V.clone()
        clean[0, 0, j0, c], dirty[0, 0, j0, c] = 0.0, bad
        want, P = oracle_mod.attention_exact(parity.to_np(Q), parity.to_np(K), parity.to_np(clean), causal=False, return_map=True)
        O = torch.zeros(1, Hq, S, D, device="cuda")
        ac.attention_exact(Q.cuda(), K.cuda(), dirty.cuda(), O, causal=False)
        maps = torch.from_numpy(P.astype(np.float32)).reshape(1, 1, Hq, S, S)
        db = ac.attncache_build_db(torch.zeros(1, 16).cuda(), maps.cuda(), n_kv_heads=Hkv, head_dim=D, causal=False)
        O2 = torch.zeros(1, 1, Hq, S, D, device="cuda")
        ac.attncache_apply(db, torch.zeros(1, dtype=torch.int32).cuda(), dirty[:, None].cuda(), O2)
        db.close()
        for got in (O.cpu().numpy(), O2[:, 0].cpu().numpy()):
            assert not np.isfinite(got[..., c]).any()
            got[..., c] = want[..., c]
            assert np.abs(got - want).max() <= parity.TOL[torch.float32]


def test_three_workgroups_of_every_reuse_kernel_fit_a_compute_unit(ac):  # noqa: F811
    """168 vector registers a thread (of 512 per lane and SIMD, in eights) leave room for three waves on each SIMD, 53 KB
    of LDS for three workgroups."""
    class Attributes(ctypes.Structure):   # hipFuncAttributes
        _fields_ = [("binary", ctypes.c_int), ("cache", ctypes.c_int), ("const", ctypes.c_size_t), ("local", ctypes.c_size_t),
                    ("max_dynamic", ctypes.c_int), ("max_threads", ctypes.c_int), ("regs", ctypes.c_int),
                    ("carveout", ctypes.c_int), ("ptx", ctypes.c_int), ("shared", ctypes.c_size_t)]
    lib, seen = ctypes.CDLL(launches.LIB), 0
    out = subprocess.run(["nm", "-D", launches.LIB], text=True, capture_output=True, check=True).stdout
    for line in out.splitlines():
        kind, name = line.split()[-2:]
        if kind == "V" and "apply_f32_kernel" in name:
            at = Attributes()
            assert lib.hipFuncGetAttributes(ctypes.byref(at), ctypes.byref(ctypes.c_char.in_dll(lib, name))) == 0
            assert 0 < at.regs <= 168 and at.shared <= 160 * 1024 // 3, (name, at.regs, at.shared)
            seen += 1
    assert seen == 10
