"""The work that a user of this framework has it do, as cases that can be timed and compared.

A case names an entry point (``kind``) and its sizes.  ``listed()`` holds the cases that stand for
the whole range, ``draw()`` makes more of the same ranges, ``prepare()`` makes what a program has
in hand before the call (seeded inputs, workspace, database handle), ``run()`` is one pass through
the public entry points, ``exact()`` the same result from plain torch in 64 bits.

Inputs follow the recipe of ``paper_2510_25979_amd/synth.py``: unit-normalised Gaussian feature
vectors, planted queries at a cosine of about 0.995 next to fresh ones, maps that are the (causal)
softmax of Gaussian logits, Gaussian Q, K, V.  They are drawn here and not taken from there so that
``exact()`` uses none of the package.
"""
import math

import torch

from paper_2510_25979_amd import binding as ac

_DT = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


def listed():
    return [
        # The smallest call: a handful of requests against a small fp32 database, all three steps
        # (search, reuse of the hits, exact attention for the misses).  Launches count.
        dict(name="step-tiny-fp32", kind="step", B=4, N=1024, M=1024, E=128, emb="f32", L=1, Hq=2, Hkv=2,
             S=32, D=64, dt="f32", causal=True, packed=False, planted=0.5, theta=0.9),
        # The serving step of the 1B-shaped model: one batch of 64 sentences, all layers, half of
        # them served by cached maps, half recomputed.
        dict(name="step-1b-half-hits", kind="step", B=64, N=10000, M=96, E=256, emb="f16", L=16, Hq=32, Hkv=32,
             S=128, D=64, dt="bf16", causal=True, packed=True, planted=0.5, theta=0.9),
        # Reuse alone on long prompts (a layer at the longest sequences the paper evaluates).
        dict(name="reuse-long-layer", kind="reuse", B=16, M=16, L=1, Hq=32, Hkv=32, S=1024, D=128, dt="bf16",
             causal=True, packed=True, misses=0.0),
        # Reuse in binary32, the precision of the paper's models: ragged length (the 0-shot average),
        # three query heads on one V.
        dict(name="reuse-fp32-gqa", kind="reuse", B=16, M=24, L=2, Hq=24, Hkv=8, S=94, D=128, dt="f32",
             causal=True, packed=False, misses=0.25),
        # Exact attention of an encoder layer on short padded sentences.
        dict(name="exact-encoder-padded", kind="exact", B=64, Hq=12, Hkv=12, S=64, D=64, dt="bf16",
             causal=False, padded=True),
        # Exact attention of one layer on long prompts.
        dict(name="exact-long-layer", kind="exact", B=16, Hq=32, Hkv=32, S=1024, D=128, dt="bf16",
             causal=True, padded=False),
        # Exact attention in binary32, ragged length.
        dict(name="exact-fp32-gqa", kind="exact", B=16, Hq=24, Hkv=8, S=94, D=128, dt="f32",
             causal=True, padded=False),
        # Database building: several layers of medium prompts computed and remembered.
        dict(name="insert-layers-gqa", kind="insert", B=16, M=24, E=256, L=4, Hq=32, Hkv=8, S=288, D=128,
             causal=True, packed=True, padded=True),
        # Search of a large index by a large batch.
        dict(name="search-million", kind="search", B=256, N=1000000, E=256, emb="f16", metric="ip", k=1, theta=0.9),
        # The best few of a middle-sized index.
        dict(name="search-100k-top8", kind="search", B=64, N=100000, E=256, emb="f16", metric="ip", k=8, theta=0.9),
        # The index size the paper quotes its search latency on, in binary32 and Euclidean.
        dict(name="search-100k-l2-fp32", kind="search", B=64, N=100000, E=128, emb="f32", metric="l2", k=1, theta=0.5),
        # Feature projector of a batch of sentences.
        dict(name="project-batch", kind="project", B=64, S=128, dm=2048, hid=512, E=256, h="bf16", feat="f16",
             padded=True),
    ]


# ------------------------------------------------------------------------------- drawn cases
def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# No drawn case costs more than the largest listed one of its class.
_MAX_BYTES = 1.4e9         # one pass
_MAX_STATE = 6.0e9         # what a state holds
_MAX_FLOPS = 1.2e11        # matrix-core paths
_MAX_FLOPS_F32 = 5.0e8     # binary32 attention
_MAX_SCORES_F32 = 8.0e8    # N * B * E of a search on the vector ALUs
_MAX_SCORES_TOPK = 8.0e9   # the same of a top-k search on the matrix cores


def _heads(rng):
    hkv = rng.choice([1, 2, 4, 8, 12])
    return hkv * rng.choice([1, 1, 2, 3, 4]), hkv


def _attention_sizes(rng, f32):
    Hq, Hkv = _heads(rng)
    if f32:
        S, D = _log_int(rng, 16, 512), rng.choice([32, 64, 64, 80, 128, 128])
    else:
        S, D = 32 * _log_int(rng, 1, 32), rng.choice([64, 128])
    return dict(Hq=Hq, Hkv=Hkv, S=S, D=D, dt="f32" if f32 else "bf16", causal=rng.random() < 0.7)


def _fit(case, keys=("B", "L")):
    """Halve the named sizes until a pass and its state fit the limits above."""
    while True:
        w = work(case)
        f32 = case.get("dt") == "f32"
        state = w["bytes"]
        if "M" in case:
            state += case["M"] * case["L"] * case["Hq"] * case["S"] ** 2 * (4.0 if f32 else 2.0)
        if w["bytes"] <= _MAX_BYTES and state <= _MAX_STATE and w["flops"] <= (_MAX_FLOPS_F32 if f32 else _MAX_FLOPS):
            return case
        for key in keys:
            if case.get(key, 1) > 1:
                case[key] //= 2
                break
        else:
            case["Hq"] = case["Hkv"] = 1
        if "M" in case and case["kind"] != "step":
            case["M"] = max(2, min(case["M"], 2 * case["B"]))


def draw(rng):
    kind = rng.choice(["step", "reuse", "reuse", "exact", "exact", "insert", "search", "search", "project"])
    if kind == "search":
        f32 = rng.random() < 0.25
        c = dict(kind=kind, B=_log_int(rng, 1, 512), N=_log_int(rng, 500, 1000000),
                 E=rng.choice([64, 96, 128, 256, 256, 384, 512, 768]), emb="f32" if f32 else "f16",
                 metric="l2" if rng.random() < 0.25 else "ip", k=rng.choice([1, 1, 1, 2, 4, 8, 16]))
        c["theta"] = 0.9 if c["metric"] == "ip" else 0.5
        plain = c["emb"] == "f16" and c["metric"] == "ip" and c["E"] <= 512
        most = _MAX_SCORES_F32 if not plain else _MAX_FLOPS / 2 if c["k"] == 1 else _MAX_SCORES_TOPK
        while c["N"] * c["B"] * c["E"] > most:
            if c["B"] > 16:
                c["B"] //= 2
            else:
                c["N"] = max(500, c["N"] // 2)
        return c
    if kind == "project":
        dm = rng.choice([512, 768, 1024, 2048, 4096])
        c = dict(kind=kind, B=_log_int(rng, 1, 256), S=_log_int(rng, 8, 1024), dm=dm, hid=dm // 4,
                 E=rng.choice([128, 256, 512]), h="f32" if rng.random() < 0.25 else "bf16",
                 feat="f32" if rng.random() < 0.25 else "f16", padded=rng.random() < 0.5)
        return _fit(c, ("B", "S"))
    f32 = kind != "insert" and rng.random() < 0.25
    c = dict(kind=kind, B=_log_int(rng, 1, 128), **_attention_sizes(rng, f32))
    if kind == "exact":
        return _fit(dict(c, padded=rng.random() < 0.4), ("B",))
    c["L"] = rng.choice([1, 1, 2, 4, 8, 16, 32])
    c["packed"] = not f32 and rng.random() < 0.75
    if kind == "reuse":
        c.update(M=max(2, min(64, 2 * c["B"])), misses=rng.choice([0.0, 0.0, 0.25, 0.5]))
        return _fit(c)
    if kind == "insert":
        del c["dt"]
        c.update(M=2 * c["B"], E=rng.choice([128, 256]), padded=rng.random() < 0.5)
        return _fit(c)
    c.update(M=_log_int(rng, 8, 64), N=_log_int(rng, 500, 20000), E=rng.choice([128, 256, 512]),
             emb="f32" if f32 else "f16", planted=rng.choice([0.25, 0.5, 0.75, 1.0]), theta=0.9)
    return _fit(c)


# ------------------------------------------------------------------------------- work
def _lengths_mean(case):
    """Mean sentence length of a padded batch (see _lengths)."""
    return (max(1, case["S"] // 4) + case["S"]) / 2 if case.get("padded") else case["S"]


def _pairs(case):
    """Visible (query row, key) pairs of one head: what an attention map holds."""
    S, n = case["S"], _lengths_mean(case)
    return n * (n + 1) / 2 + (S - n) * n if case["causal"] else S * n


def _maps_bytes(case, esz):
    S = case["S"]
    return (S * (S + 1) / 2 if case["causal"] else S * S) * esz


def _reuse_work(case, tiles_b):
    esz = 4 if case["dt"] == "f32" else 2
    S, D, n = case["S"], case["D"], tiles_b * case["L"]
    return (n * (case["Hq"] * (_maps_bytes(case, esz) + S * D * esz) + case["Hkv"] * S * D * esz),
            n * case["Hq"] * 2.0 * D * _maps_bytes(case, 1))


def _exact_work(case, tiles_b):
    esz = 4 if case["dt"] == "f32" else 2
    S, D, n = case["S"], case["D"], tiles_b * case.get("L", 1)
    keys = _lengths_mean(case)
    return (n * (2 * case["Hq"] * S + 2 * case["Hkv"] * keys) * D * esz, n * case["Hq"] * 4.0 * D * _pairs(case))


def _search_work(case):
    esz = 4 if case["emb"] == "f32" else 2
    k = case.get("k", 1)
    return ((case["N"] + case["B"]) * case["E"] * esz + case["B"] * (8 * k + 4), 2.0 * case["N"] * case["B"] * case["E"])


def work(case):
    kind = case["kind"]
    if kind == "search":
        b, f = _search_work(case)
    elif kind == "reuse":
        b, f = _reuse_work(case, _n_hits(case))
    elif kind == "exact":
        b, f = _exact_work(case, case["B"])
    elif kind == "insert":
        b, f = _exact_work(dict(case, dt="bf16"), case["B"])
        b += case["B"] * (case["L"] * case["Hq"] * _maps_bytes(case, 2) + 4 * case["E"])
    elif kind == "project":
        esz = 4 if case["h"] == "f32" else 2
        B, dm, hid, E = case["B"], case["dm"], case["hid"], case["E"]
        b = B * _lengths_mean(case) * dm * esz + 4 * (hid * dm + E * hid + hid + E) + B * E * (4 if case["feat"] == "f32" else 2)
        f = B * _lengths_mean(case) * dm + 2.0 * B * hid * (dm + E)
    else:
        hits = _n_planted(case)
        bs, fs = _search_work(case)
        br, fr = _reuse_work(case, hits)
        bx, fx = _exact_work(case, case["B"] - hits)
        b, f = bs + br + bx, fs + fr + fx
    return {"bytes": float(b), "flops": float(f)}


def tolerance(case):
    """About four times the relative error against exact() that each kind shows: search 2.4e-7,
    project 2.1e-4 (binary16 features) and below 1e-6 (binary32), insert 2.2e-3, bf16 attention
    2.3e-3, binary32 attention 4.3e-7.  Indices may differ where two scores tie within rounding."""
    kind = case["kind"]
    if kind == "search":
        return {"rel": 1e-6, "differ": 0.01}
    if kind == "project":
        return {"rel": 1e-3 if case["feat"] == "f16" else 2e-6}
    if kind == "insert":
        return {"rel": 9e-3}
    out = {"rel": 1.5e-6} if case["dt"] == "f32" else {"rel": 9e-3}
    return dict(out, differ=0.01) if kind == "step" else out


# ------------------------------------------------------------------------------- inputs
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(2510 + seed)


def _randn(g, *shape, dtype=torch.float32):
    """Gaussian values; large tensors in slabs, so that the binary32 draw stays small."""
    if dtype == torch.float32 or math.prod(shape) < (1 << 26):
        return torch.randn(*shape, generator=g, device="cuda").to(dtype)
    t = torch.empty(*shape, dtype=dtype, device="cuda")
    for i in range(shape[0]):
        t[i].copy_(torch.randn(*shape[1:], generator=g, device="cuda"))
    return t


def _unit(x):
    return x / x.norm(dim=-1, keepdim=True)


def _n_planted(case):
    return int(round(case["B"] * case["planted"]))


def _n_hits(case):
    return case["B"] - int(case["B"] * case["misses"])


def _index_inputs(case, g, planted):
    """Feature vectors [N,E] and queries [B,E]: `planted` noisy copies of rows, the rest fresh."""
    N, B, E, dt = case["N"], case["B"], case["E"], _DT[case["emb"]]
    raw = torch.randn(N, E, generator=g, device="cuda")
    emb = _unit(raw).to(dt)
    rows = torch.randint(0, N, (B,), generator=g, device="cuda")
    q = raw[rows] + 0.1 * torch.randn(B, E, generator=g, device="cuda")
    fresh = torch.randn(B, E, generator=g, device="cuda")
    miss = torch.randperm(B, generator=g, device="cuda")[planted:]
    q[miss] = fresh[miss]
    return emb, _unit(q).to(dt)


def _maps(case, g):
    """Dense [M,L,Hq,S,S] maps: row-stochastic, exact zeros above the diagonal of causal ones."""
    M, L, H, S = case["M"], case["L"], case["Hq"], case["S"]
    out = torch.empty(M, L, H, S, S, dtype=_DT[case.get("dt", "bf16")], device="cuda")
    mask = torch.ones(S, S, dtype=torch.bool, device="cuda").triu_(1)
    step = max(1, (1 << 27) // (L * H * S * S))
    for m in range(0, M, step):
        x = torch.randn(min(step, M - m), L, H, S, S, generator=g, device="cuda")
        if case["causal"]:
            x.masked_fill_(mask, float("-inf"))
        out[m:m + step].copy_(torch.softmax(x, dim=-1))
    return out


def _lengths(case, g):
    """Real tokens per sentence of a right-padded batch, or None."""
    if not case.get("padded"):
        return None
    S = case["S"]
    return torch.randint(max(1, S // 4), S + 1, (case["B"],), generator=g, device="cuda", dtype=torch.int32)


def _inputs(case, seed):
    """Everything the seed decides, as plain tensors."""
    g, kind, x = _gen(seed), case["kind"], {}
    B = case["B"]
    if kind == "search":
        x["emb"], x["q"] = _index_inputs(case, g, (B + 1) // 2)
        return x
    if kind == "project":
        dm, hid, E = case["dm"], case["hid"], case["E"]
        offset = torch.randn(B, 1, dm, generator=g, device="cuda")
        x["h"] = torch.empty(B, case["S"], dm, dtype=_DT[case["h"]], device="cuda")
        for b in range(0, B, 16):
            part = x["h"][b:b + 16]
            part.copy_(offset[b:b + 16] + torch.randn(part.shape, generator=g, device="cuda"))
        x["W1"] = torch.randn(hid, dm, generator=g, device="cuda") / math.sqrt(dm)
        x["b1"] = 0.1 * torch.randn(hid, generator=g, device="cuda")
        x["W2"] = torch.randn(E, hid, generator=g, device="cuda") / math.sqrt(hid)
        x["b2"] = 0.1 * torch.randn(E, generator=g, device="cuda")
        x["len"] = _lengths(case, g)
        return x
    L, S, D, Hq, Hkv = case.get("L", 1), case["S"], case["D"], case["Hq"], case["Hkv"]
    dt = _DT[case.get("dt", "bf16")]
    lead = (B,) if kind == "exact" else (B, L)
    if kind != "reuse":
        x["Q"] = _randn(g, *lead, Hq, S, D, dtype=dt)
        x["K"] = _randn(g, *lead, Hkv, S, D, dtype=dt)
    x["V"] = _randn(g, *lead, Hkv, S, D, dtype=dt)
    if kind in ("exact", "insert"):
        x["len"] = _lengths(case, g)
    if kind in ("step", "reuse"):
        x["maps"] = _maps(case, g)
    if kind == "reuse":
        x["hit"] = torch.randint(0, case["M"], (B,), generator=g, device="cuda", dtype=torch.int32)
        x["hit"][torch.randperm(B, generator=g, device="cuda")[_n_hits(case):]] = -1
    if kind == "step":
        x["emb"], x["q"] = _index_inputs(case, g, _n_planted(case))
        x["map_of"] = (torch.arange(case["N"], device="cuda") % case["M"]).to(torch.int32)
    if kind == "insert":
        x["slot"] = torch.randperm(case["M"], generator=g, device="cuda")[:B].to(torch.int32)
        x["feat"] = _unit(torch.randn(B, case["E"], generator=g, device="cuda")).half()
    return x


def _search_buffers(s, B, k):
    s["ws"] = torch.empty(ac.attncache_workspace_bytes(s["db"].desc, B, k), dtype=torch.uint8, device="cuda")
    s["idx"] = torch.empty(B, k, dtype=torch.int32, device="cuda")
    s["score"] = torch.empty(B, k, dtype=torch.float32, device="cuda")
    s["found"] = torch.empty(B, dtype=torch.int32, device="cuda")


def _store(case, maps):
    """The maps as the database keeps them, and the arguments that say so."""
    if not case["packed"]:
        return maps, {}
    S = case["S"]
    out = torch.empty(*maps.shape[:3], ac.packed_tile_elems(S, case["causal"]), dtype=maps.dtype, device="cuda")
    ac.attncache_pack_maps(maps, out, causal=case["causal"])
    return out, {"seq_len": S}


def prepare(case, seed):
    kind, x = case["kind"], _inputs(case, seed)
    s = dict(x, case=case)
    B = case["B"]
    if kind == "search":
        stand_in = torch.zeros(1, 1, 1, 8, 8, device="cuda")   # this handle is searched only
        s["db"] = ac.attncache_build_db(x["emb"], stand_in, n_kv_heads=1, head_dim=8,
                                        metric=ac.AC_L2 if case["metric"] == "l2" else ac.AC_IP,
                                        map_of=torch.zeros(case["N"], dtype=torch.int32, device="cuda"))
        _search_buffers(s, B, case["k"])
        return s
    if kind == "project":
        s["feat"] = torch.empty(B, case["E"], dtype=_DT[case["feat"]], device="cuda")
        n = ac.attncache_project_workspace_bytes(B, case["dm"], case["hid"], case["E"])
        s["ws"] = torch.empty(n, dtype=torch.uint8, device="cuda")
        return s
    if kind == "exact":
        s["O"] = torch.zeros_like(x["Q"])
        return s
    L, S, D, Hq = case["L"], case["S"], case["D"], case["Hq"]
    s["O"] = torch.zeros(B, L, Hq, S, D, dtype=x["V"].dtype, device="cuda")
    if kind == "insert":
        per = ac.packed_tile_elems(S, case["causal"]) if case["packed"] else 0
        shape = (case["M"], L, Hq, per) if case["packed"] else (case["M"], L, Hq, S, S)
        s["maps"], kw = torch.zeros(shape, dtype=torch.bfloat16, device="cuda"), {"seq_len": S}
        s["emb"], map_of = torch.zeros(case["M"], case["E"], dtype=torch.float16, device="cuda"), None
    else:
        s["maps"], kw = _store(case, x["maps"])
        if kind == "step":
            map_of = x["map_of"]
        else:
            s["emb"], map_of = torch.zeros(case["M"], 16, device="cuda"), None
    s["db"] = ac.attncache_build_db(s["emb"], s["maps"], n_kv_heads=case["Hkv"], head_dim=D,
                                    causal=case["causal"], map_of=map_of, **kw)
    if kind == "step":
        _search_buffers(s, B, 1)
        fold = lambda t: t.view(B, -1, S, D)   # noqa: E731  layers fold into heads
        s["folded"] = tuple(fold(s[n]) for n in ("Q", "K", "V", "O"))
    return s


# ------------------------------------------------------------------------------- one pass
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "search":
        ac.attncache_search(s["db"], s["q"], case["k"], case["theta"], s["idx"], s["score"], s["found"], s["ws"])
        return {"idx": s["idx"], "score": s["score"], "hit": s["found"]}
    if kind == "project":
        ac.attncache_project(s["h"], s["W1"], s["b1"], s["W2"], s["b2"], s["feat"], s["ws"], seq_len=s["len"])
        return {"feat": s["feat"]}
    if kind == "exact":
        ac.attention_exact(s["Q"], s["K"], s["V"], s["O"], causal=case["causal"], key_len=s["len"])
        return {"O": s["O"]}
    if kind == "reuse":
        ac.attncache_apply(s["db"], s["hit"], s["V"], s["O"])
        return {"O": s["O"]}
    if kind == "insert":
        ac.attncache_insert(s["db"], s["Q"], s["K"], s["V"], s["O"], slot=s["slot"], feat=s["feat"], key_len=s["len"])
        return {"O": s["O"], "maps": s["maps"], "emb": s["emb"]}
    ac.attncache_search(s["db"], s["q"], 1, case["theta"], s["idx"], s["score"], s["found"], s["ws"])
    ac.attncache_apply(s["db"], s["found"], s["V"], s["O"])
    q, k, v, o = s["folded"]
    ac.attention_exact(q, k, v, o, causal=case["causal"], row_sel=s["found"])
    return {"idx": s["idx"], "score": s["score"], "hit": s["found"], "O": s["O"]}


# ------------------------------------------------------------------------------- 64 bits
def _exact_search(x, case, k):
    e, q = x["emb"].double(), x["q"].double()
    s = q @ e.t()
    if case.get("metric") == "l2":
        s = 2 * s - (q * q).sum(1, keepdim=True) - (e * e).sum(1)
    score, idx = torch.sort(s, dim=1, descending=True, stable=True)   # equal scores: the lower row first
    score, idx = score[:, :k].contiguous(), idx[:, :k].to(torch.int32).contiguous()
    best = score[:, 0].float()
    sim = 1 - (-score[:, 0]).sqrt().float() if case.get("metric") == "l2" else best
    entry = x["map_of"][idx[:, 0].long()] if "map_of" in x else torch.zeros_like(idx[:, 0])
    return idx, score, torch.where(sim >= case["theta"], entry, torch.full_like(entry, -1))


def _exact_attention(q, k, v, causal, length):
    """q [Hq,S,D], k and v [Hkv,S,D] of one item -> (O, map) in 64 bits."""
    g, S = q.shape[0] // k.shape[0], q.shape[1]
    k, v = (t.double().repeat_interleave(g, 0).contiguous() for t in (k, v))
    s = torch.matmul(q.double(), k.transpose(1, 2).contiguous()) / math.sqrt(q.shape[2])
    if causal:
        s.masked_fill_(torch.ones(S, S, dtype=torch.bool, device="cuda").triu_(1), float("-inf"))
    if length is not None:
        s[:, :, int(length):] = float("-inf")
    p = torch.softmax(s, -1)
    return torch.matmul(p, v), p


def _exact_packed(p, causal):
    """One item's maps [H,S,S] in the packed block layout of the map store."""
    H, S = p.shape[0], p.shape[1]
    t = p.view(H, S // 16, 16, S // 32, 4, 8).permute(0, 1, 3, 4, 2, 5)   # [H][r][cb][q][i][e]
    t = t.reshape(H, S // 16, S // 32, 512)
    if not causal:
        return t.reshape(H, -1)
    return torch.cat([t[:, r, : (r + 2) // 2].reshape(H, -1) for r in range(S // 16)], 1)


def exact(case, seed):
    x, kind = _inputs(case, seed), case["kind"]
    B = case["B"]
    if kind == "search":
        idx, score, hit = _exact_search(x, case, case["k"])
        return {"idx": idx, "score": score, "hit": hit}
    if kind == "project":
        pooled = torch.empty(B, case["dm"], dtype=torch.float64, device="cuda")
        for b in range(B):
            n = case["S"] if x["len"] is None else int(x["len"][b])
            pooled[b] = x["h"][b, :n].double().mean(0)
        y = torch.relu(pooled @ x["W1"].double().t() + x["b1"].double())
        return {"feat": _unit(y @ x["W2"].double().t() + x["b2"].double())}
    if kind == "exact":
        out = torch.empty(x["Q"].shape, dtype=torch.float64, device="cuda")
        for b in range(B):
            out[b] = _exact_attention(x["Q"][b], x["K"][b], x["V"][b], case["causal"],
                                      None if x["len"] is None else x["len"][b])[0]
        return {"O": out}
    L, S, D, Hq, Hkv = case["L"], case["S"], case["D"], case["Hq"], case["Hkv"]
    out = torch.zeros(B, L, Hq, S, D, dtype=torch.float64, device="cuda")
    if kind == "insert":
        maps = torch.zeros(case["M"], L, Hq, S * S, dtype=torch.float32, device="cuda")
        emb = torch.zeros(case["M"], case["E"], dtype=torch.float64, device="cuda")
        for b in range(B):
            slot = int(x["slot"][b])
            emb[slot] = x["feat"][b].double()
            for l in range(L):
                out[b, l], p = _exact_attention(x["Q"][b, l], x["K"][b, l], x["V"][b, l], case["causal"],
                                                None if x["len"] is None else x["len"][b])
                flat = _exact_packed(p, case["causal"]) if case["packed"] else p.reshape(Hq, -1)
                maps[slot, l, :, : flat.shape[1]] = flat.float()
        maps = maps[..., : flat.shape[1]].contiguous()
        return {"O": out, "maps": maps if case["packed"] else maps.view(case["M"], L, Hq, S, S), "emb": emb}
    got = {}
    hit = x.get("hit")
    if kind == "step":
        idx, score, hit = _exact_search(x, case, 1)
        got = {"idx": idx, "score": score, "hit": hit}
    for b in range(B):
        m = int(hit[b])
        for l in range(L):
            if m >= 0:
                v = x["V"][b, l].double().repeat_interleave(Hq // Hkv, 0).contiguous()
                out[b, l] = torch.matmul(x["maps"][m, l].double(), v)
            elif kind == "step":
                out[b, l] = _exact_attention(x["Q"][b, l], x["K"][b, l], x["V"][b, l], case["causal"], None)[0]
    return dict(got, O=out)
