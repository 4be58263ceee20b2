"""The case lists of the GPU tests reach every kernel that the library can launch, by its own launch
rules (host code on a recorder, no GPU): a rule that moves leaves no kernel untested unnoticed."""
import subprocess

import pytest

import bench
from paper_2510_25979_amd import synth
from tests import launches
from tests import test_gpu_f32_tiles as f32
from tests import test_gpu_parity_small as small
from tests import test_gpu_projector as proj
from tests import test_gpu_row_units as rows
from tests import test_gpu_search_tiles as tiles
from tests import test_gpu_short_attention as short
from tests import test_gpu_short_reuse as reuse
from tests import test_gpu_split_units as split

# fp16 rows of more than 2,360 columns, more than 64 queries and 128 groups: 5e9 products and more for
# the oracle.  The variants with one query per wave, and all three of the Euclidean metric, are reached.
NOT_RUN = {"search_valu_kernel<half, false, %d, %s>" % (q, k) for q in (2, 4) for k in ("true", "false")}


def _kernels(*prefixes):
    """Kernels of the built library: the handles that its host code passes to a launch."""
    out = subprocess.run(["nm", "-D", launches.LIB], text=True, capture_output=True, check=True).stdout
    names = launches.plain(l.split()[-1] for l in out.splitlines() if " V " in l or " D " in l)
    return {n for n in names if n.startswith(prefixes)}


def _reached(tmp_path, calls):
    seen = set()
    for call, (status, ls) in zip(calls, launches.record(calls, tmp_path)):
        assert status == 0, call
        seen |= {la[0] for la in ls}
    return seen


def _search(c):
    return ("search", *c[:4], "f16" if "16" in str(c[4]) else "f32", c[5])


def test_every_search_kernel_is_reached(tmp_path):
    cases = (tiles.VALU_CASES + tiles.VARIANT_CASES + tiles.TOPK_CASES + tiles.BOUND_CASES + small.SEARCH_CASES +
             [(*c[:3], k, *c[3:]) for _, c in tiles.OPEN_CASES for k in (1, 5)] +
             small._random_search_shapes(40, 20251128))
    missing = _kernels("search_", "finalize_") - _reached(tmp_path, [_search(c) for c in cases])
    assert missing == NOT_RUN


@pytest.mark.parametrize("kernel", ["search_stream_kernel<float", "search_stream_kernel<half", "search_valu_kernel<float",
                                    "search_row_kernel", "search_f16_kernel<0", "search_f16_kernel<16", "search_f16_big_kernel"])
def test_queries_with_nan_reach_every_kind_of_search_kernel(tmp_path, kernel):
    seen = _reached(tmp_path, [_search(c) for c in small.NAN_CASES])
    assert any(k.startswith(kernel) for k in seen)


def _dt(t):
    return str(t).split(".")[-1].replace("bfloat", "bf").replace("float", "f")


def test_every_attention_kernel_is_reached(tmp_path):
    calls = []
    for large, cases in ((False, rows.CASES), (True, rows.CASES + rows.LARGE_CASES)):
        for Hq, Hkv, S, D, causal, lens in cases:
            B = lens if isinstance(lens, int) else len(lens)
            n = rows.copies(Hq, S, B) if large else 1
            calls += [("exact", n * B, Hq, Hkv, S, D, causal, "bf16")]
            calls += [("insert", n * B, 1, Hq, Hkv, S, D, causal, packed) for packed in (False, True)]
    calls += [("exact", *c[:6], _dt(c[7])) for c in small.EXACT_CASES]
    calls += [("exact", *c[:6], _dt(c[6])) for c in small.PADDED_CASES]
    calls += [("exact", *c, "f32") for c in f32.CASES]
    calls += [("exact", len(c[6]) * n, *c[:5], _dt(c[5])) for c in split.CASES for n in (1, split.copies(c))]
    calls += [("insert", *c, packed) for c in small.INSERT_CASES for packed in (False, True)]
    calls += [("exact", *c, "bf16", routed) for c in short.EXACT_CASES for routed in (False, True)]
    calls += [("insert", *c, packed) for c in short.INSERT_CASES for packed in (False, True)]
    calls += [("apply", c[0], c[9], *c[3:8], _dt(c[10])) for c in small.APPLY_CASES]
    calls += [("apply", c[0], 2, *c[1:], "f32") for c in f32.CASES]
    for layout in (False, True):
        calls += [("apply", c[0], c[9], *c[3:8], _dt(c[10]), layout) for c in small.APPLY_CASES if "bf" in _dt(c[10])]
        calls += [("apply", B, Lc, Hkv * g, Hkv, S, D, causal, "bf16", layout) for B, Lc, Hkv, g in reuse.CASES for S in (32, 64, 96)
                  for D in (64, 128) for causal in (True, False)]
        calls += [("apply", B, Lc, Hkv * g, Hkv, 128, D, causal, "bf16", layout) for B, Lc, Hkv, g in reuse.CASES_128 for D in (64, 128)
                  for causal in (True, False)]
    missing = _kernels("exact_", "insert_", "apply_") - _reached(tmp_path, calls)
    assert not missing


def _project(c):
    return ("project", *c[:5], _dt(c[5]), _dt(c[6]), c[9])


def test_every_projector_kernel_is_reached(tmp_path):
    missing = _kernels("pool_", "dense_", "finish_") - _reached(tmp_path, [_project(c) for c in proj.CASES])
    assert not missing


@pytest.mark.parametrize("case,kernel", [
    ((300, 520, 200, 1, "f16", "ip"), "search_stream_kernel<half, false, 1"),    # 38 us on the matrix cores, 12.5 so
    ((1000, 520, 200, 1, "f16", "ip"), "search_stream_kernel<half, false, 4"),   # 39, 16
    ((4000, 520, 100, 1, "f16", "ip"), "search_stream_kernel<half, false, 4"),
    ((7500, 1536, 64, 1, "f16", "ip"), "search_f16_kernel<0, 1"),
    ((1000, 4608, 8, 1, "f16", "ip"), "search_stream_kernel<half, false, 1"),    # 368 in tiles, 32
    ((20000, 8192, 8, 1, "f16", "l2"), "search_stream_kernel<half, true, 4"),    # 943, 224
    ((20000, 8192, 8, 1, "f32", "ip"), "search_valu_kernel<float"),              # 343, 379 in streams
    ((300000, 8, 8, 1, "f16", "l2"), "search_row_kernel<half"),                  # 28 in streams, 11
    ((20000, 20, 8, 1, "f32", "ip"), "search_row_kernel<float"),
    ((20000, 37, 8, 1, "f32", "ip"), "search_stream_kernel<float, false, 4"),
    ((100000, 128, 64, 1, "f32", "l2"), "search_bound_kernel<float, true, 2"),   # 57 in tiles of all rows, 24
    ((100000, 32, 24, 1, "f32", "l2"), "search_valu_kernel<float, true, 2"),      # bounds 15.8, 14.6
    ((100000, 32, 40, 8, "f32", "ip"), "search_valu_kernel<float, false, 4"),    # bounds 26.1, 22.6
    ((2000, 128, 400, 1, "f32", "ip"), "search_valu_kernel<float, false, 1"),    # bounds 21.2, 18.9
    ((2000, 64, 400, 1, "f16", "l2"), "search_stream_kernel<half, true, 4"),     # bounds 16.4, 14.2
    ((300000, 64, 9, 1, "f32", "ip"), "search_valu_kernel<float, false, 4"),     # bounds 28.6, 27.4
    ((32000, 64, 64, 1, "f32", "ip"), "search_bound_kernel<float, false, 2"),    # 19.4 in tiles of all rows, 13.7
    ((32000, 64, 40, 1, "f16", "l2"), "search_bound_kernel<half, true, 2"),      # 15.5, 12.3
    ((640, 256, 4, 1, "f32", "ip"), "search_small_kernel<float, false, false, 2"),   # one row of a thread 9.6, two 9.0
    ((300, 512, 4, 4, "f16", "ip"), "search_small_kernel<half, false, true, 4"),     # 11.2, four 9.4
    ((100, 640, 16, 1, "f16", "ip"), "search_small_kernel<half, false, false, 1"),   # 6.2, 6.7
    ((2000, 15, 4, 1, "f32", "ip"), "search_row_kernel<float"),                      # 6.7 in one launch, 5.6
    ((2000, 16, 4, 1, "f32", "ip"), "search_small_kernel<float"),                    # 4.8, 5.3
    ((1644, 22, 179, 1, "f32", "ip"), "search_small_kernel<float"),                  # 7.6, 9.4
    ((250, 8, 4, 1, "f16", "l2"), "search_row_kernel<half"),                         # 5.2, 5.0
], ids=str)
def test_the_kernel_that_measured_best_serves_the_shape(tmp_path, case, kernel):
    (status, ls), = launches.record([("search", *case)], tmp_path)
    assert status == 0 and ls[0][0].startswith(kernel), ls


@pytest.mark.parametrize("S,D,kernel", [(1, 256, "apply_f32_small_kernel"), (5, 256, "apply_f32_small_kernel"),
                                        (16, 12, "apply_f32_small_kernel"), (16, 64, "apply_f32_kernel<1>"),
                                        (6, 256, "apply_f32_kernel<4>"), (94, 128, "apply_f32_kernel<2>")])
def test_reuse_of_maps_of_a_few_rows_takes_a_thread_per_output(tmp_path, S, D, kernel):
    # 256 heads of one row of 256: 6.6 us in tiles of 16 rows, 2.4 so
    (status, ls), = launches.record([("apply", 64, 1, 4, 4, S, D, True, "f32")], tmp_path)
    assert status == 0 and [la[0] for la in ls] == [kernel]


@pytest.mark.parametrize("case,launched", [
    ((64, 128, 2048, 512, 256), 2),     # us, four launches / fewer: 21.6 / 18.3
    ((32, 16, 4096, 1024, 256), 4),     # 22.4 / 23.7, beyond the line
    ((16, 16, 4096, 1024, 512), 3),     # 23.7 / 22.3, on it
    ((20, 83, 3432, 856, 256), 4),      # 24.5 / 30.7, rows off the 128-byte lines
    ((66, 48, 680, 696, 512), 4),       # 20.4 / 25.3
    ((130, 169, 1384, 344, 512), 4),    # 33.0 / 39.6
    ((4, 30, 2872, 712, 128), 2),       # 20.3 / 16.2
    ((3, 1887, 1024, 600, 256), 3),     # 46.6 / 19.1, long sentences
], ids=str)
def test_the_projector_takes_the_launches_that_measured_best(tmp_path, case, launched):
    (status, ls), = launches.record([("project", *case, "bf16", "f16", True)], tmp_path)
    assert status == 0 and len(ls) == launched, ls


@pytest.mark.parametrize("case", [(64, 20, 2048, 512, 256), (12, 9, 4096, 1024, 256)], ids=str)
def test_a_workspace_for_four_launches_takes_four(tmp_path, case):
    B, S, dm, hid, E = case
    least = 4 * B * (dm + 4 * hid + 4 * E)   # the pooled input and four partial results of each layer
    calls = [("project", *case, "bf16", "f32", True, *ws) for ws in ((), (least,), (least - 16,))]
    (_, few), (status, four), (refused, none) = launches.record(calls, tmp_path)
    assert len(few) < 4 and status == 0 and len(four) == 4 and refused == -6 and not none


@pytest.mark.parametrize("dt,metric", [("f16", "ip"), ("f16", "l2"), ("f32", "ip")])
def test_selections_of_256_threads_are_small(tmp_path, dt, metric):
    """What lets them do without a bound that rises: no more than 1,024 groups, of 32 rows at least, of which 256 rows are no
    more than eight."""
    calls = [("search", N, E, 300, min(k, N), dt, metric) for N in (200, 250, 257, 513, 4096, 32768, 32769, 65536, 65600)
             for E in (40, 64, 256) for k in (2, 3, 4, 8, 9, 16, 64)]
    for call, (status, ls) in zip(calls, launches.record(calls, tmp_path)):
        small = any(la[0].startswith("finalize_topk_kernel") and ", 256, " in la[0] for la in ls)
        assert status == 0 and (not small or call[4] <= 8 or call[1] <= 256), call


def test_the_projector_workspace_holds_every_length_and_smaller_batch(tmp_path):
    """Where the launches depend on the sentences' length, the workspace, which does not know it, is enough for the fewest."""
    import ctypes
    lib = ctypes.CDLL(launches.LIB)
    lib.attncache_project_workspace_bytes.restype = ctypes.c_size_t
    for B, dm, hid, E in [(16, 1744, 872, 480), (20, 3432, 856, 256), (6, 1024, 600, 256), (70, 2048, 512, 256)]:
        ws = lib.attncache_project_workspace_bytes(B, dm, hid, E)
        calls = [("project", b, S, dm, hid, E, "bf16", "f16", True, *bytes) for b in (1, B // 2, B) for S in (1, 100, 3000)
                 for bytes in ((), (ws,))]
        got = launches.record(calls, tmp_path)
        assert got[::2] == got[1::2] and all(status == 0 for status, _ in got)


@pytest.mark.parametrize("case,kernel", [
    ((64, 16, 32, 32, 128, 64, True, True), "insert_bf16_short_kernel<64, true, true"),
    ((64, 12, 32, 32, 128, 128, True, True), "insert_bf16_short_kernel<128, true, true"),   # us, two passes over the keys 651, one 639
    ((64, 16, 32, 32, 128, 128, True, True), "insert_bf16_kernel<128, true, true"),         # 852, 874
    ((64, 16, 32, 32, 128, 64, True, False), "insert_bf16_kernel<64, true, false"),         # 618, 788
    ((64, 8, 64, 16, 128, 64, True, False), "insert_bf16_short_kernel<64, true, false"),    # 563, 513
    ((64, 16, 32, 16, 96, 64, True, False), "insert_bf16_short_kernel<64, true, false"),    # 372, 360
    ((64, 16, 32, 16, 128, 128, True, True), "insert_bf16_kernel<128, true, true"),         # 713, 746
    ((64, 8, 128, 16, 128, 128, True, True), "insert_bf16_short_kernel<128, true, true"),   # 1,216, 1,188
    ((64, 8, 32, 32, 96, 128, True, False), "insert_bf16_kernel<128, true, false"),         # 354, 382
    ((64, 8, 32, 16, 128, 128, True, False), "insert_bf16_short_kernel<128, true, false"),  # 415, 405
    ((128, 1, 32, 16, 128, 64, True, False), "insert_bf16_kernel<64, true, false"),         # 55.5, 57.7
    ((32, 1, 16, 8, 128, 64, True, False), "insert_bf16_short_kernel<64, true, false"),     # 13.0, 12.4
    ((64, 8, 32, 16, 128, 64, True, False), "insert_bf16_short_kernel<64, true, false"),    # 296, 281
    ((128, 1, 32, 32, 96, 64, True, False), "insert_bf16_short_kernel<64, true, false"),    # 46.8, 45.1
    ((256, 1, 32, 32, 96, 64, True, False), "insert_bf16_kernel<64, true, false"),          # 111, 116
    ((64, 16, 32, 32, 128, 64, False, False), "insert_bf16_short_kernel<64, false, false"),   # 606, 581
    ((64, 32, 32, 16, 64, 128, True, False), "insert_bf16_kernel<128, true, false"),        # 719, 753
    ((64, 32, 32, 16, 64, 128, True, True), "insert_bf16_short_kernel<128, true, true"),    # 686, 650
    # and small ones: the workgroups of the other kernels would begin a second round
    ((40, 1, 8, 4, 32, 64, True, True), "insert_bf16_short_kernel<64, true, true"),         # 5.7, 5.0
    ((16, 1, 8, 4, 64, 64, True, True), "insert_bf16_split_kernel<64, true, true"),         # 5.1, 5.7
    ((12, 1, 8, 4, 96, 128, True, True), "insert_bf16_short_kernel<128, true, true"),       # 9.2, 7.7
    ((22, 1, 8, 4, 96, 64, True, True), "insert_bf16_short_kernel<64, true, true"),         # 9.3, 6.6
    ((16, 1, 8, 1, 128, 64, True, True), "insert_bf16_split_kernel<64, true, true"),        # 7.0, 7.3
    ((96, 1, 8, 8, 64, 64, True, True), "insert_bf16_kernel<64, true, true"),               # 7.0, 7.7
    ((97, 1, 8, 8, 64, 64, True, True), "insert_bf16_short_kernel<64, true, true"),         # 9.7, 7.8
    ((65, 1, 8, 8, 32, 128, True, True), "insert_bf16_short_kernel<128, true, true"),       # 8.9, 6.7
], ids=str)
def test_large_inserts_of_short_sequences_take_the_kernel_that_measured_best(tmp_path, case, kernel):
    (status, ls), = launches.record([("insert", *case)], tmp_path)
    assert status == 0 and ls[0][0].startswith(kernel), ls


@pytest.mark.parametrize("case,grid", [
    # B, layers, heads, K/V heads, S, D, causal, packed; workgroups                              us, one workgroup a tile / workgroups of four units
    ((64, 32, 32, 16, 128, 128, True, True), 2 * 32768),   # 886 / 774
    ((64, 32, 32, 16, 128, 128, False, False), 2 * 32768),   # 1,015 / 914
    ((64, 4, 32, 16, 128, 128, True, True), 4096),         # 86.7 / 86.9
    ((64, 16, 32, 16, 96, 128, True, True), 16384),        # 127 / 135 (six units)
    ((63, 21, 72, 9, 32, 64, True, False), 2 * 11912),     # (11,907 tiles, rounded up to eight)
    ((16, 4, 16, 8, 128, 128, True, True), 512),           # 11.9 / 16.8
    ((16, 2, 16, 8, 128, 128, True, True), 2 * 256),
    ((16, 1, 64, 8, 128, 128, True, True), 8 * 128),       # 18.8 / 17.1
    ((16, 2, 64, 8, 64, 128, True, True), 4 * 256),        # 11.1 / 10.9
], ids=str)
def test_workgroups_of_short_reuse(tmp_path, case, grid):
    (status, ls), = launches.record([("apply", *case[:7], "bf16", case[7])], tmp_path)
    assert status == 0 and [(la[0].split("<")[0], la[1]) for la in ls] == [("apply_bf16_short_kernel", grid)]


@pytest.mark.parametrize("case,kernel", [
    # B, layers, heads, K/V heads                      us, two halves / units of 32 rows
    ((8, 8, 32, 8), "apply_bf16_short_kernel<64"),     # (512 tiles)
    ((12, 8, 32, 8), "apply_bf16_kernel<true>"),       # 18.1 / 18.9
    ((64, 8, 32, 8), "apply_bf16_kernel<true>"),       # 96.5 / 100
    ((128, 8, 24, 8), "apply_bf16_short_kernel<64"),   # 165 / 157
    ((128, 8, 32, 8), "apply_bf16_short_kernel<64"),   # 235 / 211
    ((64, 8, 96, 8), "apply_bf16_short_kernel<64"),    # 351 / 301
    ((128, 8, 8, 8), "apply_bf16_kernel<false>"),      # 61.3 / 63.8
    ((512, 8, 8, 8), "apply_bf16_kernel<false>"),      # 290 / 289
], ids=str)
def test_packed_causal_maps_of_128_x_64_take_the_kernel_that_measured_best(tmp_path, case, kernel):
    (status, ls), = launches.record([("apply", *case, 128, 64, True, "bf16", True)], tmp_path)
    assert status == 0 and ls[0][0].startswith(kernel), ls


@pytest.mark.parametrize("case,grid", [
    # B, heads, K/V heads, S, D, causal; workgroups                us, one workgroup a K/V head / workgroups of four units
    ((512, 128, 16, 32, 128, True), 2 * 8192),       # 238 / 207
    ((128, 256, 16, 32, 128, True), 4 * 2048),       # 100 / 99
    ((512, 128, 16, 32, 64, True), 2 * 8192),        # 105 / 105
    ((256, 128, 16, 32, 64, True), 4096),            # 47.5 / 48.4
    ((512, 64, 16, 64, 128, True), 8192),            # 246 / 254
    ((1367, 24, 2, 32, 128, False), 3 * 2736),       # (2,734 K/V heads, rounded up to eight)
], ids=str)
def test_workgroups_of_short_exact_attention(tmp_path, case, grid):
    (status, ls), = launches.record([("exact", *case, "bf16")], tmp_path)
    assert status == 0 and [(la[0].split("<")[0], la[1]) for la in ls] == [("exact_bf16_short_kernel", grid)]


@pytest.mark.parametrize("case,kernel", [
    ((1024, 32, 16, 128, 128, True), "exact_bf16_kernel<128, true, true"),          # us, resident 586, short 620
    ((512, 32, 16, 128, 128, True), "exact_bf16_short_kernel<128, true, 4"),        # 298, 296
    ((2048, 64, 16, 128, 128, True), "exact_bf16_short_kernel<128, true, 4"),       # 1,970, 1,981
    ((2048, 32, 16, 128, 64, True), "exact_bf16_short_kernel<64, true, 4"),         # 577, 543
], ids=str)
def test_large_exact_launches_of_128_rows_take_the_kernel_that_measured_best(tmp_path, case, kernel):
    (status, ls), = launches.record([("exact", *case, "bf16")], tmp_path)
    assert status == 0 and ls[0][0].startswith(kernel), ls


@pytest.mark.parametrize("heads", [{}, dict(n_q_heads=8, n_kv_heads=8), dict(n_q_heads=32, n_kv_heads=16)], ids=str)
@pytest.mark.parametrize("scale", [{}, dict(batch=1), dict(batch=5, n_layers=1), dict(seq_len=64), dict(seq_len=32, n_layers=2),
                                   dict(head_dim=64), dict(head_dim=128, batch=16), dict(seq_len=96, n_layers=3)], ids=str)
def test_the_benchmark_names_the_kernels_that_run(tmp_path, scale, heads):
    calls, names = [], []
    for w in synth.WORKLOADS.values():
        w = w.scaled(**scale, **heads)
        bf16 = w.map_dtype == "bf16"
        size = (w.n_q_heads, w.n_kv_heads, w.seq_len, w.head_dim, w.causal)
        for layout in ("packed", "dense") if bf16 else ("dense",):
            calls.append(("apply", w.batch, w.n_layers, *size, w.map_dtype, layout == "packed"))
            names.append(bench.apply_kernel_name(w, layout))
        calls.append(("exact", w.batch, w.n_layers * w.n_q_heads, w.n_layers * w.n_kv_heads, *size[2:], w.map_dtype))
        names.append(bench.exact_kernel_name(w))
        if bf16:
            calls.append(("insert", w.batch, w.n_layers, *size, True))
            names.append(bench.insert_kernel_name(w))
    for call, name, (status, ls) in zip(calls, names, launches.record(calls, tmp_path)):
        ran = ls[0][0]
        if ran.startswith("exact_bf16_kernel<"):
            ran = "exact_bf16_kernel (%s)" % ("resident" if ran.endswith("true>") else "streaming")
        assert status == 0 and ran.split("<")[0] == name, (call, ran, name)
