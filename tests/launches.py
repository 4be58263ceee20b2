"""Which kernels a call launches, and how: the library's host code on a recorder in the place of the
HIP runtime (launch_recorder.c), in a process of its own, without a GPU.

record(calls) -> one (status, [(kernel, grid_x, grid_y, grid_z, block, lds), ...]) per call; apply_f32_small_kernel
adds the (query, layer, head) that its launch starts with.  A call is
("search", N, E, B, k, "f16"|"f32", "ip"|"l2"), ("exact", B, Hq, Hkv, S, D, causal, "bf16"|"f32"[, routed]),
("insert", B, Lc, Hq, Hkv, S, D, causal, packed), ("apply", B, Lc, Hq, Hkv, S, D, causal, "bf16"|"f32"[, packed]) or
("project", B, S, dm, hid, E, "bf16"|"f32", "f16"|"f32", biases[, bytes of workspace])."""
import ctypes
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2510_25979_amd", "libattncache.so")
PTR, F32, F16, BF16 = 4096, 0, 1, 2   # never dereferenced
HUGE = 1 << 62


def plain(symbols):
    """Kernel names as they are written.  c++filt does not know _Float16 and bf16: builtin types stand in for them."""
    text = "\n".join(symbols).replace("DF16_", "Dh").replace("DF16b", "g")
    out = subprocess.run(["c++filt"], input=text, text=True, capture_output=True, check=True).stdout
    return [n.replace("void ac::", "").replace("ac::", "").replace("__float128", "bf16").split("(")[0] for n in out.splitlines()]


def record(calls, build_dir, lib=LIB):
    rec = os.path.join(str(build_dir), "liblaunch_recorder.so")
    if not os.path.exists(rec):
        subprocess.run(["gcc", "-O1", "-Wall", "-Werror", "-Wno-unused-result", "-shared", "-fPIC", "-I/opt/rocm/include",
                        os.path.join(HERE, "launch_recorder.c"), "-o", rec, "-ldl"], check=True)
    out = subprocess.run([sys.executable, os.path.abspath(__file__), rec, lib], input=json.dumps(calls), text=True,
                         capture_output=True, check=True).stdout
    got = json.loads(out)
    names = sorted({la[0] for _, ls in got for la in ls})
    nice = dict(zip(names, plain(names)))
    return [(st, [(nice[la[0]], *la[1:]) for la in ls]) for st, ls in got]


def _main(rec, path):
    R = ctypes.CDLL(rec, mode=ctypes.RTLD_GLOBAL)
    R.recorded.restype = ctypes.c_char_p
    L = ctypes.CDLL(path)
    i32, f32, vp, sz = ctypes.c_int32, ctypes.c_float, ctypes.c_void_p, ctypes.c_size_t

    def db(N, E, emb, metric, M, Lc, Hq, Hkv, D, S, dt, causal, packed):
        d = (i32 * 14)(N, E, emb, metric, M, Lc, Hq, Hkv, D, S, dt, causal, 0, packed)
        h = vp()
        st = L.attncache_build_db(d, vp(PTR), vp(PTR), vp(PTR), None, sz(0), None, ctypes.byref(h))
        assert st == 0, st
        return h

    p, out = vp(PTR), []
    for fn, *c in json.load(sys.stdin):
        R.forget()
        h = None
        if fn == "search":
            N, E, B, k, emb, metric = c
            h = db(N, E, F16 if emb == "f16" else F32, int(metric == "l2"), 1, 1, 1, 1, 8, 32, F32, 1, 0)
            st = L.attncache_search(h, p, B, k, f32(0.5), p, p, p, p, sz(HUGE), None)
        elif fn == "exact":
            B, Hq, Hkv, S, D, causal, dt, *routed = c
            st = L.attention_exact(p, p, p, p, p if any(routed) else None, None, B, Hq, Hkv, S, D, BF16 if dt == "bf16" else F32, int(causal),
                                   f32(0), None)
        elif fn == "insert":
            B, Lc, Hq, Hkv, S, D, causal, packed = c
            h = db(1, 16, F16, 0, 1, Lc, Hq, Hkv, D, S, BF16, int(causal), int(packed))
            st = L.attncache_insert(h, None, p, None, None, p, p, p, p, B, 0, Lc, f32(0), None)
        elif fn == "project":
            B, S, dm, hid, E, dt, feat, biases, *ws = c
            bias = p if biases else None
            st = L.attncache_project(p, p, p, bias, p, bias, p, B, S, dm, hid, E, BF16 if dt == "bf16" else F32,
                                     F16 if feat == "f16" else F32, 1, p, sz(ws[0] if ws else HUGE), None)
        else:
            B, Lc, Hq, Hkv, S, D, causal, dt, *packed = c
            h = db(1, 16, F16, 0, 1, Lc, Hq, Hkv, D, S, BF16 if dt == "bf16" else F32, int(causal), int(any(packed)))
            st = L.attncache_apply(h, p, p, p, B, 0, Lc, None)
        if h:
            L.attncache_destroy_db(h)
        rows = [r.split(" ") for r in R.recorded().decode().splitlines()]
        out.append((st, [(r[0], *map(int, r[1:])) for r in rows]))
    json.dump(out, sys.stdout)


if __name__ == "__main__":
    _main(*sys.argv[1:])
