"""What libee launches for a call, on a machine without a GPU.

`launches(scenarios)` runs the calls of every scenario in a process of its own, in which tests/launch_recorder.cpp stands in
for the HIP runtime: the library's host code (argument checks, launch rules, sizes) is the real one, the kernels are
recorded and not run.  A scenario is a dict
  cfg    n_layers, d_model, n_q_heads, n_kv_heads, d_ffn, vocab, exit_layers (bf16, head size 128, unless given)
  rows   rows of the batch;  cap: positions per cache row;  kv_rows: cache rows (the batch's unless given)
  calls  list of [entry point without ee_, arguments after the handles ...]
and the result is, per call, (return code, list of launches); a launch is a dict of `kernel` (name without its parameters),
`grid`, `args` (parameter types -> values in order: numbers, addresses, the first 8 bytes of a structure)."""
import ctypes as C
import importlib.util
import json
import os
import re
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
PKG = os.path.join(os.path.dirname(HERE), "paper_2504_10724_amd")


def launches(scenarios, lib=None):
    with tempfile.TemporaryDirectory() as d:
        so = os.path.join(d, "launch_recorder.so")
        subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", os.path.join(HERE, "launch_recorder.cpp"), "-o", so], check=True)
        r = subprocess.run([sys.executable, os.path.abspath(__file__), so, lib or os.path.join(PKG, "libee.so")], input=json.dumps(scenarios), text=True,
                           capture_output=True, timeout=300)
        assert r.returncode == 0, r.stderr[-2000:]
        return json.loads(r.stdout)


# ------------------------------------------------------------------ in the other process
def _capi():
    spec = importlib.util.spec_from_file_location("capi", os.path.join(PKG, "capi.py"))
    m = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(m)
    return m


def _recorded(rec):
    out, dims, vals = [], (C.c_uint32 * 6)(), (C.c_int64 * 64)()
    for i in range(rec.rec_count()):
        name = rec.rec_name(i).decode()
        rec.rec_dims(i, dims)
        n = rec.rec_args(i, vals, 64)
        kernel, types = re.match(r"(?:void )?(\w+(?:<.*?>)?)\((.*)\)$", name).groups()
        out.append(dict(kernel=kernel, grid=list(dims[:3]), args=list(vals[:n]), types=re.sub(r"<[^>]*>", "", types).split(", ")))
    rec.rec_clear()
    return out


class _Addresses:
    """addresses that the host never reads, far enough apart and aligned as device memory is"""

    def __init__(self):
        self.at = 1 << 40

    def take(self, nbytes):
        p = self.at
        self.at += (nbytes + 4095) // 4096 * 4096
        return p


def _run(ee, lib, rec, s):
    c, mem = dict(dtype=ee.EE_BF16, head_dim=128, rms_eps=1e-5, rope_theta=1e4, max_pos=4096), _Addresses()
    c.update(s["cfg"])
    cfg = ee.ee_model_config()
    for k, v in c.items():
        if k != "exit_layers":
            setattr(cfg, k, v)
    cfg.n_exits = len(c["exit_layers"])
    for i, l in enumerate(c["exit_layers"]):
        cfg.exit_layers[i] = l
    m, kv, b, vb = (C.c_void_p() for _ in range(4))
    ok = lambda rc: (rc == 0) or sys.exit(lib.ee_last_error().decode())      # noqa: E731
    ok(lib.ee_model_create(C.byref(cfg), C.byref(m)))
    for l in range(1, cfg.n_layers + 1):
        w = ee.ee_layer_weights(*[mem.take(1 << 30) for _ in range(6)])
        ok(lib.ee_model_set_layer(m, l, C.byref(w)))
    for e in range(cfg.n_exits):
        ok(lib.ee_model_set_exit(m, e, C.cast(mem.take(1 << 20), C.c_void_p), mem.take(1 << 30)))
    ok(lib.ee_model_set_embed(m, mem.take(1 << 30)))
    rows, kv_rows = s["rows"], s.get("kv_rows", s["rows"])
    caps = (C.c_int32 * kv_rows)(*[s.get("cap", 64)] * kv_rows)
    pool = lib.ee_kv_pool_bytes(m, cfg.n_layers, caps, kv_rows)
    ok(lib.ee_kv_bind(m, mem.take(pool), pool, cfg.n_layers, caps, kv_rows, C.byref(kv)))
    st, ws = lib.ee_batch_state_bytes(m, rows), lib.ee_workspace_bytes(m, rows)
    ok(lib.ee_batch_bind(m, rows, mem.take(st), st, mem.take(ws), ws, C.byref(b)))
    rec.rec_clear()
    any_ = mem.take(1 << 30)
    th = (C.c_float * 16)(*[0.5] * 16)
    out = []
    for name, *a in s["calls"]:
        h = {"layer_forward": lambda: (m, a[0], kv, b, None), "exit_head": lambda: (m, a[0], 0.5, 0, b, a[1] if len(a) > 1 else None, None),
             "fill_skipped_kv": lambda: (m, a[0], a[1], kv, b, None), "decode_step": lambda: (m, kv, b, th, cfg.n_exits, None),
             "decode_segment": lambda: (m, kv, b, th, cfg.n_exits, a[0], None), "decode_finish": lambda: (m, kv, b, a[0], None),
             "prefill": lambda: (m, kv, b, any_, any_, any_, a[0], None),
             "backfill_kv": lambda: (m, a[0], a[1], kv, b, any_, any_, any_, a[2], None)}[name]()
        rc = getattr(lib, "ee_" + name)(*h)
        out.append([rc, _recorded(rec)])
    for h, f in ((b, lib.ee_batch_destroy), (kv, lib.ee_kv_destroy), (m, lib.ee_model_destroy)):
        f(h)
    return out


if __name__ == "__main__":
    rec_, ee_ = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL), _capi()
    rec_.rec_name.restype = C.c_char_p
    ee_.LIB_PATH = sys.argv[2]
    json.dump([_run(ee_, ee_.load(), rec_, s) for s in json.load(sys.stdin)], sys.stdout)
