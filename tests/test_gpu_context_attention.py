"""GPU parity of the context-pass attention at the edges of its tiling (k_bf16_attn_ctx): tiles of one and two
blocks of 16 MFMA columns per wave, contexts that end on and beside the 32- and 64-position borders, tiles that
two cache rows share, tiles of many rows (served entry group by entry group) and calls just below the size from
which the tiled kernel runs.  Bar: the context pass's 2e-2 for hidden states and cache (a chain of bf16 operand
roundings; see test_gpu_prefill.py)."""
import numpy as np
import pytest
import torch

import synth
from helpers import OracleSide
from oracle import ee_oracle as orc
from parity import GpuSide, rows_close, TOL
from paper_2504_10724_amd import session as S

pytestmark = pytest.mark.gpu

BASE = synth.CONFIGS["llama2_7b"].with_(n_layers=2, resident=2, d_model=256, d_ffn=256, vocab=512, exit_layers=(1, 2),
                                        thresholds=(0.5, 0.0), steps=1)


# heads (q, kv), lengths of the contexts; all their tokens go in one call.  G = 8: tiles of 8 C entries, G = 1: 64 C,
# G = 3: 20 C (five entries fill 15 of 16 columns)
@pytest.mark.parametrize("hq,hkv,lengths", [
    (64, 8, [31, 32, 33, 63, 64, 65]),              # 288 entries, C = 1: borders of groups and stages
    (64, 8, [700, 329]),                            # 1029 entries, C = 2, a tile of two rows, a partial last tile
    (64, 8, [1] * 260),                             # C = 1, every tile of eight rows: entry groups
    (64, 8, [97, 150]),                             # 247 entries: below the tiled kernel
    (32, 32, [480, 35]),                            # G = 1, 515 entries, C = 1
    (32, 32, [1000, 24, 1]),                        # G = 1, C = 2, a tile of three rows
    (48, 16, [400, 41]),                            # G = 3, C = 1
], ids=lambda v: "x".join(map(str, v[:3])) if isinstance(v, list) else str(v))
def test_context_attention_tiles(hq, hkv, lengths):
    n = sum(lengths)
    s = BASE.with_(name=f"ctx_{hq}_{hkv}_{n}", n_q_heads=hq, n_kv_heads=hkv, batch=len(lengths), ctx_lo=1, ctx_hi=max(lengths))
    print(f"[case] context attention {s.name}", flush=True)
    check = range(len(lengths)) if len(lengths) < 8 else [0, 7, 8, 255, 259]
    o = OracleSide(s, rows=list(check), cap=max(lengths), fill_ctx=False)
    g = GpuSide(s, weights=o.weights, synth_rows=[], max_pos=1024)
    kv = S.KVCache(g.model, s.resident, [(x + 31) // 32 * 32 for x in lengths])
    kv.pool.view(torch.bfloat16).fill_(float("nan"))        # what was never written must not be read
    b = S.Batch(g.model, n)
    b.reset(np.zeros(n, np.int32), np.zeros(n, np.int32), None)
    toks = {r: synth.context_tokens(s, r, x) for r, x in enumerate(lengths)}
    (tok, pos, seq), = list(S.prefill_chunks(toks, n))
    assert S.prefill(g.model, kv, b, tok, pos, seq) == 0
    torch.cuda.synchronize()
    assert int(b.field("status").cpu()[0]) == 0
    h = b.field("h").cpu().numpy()
    assert np.isfinite(h).all()
    for i, r in enumerate(check):
        rc, want = orc.prefill(o.model, o.kv, i, toks[r], want_h=True)
        assert rc == 0
        worst, ok = rows_close(h[seq == r], want, TOL["bf16"])
        assert ok, f"cache row {r}: worst entry error {worst:.2e}"
        K, V = kv.read_context(2, r, lengths[r])
        for got, ref in ((K, o.kv.K), (V, o.kv.V)):
            worst, ok = rows_close(got.reshape(1, -1), ref[1, i, :, :lengths[r]].reshape(1, -1), TOL["bf16"])
            assert ok, f"cache row {r}: worst cache error {worst:.2e}"
