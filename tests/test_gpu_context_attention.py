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


# a batch of 1152 entries takes the whole context but its last tokens in one call, those in the next: the
# tiling goes by the call's entries (1088 of them: C = 2, 64: not tiled; 700 and 300: C = 1; G = 1, 800: C = 1, 330: not tiled)
@pytest.mark.parametrize("hq,hkv,first,rest", [(64, 8, 1088, 64), (64, 8, 700, 300), (32, 32, 800, 330)])
def test_short_call_in_a_large_batch(hq, hkv, first, rest):
    n = first + rest
    s = BASE.with_(name=f"short_{hq}_{hkv}_{n}", n_q_heads=hq, n_kv_heads=hkv, batch=1, ctx_lo=1, ctx_hi=n)
    print(f"[case] {rest} entries after {first} in a batch of 1152", flush=True)
    o = OracleSide(s, rows=[0], cap=n, fill_ctx=False)
    g = GpuSide(s, weights=o.weights, synth_rows=[], max_pos=2048)
    kv, b = S.KVCache(g.model, s.resident, [(n + 31) // 32 * 32]), S.Batch(g.model, 1152)
    kv.pool.view(torch.bfloat16).fill_(float("nan"))
    b.reset(np.zeros(1152, np.int32), np.zeros(1152, np.int32), None)
    toks = synth.context_tokens(s, 0, n)
    got = []
    for lo, hi in ((0, first), (first, n)):
        i = np.arange(lo, hi, dtype=np.int32)
        assert S.prefill(g.model, kv, b, np.asarray(toks[lo:hi], np.int32), i, np.zeros(hi - lo, np.int32)) == 0
        got.append(b.field("h").cpu().numpy()[:hi - lo])
    assert int(b.field("status").cpu()[0]) == 0
    rc, want = orc.prefill(o.model, o.kv, 0, toks, want_h=True)
    assert rc == 0
    worst, ok = rows_close(np.concatenate(got), want, TOL["bf16"])
    assert ok, f"worst entry error {worst:.2e}"
    K, V = kv.read_context(2, 0, n)
    for a, ref in ((K, o.kv.K), (V, o.kv.V)):
        worst, ok = rows_close(a.reshape(1, -1), ref[1, 0, :, :n].reshape(1, -1), TOL["bf16"])
        assert ok, f"worst cache error {worst:.2e}"


@pytest.mark.parametrize("n", [515, 1100])                  # one and two blocks of columns per wave
def test_mean_of_two_values_is_rounded_once(n):
    """All scores 0, values 254/128 and 255/128 in turn: the mean over an even number of positions lies half way between
    these two bf16 neighbours and has to become 254/128 (the even one) for every number of positions; a result that is
    off by one unit of fp32 before it is rounded becomes 255/128 for some of them."""
    print(f"[case] mean over 1 .. {n} positions", flush=True)
    d, heads = 64, 32
    m = S.Model(n_layers=1, d_model=d, n_q_heads=heads, n_kv_heads=heads, head_dim=128, d_ffn=64, vocab=32, dtype="bf16",
                exit_layers=[1], max_pos=2048)
    # two tokens with one value each; the gain makes their normalised value 1
    emb = torch.zeros(32, d)
    emb[0, 0] = emb[1, 1] = 1.0
    W_qkv, W_o = torch.zeros(3 * heads * 128, d), torch.zeros(d, heads * 128)
    W_qkv[2 * heads * 128:, 0], W_qkv[2 * heads * 128:, 1] = 254 / 128, 255 / 128
    W_o[torch.arange(heads) + 2, torch.arange(heads) * 129 % (heads * 128)] = 1.0       # one feature of each head
    b16 = lambda t: t.bfloat16()      # noqa: E731
    m.set_layer(1, g_attn=torch.full((d,), float(np.sqrt(1.0 / d + 1e-5))), W_qkv=b16(W_qkv), W_o=b16(W_o), g_ffn=torch.ones(d),
                W_gate=b16(torch.zeros(64, d)), W_up=b16(torch.zeros(64, d)), W_down=b16(torch.zeros(d, 64)))
    m.set_embed(b16(emb))
    kv, b = S.KVCache(m, 1, [(n + 31) // 32 * 32]), S.Batch(m, n)
    b.reset(np.zeros(n, np.int32), np.zeros(n, np.int32), None)
    i = np.arange(n, dtype=np.int32)
    assert S.prefill(m, kv, b, i % 2, i, np.zeros(n, np.int32)) == 0
    got = b.field("h").cpu().numpy()[:, 2:2 + heads]
    even = i % 2 == 1                                       # an even number of positions
    assert np.array_equal(got[even], np.full((even.sum(), heads), 254 / 128, np.float32)), i[even][(got[even] != 254 / 128).any(-1)] + 1
    mean = (254 + ((i + 1) // 2) / (i + 1.0)) / 128
    want = torch.from_numpy(mean).float().bfloat16().float().numpy()
    assert np.array_equal(got[~even], np.repeat(want[~even, None], heads, 1))
