"""GPU parity on both sides of two launch rules of the bf16 products: the q|k|v product of a context pass whose
column tiles fill whole rounds of workgroups in one launch and are K-sliced in a second (the append kernel then reads
finished columns and slice planes), and the keys and values of several skipped layers on the 256-column tile kernel
or the weight-streaming one."""
import numpy as np
import pytest
import torch

import synth
from helpers import OracleSide
from oracle import ee_oracle as orc
from parity import GpuSide, rows_close, TOL
from paper_2504_10724_amd import session as S

pytestmark = pytest.mark.gpu


# 40 column tiles of 256: 6 row groups are 240 tiles, 7 are 280 (both one launch), 8 are 320 (32 column tiles, the
# queries, + 8 in slices, the keys and values), the last row group with one entry and full; 48 column tiles: queries and
# keys + 16 in slices, the values
@pytest.mark.parametrize("n,hq,hkv", [(1536, 64, 8), (1537, 64, 8), (1760, 64, 8), (1793, 64, 8), (2048, 64, 8), (1793, 32, 32)])
def test_qkv_of_a_context_pass_in_one_and_two_launches(n, hq, hkv):
    s = synth.CONFIGS["llama2_70b"].with_(name=f"qkv_{n}_{hkv}", n_layers=2, resident=2, d_model=1024, n_q_heads=hq,
                                          n_kv_heads=hkv, d_ffn=256, vocab=512, exit_layers=(1, 2), thresholds=(0.5, 0.0),
                                          batch=40, ctx_lo=1, ctx_hi=52, steps=1)
    print(f"[case] {s.name}", flush=True)
    lengths = [n // 40 + (1 if r < n % 40 else 0) for r in range(40)]
    check = [0, 1, 25, 39]
    o = OracleSide(s, rows=check, cap=64, fill_ctx=False)
    g = GpuSide(s, weights=o.weights, synth_rows=[], max_pos=64)
    kv = S.KVCache(g.model, 2, [64] * 40)
    b = S.Batch(g.model, n)
    b.reset(np.zeros(n, np.int32), np.zeros(n, np.int32), None)
    toks = {r: synth.context_tokens(s, r, x) for r, x in enumerate(lengths)}
    (tok, pos, seq), = list(S.prefill_chunks(toks, n))
    assert S.prefill(g.model, kv, b, tok, pos, seq) == 0
    torch.cuda.synchronize()
    h = b.field("h").cpu().numpy()
    for i, r in enumerate(check):
        rc, want = orc.prefill(o.model, o.kv, i, toks[r], want_h=True)
        assert rc == 0
        worst, ok = rows_close(h[seq == r], want, TOL["bf16"])
        assert ok, f"cache row {r}: worst entry error {worst:.2e}"
        K, V = kv.read_context(2, r, lengths[r])
        for got, ref in ((K, o.kv.K), (V, o.kv.V)):
            worst, ok = rows_close(got.reshape(1, -1), ref[1, i, :, :lengths[r]].reshape(1, -1), TOL["bf16"])
            assert ok, f"cache row {r}: worst cache error {worst:.2e}"


# 32 tiles of 256 columns per layer: 7 layers are 224 (tile kernel from the first row on), 6 are 192 (75 % of a round:
# streaming up to 64 rows, then the kernel whose waves stream alone), 10 are 320 and 40 MiB (that kernel from the first
# row up to 128); of 8 kv heads 3 layers are 48 tiles of 128 (streaming up to 64 rows); from 129 rows on the tiles take all
@pytest.mark.parametrize("layers,hkv", [(7, 32), (8, 32), (11, 32), (4, 8)])
@pytest.mark.parametrize("rows", [1, 33, 64, 65, 129])
def test_skipped_layers_of_few_rows(layers, hkv, rows):
    print(f"[case] fill of {layers - 1} layers, {hkv} kv heads, {rows} rows", flush=True)
    d, hd = 256, 128
    gen = torch.Generator().manual_seed(rows * 100 + layers)
    rnd = lambda *shape, std=0.02: (torch.randn(*shape, generator=gen) * std).bfloat16()      # noqa: E731
    m = S.Model(n_layers=layers, d_model=d, n_q_heads=hkv, n_kv_heads=hkv, head_dim=hd, d_ffn=64, vocab=64, dtype="bf16",
                exit_layers=[1, layers], max_pos=64)
    qkv, gains = {}, {}
    for l in range(1, layers + 1):
        qkv[l], gains[l] = rnd(3 * hkv * hd, d), 1 + 0.1 * torch.randn(d, generator=gen)
        m.set_layer(l, g_attn=gains[l], W_qkv=qkv[l], W_o=rnd(d, hkv * hd), g_ffn=torch.ones(d), W_gate=rnd(64, d),
                    W_up=rnd(64, d), W_down=rnd(d, 64))
    for e in range(2):
        m.set_exit(e, g=torch.ones(d), W=rnd(64, d))
    emb = rnd(64, d, std=1.0)
    m.set_embed(emb)
    kv, b = S.KVCache(m, layers, [32] * rows), S.Batch(m, rows)
    tok, pos = np.arange(rows) % 64, np.arange(rows) % 32
    b.reset(tok, pos, None)
    b.begin_step()
    assert S.exit_head(m, 0, 0.0, False, b) == 0 and S.compact_active(b, 0, 1) == 0
    assert S.fill_skipped_kv(m, 1, layers, kv, b) == 0
    h = emb[torch.from_numpy(tok).long()].double()
    inv = 10000.0 ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64) / hd)
    ang = torch.from_numpy(pos).double()[:, None] * inv
    c, s_ = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    for l in (2, layers):
        x = (h / torch.sqrt(h.square().mean(-1, keepdim=True) + 1e-5) * gains[l].double()).float().bfloat16().double()
        y = (x @ qkv[l][hkv * hd:].double().T).view(rows, 2, hkv, hd)
        k, v = y[:, 0], y[:, 1]
        k = torch.cat([k[..., :64] * c - k[..., 64:] * s_, k[..., 64:] * c + k[..., :64] * s_], -1)
        for r in sorted({0, rows // 2, rows - 1}):
            K, V = kv.read_context(l, r, 32)
            for got, want in ((K[:, pos[r]], k[r]), (V[:, pos[r]], v[r])):
                err = np.abs(got - want.numpy()).max() / np.abs(want.numpy()).max()
                assert err <= 1e-2, (l, r, err)              # one bf16 rounding, as for every cache entry


# 16 rows of 8 kv heads: up to 8 shares.  Rows of one to eleven groups of 256 positions beside each other, all live (4
# shares), 6 (8 by the live pairs), one; 74 pairs of 2 kv heads; 40 rows of 8 (320 pairs: 2 shares)
@pytest.mark.parametrize("rows,hq,hkv,live", [(16, 64, 8, 16), (16, 64, 8, 6), (16, 64, 8, 1), (37, 4, 2, 37), (40, 64, 8, 40),
                                              (12, 32, 32, 12)])
def test_shared_positions_against_unshared(rows, hq, hkv, live):
    """the same rows in a batch whose capacity leaves every row to one workgroup: other sums only"""
    print(f"[case] shares: {live} of {rows} rows, {hq}/{hkv} heads", flush=True)
    gen = torch.Generator().manual_seed(9)
    d = 512
    rnd = lambda *shape: (torch.randn(*shape, generator=gen) * 0.02).bfloat16()      # noqa: E731
    m = S.Model(n_layers=1, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=128, d_ffn=64, vocab=64, dtype="bf16",
                exit_layers=[1], max_pos=4096)
    one = torch.ones(d)
    m.set_layer(1, g_attn=one, W_qkv=rnd((hq + 2 * hkv) * 128, d), W_o=rnd(d, hq * 128), g_ffn=one, W_gate=rnd(64, d),
                W_up=rnd(64, d), W_down=rnd(d, 64))
    m.set_embed(rnd(64, d))
    lengths = [(1, 31, 256, 511, 512, 513, 900, 1100, 1280, 1535, 2047, 2815)[r % 12] for r in range(rows)]
    out = []
    for B in (rows, (512 + hkv - 1) // hkv):
        kv, b = S.KVCache(m, 1, [(x + 32) // 32 * 32 for x in lengths] + [32] * (B - rows)), S.Batch(m, B)
        kv.pool.view(torch.bfloat16).normal_(0.0, 1.0, generator=torch.Generator(device="cuda").manual_seed(3))
        b.reset(np.arange(B) % 64, np.array(lengths + [0] * (B - rows), np.int32), None)
        b.begin_step()
        b.field("n_active").fill_(live)
        before = b.field("h")[:live].cpu().numpy().copy()
        # the pool's layout goes by the capacities of the rows before: the first rows are the same in both
        assert S.layer_forward(m, 1, kv, b) == 0
        out.append(b.field("h")[:live].cpu().numpy() - before)
    assert np.isfinite(out[0]).all()
    worst, ok = rows_close(out[0], out[1], TOL["bf16"])
    assert ok, worst


# two row groups (the second with 4, 44 and 256 rows): 576, 688 and 688 tile-rows of q|k|v, gate/up and head are one round of
# 192, 230 and 230 workgroups at 192 columns (the last of 688 with 4 of 6 tile-rows) and 144, 172 and 172 at 256
@pytest.mark.parametrize("rows", [260, 300, 512])
def test_products_of_several_row_groups_on_192_columns(rows):
    from test_gpu_parity import test_calls_one_by_one as calls_one_by_one
    calls_one_by_one(synth.CONFIGS["llama2_7b"].with_(
        name=f"cols_b{rows}", n_layers=2, resident=2, d_model=256, n_q_heads=112, n_kv_heads=16, d_ffn=11008, vocab=22016,
        exit_layers=(1, 2), thresholds=(0.5, 0.0), batch=rows, ctx_lo=1, ctx_hi=12, steps=1))
