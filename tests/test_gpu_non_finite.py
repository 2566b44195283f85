"""Non-finite values on the GPU: what one NaN or infinity may reach and what it may not.  A logit that is NaN is
never a row's token; a row whose logits are all NaN gives token 0 and meets no threshold; rows beside it are
untouched.  In a context pass a token with a NaN, or an entry refused for its position, reaches the entries that come
after it in its context and the 16 / G entries that share its pass over the cache (G query heads per kv head), no more."""
import numpy as np
import pytest
import torch

from parity import rows_close, TOL
from paper_2504_10724_amd import session as S

pytestmark = pytest.mark.gpu


def _head_only(dtype, d, V, W, emb):
    """a model of one layer whose head W is asked about the embeddings themselves"""
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    hd = 128 if dtype == "bf16" else 8
    m = S.Model(n_layers=1, d_model=d, n_q_heads=1, n_kv_heads=1, head_dim=hd, d_ffn=64, vocab=V, dtype=dtype,
                exit_layers=[1], max_pos=32)
    m.set_exit(0, g=torch.ones(d), W=W.to(t))
    m.set_embed(emb.to(t))
    return m


def _ask(m, rows):
    b = S.Batch(m, rows)
    b.reset(np.arange(rows), np.zeros(rows, np.int32), None)
    b.begin_step()
    assert S.exit_head(m, 0, 0.0, False, b) == 0
    torch.cuda.synchronize()
    return [b.field(k).cpu() for k in ("head_tok", "head_conf", "head_exit")]


# columns in the first stride of the block (its first lane, another lane, another wave), a later stride, the last one
@pytest.mark.parametrize("cols", [[0], [3], [64, 200], [0, 256], [299], list(range(0, 300, 2))],
                         ids=lambda c: f"{len(c)}from{c[0]}")
@pytest.mark.parametrize("value", [float("nan"), float("-inf")], ids=str)
def test_f32_head_with_non_finite_columns(cols, value):
    print(f"[case] f32 head, columns {cols[:4]} {value}", flush=True)
    gen = torch.Generator().manual_seed(5)
    d, V, rows = 16, 300, 9
    emb = torch.randn(V, d, generator=gen)
    emb[:, 0] = emb[:, 0].abs() + 0.1
    W = torch.randn(V, d, generator=gen)
    W[cols] = 0.0
    W[cols, 0] = value
    tok, conf, leaves = _ask(_head_only("f32", d, V, W, emb), rows)
    h = emb[:rows].double()
    z = (h / torch.sqrt(h.square().mean(-1, keepdim=True) + 1e-5)) @ W.double().T
    z[:, cols] = -np.inf
    assert torch.equal(tok.long(), z.argmax(-1))
    if np.isnan(value):
        assert torch.isnan(conf).all() and not leaves.any()
    else:
        assert torch.allclose(conf.double(), torch.softmax(z, -1).max(-1).values, rtol=1e-4) and leaves.all()


# weight-streaming kernel (no multiple of 128) with one and several column tiles, tile kernel; a row of NaN among others
@pytest.mark.parametrize("dtype,V", [("bf16", 32), ("bf16", 96), ("bf16", 512), ("f32", 300)])
def test_a_row_of_nan_logits_gives_token_0(dtype, V):
    print(f"[case] {dtype} head, V = {V}, a row of NaN", flush=True)
    gen = torch.Generator().manual_seed(6)
    d, rows = 64, 5
    emb, W = torch.randn(V, d, generator=gen), torch.randn(V, d, generator=gen)
    m = _head_only(dtype, d, V, W, emb)
    tok, conf, leaves = _ask(m, rows)
    assert leaves.all()
    emb[2, 7] = float("nan")
    m.set_embed(emb.to(m.tdtype))
    tok2, conf2, leaves2 = _ask(m, rows)
    others = [0, 1, 3, 4]
    assert torch.equal(tok2[others], tok[others]) and torch.equal(conf2[others], conf[others]) and leaves2[others].all()
    assert int(tok2[2]) == 0 and torch.isnan(conf2[2]) and not leaves2[2]


# 288 entries: 8 of G = 8 in a tile; 1029: 16; G = 1, 515 entries: 64, 1100: 128.  Two cache rows, the border inside a tile
@pytest.mark.parametrize("hq,hkv,lengths", [(64, 8, [150, 138]), (64, 8, [700, 329]), (32, 32, [480, 35]), (32, 32, [700, 400])],
                         ids=str)
@pytest.mark.parametrize("refused", [False, True], ids=["nan", "refused"])
def test_context_pass_keeps_a_bad_entry_to_itself(hq, hkv, lengths, refused):
    n, d, V = sum(lengths), 256, 512
    print(f"[case] context pass of {n} entries, {hq}/{hkv} heads, one {'refused' if refused else 'NaN'}", flush=True)
    gen = torch.Generator().manual_seed(7)
    rnd = lambda *shape: (torch.randn(*shape, generator=gen) * 0.02).bfloat16()      # noqa: E731
    m = S.Model(n_layers=1, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=128, d_ffn=256, vocab=V, dtype="bf16",
                exit_layers=[1], max_pos=1024)
    one = torch.ones(d)
    m.set_layer(1, g_attn=one, W_qkv=rnd((hq + 2 * hkv) * 128, d), W_o=rnd(d, hq * 128), g_ffn=one, W_gate=rnd(256, d),
                W_up=rnd(256, d), W_down=rnd(d, 256))
    emb = rnd(V, d)
    emb[V - 1] = float("nan")
    m.set_embed(emb)
    kv, b = S.KVCache(m, 1, [(x + 63) // 32 * 32 for x in lengths]), S.Batch(m, n)
    b.reset(np.zeros(n, np.int32), np.zeros(n, np.int32), None)
    tok = torch.randint(0, V - 1, (n,), generator=gen).int().numpy()
    pos = np.concatenate([np.arange(x) for x in lengths]).astype(np.int32)
    seq = np.repeat(np.arange(2), lengths).astype(np.int32)

    def call(t, p):
        kv.pool.view(torch.bfloat16).fill_(float("nan"))
        assert S.prefill(m, kv, b, t, p, seq) == 0
        torch.cuda.synchronize()
        return b.field("h").cpu().numpy().copy(), int(b.field("status").cpu()[0])
    want, status = call(tok, pos)
    assert np.isfinite(want).all() and status == 0
    per_pass = 16 // (hq // hkv)
    for bad in (lengths[0] - 29, lengths[0] + 21):
        t, p = tok.copy(), pos.copy()
        if refused:
            p[bad] = 1000                                   # beyond the capacity of its cache row
        else:
            t[bad] = V - 1
        h, status = call(t, p)
        assert status == (1 if refused else 0)
        b.field("status").zero_()
        i = np.arange(n)
        # the entries after it in its context read its key and value (refused: what was never written there)
        clean = ((seq != seq[bad]) | (i < bad)) & (i // per_pass != bad // per_pass)
        assert np.isfinite(h[clean]).all(), f"entries {i[clean & ~np.isfinite(h).all(-1)]}"
        worst, ok = rows_close(h[clean], want[clean], TOL["bf16"])
        assert ok, worst
