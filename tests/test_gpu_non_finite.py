"""Non-finite values on the GPU: what one NaN or infinity may reach and what it may not.  A logit that is NaN is
never a row's token; a row whose logits are all NaN gives token 0 and meets no threshold; rows beside it are
untouched."""
import numpy as np
import pytest
import torch

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
@pytest.mark.parametrize("cols", [[0], [3], [64, 200], [0, 256], [299], list(range(0, 300, 2))], ids=str)
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
