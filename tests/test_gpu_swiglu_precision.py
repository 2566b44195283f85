"""The SwiGLU product silu(g) u of the bf16 path, bit for bit as good as one fp32 evaluation rounded to bf16.  Weights
and inputs are chosen so that g and u reach the epilogue exactly: the embedding of a row has one value that is not
zero, so g = x w_gate and u = x w_up are products of two bf16 numbers (16 bits, no sum), and the down projection
copies each of the F results into a column of its own of a residual stream that is zero there."""
import numpy as np
import pytest
import torch

from paper_2504_10724_amd import session as S

pytestmark = pytest.mark.gpu


# F on the 256-row tile kernels, and off the 128-wide grid (weight-streaming kernel)
@pytest.mark.parametrize("F", [4096, 1088])
def test_swiglu_is_rounded_once(F):
    d, rows = F + 64, 32
    print(f"[case] SwiGLU F = {F}", flush=True)
    gen = torch.Generator().manual_seed(8)
    emb = torch.zeros(rows, d)
    emb[torch.arange(rows), torch.arange(rows)] = 1.0
    # RMSNorm of such a row: 1 / sqrt(1 / d + eps), the same for all; the gain makes it a bf16 number away from a tie
    x = (1.0 / np.sqrt(1.0 / d + 1e-5))
    gain = torch.full((d,), np.float32(1.0 / x))
    W_gate, W_up, W_down = torch.zeros(F, d), torch.zeros(F, d), torch.zeros(d, F)
    W_gate[:, :rows] = torch.empty(F, rows).uniform_(-80.0, 20.0, generator=gen).bfloat16().float()
    W_up[:, :rows] = (torch.empty(F, rows).uniform_(1.0, 2.0, generator=gen)).bfloat16().float()
    W_down[torch.arange(F) + 64, torch.arange(F)] = 1.0
    m = S.Model(n_layers=1, d_model=d, n_q_heads=1, n_kv_heads=1, head_dim=128, d_ffn=F, vocab=32, dtype="bf16",
                exit_layers=[1], max_pos=32)
    b16 = lambda t: t.bfloat16()      # noqa: E731
    m.set_layer(1, g_attn=torch.ones(d), W_qkv=b16(torch.zeros(384, d)), W_o=b16(torch.zeros(d, 128)), g_ffn=gain,
                W_gate=b16(W_gate), W_up=b16(W_up), W_down=b16(W_down))
    m.set_embed(b16(emb))
    kv, b = S.KVCache(m, 1, [32] * rows), S.Batch(m, rows)
    b.reset(np.arange(rows), np.zeros(rows, np.int32), None)
    b.begin_step()
    assert S.layer_forward(m, 1, kv, b) == 0
    got = b.field("h").cpu()[:, 64:].double()
    g, u = W_gate[:, :rows].T.double(), W_up[:, :rows].T.double()
    want = g / (1.0 + torch.exp(-g)) * u
    # half a unit in the last place of a bf16 number, and what comes before the rounding in fp32: exponential (1 ulp),
    # sum, division and product (half an ulp each): 2.5 x 2^-23 relative to the result
    half = torch.exp2(torch.floor(torch.log2(want.abs())) - 8.0)
    over = (((got - want).abs() - half) / want.abs()).max().item()
    print(f"  largest error beyond half a bf16 ulp: {over:.2e} of the value", flush=True)
    assert over <= 2.5 * 2.0 ** -23
