"""Caller's arrays that are not aligned for 16-byte access: an embedding that starts in the middle of a 16-byte piece
(its rows are read value by value, and the step's first norm is a launch of its own), debug logits likewise (single
stores).  The results are those of the aligned arrays, bit for bit."""
import ctypes as C

import numpy as np
import pytest
import torch

import synth
from helpers import OracleSide, small_shape
from parity import GpuSide
from paper_2504_10724_amd import capi
from paper_2504_10724_amd import session as S

pytestmark = pytest.mark.gpu

BF16 = synth.CONFIGS["llama2_7b"].with_(name="align_bf16", n_layers=2, resident=2, d_model=512, n_q_heads=4, n_kv_heads=2,
                                        d_ffn=1024, vocab=2048, exit_layers=(1, 2), thresholds=(0.5, 0.0), batch=21,
                                        ctx_lo=5, ctx_hi=70, steps=1)
F32 = small_shape(name="align_f32", d_model=40, vocab=64, batch=5)


def _shifted(t):
    """the same values one element further into an allocation"""
    buf = torch.empty(t.numel() + 8, dtype=t.dtype, device="cuda")
    out = buf[1:1 + t.numel()].view(t.shape)
    out.copy_(t)
    assert out.data_ptr() % 16
    return out


@pytest.mark.parametrize("s", [BF16, F32], ids=lambda s: s.name)
def test_embedding_off_alignment(s):
    print(f"[case] embedding off alignment, {s.name}", flush=True)
    o = OracleSide(s)
    sides = [GpuSide(s, weights=o.weights) for _ in range(2)]
    emb = _shifted(sides[1].model._keep["embed"])
    capi.check(sides[1].model.lib.ee_model_set_embed(sides[1].model.h, C.c_void_p(emb.data_ptr())))
    for g in sides:
        g.batch.set_row_scale(synth.row_scale(s, 0))
        assert S.decode_step(g.model, g.kv, g.batch, s.thresholds) == 0
    torch.cuda.synchronize()
    for k in ("h", "out_tok", "out_layer", "out_conf"):
        assert torch.equal(sides[0].batch.field(k), sides[1].batch.field(k)), k
    for l in range(1, s.resident + 1):
        for r in range(s.batch):                            # the positions that have been written, the new one among them
            for x, y in zip(*(g.kv.read_context(l, r, int(o.ctx[r]) + 1) for g in sides)):
                assert np.array_equal(x, y), (l, r)
    # a context pass of three entries, one of each of three cache rows
    tok, pos, seq = np.array([1, 5, 9]), np.asarray(o.ctx[:3]) + 1, np.arange(3)
    for g in sides:
        assert S.prefill(g.model, g.kv, g.batch, tok, pos, seq) == 0
    assert torch.equal(sides[0].batch.field("h")[:3], sides[1].batch.field("h")[:3])


@pytest.mark.parametrize("V", [2048, 2080])                 # tile kernel, weight-streaming kernel
def test_logits_off_alignment(V):
    print(f"[case] logits off alignment, V = {V}", flush=True)
    s = BF16.with_(name=f"align_logits_{V}", vocab=V)
    o = OracleSide(s)
    g = GpuSide(s, weights=o.weights)
    g.batch.set_row_scale(synth.row_scale(s, 0))
    g.batch.begin_step()
    want = torch.zeros((s.batch, V), device="cuda")
    buf = torch.full((s.batch * V + 8,), 7.0, device="cuda")
    got = buf[1:1 + s.batch * V].view(s.batch, V)
    assert want.data_ptr() % 16 == 0 and got.data_ptr() % 16 == 4
    for z in (want, got):
        assert S.exit_head(g.model, 0, 0.5, 0, g.batch, z) == 0
    torch.cuda.synchronize()
    assert torch.equal(want, got) and bool((want != 0).any(1).all())
    assert buf[0] == 7.0 and bool((buf[1 + s.batch * V:] == 7.0).all())
