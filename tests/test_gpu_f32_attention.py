"""GPU parity of the fp32 attention on few rows with long contexts, rows much shorter than the longest beside them, and on both
sides of the cache sizes and row counts from which a workgroup has eight or sixteen waves, or scores go through LDS; head sizes of 1, 5, 16 and 64 lanes
per position.  Whole steps against the oracle, bar of every fp32 step."""
import numpy as np
import pytest

from helpers import OracleSide, small_shape
from parity import GpuSide, compare_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,hq,hkv,batch,lo,hi", [
    (64, 4, 4, 1, 1500, 1500), (64, 4, 2, 8, 1, 1100), (20, 4, 2, 3, 500, 700), (256, 2, 1, 2, 300, 600), (4, 2, 2, 5, 2, 520),
    (64, 4, 4, 40, 100, 127), (64, 4, 4, 40, 100, 130),
    (64, 4, 4, 65, 100, 300), (16, 8, 8, 97, 100, 300), (16, 8, 8, 65, 20, 300),
    (16, 8, 8, 97, 1, 520), (20, 8, 4, 100, 300, 520), (4, 8, 2, 137, 1, 520), (4, 8, 2, 138, 1, 520)])
def test_f32_attention_of_long_rows(hd, hq, hkv, batch, lo, hi):
    s = small_shape(name="f32_attention", d_model=64, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, d_ffn=96, vocab=128, batch=batch, ctx_lo=lo,
                    ctx_hi=hi, steps=2, thresholds=(0.05, 0.0))
    print(f"[case] f32 attention hd {hd} {hq}/{hkv} heads, {batch} rows of {lo}..{hi}", flush=True)
    o = OracleSide(s)
    g = GpuSide(s, weights=o.weights, cap_multiple=1)
    sticky = np.zeros(s.batch, bool)
    for step in range(s.steps):
        rep = compare_step(s, o, g, step, sticky=sticky)
        assert rep["mismatch"] == 0, rep["detail"]


# 8 heads: calls of 96 entries are 768 pairs, of 97 more; contexts of 530 tokens leave room for more than 512 positions
@pytest.mark.parametrize("hd,rows_per_call,lengths", [(16, 96, 530), (16, 97, 530), (20, 200, 530), (64, 150, 530), (16, 150, 500)])
def test_f32_context_pass_of_many_entries(hd, rows_per_call, lengths):
    from test_gpu_prefill import test_context_pass_cache_and_hidden_states as context_pass
    context_pass(small_shape(name=f"f32_context_hd{hd}", d_model=64, n_q_heads=8, n_kv_heads=4, head_dim=hd, d_ffn=96, vocab=128, batch=2,
                             ctx_lo=lengths, ctx_hi=lengths, steps=1), rows_per_call)
