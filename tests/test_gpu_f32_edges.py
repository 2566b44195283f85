"""GPU parity of the fp32 path at the edges of its kernels: K that is no multiple of 4 (element-wise loads) or of
16 (a partial last chunk), fewer and more chunks than waves, 16-row and 16-column remainders, head sizes whose
lanes do not fill a power of two, and one value per lane.  Whole decode steps against the oracle; bar as for every
fp32 step (decisions bit for bit, hidden states within 2e-4)."""
import numpy as np
import pytest

from helpers import OracleSide, small_shape
from parity import GpuSide, compare_step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(d_model=54, n_q_heads=6, n_kv_heads=3, head_dim=10, d_ffn=77, vocab=61, batch=17),     # nothing divides by 4
    dict(d_model=40, n_q_heads=4, n_kv_heads=2, head_dim=20, d_ffn=68, vocab=300, batch=33),    # 5 of 8 lanes per position
    dict(d_model=516, n_q_heads=2, n_kv_heads=1, head_dim=256, d_ffn=524, vocab=17, batch=1),   # a wave per position
    dict(d_model=12, n_q_heads=2, n_kv_heads=2, head_dim=4, d_ffn=4, vocab=16, batch=16),       # one chunk, one lane
], ids=lambda k: f"d{k['d_model']}_hd{k['head_dim']}")
def test_f32_shapes(kw):
    s = small_shape(name="f32_edges", ctx_lo=1, ctx_hi=130, steps=2, thresholds=(0.05, 0.0), **kw)
    print(f"[case] f32 edges {kw}", flush=True)
    o = OracleSide(s)
    g = GpuSide(s, weights=o.weights, cap_multiple=1)
    sticky = np.zeros(s.batch, bool)
    for step in range(s.steps):
        rep = compare_step(s, o, g, step, sticky=sticky)
        assert rep["mismatch"] == 0, rep["detail"]
