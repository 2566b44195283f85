"""Confidence of the bf16 exit head against fp64 where rounding errors do not average out: in every tile of 32 logits one is the
maximum, one is -infinity and the other 30 lie at the same distance below the maximum.  The weight-streaming kernel (16 rows),
the one whose waves stream alone (100 and 200) and tiles of 128 (300) and 256 columns (600)."""
import numpy as np
import pytest
import torch

from paper_2504_10724_amd import session as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,vocab,d", [(16, 4096, 256), (100, 8192, 256), (200, 8192, 256), (300, 8192, 256), (600, 32768, 256)])
def test_confidence_of_equal_distances(rows, vocab, d):
    print(f"[case] confidence of equal distances, {rows} rows, {vocab} logits", flush=True)
    m = S.Model(n_layers=1, d_model=d, n_q_heads=2, n_kv_heads=2, head_dim=128, d_ffn=64, vocab=vocab, dtype="bf16", exit_layers=[1],
                max_pos=64, rms_eps=0.0)
    emb, W = torch.zeros(vocab, d), torch.zeros(vocab, d)
    emb[:, 0] = 1.0                                          # normalised: sqrt(d) = 16 in column 0, exactly
    W[:, 0] = -1.0 / 16
    W[::32, 0] = 0.0
    W[5::32, 0] = -float("inf")
    m.set_embed(emb.bfloat16())
    m.set_exit(0, g=torch.ones(d), W=W.bfloat16())
    b = S.Batch(m, rows)
    b.reset(np.zeros(rows, np.int32), np.zeros(rows, np.int32), None)
    rng, err = np.random.default_rng(rows), []
    for _ in range(20):
        dist = rng.uniform(0.2, 10.0, rows).astype(np.float32)     # the row's logit scale
        b.set_row_scale(dist)
        b.begin_step()
        assert S.exit_head(m, 0, 0.5, False, b) == 0
        conf = b.field("head_conf").cpu().numpy().astype(np.float64)
        err.append(conf * (vocab // 32) * (1.0 + 30.0 * np.exp(-dist.astype(np.float64))) - 1.0)
    err = np.abs(np.concatenate(err))
    print(f"  relative error: largest {err.max():.2e}, root mean square {np.sqrt((err ** 2).mean()):.2e}", flush=True)
    # a term is within 1.4e-7 of its value (the exponential and one multiply-add), a tile's sum rounds five times on a term's
    # way, the row's four waves once, the reciprocal once: 1.4e-7 + 7 * 2^-24.
    # (32 terms added one by one, or a distance rounded once more before the exponential, give up to 9e-7.)
    assert err.max() <= 1.4e-7 + 7 * 2.0 ** -24
