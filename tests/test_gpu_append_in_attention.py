"""Decode attention that rotates and appends itself (few (row, kv head) pairs) against the append kernel and the attention
behind it: the same rows in a batch whose capacity takes the separate launches.  One, four and sixteen query heads per kv head,
rows whose new position opens or closes a group of 32 positions, lies in the first group or behind several, rows left of a
batch, and rows whose position is refused; capacities on both sides of the one from which the attention behind the append
kernel has four waves per row."""
import numpy as np
import pytest
import torch

from parity import rows_close, TOL
from paper_2504_10724_amd import session as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv", [(16, 16), (64, 16), (256, 16)])
@pytest.mark.parametrize("live", [40, 7])
@pytest.mark.parametrize("longest", [255, 300])
def test_append_in_attention_equals_its_own_launch(hq, hkv, live, longest):
    print(f"[case] append in attention {hq}/{hkv} heads, {live} rows of up to {longest}", flush=True)
    gen = torch.Generator().manual_seed(9)
    d, rows = 256, 40                                        # 640 pairs; 64 rows are 1024
    rnd = lambda *shape: (torch.randn(*shape, generator=gen) * 0.05).bfloat16()      # noqa: E731
    m = S.Model(n_layers=1, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=128, d_ffn=64, vocab=64, dtype="bf16",
                exit_layers=[1], max_pos=512)
    one = torch.ones(d)
    m.set_layer(1, g_attn=one, W_qkv=rnd((hq + 2 * hkv) * 128, d), W_o=rnd(d, hq * 128), g_ffn=one, W_gate=rnd(64, d),
                W_up=rnd(64, d), W_down=rnd(d, 64))
    m.set_embed(rnd(64, d))
    pos = [min(longest, (0, 1, 30, 31, 32, 33, 95, 96, 127, 128, 200, 255, 256, 300)[r % 14]) for r in range(rows)]
    cap = [(p + 32) // 32 * 32 for p in pos]
    refused = [2, 5]                                         # at their capacity: nothing may be appended
    for r in refused:
        pos[r] = cap[r]
    out = []
    for B in (rows, 64):
        kv, b = S.KVCache(m, 1, cap + [32] * (B - rows)), S.Batch(m, B)
        kv.pool.view(torch.bfloat16).normal_(0.0, 1.0, generator=torch.Generator(device="cuda").manual_seed(3))
        before = kv.pool.clone()
        b.reset(np.arange(B) % 64, np.array(pos + [0] * (B - rows), np.int32), None)
        b.begin_step()
        b.field("n_active").fill_(live)
        assert S.layer_forward(m, 1, kv, b) == 0
        new = [[np.asarray(x) for x in kv.read_context(1, r, 1, pos0=pos[r])] for r in range(live) if r not in refused]
        changed = int((kv.pool.view(torch.int16) != before.view(torch.int16)).sum())
        assert int(b.field("status")[0]) == 1
        # nothing but the new positions changes; a value may by chance be what was there
        most = (live - sum(r < live for r in refused)) * 2 * hkv * 128
        assert 0.98 * most <= changed <= most
        out.append((b.field("h")[:live].cpu().numpy(), np.array(new)))
    good = [r for r in range(live) if r not in refused]
    worst, ok = rows_close(out[0][0][good], out[1][0][good], TOL["bf16"])
    assert ok and np.isfinite(out[0][0][good]).all(), worst
    err = np.abs(out[0][1] - out[1][1]).max() / np.abs(out[1][1]).max()
    assert err <= 1e-2, err                                  # one bf16 rounding
