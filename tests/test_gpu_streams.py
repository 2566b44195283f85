"""A call takes the layers as they are when it is made: a step that waits on its stream is not changed by what the host sets
afterwards, as long as the buffers it was given stay."""
import numpy as np
import pytest
import torch

from paper_2504_10724_amd import session as S

pytestmark = pytest.mark.gpu


def test_fp32_fill_of_skipped_layers_keeps_the_weights_it_was_called_with():
    print("[case] fp32 fill of 39 layers waits while the host sets other weights", flush=True)
    d, hd, heads, layers, rows = 64, 16, 4, 40, 5
    gen = torch.Generator().manual_seed(3)
    rnd = lambda *shape: torch.randn(*shape, generator=gen) * 0.1      # noqa: E731
    m = S.Model(n_layers=layers, d_model=d, n_q_heads=heads, n_kv_heads=heads, head_dim=hd, d_ffn=32, vocab=64, dtype="f32", exit_layers=[1, layers],
                max_pos=64)

    def set_layers():
        w = {}
        for l in range(1, layers + 1):
            w[l] = 1.0 + rnd(d), rnd(3 * heads * hd, d)
            m.set_layer(l, g_attn=w[l][0], W_qkv=w[l][1], W_o=rnd(d, heads * hd), g_ffn=torch.ones(d), W_gate=rnd(32, d), W_up=rnd(32, d),
                        W_down=rnd(d, 32))
        return w
    first = set_layers()
    kept = dict(m._keep)                                     # the caller keeps the buffers of the layers that are replaced
    m.set_exit(0, g=torch.ones(d), W=rnd(64, d))
    emb = rnd(64, d)
    m.set_embed(emb)
    kv, b = S.KVCache(m, layers, [8] * rows), S.Batch(m, rows)
    b.reset(np.arange(rows), np.zeros(rows, np.int32), None)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        b.begin_step()
        assert S.exit_head(m, 0, 0.0, False, b) == 0 and S.compact_active(b, 0, 1) == 0
        torch.cuda._sleep(400_000_000)                       # the fill waits on its stream
        assert S.fill_skipped_kv(m, 1, layers, kv, b) == 0
        done = torch.cuda.Event()
        done.record()
    set_layers()
    waited = not done.query()
    side.synchronize()
    assert kept and waited, "the other weights came after the fill had run"
    h = emb[:rows].double()
    for l in (2, 33, 34, layers):
        g, w = first[l]
        y = (h / torch.sqrt(h.square().mean(-1, keepdim=True) + 1e-5) * g.double()) @ w[heads * hd:].double().T
        for r in range(rows):                                # position 0: no rotation
            K, V = kv.read_context(l, r, 1)
            got = np.concatenate([K.reshape(-1), V.reshape(-1)])
            err = float(np.abs(got - y[r].numpy()).max() / np.abs(y[r].numpy()).max())
            assert err <= 1e-5, (l, r)
