"""GPU parity of the keys and values of ONE skipped layer in batches whose capacity takes the product to each of its kernels:
the one whose waves stream alone (up to 128 rows, and up to 256 where the tiles are few), 128 columns (257 and 1024), 192
columns (1025 to 1280; 43 column tiles of which the last has four of six tile-rows) and 256 columns (1281).  All
rows have left, or a few entries of a large batch are filled from kept states.  And of seven and eight layers in one launch of
256-column tiles whose row tiles are nearly all live."""
import numpy as np
import pytest
import torch

from paper_2504_10724_amd import session as S
from test_gpu_launch_rules import test_skipped_layers_of_few_rows as fill_and_compare

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows", [1, 65, 200, 257, 1024, 1025, 1100, 1280, 1281])
def test_one_skipped_layer(rows):
    fill_and_compare(2, 32, rows)


# 224 and 256 workgroups, a table of weights: full row groups, and seven row tiles of eight
@pytest.mark.parametrize("layers,rows", [(8, 200), (8, 225), (8, 256), (9, 256)])
def test_several_skipped_layers_of_many_rows(layers, rows):
    fill_and_compare(layers, 32, rows)


# 4608 values and 8 kv heads: nine slices, added up by a launch of their own (129 rows and more)
@pytest.mark.parametrize("capacity,entries,d,hkv", [(1100, 5, 512, 32), (1100, 300, 512, 32), (1100, 1100, 512, 32), (129, 129, 4608, 8),
                                                    (250, 40, 4608, 8)])
def test_one_more_layer_for_cached_tokens(capacity, entries, d, hkv):
    print(f"[case] backfill of one layer, {entries} entries in a batch of {capacity}", flush=True)
    hd, n_kv = 128, 40
    gen = torch.Generator().manual_seed(capacity + entries)
    rnd = lambda *shape, std=0.02: (torch.randn(*shape, generator=gen) * std).bfloat16()      # noqa: E731
    m = S.Model(n_layers=2, d_model=d, n_q_heads=hkv, n_kv_heads=hkv, head_dim=hd, d_ffn=64, vocab=64, dtype="bf16", exit_layers=[1, 2],
                max_pos=64)
    qkv, gains = {}, {}
    for l in (1, 2):
        qkv[l], gains[l] = rnd(3 * hkv * hd, d), 1 + 0.1 * torch.randn(d, generator=gen)
        m.set_layer(l, g_attn=gains[l], W_qkv=qkv[l], W_o=rnd(d, hkv * hd), g_ffn=torch.ones(d), W_gate=rnd(64, d), W_up=rnd(64, d),
                    W_down=rnd(d, 64))
    kv, b = S.KVCache(m, 2, [32] * n_kv), S.Batch(m, capacity)
    b.reset(np.zeros(capacity, np.int32), np.zeros(capacity, np.int32), None)
    h = torch.randn(n_kv * 32, d, generator=gen)
    store = S.HiddenStore(m, kv)
    store.buf.copy_(h.view(-1))
    at = torch.randperm(n_kv * 32, generator=gen)[:entries]
    dev = lambda x: x.to(torch.int32).cuda()      # noqa: E731
    assert S.backfill_kv(m, 1, 2, kv, b, store, dev(at % 32), dev(at // 32)) == 0
    torch.cuda.synchronize()
    assert int(b.field("status")[0]) == 0
    h = h.double()
    x = (h / torch.sqrt(h.square().mean(-1, keepdim=True) + 1e-5) * gains[2].double()).float().bfloat16().double()
    y = (x @ qkv[2][hkv * hd:].double().T).view(n_kv, 32, 2, hkv, hd)
    k, v = y[:, :, 0], y[:, :, 1]
    ang = torch.arange(32, dtype=torch.float64)[:, None] * 10000.0 ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64) / hd)
    c, s_ = torch.cos(ang)[None, :, None], torch.sin(ang)[None, :, None]
    k = torch.cat([k[..., :64] * c - k[..., 64:] * s_, k[..., 64:] * c + k[..., :64] * s_], -1)
    for r in sorted({int(at[0]) // 32, int(at[-1]) // 32, n_kv - 1}):
        pos = sorted(int(p) % 32 for p in at if int(p) // 32 == r)
        K, V = kv.read_context(2, r, 32)
        for got, want in ((K, k[r]), (V, v[r])):
            want = want.permute(1, 0, 2)[:, pos].numpy()
            if pos:
                assert np.abs(got[:, pos] - want).max() <= 1e-2 * np.abs(want).max(), r      # one bf16 rounding
