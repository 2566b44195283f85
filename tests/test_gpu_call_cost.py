"""What a call costs follows the rows it has, not the capacity of the batch or the cache it runs in.  Each test times
one class of kernels (HIP events inside the library, the shortest of 30 runs after 20 others) on two sides that do the same work; the bound
lies between what they differ by and what a launch rule that goes by the capacity made of it."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2504_10724_amd import capi
from paper_2504_10724_amd import session as S

pytestmark = pytest.mark.gpu

ATTENTION, QKV, DOWN = (1 << capi.KERNEL_CLASSES.index(k) for k in ("attention", "gemm_qkv", "gemm_down"))
SHAPES = {"70b": (8192, 64, 8), "7b": (4096, 32, 32), "small": (2048, 16, 4)}      # d, query heads, kv heads (the FFN is kept small)


def _model(shape, layers=1, ffn=256):
    d, hq, hkv = SHAPES[shape]
    m = S.Model(n_layers=layers, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=128, d_ffn=ffn, vocab=512, dtype="bf16",
                exit_layers=[layers], max_pos=4096)
    rnd = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02)      # noqa: E731
    one = torch.ones(d, device="cuda")
    for l in range(1, layers + 1):
        m.set_layer(l, g_attn=one, W_qkv=rnd((hq + 2 * hkv) * 128, d), W_o=rnd(d, hq * 128), g_ffn=one, W_gate=rnd(ffn, d),
                    W_up=rnd(ffn, d), W_down=rnd(d, ffn))
    m.set_exit(0, g=one, W=rnd(512, d))
    m.set_embed(rnd(512, d))
    return m


def _time(call, kernels):
    """microseconds of the launches of one class in a call"""
    lib, n, ms, got = capi.load(), C.c_int(), C.c_float(), []
    capi.check(lib.ee_timing_enable(kernels))
    try:
        for k in range(50):
            capi.check(lib.ee_timing_reset())
            call()
            capi.check(lib.ee_timing_read(kernels.bit_length() - 1, C.byref(n), C.byref(ms)))
            got.append(ms.value * 1e3)
    finally:
        lib.ee_timing_enable(0)
    return min(got[20:])


def _context_call(m, batch, lengths, start):
    """one call of lengths[r] tokens for cache row r, which holds `start` positions"""
    kv, b, n = S.KVCache(m, 1, [(start + x + 31) // 32 * 32 for x in lengths]), S.Batch(m, batch), sum(lengths)
    kv.pool.view(torch.bfloat16).normal_()
    b.reset(np.zeros(batch, np.int32), np.zeros(batch, np.int32), None)
    dev = lambda x: torch.as_tensor(np.asarray(x, np.int32)).cuda()      # noqa: E731
    tok, seq = dev(np.arange(n) % 512), dev(np.repeat(np.arange(len(lengths)), lengths))
    pos = dev(np.concatenate([start + np.arange(x) for x in lengths]))
    return lambda: capi.check(S.prefill(m, kv, b, tok, pos, seq))


@pytest.mark.parametrize("shape,batch,lengths,start", [("70b", 1024, [50, 50], 3000), ("70b", 2048, [64], 1936),
                                                       ("7b", 2048, [64], 1936)])
def test_context_attention_of_a_short_call(shape, batch, lengths, start):
    m = _model(shape)
    small = _time(_context_call(m, sum(lengths), lengths, start), ATTENTION)
    large = _time(_context_call(m, batch, lengths, start), ATTENTION)
    print(f"[case] attention of {sum(lengths)} entries, {shape}: {small:.1f} us alone, {large:.1f} in a batch of {batch}", flush=True)
    assert large <= 1.5 * small


def test_qkv_of_a_short_call():
    """2048 rows of the 7B shape have more 256-column tiles than fit a round of workgroups, 1025 have not"""
    m = _model("7b")
    small = _time(_context_call(m, 1025, [64], 0), QKV)
    large = _time(_context_call(m, 2048, [64], 0), QKV)
    print(f"[case] q|k|v of 64 entries: {small:.1f} us in a batch of 1025, {large:.1f} in one of 2048", flush=True)
    assert large <= 1.25 * small


@pytest.mark.parametrize("shape", ["70b", "7b"])
def test_qkv_does_not_rise_below_2048_entries(shape):
    """eight row groups: the column tiles of a full round run in one launch and the rest in slices; with seven groups
    that would leave some XCDs with more workgroups than CUs"""
    m = _model(shape)
    t = {n: _time(_context_call(m, n, [n], 0), QKV) for n in (1600, 2048)}
    print(f"[case] q|k|v, {shape}: {t[1600]:.1f} us for 1600 entries, {t[2048]:.1f} for 2048", flush=True)
    assert t[1600] <= 1.15 * t[2048]


def _layer_call(m, batch, live, positions):
    kv, b = S.KVCache(m, 1, [4096] * batch), S.Batch(m, batch)
    kv.pool.view(torch.bfloat16).normal_()
    b.reset(np.zeros(batch, np.int32), np.full(batch, positions - 1), None)
    b.begin_step()
    b.field("n_active").fill_(live)
    return lambda: capi.check(S.layer_forward(m, 1, kv, b))


@pytest.mark.parametrize("live,positions", [(1, 3900), (2, 3900)])
def test_attention_of_the_rows_that_are_left(live, positions):
    """rows that have left no longer count when the positions of the others are shared out"""
    m = _model("70b")
    small = _time(_layer_call(m, live, live, positions), ATTENTION)
    large = _time(_layer_call(m, 16, live, positions), ATTENTION)
    print(f"[case] attention of {live} rows: {small:.1f} us, as what is left of 16: {large:.1f}", flush=True)
    assert large <= 1.4 * small


FILL = 1 << capi.KERNEL_CLASSES.index("fill_kv")


def _fill_call(m, rows, left, layers):
    kv, b = S.KVCache(m, layers + 1, [64] * rows), S.Batch(m, rows)
    b.reset(np.zeros(rows, np.int32), np.arange(rows) % 60, None)
    b.begin_step()
    b.field("exited_idx").copy_(torch.arange(rows, dtype=torch.int32))
    b.field("n_exited").fill_(left)
    return lambda: capi.check(S.fill_skipped_kv(m, 1, layers + 1, kv, b))


# 160 tiles of 128 columns and 192: more than the streaming kernel runs at a time with 65 rows and more
@pytest.mark.parametrize("shape,layers,rows,left", [("70b", 10, 128, 128), ("7b", 3, 65, 40), ("7b", 6, 128, 30)])
def test_fill_just_above_64_rows(shape, layers, rows, left):
    """129 rows run on the tile kernel whatever the number of layers"""
    m = _model(shape, layers + 1)
    few = _time(_fill_call(m, rows, left, layers), FILL)
    more = _time(_fill_call(m, 129, left, layers), FILL)
    print(f"[case] fill of {layers} layers, {left} rows: {few:.1f} us in a batch of {rows}, {more:.1f} in one of 129", flush=True)
    assert few <= 1.15 * more


def test_fill_of_layers_that_spill_into_a_second_round():
    """40 layers of the 70B shape are 320 tiles; one row of them costs about what 20 layers cost twice"""
    m = _model("70b", 41)
    t = {n: _time(_fill_call(m, 16, 1, n), FILL) for n in (20, 40)}
    print(f"[case] fill of one row: 20 layers {t[20]:.1f} us, 40 layers {t[40]:.1f}", flush=True)
    assert t[40] <= 2.02 * t[20]


@pytest.mark.parametrize("rows,positions", [(1, 20), (8, 62), (20, 62), (64, 20)])
def test_fp32_layer_of_short_rows_in_a_large_cache(rows, positions):
    """room for 2000 positions more per row costs a layer of the fp32 workload's shape at most what more waves per row cost"""
    d, heads, hd, ffn = 256, 4, 64, 688
    m = S.Model(n_layers=1, d_model=d, n_q_heads=heads, n_kv_heads=heads, head_dim=hd, d_ffn=ffn, vocab=64, dtype="f32", exit_layers=[1],
                max_pos=4096)
    rnd = lambda *s: torch.empty(s, device="cuda").normal_(0.0, 0.02)      # noqa: E731
    one = torch.ones(d, device="cuda")
    m.set_layer(1, g_attn=one, W_qkv=rnd(3 * heads * hd, d), W_o=rnd(d, heads * hd), g_ffn=one, W_gate=rnd(ffn, d), W_up=rnd(ffn, d), W_down=rnd(d, ffn))
    m.set_embed(rnd(64, d))
    t = {}
    for room in (0, 2000):
        kv, b = S.KVCache(m, 1, [positions + 8 + room] * rows), S.Batch(m, rows)
        kv.pool.view(torch.float32).normal_()
        b.reset(np.zeros(rows, np.int32), np.full(rows, positions - 1), None)
        b.begin_step()
        got = []
        for _ in range(20):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            start.record()
            for _ in range(100):
                capi.check(S.layer_forward(m, 1, kv, b))
            end.record()
            torch.cuda.synchronize()
            got.append(start.elapsed_time(end) * 10.0)
        t[room] = min(got[3:])
    print(f"[case] fp32 layer of {rows} rows of {positions} positions: {t[0]:.1f} us, {t[2000]:.1f} with room for 2000 more", flush=True)
    assert t[2000] <= 1.15 * t[0]


# a second row group of 144 rows, and of 256.  With the two groups on two loops 400 rows took 1.05 times as long as 512, now 0.91 to 1.00
@pytest.mark.parametrize("shape,ffn,kernels", [("small", 5632, DOWN), ("7b", 11008, DOWN), ("70b", 256, QKV)],
                         ids=["2048-wide-down", "7b-down", "70b-qkv"])
def test_products_of_400_rows_take_no_longer_than_of_512(shape, ffn, kernels):
    print(f"[case] products of 400 and 512 rows, {shape}, FFN {ffn}", flush=True)
    m, us = _model(shape, ffn=ffn), []
    for rows in (400, 512):
        kv, b = S.KVCache(m, 1, [32] * rows), S.Batch(m, rows)
        b.reset(np.arange(rows), np.zeros(rows, np.int32), None)
        b.begin_step()
        us.append(_time(lambda: capi.check(S.layer_forward(m, 1, kv, b)), kernels))
    print(f"[times] {us[0]:.1f} us, {us[1]:.1f} us", flush=True)
    assert us[0] <= 1.03 * us[1], us
