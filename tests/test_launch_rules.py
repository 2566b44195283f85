"""The launch rules, on the library's host code alone (no GPU): what is launched for a call, and with which arguments."""
import pytest

from host_launches import launches

# query heads, kv heads, d, FFN: the widths of the workloads, heads between them, a smaller model, one off the 128-wide tile grid
SHAPES = [(32, 32, 4096, 11008), (64, 8, 8192, 28672), (40, 40, 5120, 13824), (48, 48, 6144, 16384), (24, 24, 3072, 8192), (16, 4, 2048, 5632),
          (32, 32, 512, 1024), (4, 2, 576, 1088)]
FILLS = [SHAPES[0], SHAPES[1], SHAPES[5], SHAPES[7]]
ROWS = [1, 7, 32, 33, 64, 65, 96, 128, 129, 200, 256, 257, 400, 512, 513, 600, 768, 769, 1000, 1024, 1025, 1100, 1280, 1281, 1537, 1792, 2048,
        2049, 2304, 2816, 2817, 4096, 4097, 4352, 5000, 5888, 8192, 20000, 65535]


def _cfg(shape, layers, exits):
    hq, hkv, d, f = shape
    return dict(n_layers=layers, d_model=d, n_q_heads=hq, n_kv_heads=hkv, d_ffn=f, vocab=32000, exit_layers=exits)


def _arg(launch, kind, nth=0):
    return [a for a, t in zip(launch["args"], launch["types"]) if t == kind][nth]


def _products(launches_):
    return [x for x in launches_ if x["kernel"].startswith("k_bf16_gemm")]


@pytest.mark.parametrize("shape", SHAPES, ids=str)
def test_every_product_is_given_its_weights(shape):
    """the weights as an address, or a table of addresses on a kernel that reads it: keys and values of one skipped layer and of
    several, of few entries in a large batch, of a step with exits on neighbouring layers, and every product of a context pass"""
    calls = [["fill_skipped_kv", 1, 2], ["fill_skipped_kv", 1, 4], ["backfill_kv", 3, 4, 1], ["decode_step"], ["prefill", 1], ["exit_head", 0]]
    got = launches([dict(cfg=_cfg(shape, 4, [1, 2, 4]), rows=n, calls=calls + [["prefill", n]]) for n in ROWS])
    for n, per_call in zip(ROWS, got):
        for call, (rc, ran) in zip(calls + [["prefill", n]], per_call):
            assert rc == 0 and _products(ran), (n, call)
            for x in _products(ran):
                weights, table = _arg(x, "HIP_vector_type const*", 1), _arg(x, "ZBatch") if "ZBatch" in x["types"] else 0
                assert weights or table, (n, call, x["kernel"])


@pytest.mark.parametrize("shape", [x for x in SHAPES if x[2] >= 2048], ids=str)      # narrower products are not sliced
def test_the_append_kernel_reads_the_planes_the_product_wrote(shape):
    """q|k|v of a context pass and of a step, keys and values of one skipped layer and of several; or none, where a launch has added
    them up"""
    calls = [["fill_skipped_kv", 1, 2], ["fill_skipped_kv", 1, 4], ["backfill_kv", 3, 4, 1], ["layer_forward", 1]]
    got = launches([dict(cfg=_cfg(shape, 4, [1, 2, 4]), rows=n, calls=calls + [["prefill", n]]) for n in ROWS])
    qkv, sliced = (shape[0] + 2 * shape[1]) * 128, 0
    for n, per_call in zip(ROWS, got):
        for call, (rc, ran) in zip(calls + [["prefill", n]], per_call):
            columns = qkv if call[0] in ("layer_forward", "prefill") else 2 * shape[1] * 128
            for i, x in enumerate(ran):
                if x["kernel"] != "k_bf16_rope_append":
                    continue
                splits, plane, planes, ld, start = x["args"][-5:]
                made = next(y for y in reversed(ran[:i]) if y["kernel"].startswith(("k_bf16_gemm", "k_splitk_finish")))
                if made["kernel"].startswith("k_splitk") or "long" not in made["types"] or made["args"][made["types"].index("int const*") - 1] == 1:
                    assert splits == 1 and start == columns, (n, call)
                    continue
                at = made["types"].index("long")
                sliced += 1
                assert made["args"][at - 3 - 1] == splits > 1 and made["args"][at - 1:at + 2] == [planes, plane, ld], (n, call)
                assert ld == columns - start and plane >= n * ld, (n, call)
    assert sliced


def test_large_batches_are_not_sliced():
    """products off the 128-wide tile grid: K is sliced where few rows give few workgroups; 2000 rows of 130 tile-rows give two for
    every CU, and up to the largest batch only a last round that is nearly empty is worth a second plane"""
    rows = [65, 2000, 3000, 4000, 4100, 6000, 8000, 12000, 20000, 40000, 65535]
    got = launches([dict(cfg=dict(n_layers=1, d_model=4160, n_q_heads=32, n_kv_heads=32, d_ffn=11008, vocab=32000, exit_layers=[1]), rows=n, cap=32,
                         calls=[["layer_forward", 1]]) for n in rows])
    for nth in (0, 1, 3):                                    # q|k|v, O and down
        slices = [_products(c[0][1])[nth]["args"][6] for c in got]
        assert slices[0] > 1 and max(slices[1:]) <= 2 and slices[-1] == 1, slices


def _sums(launch):
    """the order in which a product adds its columns up: kernels of one kind differ in the tiles they take, not in this"""
    kind = next(k for k in ("few", "cols", "dma") if k in launch["kernel"]) if "_gemm_" in launch["kernel"] else "stream"
    splits = 1 if kind in ("cols", "stream") else launch["args"][6]
    return "tile" if kind in ("cols", "dma") else kind, splits


@pytest.mark.parametrize("exits", [[1, 11, 21, 31, 41], [2, 3, 4, 5, 41], [1, 3, 5, 9, 12, 13, 40, 41], [8, 16, 24, 32]], ids=str)
@pytest.mark.parametrize("shape", FILLS, ids=str)
def test_the_end_of_a_step_in_pieces_fills_layers_as_the_step_does(shape, exits):
    """keys and values of skipped layers: per layer the same kind of sums after ee_decode_finish as in ee_decode_step"""
    rows = [1, 33, 64, 65, 128, 129, 256, 300, 1100]
    cfg = dict(_cfg(shape, exits[-1], exits), vocab=512)
    calls = [["decode_step"]] + [["decode_finish", e] for e in range(len(exits))]
    for n, ((rc, step), *finish) in zip(rows, launches([dict(cfg=cfg, rows=n, cap=32, calls=calls) for n in rows])):
        fills = lambda ran: [_sums(x) for x in _products(ran) if _arg(x, "HIP_vector_type const*", 1) == 0 for _ in range(x["grid"][2])]   # noqa: E731
        want = fills(step)
        assert rc == 0 and len(want) == exits[-1] - exits[0]
        for e, (rc, ran) in enumerate(finish):
            left = exits[-1] - exits[min(e + 1, len(exits) - 1)]
            assert rc == 0 and fills(ran) == want[len(want) - left:], (n, e)


@pytest.mark.parametrize("vocab,tiles", [(32000, False), (40960, False), (51200, True), (65536, True), (76800, False), (98304, False),
                                         (102400, True), (128256, True), (131072, True), (151936, False)])
def test_heads_of_few_rows_whose_tiles_fill_their_rounds_keep_them(vocab, tiles):
    rows = [1, 32, 64, 100, 128]
    cfg = dict(n_layers=1, d_model=4096, n_q_heads=32, n_kv_heads=8, d_ffn=14336, vocab=vocab, exit_layers=[1])
    for n, ((rc, ran),) in zip(rows, launches([dict(cfg=cfg, rows=n, calls=[["exit_head", 0]]) for n in rows])):
        assert rc == 0 and _products(ran)[0]["kernel"].startswith("k_bf16_gemm_dma8" if tiles else "k_bf16_gemm_few"), n


@pytest.mark.parametrize("rows,vocab,tiles", [(129, 14080, False), (129, 16000, True), (160, 16000, True), (161, 16000, False), (256, 16384, False)])
def test_two_row_groups_of_128_where_they_leave_fewer_cus_idle(rows, vocab, tiles):
    cfg = dict(n_layers=1, d_model=4096, n_q_heads=32, n_kv_heads=8, d_ffn=14336, vocab=vocab, exit_layers=[1])
    ((rc, ran),), = launches([dict(cfg=cfg, rows=rows, calls=[["exit_head", 0]])])
    assert rc == 0 and _products(ran)[0]["kernel"].startswith("k_bf16_gemm_dma2" if tiles else "k_bf16_gemm_few")


@pytest.mark.parametrize("shape,layers,rows,kind", [
    # more than 128 rows: the tile kernels whatever the number of layers
    ((64, 8, 8192, 28672), 2, 129, "dma"), ((64, 8, 8192, 28672), 40, 129, "dma"), ((16, 4, 2048, 5632), 2, 256, "dma"),
    # 97 to 128 rows: tiles of 128 columns that fill three quarters of their rounds, 192 and 160
    ((32, 32, 4096, 11008), 3, 96, "few"), ((32, 32, 4096, 11008), 3, 97, "dma"), ((64, 8, 8192, 28672), 12, 128, "dma"),
    ((64, 8, 8192, 28672), 10, 128, "few"), ((32, 32, 4096, 11008), 5, 128, "few"),
    # up to 32 rows: 64 tile-rows per layer (70B), 32
    ((64, 8, 8192, 28672), 2, 32, "stream"), ((64, 8, 8192, 28672), 2, 33, "few"), ((64, 8, 8192, 28672), 3, 32, "few"),
    ((16, 4, 2048, 5632), 8, 16, "stream"), ((16, 4, 2048, 5632), 8, 32, "stream"), ((16, 4, 2048, 5632), 10, 1, "few"),
    ((32, 8, 4096, 14336), 4, 16, "few"), ((32, 8, 4096, 14336), 4, 17, "stream")])
def test_kernel_of_a_fill_of_several_layers(shape, layers, rows, kind):
    cfg = dict(_cfg(shape, layers + 1, [1, layers + 1]), vocab=512)
    ((rc, ran),), = launches([dict(cfg=cfg, rows=rows, cap=32, calls=[["fill_skipped_kv", 1, layers + 1]])])
    assert rc == 0 and ("_gemm_" + kind if kind != "stream" else "k_bf16_gemm<") in _products(ran)[0]["kernel"]


@pytest.mark.parametrize("rows,planes", [(128, "few"), (129, 16), (256, 16), (257, 8), (1000, 4)])
def test_many_planes_of_one_skipped_layer_are_added_up_before_the_append(rows, planes):
    cfg = dict(_cfg((64, 8, 8192, 28672), 2, [1, 2]), vocab=512)
    ((rc, ran),), = launches([dict(cfg=cfg, rows=rows, cap=32, calls=[["fill_skipped_kv", 1, 2]])])
    splits = _products(ran)[0]["args"][6]
    assert rc == 0 and (planes == "few" or splits == planes)
    assert any(x["kernel"].startswith("k_splitk_finish") for x in ran) == (splits > 8)


@pytest.mark.parametrize("exits", [[1, 11, 21, 31, 41], [8, 16, 24, 32], [2, 4, 6, 8], [3, 5, 12, 42]], ids=str)
@pytest.mark.parametrize("shape", FILLS, ids=str)
def test_fills_up_to_the_last_exit_are_those_of_the_step(shape, exits):
    """a step made of its calls fills (exit, R] at every exit, ee_decode_step from one exit to the next: the same kind of sums"""
    rows = [1, 33, 64, 65, 128, 129, 256, 300, 1100]
    cfg = dict(_cfg(shape, exits[-1], exits), vocab=512)
    calls = [["decode_step"]] + [["fill_skipped_kv", l, exits[-1]] for l in exits[:-1]]
    for n, ((rc, step), *fill) in zip(rows, launches([dict(cfg=cfg, rows=n, cap=32, calls=calls) for n in rows])):
        fills = lambda ran: [_sums(x) for x in _products(ran) if _arg(x, "HIP_vector_type const*", 1) == 0 for _ in range(x["grid"][2])]   # noqa: E731
        want = fills(step)
        assert rc == 0 and len(want) == exits[-1] - exits[0]
        for l, (rc, ran) in zip(exits, fill):
            assert rc == 0 and fills(ran) == want[len(want) - (exits[-1] - l):], (n, l)


# 16, 74, 96 and 32 (row, kv head) pairs: few enough that places stay empty, and still no share below two groups of 32 positions per wave
@pytest.mark.parametrize("hq,hkv,rows,cap,most", [(4, 2, 8, 704, 2), (4, 2, 8, 928, 3), (4, 2, 37, 928, 3), (64, 8, 12, 736, 2), (32, 32, 1, 992, 3),
                                                  (32, 32, 1, 1024, 4), (4, 2, 8, 640, 1)])
def test_positions_are_shared_in_pieces_of_256(hq, hkv, rows, cap, most):
    """how a row's positions are shared decides in which order its partial softmax sums are added, so it decides the bits"""
    cfg = dict(_cfg((hq, hkv, 512, 1024), 1, [1]), vocab=512)
    ((rc, ran),), = launches([dict(cfg=cfg, rows=rows, cap=cap, calls=[["layer_forward", 1]])])
    attention = next(x for x in ran if x["kernel"] == "k_bf16_attn_decode")
    assert rc == 0 and attention["grid"] == [hkv, rows, most]
    assert any(x["kernel"] == "k_bf16_attn_merge" for x in ran) == (most > 1)
