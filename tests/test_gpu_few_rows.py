"""GPU parity of the products whose waves stream on their own (few rows, shapes off the 128-wide tile grid): K of 17 and 31
steps of 64 (slices of unequal length, fewer tiles than a wave's ring holds), 34, 62, 65 and 124 tile-rows (a last workgroup
with one to three), live rows on both sides of the 8-row pieces an activation tile is fetched in and of its 32 rows, one
to four row tiles with fewer left after the compaction, several row groups, the keys and values of one skipped layer
(slices the append kernel adds) and of four.  Call by call against the oracle, at its bars."""
import pytest

import synth
from test_gpu_parity import test_calls_one_by_one as calls_one_by_one

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,rows,d,ffn,vocab", [
    (2, 5, 1088, 1984, 2080), (2, 31, 1088, 1984, 2080), (2, 33, 1088, 1984, 2080), (2, 64, 1088, 1984, 2080),
    (5, 8, 1088, 1984, 2080), (5, 9, 1088, 1984, 2080), (5, 40, 1088, 1984, 2080), (5, 63, 1088, 1984, 2080),
    (2, 65, 1088, 1984, 2080), (5, 96, 1088, 1984, 2080), (2, 97, 1088, 1984, 2080), (5, 128, 1088, 1984, 2080),
    (2, 129, 1088, 1984, 2080), (2, 257, 1088, 1984, 2080),
    # on the tile grid: 65 to 128 rows, and two row groups where the tile kernels would leave half of the CUs idle
    (2, 70, 1280, 2048, 2048), (5, 128, 1280, 2048, 2048), (2, 129, 1280, 2048, 2048), (5, 256, 1280, 2048, 2048)])
def test_calls_of_few_rows(layers, rows, d, ffn, vocab):
    calls_one_by_one(synth.CONFIGS["llama2_7b"].with_(
        name=f"few_rows_l{layers}_b{rows}_d{d}", n_layers=layers, resident=layers, d_model=d, n_q_heads=16, n_kv_heads=16, d_ffn=ffn,
        vocab=vocab, exit_layers=(1, layers), thresholds=(0.7, 0.0), batch=rows, ctx_lo=3, ctx_hi=40, steps=2))
