"""GPU parity of the products of at most 64 rows whose waves stream on their own: K of 17 and 31 steps of 64 (slices of
unequal length, fewer tiles than a wave's ring holds), 34, 62, 65 and 124 tile-rows (a last workgroup with one to three),
live rows on both sides of the 8-row pieces an activation tile is fetched in and of its 32 rows, one row tile left of two
after the compaction, and the keys and values of one skipped layer (slices the append kernel adds) and of four.  Call by
call against the oracle, at its bars."""
import pytest

import synth
from test_gpu_parity import test_calls_one_by_one as calls_one_by_one

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,rows", [(2, 5), (2, 31), (2, 33), (2, 64), (5, 8), (5, 9), (5, 40), (5, 63)])
def test_calls_of_few_rows(layers, rows):
    calls_one_by_one(synth.CONFIGS["llama2_7b"].with_(
        name=f"few_rows_l{layers}_b{rows}", n_layers=layers, resident=layers, d_model=1088, n_q_heads=16, n_kv_heads=16, d_ffn=1984,
        vocab=2080, exit_layers=(1, layers), thresholds=(0.7, 0.0), batch=rows, ctx_lo=3, ctx_hi=40, steps=2))
