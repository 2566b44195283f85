"""The tile kernels' two loops (waves of a SIMD in turns where most row tiles are live, else each wave on its own) add up in one
order: rows of the same token are the same bits, whichever loop and place in the tile they get.  Row tiles on both sides of
the rule, a last 16-row tile with one row, row groups of which the last one takes the other loop or the same; stores, residual updates,
SwiGLU and exit statistics with logits.  The exit statistics of full tiles besides: logits off 16-byte alignment, equal maxima, infinities
and NaN."""
import numpy as np
import pytest
import torch

from paper_2504_10724_amd import session as S

pytestmark = pytest.mark.gpu

TOKENS = 61          # no divisor of a tile: equal rows sit at different places of their tiles


def model(d, heads, kv_heads, ffn, vocab):
    gen = torch.Generator(device="cuda").manual_seed(5)
    w = lambda n, k: torch.empty((n, k), dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=gen)      # noqa: E731
    m = S.Model(n_layers=1, d_model=d, n_q_heads=heads, n_kv_heads=kv_heads, head_dim=128, d_ffn=ffn, vocab=vocab, dtype="bf16",
                exit_layers=[1], max_pos=32)
    one = torch.ones(d, device="cuda")
    m.set_layer(1, g_attn=one, W_qkv=w((heads + 2 * kv_heads) * 128, d), W_o=w(d, heads * 128), g_ffn=one, W_gate=w(ffn, d), W_up=w(ffn, d),
                W_down=w(d, ffn))
    m.set_exit(0, g=one, W=w(vocab, d))
    m.set_embed(w(vocab, d))
    return m


def same_rows(x, ref, what):
    """row i of x is row i % TOKENS of ref, bit for bit"""
    want = ref[torch.arange(len(x), device=x.device) % TOKENS]
    assert torch.isfinite(x.float()).all(), what
    differ = torch.nonzero((x != want).reshape(len(x), -1).any(-1)).flatten().tolist()
    assert not differ, (what, differ[:8])


def live_rows(d, ffn, rows, counts):
    """a layer and its head on the first `live` of the rows, for each of the counts: the rows of the first count again"""
    m = model(d, 8, 8, ffn, 51200)
    kv, b = S.KVCache(m, 1, [32] * rows), S.Batch(m, rows)
    logits, ref = torch.empty((rows, 51200), device="cuda"), None
    for live in counts:
        print(f"[case] d = {d}, {live} of {rows} rows", flush=True)
        b.reset(np.arange(rows) % TOKENS, np.zeros(rows, np.int32), None)
        b.begin_step()
        b.field("n_active").fill_(live)
        assert S.layer_forward(m, 1, kv, b) == 0 and S.exit_head(m, 0, 0.5, False, b, logits) == 0
        got = [b.field("h")[:live].clone(), logits[:live].clone(), b.field("head_conf")[:live].clone(), b.field("head_tok")[:live].clone()]
        ref = ref or got                                     # 160 rows: no row tile in turns
        for x, r, what in zip(got, ref, ("state", "logits", "confidence", "token")):
            same_rows(x, r, (what, live))


# 224 tiles of 256 columns and the down projection in K slices; 230 workgroups of 192 columns, the last with two tile-rows of six
@pytest.mark.parametrize("d,ffn", [(1024, 28672), (512, 22016)])
def test_one_row_group(d, ffn):
    live_rows(d, ffn, 256, (160, 161, 176, 177, 192, 193, 208, 209, 224, 225, 240, 241, 256))


# the last group with fewer than five row tiles (its own loop), with five, six and seven; the down projection in slices of 56 stages and of 10 or 11
@pytest.mark.parametrize("d,ffn", [(2048, 28672), (512, 22016)])
def test_two_row_groups(d, ffn):
    live_rows(d, ffn, 512, (160, 257, 300, 384, 385, 401, 416, 417, 433, 448, 449, 480, 512))


# the last row group has 100 rows (its own loop), 208 and 255; 1124 entries of the narrower model: 192 columns
@pytest.mark.parametrize("d,heads,kv_heads,ffn,n", [(4096, 32, 32, 11008, 1124), (4096, 32, 32, 11008, 2047), (8192, 64, 8, 28672, 1892),
                                                    (8192, 64, 8, 28672, 2000)])
def test_several_row_groups(d, heads, kv_heads, ffn, n):
    print(f"[case] {n} entries, d = {d}", flush=True)
    m = model(d, heads, kv_heads, ffn, 32000)
    kv, b = S.KVCache(m, 1, [32] * n), S.Batch(m, n)
    b.reset(np.zeros(n, np.int32), np.zeros(n, np.int32), None)
    logits = torch.empty((n, 32000), device="cuda")
    assert S.prefill(m, kv, b, np.arange(n) % TOKENS, np.zeros(n, np.int32), np.arange(n)) == 0
    assert S.exit_head(m, 0, 0.0, True, b, logits) == 0
    for x, what in ((b.field("h"), "state"), (logits, "logits"), (b.field("head_conf"), "confidence"), (b.field("head_tok"), "token")):
        same_rows(x, x, what)


def head(W, emb):
    """a model of which only the head is asked, about the embeddings themselves"""
    V, d = W.shape
    m = S.Model(n_layers=1, d_model=d, n_q_heads=1, n_kv_heads=1, head_dim=128, d_ffn=64, vocab=V, dtype="bf16", exit_layers=[1], max_pos=32)
    m.set_exit(0, g=torch.ones(d), W=W)
    m.set_embed(emb)
    return m


def ask(m, b, live, logits):
    b.begin_step()
    b.field("n_active").fill_(live)
    assert S.exit_head(m, 0, 0.0, False, b, logits) == 0
    torch.cuda.synchronize()
    return [b.field(k)[:live].clone() for k in ("head_tok", "head_conf", "head_exit")]


def test_logits_off_alignment():
    """200 tiles of 256 columns, 225 and 256 rows: the aligned array's values, and nothing around them"""
    print("[case] logits off alignment, 225 and 256 rows", flush=True)
    gen, V, rows = torch.Generator().manual_seed(8), 51200, 256
    m = head((torch.randn(V, 256, generator=gen) * 0.02).bfloat16(), torch.randn(V, 256, generator=gen).bfloat16())
    b = S.Batch(m, rows)
    b.reset(np.arange(rows), np.zeros(rows, np.int32), None)
    for live in (225, 256):
        want = torch.zeros((rows, V), device="cuda")
        buf = torch.full((rows * V + 8,), 7.0, device="cuda")
        got = buf[1:1 + rows * V].view(rows, V)
        assert want.data_ptr() % 16 == 0 and got.data_ptr() % 16 == 4
        x, y = (ask(m, b, live, z) for z in (want, got))
        assert all(torch.equal(p, q) for p, q in zip(x, y))
        assert torch.equal(want[:live], got[:live]) and bool((want[:live] != 0).any(1).all())
        assert buf[0] == 7.0 and bool((buf[1 + live * V:] == 7.0).all())


@pytest.mark.parametrize("column", [None, 3, 51199], ids=str)
def test_equal_maxima_and_non_finite_values(column):
    """Every row has two equal largest logits in one 32-column tile: the lower column is its token.  Columns of -infinity change nothing.
    A row of NaN gives token 0 and does not leave; a column of NaN is nobody's token, and nobody leaves.  In turns (225 rows)
    and not (160), the same bits."""
    print(f"[case] equal maxima, -infinity, rows of NaN, column {column} of NaN", flush=True)
    gen, V, d, rows = torch.Generator().manual_seed(9), 51200, 256, 225
    emb, W = torch.randn(V, d, generator=gen), torch.randn(V, d, generator=gen)
    emb[:, 0] = emb[:, 0].abs() + 0.1
    emb = emb.bfloat16()
    token = []
    for j in range(rows):
        lo = j % 31
        at = 32 * (j + 8) + lo
        W[[at, at + 1 + 7 * j % (31 - lo)]] = 3 * emb[j].float()         # |x|^2 is about 256, the other logits' spread 16
        token.append(at)
    W[[64, 65, 95, 20000]] = 0.0
    W[[64, 65, 95, 20000], 0] = -float("inf")
    if column is not None:
        W[column] = 0.0
        W[column, 0] = float("nan")
    bad = [7, 100, 159, 200, 224]
    emb[bad, 9] = float("nan")
    token = torch.tensor(token)
    token[bad] = 0
    m = head(W.bfloat16(), emb)
    b = S.Batch(m, rows)
    b.reset(np.arange(rows), np.zeros(rows, np.int32), None)
    logits = [torch.zeros((rows, V), device="cuda") for _ in range(2)]
    alone, turns = ask(m, b, 160, logits[0]), ask(m, b, rows, logits[1])
    for x, y in zip(alone + [logits[0][:160]], turns + [logits[1]]):
        assert torch.equal(x.float().nan_to_num(nan=-1.0), y[:160].float().nan_to_num(nan=-1.0))
    assert torch.equal(turns[0].cpu().long(), token)
    good = torch.ones(rows, dtype=torch.bool)
    good[bad] = False
    conf, leaves = turns[1].cpu(), turns[2].cpu().bool()
    if column is None:
        assert torch.allclose(conf[good], torch.full_like(conf[good], 0.5), rtol=1e-4) and bool(leaves[good].all())
        assert bool(torch.isnan(conf[~good]).all()) and not bool(leaves[~good].any())
    else:
        assert bool(torch.isnan(conf).all()) and not bool(leaves.any())
