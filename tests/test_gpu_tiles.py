"""GPU parity of one forward and one backward at sizes where a kernel variant's
tiles, k-tiles or dispatch rule can go wrong, against the oracle (the
tolerances are those of the parity tests: bf16 rounding of stored activations)."""
import numpy as np
import pytest

from parity import Inputs, compare_replays, forced_oracle, gpu_replay, rel_err, small_cfg, tol
from test_gpu_stage import _one_event_pair, binding  # noqa: F401  (binding: the fixture)

pytestmark = pytest.mark.gpu


def _check(binding, c):  # noqa: F811
    (g_out, g_in, G), (o_out, o_in, o_G) = _one_event_pair(binding, c)
    assert rel_err(np.atleast_1d(g_out).ravel(), np.atleast_1d(o_out).ravel()) <= tol(c, "act")
    if o_in is not None:
        assert rel_err(g_in, o_in) <= tol(c, "grad")
    for n in o_G:
        assert rel_err(G[n], o_G[n]) <= tol(c, "grad"), n


# 256 x 256 ping-pong tiles with both operands K-major (FFN1 forward, FFN2 input
# gradient: 16 x 16 ragged tiles, whole rounds of the CUs): 1 to 5 k-tiles over
# d, with and without a partial last one
@pytest.mark.parametrize("d", [32, 64, 128, 160, 288])
def test_pingpong_kmajor(binding, d):  # noqa: F811
    _check(binding, small_cfg("tall_bf16", d_model=d, n_heads=d // 32))


# the same tiles in every forward and input-gradient product of a block (T
# 16600: 65 row tiles, two rounds of 256 x 128 tiles against one of 256 x 256)
@pytest.mark.parametrize("d", [480, 512])
def test_pingpong_all_products(binding, d):  # noqa: F811
    _check(binding, small_cfg("dh32_bf16", d_model=d, n_heads=d // 32, d_ff=64, seq=83, micro_batch=200))


# 256 x 128 ring tiles in more than one round, the last one partial and ragged (T 25500: 100 row
# tiles; N 1920 six rounds and N 640 two of them): bias, residual and plain products over 1, 10 and
# 30 k-tiles, then the GELU product and the gelu' one (128 x 128 tiles, two per CU)
@pytest.mark.parametrize("d,f", [(640, 64), (32, 640)])
def test_ring_rounds(binding, d, f):  # noqa: F811
    _check(binding, small_cfg("dh32_bf16", d_model=d, n_heads=d // 32, d_ff=f, seq=85, micro_batch=300))


# products split by columns (T 16200: 64 row tiles; N 1440 as 1024 in one round of
# 256 x 256 tiles and 416 apart): bias, GELU, and gelu' with its column sums
def test_column_split(binding):  # noqa: F811
    _check(binding, small_cfg("dh32_bf16", d_model=480, n_heads=15, d_ff=1440, seq=81, micro_batch=200))


# the same tiles with both operands MN-major (grouped weight gradients): 1 to 4
# k-tiles over T, T a multiple of 8 or odd
@pytest.mark.parametrize("seq,mu", [(20, 2), (64, 1), (36, 2), (25, 3), (64, 2), (67, 3)])
def test_pingpong_grouped(binding, seq, mu):  # noqa: F811
    _check(binding, small_cfg("tall_bf16", d_model=1024, n_heads=16, head_dim=64, d_ff=4096, seq=seq, micro_batch=mu))


# grouped weight gradients on the ring kernel's tiles over an odd T: 64 x 64, then 256 x 128 (d 544:
# ragged, W_1 and W_2 in XCD blocks)
@pytest.mark.parametrize("seq,mu", [(33, 1), (33, 3), (101, 5)])
def test_grouped_odd_tokens(binding, seq, mu):  # noqa: F811
    _check(binding, small_cfg("ragged_bf16", seq=seq, micro_batch=mu))
    _check(binding, small_cfg("dh32_bf16", d_model=544, n_heads=17, d_ff=2048, seq=seq, micro_batch=mu))


# LM head on the pipelined kernels at vocabularies that are not multiples of 8:
# input gradient over K = V with a partial last chunk and k-tile; weight
# gradient with and without a whole round of 256 x 256 tiles (64 row tiles at
# d 1024) and a remainder; logits kept and not kept
@pytest.mark.parametrize("fused", [0, 1])
@pytest.mark.parametrize("V,d,seq,mu", [(63, 128, 72, 2), (257, 64, 33, 1), (1003, 128, 100, 2), (16384, 1024, 36, 2),
                                        (16391, 1024, 25, 3), (17001, 1024, 36, 2)])
def test_lm_head(binding, V, d, seq, mu, fused):  # noqa: F811
    _check(binding, small_cfg("last_bf16", vocab=V, d_model=d, n_heads=d // 64, head_dim=64, d_ff=256, seq=seq,
                              micro_batch=mu, fused_head=fused))


# ping-pong tiles over segments (window products), one micro-batch: 256 x 128 tiles over 1 to 6
# k-tiles and split over K (T 1088); 256 x 256 tiles, ragged on both sides, for the QKV product over
# 1 to 3 k-tiles (d 2016) and split over K (d 1504)
@pytest.mark.parametrize("d,T", [(288, 64), (288, 128), (288, 320), (96, 384), (512, 384), (512, 1088), (2016, 64),
                                 (2016, 128), (2016, 192), (1504, 1152)])
def test_pingpong_window(binding, d, T):  # noqa: F811
    _check(binding, small_cfg("win_bf16", n_layers=1 if d > 512 else 2, d_model=d, n_heads=d // 32, head_dim=32,
                              d_ff=96 if d > 512 else 416, seq=T // 2, micro_batch=2))


# the same over many segments of one k-tile each: 18 micro-batches of 64 tokens in a window, split
# over K at a segment's first row
def test_pingpong_window_short_segments(binding):  # noqa: F811
    c = small_cfg("winwide_bf16", seq=32, K=18, M=18)
    inp = Inputs(c, 1, c["M"])
    g = gpu_replay(c, inp)
    compare_replays(c, g, forced_oracle(c, inp, g), theta0=inp.params)


# bf16 products on the tiles of small grids, ragged on every side: 64 x 64 up to
# one round of the CUs, then 128 x 64 (each epilogue: N = d, 3 d and f), then 128 x 128
@pytest.mark.parametrize("d,f,seq,mu", [(32, 64, 1, 1), (96, 160, 65, 1), (448, 1792, 33, 3), (320, 992, 100, 11),
                                        (960, 64, 100, 11), (320, 992, 200, 11), (960, 96, 200, 11)])
def test_small_grids_bf16(binding, d, f, seq, mu):  # noqa: F811
    _check(binding, small_cfg("dh32_bf16", d_model=d, n_heads=d // 32, d_ff=f, seq=seq, micro_batch=mu))


# FFN weights too wide for the transposed copies: input gradients on MN-major weights
@pytest.mark.parametrize("seq,mu", [(33, 1), (100, 3)])
def test_untransposed_weights(binding, seq, mu):  # noqa: F811
    _check(binding, small_cfg("dh32_bf16", d_model=96, n_heads=3, d_ff=32768, seq=seq, micro_batch=mu))


# fp32 products on 32 x 32, 64 x 64 and 128 x 128 tiles, and split weight gradients
@pytest.mark.parametrize("d,f,seq,mu", [(32, 64, 1, 1), (96, 160, 65, 1), (64, 2080, 125, 8), (32, 4128, 250, 8)])
def test_small_grids_fp32(binding, d, f, seq, mu):  # noqa: F811
    _check(binding, small_cfg("ragged_fp32", n_layers=1, d_model=d, n_heads=d // 32, d_ff=f, seq=seq, micro_batch=mu))


# dropout draws shared between lanes (two queries x four keys per draw) at each
# head dim, with key and query counts that end inside a draw, a 16-row tile and a block
@pytest.mark.parametrize("dh", [32, 64, 128])
@pytest.mark.parametrize("seq", [1, 2, 5, 63, 66, 131])
def test_dropout_draws(binding, dh, seq):  # noqa: F811
    _check(binding, small_cfg("drop_ragged_bf16", n_layers=1, d_model=2 * dh, n_heads=2, head_dim=dh, d_ff=64, seq=seq,
                              micro_batch=2))


# attention on the larger workgroups (more than two rounds of 64-row ones: 120
# heads of 300 rows), whose last blocks are ragged; small grids are everywhere else
@pytest.mark.parametrize("name", ["ragged_bf16", "drop_ragged_bf16"])
@pytest.mark.parametrize("dh", [32, 64, 128])
def test_attention_large_grid(binding, dh, name):  # noqa: F811
    _check(binding, small_cfg(name, n_layers=1, d_model=4 * dh, n_heads=4, head_dim=dh, d_ff=64, seq=300, micro_batch=30))


# embeddings: one 8-column chunk per lane with idle lanes, two steps of 512
# columns with a partial last one, more than one workgroup of columns and a
# partial one, the last token's workgroup partly idle; one sequence, 8 and 9
# (a second step of loads); ids repeat
@pytest.mark.parametrize("name", ["first_bf16", "first_fp32"])
@pytest.mark.parametrize("d,seq,mu", [(32, 1, 1), (288, 37, 8), (544, 21, 9)])
def test_embeddings(binding, name, d, seq, mu):  # noqa: F811
    _check(binding, small_cfg(name, d_model=d, n_heads=d // 32, head_dim=32, d_ff=64, seq=seq, micro_batch=mu))
