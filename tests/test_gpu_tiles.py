"""GPU parity of one forward and one backward at sizes where a kernel variant's
tiles, k-tiles or dispatch rule can go wrong, against the oracle (the
tolerances are those of the parity tests: bf16 rounding of stored activations)."""
import numpy as np
import pytest

from parity import rel_err, small_cfg, tol
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


# the same tiles with both operands MN-major (grouped weight gradients): 1 to 4
# k-tiles over T
@pytest.mark.parametrize("T", [40, 64, 72, 128, 200])
def test_pingpong_grouped(binding, T):  # noqa: F811
    _check(binding, small_cfg("tall_bf16", d_model=1024, n_heads=16, head_dim=64, d_ff=4096, seq=T // 2,
                              micro_batch=2))


# 256 x 128 ping-pong tiles over segments (window products): 1 to 6 k-tiles, one micro-batch
@pytest.mark.parametrize("T", [64, 128, 320, 384])
def test_pingpong_window(binding, T):  # noqa: F811
    _check(binding, small_cfg("win_bf16", d_model=288, n_heads=9, head_dim=32, d_ff=416, seq=T // 2, micro_batch=2))
