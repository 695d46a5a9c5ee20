"""The LM head's cross-entropy at the edges of the number range, on logits that
are set exactly: with a final LayerNorm of gain 0 its output is its bias b, so
the logit of column v is w_lm[v] . b for every token."""
import numpy as np
import pytest

from parity import Inputs, rel_err, small_cfg, to_host, to_torch, tol, unflatten
from test_gpu_stage import binding  # noqa: F401  (the fixture)
from oracle import stage as ostage

pytestmark = pytest.mark.gpu


def _pair(binding, c, inp):  # noqa: F811
    """F_0 then B_0 with K = 2: loss, input gradient and G."""
    import torch
    st = binding.Stage(c, K=2, delay=0)
    st.load_params(inp.params)
    out = torch.zeros(1, dtype=torch.float32, device="cuda")
    gi = torch.zeros(c["micro_batch"] * c["seq"], c["d_model"], dtype=st.act_dtype, device="cuda")
    st.forward(0, to_torch(inp.x_dev[0]), out, to_torch(inp.tgt[0]))
    st.backward(0, None, gi)
    G = unflatten(c, st.read(binding.GRADS))
    st.sync()
    st.close()
    return float(out.item()), to_host(gi), G


# Logits that overflow to -inf are zero probabilities, also where they fill a whole 64-column
# group of the statistics (columns 64 .. 127), its valid part (192 .. 199) or all of it but one.
@pytest.mark.parametrize("fused", [0, 1])
@pytest.mark.parametrize("dead", [(64, 128), (192, 200), (65, 128), (0, 64)])
def test_minus_infinity_logits(binding, dead, fused):  # noqa: F811
    c = small_cfg("last_bf16", vocab=200, fused_head=fused)
    inp = Inputs(c, 3, 1)
    inp.params["lnf_g"][:] = 0.0
    inp.params["lnf_b"][:] = 1.0
    inp.params["w_lm"][dead[0]:dead[1]] = -3e38   # 128 of them: below the fp32 range
    inp.tgt[0] = np.where((inp.tgt[0] >= dead[0]) & (inp.tgt[0] < dead[1]), (dead[0] + 100) % 200, inp.tgt[0]).astype(np.int32)
    loss, gi, G = _pair(binding, c, inp)
    theta = inp.oracle_params()
    o_loss, saved = ostage.stage_fwd(c, theta, inp.x[0], inp.tgt[0])
    _, o_G = ostage.stage_bwd(c, theta, saved, None, 2)
    assert abs(loss - o_loss) <= tol(c, "act") * abs(o_loss)
    assert np.all(np.isfinite(gi))
    for n in ("w_lm", "lnf_b"):
        assert rel_err(G[n], o_G[n]) <= tol(c, "grad"), n
    assert not np.any(G["w_lm"][dead[0]:dead[1]])


def _bf16_rne(x):
    m, e = np.frexp(x)   # 8 significant bits
    return np.ldexp(np.rint(m * 256) / 256, e)


# The logit gradient of one token, exp(z) / 2 in bf16, at logits z between -80 and -24 whose
# gradient lies 2^-22 to 2^-20 from a rounding boundary. An exponential within one ulp (2^-23)
# rounds every one of them correctly; one whose argument is first multiplied by log2 e and
# rounded is off by up to |z| 2^-24 and gets about a quarter of them wrong. The loss is log(1 + 2e-9):
# z - lse rounds to z.
@pytest.mark.parametrize("fused", [0, 1])
def test_logit_gradient_exponential(binding, fused):  # noqa: F811
    a, b = np.meshgrid(-(24.0 + np.arange(56 * 2) / 2), np.arange(128 * 16) / 4096, indexing="ij")
    z = (a + b).ravel()
    g = 0.5 * np.exp(z)
    m = np.frexp(g)[0] * 256
    off = np.abs(m - np.floor(m) - 0.5) / m   # relative distance from the nearest boundary
    pick = np.flatnonzero((off > 2.0 ** -22) & (off < 2.0 ** -20))
    assert pick.size >= 50
    V = 1 + pick.size
    c = small_cfg("last_bf16", vocab=V, d_model=64, n_heads=1, head_dim=64, d_ff=64, seq=1, micro_batch=1,
                  fused_head=fused)
    inp = Inputs(c, 0, 1)
    p = inp.params
    p["lnf_g"][:], p["lnf_b"][:], p["w_lm"][:] = 0.0, 0.0, 0.0
    p["lnf_b"][:3] = 1.0, 2.0 ** -8, 2.0 ** -12
    ai, bi = np.divmod(pick, 128 * 16)
    p["w_lm"][1:, 0] = -(24.0 + ai / 2)   # each exact in bf16, and so are their products' sum in fp32
    p["w_lm"][1:, 1] = bi // 16
    p["w_lm"][1:, 2] = bi % 16
    inp.tgt[0][:] = 0   # logit 0
    _, _, G = _pair(binding, c, inp)
    np.testing.assert_array_equal(G["w_lm"][1:, 0], _bf16_rne(g[pick]))
