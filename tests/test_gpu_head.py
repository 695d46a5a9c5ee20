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
