"""The layer backward's deferred reductions: with every weight gradient split
(small outputs, many tokens) the composite must give bit for bit what the
per-kernel entry points give, which reduce right after each product, both
overwriting and accumulating."""

import pytest
import torch

from helpers import announce
from paper_2408_03505_amd import binding as B
from paper_2408_03505_amd.synthetic import PARAM_ORDER, layer_inputs

pytestmark = pytest.mark.gpu

# (batch, seq, hidden, heads, head_dim, mlp): all four weight gradients split;
# then a mix (1000 tokens: none split), odd column counts for the block ranges
CASES = [(8, 197, 256, 4, 64, 520), (5, 211, 200, 2, 80, 328), (2, 500, 192, 3, 64, 768)]


def _by_kernels(cfg, p, x, dout, saved, want, accumulate):
    """The layer's gradients into want, by the per-kernel entry points."""
    s = B.saved_views(cfg, saved)
    acc = dict(accumulate=accumulate)
    du = B.enc_mlp_down_bwd_data(dout, p["w_2"], s["u"])
    B.enc_mlp_down_bwd_weight(dout, s["g"], want["w_2"], want["b_2"], **acc)
    dy2 = B.enc_mlp_up_bwd_data(du, p["w_1"])
    B.enc_mlp_up_bwd_weight(du, s["y2"], want["w_1"], want["b_1"], **acc)
    dh, _, _ = B.enc_ln_bwd(dy2, s["h"], s["mean2"], s["rstd2"], p["ln2_g"], dresid=dout, dgamma=want["ln2_g"],
                            dbeta=want["ln2_b"], **acc)
    do = B.enc_oproj_bwd_data(dh, p["w_o"])
    B.enc_oproj_bwd_weight(dh, s["o"], want["w_o"], want["b_o"], **acc)
    dqkv = B.enc_attn_bwd(cfg["batch"], cfg["seq"], cfg["heads"], cfg["head_dim"], s["qkv"], s["o"], s["lse"], do)
    dy1 = B.enc_qkv_bwd_data(dqkv, p["w_qkv"])
    B.enc_qkv_bwd_weight(dqkv, s["y1"], want["w_qkv"], want["b_qkv"], **acc)
    B.enc_ln_bwd(dy1, x, s["mean1"], s["rstd1"], p["ln1_g"], dresid=dh, dgamma=want["ln1_g"], dbeta=want["ln1_b"],
                 **acc)


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("accumulate", (False, True))
def test_composite_reductions_match_the_kernels(case, accumulate):
    cfg = dict(zip(("batch", "seq", "hidden", "heads", "head_dim", "mlp"), case), ln_eps=1e-6)
    M = cfg["batch"] * cfg["seq"]
    split = [B.linear_bwd_weight_workspace_bytes(M, n, k) > 0 for n, k in (s for s in B.param_shapes(cfg).values()
                                                                           if len(s) == 2)]
    assert all(split) if M >= 1024 else not any(split)
    x, params, dout = layer_inputs(cfg, seed=3)
    p = {n: params[n].cuda() for n in PARAM_ORDER}
    x, dout = x.cuda(), dout.cuda()
    announce(f"layer {case} accumulate={accumulate}")
    _, saved = B.encoder_layer_fwd(cfg, p, x)
    grads = {n: torch.full(s, 0.5, device="cuda") for n, s in B.param_shapes(cfg).items()}
    want = {n: g.clone() for n, g in grads.items()}
    B.encoder_layer_bwd(cfg, p, x, saved, dout, grads=grads, accumulate=accumulate)
    _by_kernels(cfg, p, x, dout, saved, want, accumulate)
    torch.cuda.synchronize()
    for n in PARAM_ORDER:
        assert torch.equal(grads[n], want[n]), n


@pytest.mark.parametrize("accumulate", (False, True))
def test_gradients_that_share_a_buffer_are_written_in_order(accumulate):
    """Tied gradients: both LayerNorms' scales, their biases and two of the
    projections' biases into one buffer each."""
    cfg = dict(zip(("batch", "seq", "hidden", "heads", "head_dim", "mlp"), CASES[0]), ln_eps=1e-6)
    x, params, dout = layer_inputs(cfg, seed=4)
    p = {n: params[n].cuda() for n in PARAM_ORDER}
    x, dout = x.cuda(), dout.cuda()
    announce(f"layer {CASES[0]} tied gradients accumulate={accumulate}")
    _, saved = B.encoder_layer_fwd(cfg, p, x)

    def tied():
        g = {n: torch.full(s, 0.5, device="cuda") for n, s in B.param_shapes(cfg).items()}
        g.update(ln2_g=g["ln1_g"], ln2_b=g["ln1_b"], b_2=g["b_o"])
        return g

    grads, want = tied(), tied()
    B.encoder_layer_bwd(cfg, p, x, saved, dout, grads=grads, accumulate=accumulate)
    _by_kernels(cfg, p, x, dout, saved, want, accumulate)
    torch.cuda.synchronize()
    for n in PARAM_ORDER:
        assert torch.equal(grads[n], want[n]), n
