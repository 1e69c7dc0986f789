"""The 256-row GEMM tiles' pipeline at its edges: contractions of one to five
and a few more 64-wide steps (prologue, steady state and drain in every
combination), ragged rows, columns and token counts, in all three layouts.
Integer inputs: fp32 accumulation and the bf16 results are exact, so outputs
must equal the exact product bit for bit."""

import pytest
import torch

from helpers import announce
from paper_2408_03505_amd import binding as B
from paper_2408_03505_amd.synthetic import random_int_bf16, random_sparse_sign_bf16

pytestmark = pytest.mark.gpu

# output sizes that take each tile (checked below), with ragged last tiles
SHAPES = {(256, 256): (4000, 3880), (256, 192): (4088, 3064)}
STEPS = (1, 2, 3, 4, 5, 8, 9)


def _bf(t):
    return t.to(torch.bfloat16)


@pytest.mark.parametrize("tile", list(SHAPES))
@pytest.mark.parametrize("steps", STEPS)
def test_forward_and_input_gradient_steps(tile, steps):
    M, N = SHAPES[tile]
    N -= N % 24  # the QKV entry points take 3 * A columns, A a multiple of 8
    K = 64 * steps
    assert B.linear_plan(B.LAYOUT_FWD, M, N, K) == (*tile, 1)
    assert B.linear_plan(B.LAYOUT_DGRAD, M, N, K) == (*tile, 1)
    x, w = random_sparse_sign_bf16((M, K), 1, 0.2), random_sparse_sign_bf16((N, K), 2, 0.2)
    bias, u0 = random_int_bf16((N,), 3), torch.zeros(M, N, dtype=torch.bfloat16)
    want = x.float() @ w.float().T
    assert float(want.abs().max()) < 120  # exact in bf16, with the bias
    announce(f"enc_qkv_fwd {M}x{N}x{K}")
    got = B.enc_qkv_fwd(x.cuda(), w.cuda(), bias.cuda())
    torch.cuda.synchronize()
    assert torch.equal(got.cpu(), _bf(want + bias.float()))
    announce(f"enc_oproj_fwd {M}x{N}x{K}")
    res = random_int_bf16((M, N), 4)
    got = B.enc_oproj_fwd(x.cuda(), w.cuda(), bias.cuda(), res.cuda())
    torch.cuda.synchronize()
    assert torch.equal(got.cpu(), _bf(want + bias.float() + res.float()))
    wt = w.T.contiguous().cuda()  # [K, N]: the input gradient's weight layout
    announce(f"enc_mlp_up_bwd_data {M}x{N}x{K}")
    got = B.enc_mlp_up_bwd_data(x.cuda(), wt)
    torch.cuda.synchronize()
    assert torch.equal(got.cpu(), _bf(want))
    announce(f"enc_mlp_down_bwd_data {M}x{N}x{K}")
    got = B.enc_mlp_down_bwd_data(x.cuda(), wt, u0.cuda())  # GELU'(0) = 1/2
    torch.cuda.synchronize()
    # (the erf approximation's 1.5e-7 cannot move a bf16 rounding of an exact half-integer)
    assert torch.equal(got.cpu(), _bf(want * 0.5))


@pytest.mark.parametrize("tile", list(SHAPES))
@pytest.mark.parametrize("tokens", (1, 63, 64, 65, 129, 192, 257, 320, 511, 577))
def test_weight_gradient_tokens(tile, tokens):
    N, K = SHAPES[tile]
    assert B.linear_plan(B.LAYOUT_WGRAD, tokens, N, K) == (*tile, 1)
    dy, x = random_int_bf16((tokens, N), 5), random_int_bf16((tokens, K), 6)
    want = dy.float().T @ x.float()
    for acc in (False, True):
        announce(f"enc_linear_bwd_weight {tokens} tokens -> {N}x{K} accumulate={acc}")
        dW = torch.full((N, K), 3.0, device="cuda")
        db = torch.full((N,), 5.0, device="cuda")
        B.enc_linear_bwd_weight(dy.cuda(), x.cuda(), dW=dW, db=db, accumulate=acc)
        torch.cuda.synchronize()
        assert torch.equal(dW.cpu(), want + (3.0 if acc else 0.0))
        assert torch.equal(db.cpu(), dy.float().sum(0) + (5.0 if acc else 0.0))
