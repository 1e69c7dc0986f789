"""The GEMM tiles' pipelines at their edges: contractions of one to a few
64-wide steps more than the deepest ring (prologue, steady state and drain in
every combination), ragged rows, columns and token counts, in all three
layouts, on every tile the launch plan has.  Integer inputs: fp32 accumulation
and the bf16 results are exact, so outputs must equal the exact product bit
for bit."""

import itertools

import pytest
import torch

from helpers import announce
from paper_2408_03505_amd import binding as B
from paper_2408_03505_amd.synthetic import random_int_bf16, random_sparse_sign_bf16

pytestmark = pytest.mark.gpu

TILES = [(256, 256), (256, 192), (128, 256), (128, 192), (192, 128), (128, 128), (64, 192), (64, 128), (64, 64)]
STEPS = (1, 2, 3, 4, 5, 6, 8, 11, 13)
TOKENS = (1, 63, 64, 65, 129, 192, 257, 320, 383, 511, 577, 830)
# output sizes tried, smallest product first; columns are whole 3 x 8 blocks
_ROWS = (40, 120, 248, 520, 1000, 1576, 2040, 3064, 4088, 6296)
_COLS = (72, 192, 384, 768, 1152, 1560, 2304, 3072, 3888, 4104)
_SIZES = sorted(itertools.product(_ROWS, _COLS), key=lambda t: t[0] * t[1])


def _cases(layout, contractions):
    """(tile, rows, cols, contraction): per tile and contraction the smallest
    size tried that runs on the tile, unsplit (host queries only)."""
    out = []
    for k in contractions:
        seen = set()
        for r, c in _SIZES:
            bm, bn, sp = B.linear_plan(layout, r, c, k) if layout != B.LAYOUT_WGRAD else B.linear_plan(layout, k, r, c)
            if sp == 1 and (bm, bn) not in seen:
                seen.add((bm, bn))
                out.append(((bm, bn), r, c, k))
    return out


def test_every_tile_is_covered():
    for layout, ks in ((B.LAYOUT_FWD, [64 * s for s in STEPS]), (B.LAYOUT_DGRAD, [64 * s for s in STEPS]),
                       (B.LAYOUT_WGRAD, TOKENS)):
        tiles = {c[0] for c in _cases(layout, ks)}
        assert len(tiles) >= 7 and tiles <= set(TILES), (layout, tiles)


def _operands(M, N, K):
    return random_sparse_sign_bf16((M, K), 1, 0.1), random_sparse_sign_bf16((N, K), 2, 0.1)


@pytest.mark.parametrize("steps", STEPS)
def test_forward_steps(steps):
    for tile, M, N, K in _cases(B.LAYOUT_FWD, [64 * steps]):
        x, w = _operands(M, N, K)
        bias, res = random_int_bf16((N,), 3), random_int_bf16((M, N), 4)
        want = x.float() @ w.float().T
        assert float(want.abs().max()) < 120  # exact in bf16, with the bias and the residual
        announce(f"enc_qkv_fwd {M}x{N}x{K} on {tile}")
        got = B.enc_qkv_fwd(x.cuda(), w.cuda(), bias.cuda(), split=False)
        torch.cuda.synchronize()
        assert torch.equal(got.cpu(), (want + bias.float()).to(torch.bfloat16))
        announce(f"enc_oproj_fwd {M}x{N}x{K} on {tile}")
        got = B.enc_oproj_fwd(x.cuda(), w.cuda(), bias.cuda(), res.cuda(), split=False)
        torch.cuda.synchronize()
        assert torch.equal(got.cpu(), (want + bias.float() + res.float()).to(torch.bfloat16))


@pytest.mark.parametrize("steps", STEPS)
def test_input_gradient_steps(steps):
    for tile, M, N, K in _cases(B.LAYOUT_DGRAD, [64 * steps]):
        x, w = _operands(M, N, K)
        want = x.float() @ w.float().T
        wt = w.T.contiguous().cuda()  # [K, N]: the input gradient's weight layout
        announce(f"enc_mlp_up_bwd_data {M}x{N}x{K} on {tile}")
        got = B.enc_mlp_up_bwd_data(x.cuda(), wt, split=False)
        torch.cuda.synchronize()
        assert torch.equal(got.cpu(), want.to(torch.bfloat16))
        announce(f"enc_mlp_down_bwd_data {M}x{N}x{K} on {tile}")
        u = torch.full((M, N), 8.0, dtype=torch.bfloat16, device="cuda")  # GELU'(8) == 1 in fp32
        got = B.enc_mlp_down_bwd_data(x.cuda(), wt, u, split=False)
        torch.cuda.synchronize()
        assert torch.equal(got.cpu(), want.to(torch.bfloat16))


@pytest.mark.parametrize("tokens", TOKENS)
def test_weight_gradient_tokens(tokens):
    for tile, N, K, _ in _cases(B.LAYOUT_WGRAD, [tokens]):
        dy, x = random_int_bf16((tokens, N), 5), random_int_bf16((tokens, K), 6)
        want = dy.float().T @ x.float()
        for acc in (False, True):
            announce(f"enc_linear_bwd_weight {tokens} tokens -> {N}x{K} accumulate={acc} on {tile}")
            dW = torch.full((N, K), 3.0, device="cuda")
            db = torch.full((N,), 5.0, device="cuda")
            B.enc_linear_bwd_weight(dy.cuda(), x.cuda(), dW=dW, db=db, accumulate=acc, split=False)
            torch.cuda.synchronize()
            assert torch.equal(dW.cpu(), want + (3.0 if acc else 0.0))
            assert torch.equal(db.cpu(), dy.float().sum(0) + (5.0 if acc else 0.0))
