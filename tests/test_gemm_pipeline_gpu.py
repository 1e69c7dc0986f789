"""The GEMM tiles' pipelines at their edges: contractions of one to a few
64-wide steps more than the deepest ring (prologue, steady state and drain in
every combination), ragged rows, columns and token counts, in all three
layouts, on every tile that the launch plan gives a product, whole and as
splits of the contraction.  Integer inputs: fp32 accumulation and the bf16
results are exact, so outputs must equal the exact product bit for bit; the
GELU and GELU' epilogues are held to the float64 oracle."""

import numpy as np
import pytest
import torch

import oracle
from helpers import announce, f64
from paper_2408_03505_amd import binding as B
from paper_2408_03505_amd.synthetic import random_int_bf16, random_sparse_sign_bf16

gpu = pytest.mark.gpu

# stages of k-steps that each tile's pipeline holds
STAGES = {(256, 256): 2, (256, 192): 2, (128, 256): 3, (128, 192): 4, (192, 128): 2, (128, 128): 2, (64, 192): 4,
          (64, 128): 3, (64, 64): 4}
STEPS = (1, 2, 3, 4, 5, 6, 8, 11, 12, 13, 14, 17, 18, 19, 33, 34, 35)
# token counts with these numbers of k-steps, whole, nearly whole and nearly empty last ones
TOKENS = (1, 63, 64, 65, 129, 192, 193, 257, 320, 383, 511, 577, 700, 768, 830, 833, 896, 1025, 1152, 1215, 2049, 2175,
          2240)
LAYOUTS = {"fwd": B.LAYOUT_FWD, "dgrad": B.LAYOUT_DGRAD, "wgrad": B.LAYOUT_WGRAD, "fwd_gelu": B.LAYOUT_FWD_GELU,
           "dgrad_gelu": B.LAYOUT_DGRAD_GELU}
# output sizes, smallest first; between them and the contractions above every
# tile runs in every layout that it is offered to
_SIZES = sorted([(40, 72), (120, 192), (248, 768), (264, 6696), (776, 7128), (1000, 1152), (4192, 264), (6576, 528),
                 (6576, 1032), (6592, 1800), (7248, 1056)], key=lambda t: t[0] * t[1])


def _plan(layout, rows, cols, k):
    a = (k, rows, cols) if layout == B.LAYOUT_WGRAD else (rows, cols, k)
    return B.linear_plan(layout, *a)


def _cases(layout, k):
    """(tile, rows, cols): per tile the smallest size that runs on it, unsplit,
    at this contraction (host queries only)."""
    out = {}
    for r, c in _SIZES:
        bm, bn, sp = _plan(layout, r, c, k)
        if sp == 1:
            out.setdefault((bm, bn), (r, c))
    return [(tile, r, c) for tile, (r, c) in out.items()]


# the forward GELU is never given 192x128 tiles
@pytest.mark.parametrize("name", LAYOUTS)
def test_every_tile_is_covered(name):
    offered = set(STAGES) - ({(192, 128)} if name == "fwd_gelu" else set())
    seen = {}
    for k in TOKENS if name == "wgrad" else [64 * s for s in STEPS]:
        for tile, _, _ in _cases(LAYOUTS[name], k):
            seen.setdefault(tile, set()).add(-(-k // 64))
    assert set(seen) == offered
    for tile, steps in seen.items():
        # every phase of the ring at the last k-step, and a steady state
        assert {s % STAGES[tile] for s in steps} == set(range(STAGES[tile])), (tile, steps)
        assert max(steps) >= 2 * STAGES[tile] + 2, (tile, steps)


def _operands(M, N, K):
    return random_sparse_sign_bf16((M, K), 1, 0.1), random_sparse_sign_bf16((N, K), 2, 0.1)


def _product(x, w):
    want = x.float() @ w.float().T
    assert float(want.abs().max()) < 120  # exact in bf16, with the bias and the residual
    return want


@gpu
@pytest.mark.parametrize("steps", STEPS)
def test_forward_steps(steps):
    for tile, M, N in _cases(B.LAYOUT_FWD, 64 * steps):
        x, w = _operands(M, N, 64 * steps)
        bias, res = random_int_bf16((N,), 3), random_int_bf16((M, N), 4)
        want = _product(x, w)
        announce(f"enc_qkv_fwd {M}x{N}x{64 * steps} on {tile}")
        got = B.enc_qkv_fwd(x.cuda(), w.cuda(), bias.cuda(), split=False)
        torch.cuda.synchronize()
        assert torch.equal(got.cpu(), (want + bias.float()).to(torch.bfloat16))
        announce(f"enc_oproj_fwd {M}x{N}x{64 * steps} on {tile}")
        got = B.enc_oproj_fwd(x.cuda(), w.cuda(), bias.cuda(), res.cuda(), split=False)
        torch.cuda.synchronize()
        assert torch.equal(got.cpu(), (want + bias.float() + res.float()).to(torch.bfloat16))


# Rounding to bf16 is off by at most 2^-8 of the value.  Before it, GELU(v) is
# off by |v| times the 0.75e-7 of the tail formula and a few fp32 roundings, and
# GELU'(u) by about 1e-7 (4e-7 and 1e-6 allowed).
def _near(got, want, scale):
    assert np.all(np.abs(f64(got) - want) <= 2.0 ** -8 * np.abs(want) * 1.001 + 1e-6 * scale)


@gpu
@pytest.mark.parametrize("steps", STEPS)
def test_forward_gelu_steps(steps):
    for tile, M, N in _cases(B.LAYOUT_FWD_GELU, 64 * steps):
        x, w = _operands(M, N, 64 * steps)
        bias = random_int_bf16((N,), 3)
        want = _product(x, w) + bias.float()
        announce(f"enc_mlp_up_fwd {M}x{N}x{64 * steps} on {tile}")
        u, g = B.enc_mlp_up_fwd(x.cuda(), w.cuda(), bias.cuda(), split=False)
        torch.cuda.synchronize()
        assert torch.equal(u.cpu(), want.to(torch.bfloat16))
        v = want.double().numpy()
        _near(g, oracle.gelu(v), np.maximum(np.abs(v), 1.0))


@gpu
@pytest.mark.parametrize("steps", STEPS)
def test_input_gradient_steps(steps):
    for tile, M, N in _cases(B.LAYOUT_DGRAD, 64 * steps):
        x, w = _operands(M, N, 64 * steps)
        want = _product(x, w)
        announce(f"enc_mlp_up_bwd_data {M}x{N}x{64 * steps} on {tile}")
        got = B.enc_mlp_up_bwd_data(x.cuda(), w.T.contiguous().cuda(), split=False)
        torch.cuda.synchronize()
        assert torch.equal(got.cpu(), want.to(torch.bfloat16))


@gpu
@pytest.mark.parametrize("steps", STEPS)
def test_input_gradient_gelu_steps(steps):
    for tile, M, N in _cases(B.LAYOUT_DGRAD_GELU, 64 * steps):
        x, w = _operands(M, N, 64 * steps)
        want = _product(x, w).double().numpy()
        u = torch.randn((M, N), generator=torch.Generator().manual_seed(7)).to(torch.bfloat16)
        announce(f"enc_mlp_down_bwd_data {M}x{N}x{64 * steps} on {tile}")
        got = B.enc_mlp_down_bwd_data(x.cuda(), w.T.contiguous().cuda(), u.cuda(), split=False)
        torch.cuda.synchronize()
        _near(got, want * oracle.gelu_grad(f64(u)), np.abs(want))


def _weight_gradient(tokens, N, K, accumulate, split, where):
    dy, x = random_int_bf16((tokens, N), 5), random_int_bf16((tokens, K), 6)
    announce(f"enc_linear_bwd_weight {tokens} tokens -> {N}x{K} accumulate={accumulate} on {where}")
    dW = torch.full((N, K), 3.0, device="cuda")
    db = torch.full((N,), 5.0, device="cuda")
    B.enc_linear_bwd_weight(dy.cuda(), x.cuda(), dW=dW, db=db, accumulate=accumulate, split=split)
    torch.cuda.synchronize()
    assert torch.equal(dW.cpu(), dy.float().T @ x.float() + (3.0 if accumulate else 0.0))
    assert torch.equal(db.cpu(), dy.float().sum(0) + (5.0 if accumulate else 0.0))


@gpu
@pytest.mark.parametrize("tokens", TOKENS)
def test_weight_gradient_tokens(tokens):
    for tile, N, K in _cases(B.LAYOUT_WGRAD, tokens):
        for acc in (False, True):
            _weight_gradient(tokens, N, K, acc, False, tile)


# (rows, columns, contraction) of products that split, one or more per tile
# that splits run
SPLITS = {(128, 128): [(40, 120, 1216), (2888, 504, 4608)], (64, 192): [(7, 7176, 23040), (1, 7200, 14912)],
          (64, 128): [(136, 5688, 1024), (3600, 456, 1536)], (64, 64): [(72, 2736, 1536), (1168, 72, 3648)]}
WGRAD_SPLITS = {(128, 128): (40, 72, 2309), (128, 192): (40, 4344, 4096), (128, 256): (136, 6648, 4096),
                (192, 128): (136, 6680, 3648), (256, 192): (3624, 568, 8692), (256, 256): (5704, 448, 8246)}


def test_the_split_sizes_run_on_the_tiles_they_name():
    for tile, sizes in SPLITS.items():
        for M, N, K in sizes:
            for layout in (B.LAYOUT_FWD, B.LAYOUT_DGRAD, B.LAYOUT_FWD_GELU, B.LAYOUT_DGRAD_GELU):
                plan = _plan(layout, M, N, K)
                assert plan[:2] == tile and plan[2] > 1, (M, N, K, plan)
    for tile, (N, K, tokens) in WGRAD_SPLITS.items():
        plan = _plan(B.LAYOUT_WGRAD, N, K, tokens)
        assert plan[:2] == tile and plan[2] > 1, (N, K, tokens, plan)


@gpu
@pytest.mark.parametrize("tile", SPLITS)
def test_split_products(tile):
    for M, N, K in SPLITS[tile]:
        x, w = _operands(M, N, K)
        bias = random_int_bf16((N,), 3)
        want = _product(x, w)
        announce(f"enc_mlp_up_fwd {M}x{N}x{K} split on {tile}")
        u, g = B.enc_mlp_up_fwd(x.cuda(), w.cuda(), bias.cuda())
        torch.cuda.synchronize()
        v = want + bias.float()
        assert torch.equal(u.cpu(), v.to(torch.bfloat16))
        _near(g, oracle.gelu(v.double().numpy()), np.maximum(np.abs(v.numpy()), 1.0))
        announce(f"enc_mlp_up_bwd_data {M}x{N}x{K} split on {tile}")
        got = B.enc_mlp_up_bwd_data(x.cuda(), w.T.contiguous().cuda())
        torch.cuda.synchronize()
        assert torch.equal(got.cpu(), want.to(torch.bfloat16))


@gpu
@pytest.mark.parametrize("tile", WGRAD_SPLITS)
def test_split_weight_gradients(tile):
    N, K, tokens = WGRAD_SPLITS[tile]
    for acc in (False, True):
        _weight_gradient(tokens, N, K, acc, True, tile)
