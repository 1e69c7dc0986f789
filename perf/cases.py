"""The work that users of the encoder kernels have them do, as measurable cases.

A case is a plain dict; `kind` picks the calls:

  layer_step     encoder_layer_fwd + encoder_layer_bwd on one micro-batch, or on
                 `micro` micro-batches whose gradients accumulate
  layer_fwd      encoder_layer_fwd alone (a frozen encoder)
  parallel_step  encoder_parallel_fwd + _bwd (the ViT-22B-style block)
  encoder_step   patch embedding, a stack of layers and the final LayerNorm,
                 forward and backward
  attn_step      enc_attn_fwd + enc_attn_bwd, as a scheduler places them
  norm_step      enc_ln_fwd + enc_ln_bwd with the residual gradient
  mlp_fwd        enc_mlp_up_fwd + enc_mlp_down_fwd
  qkv_bwd        enc_qkv_bwd_data + enc_qkv_bwd_weight

Every program here keeps its outputs, saved tensors and workspaces from call to
call, as a training loop does.
"""

import math

import torch

from paper_2408_03505_amd import binding as B

BF, F32, F64 = torch.bfloat16, torch.float32, torch.float64
EPS = 1e-6


def _layer(name, kind, batch, seq, hidden, heads, head_dim, mlp, **more):
    return dict(name=name, kind=kind, batch=batch, seq=seq, hidden=hidden, heads=heads, head_dim=head_dim, mlp=mlp,
                **more)


def listed():
    return [
        # The smallest training call: a ViT-Tiny layer on two 224-pixel images.
        # Twenty short launches; latency is all of it.
        _layer("layer_step_tiny", "layer_step", 2, 197, 192, 3, 64, 768, micro=1),
        # A ViT-Base layer in training, 32 images with a class token (6304 rows,
        # a ragged number of tiles).
        _layer("layer_step_base", "layer_step", 32, 197, 768, 12, 64, 3072, micro=1),
        # A ViT-Huge layer in training: head dimension 80, 257 tokens.
        _layer("layer_step_huge", "layer_step", 16, 257, 1280, 16, 80, 5120, micro=1),
        # One GPU's 1/8 tensor-parallel shard of a ViT-22B layer; two
        # micro-batches of one iteration, the second adding to the gradients.
        _layer("layer_step_22b_tp8", "layer_step", 8, 256, 6144, 6, 128, 3072, micro=2),
        # The full ViT-22B layer in training: the largest unit of work.
        _layer("layer_step_22b", "layer_step", 8, 256, 6144, 48, 128, 24576, micro=1),
        # A frozen ViT-10B layer (forward only) on four images with a class token.
        _layer("layer_fwd_10b", "layer_fwd", 4, 257, 4096, 32, 128, 16384),
        # The ViT-22B-style block (parallel branches, QK normalisation) on the
        # tensor-parallel shard, in training.
        _layer("parallel_step_22b_tp8", "parallel_step", 8, 256, 6144, 6, 128, 3072),
        # A whole ViT-Base encoder on eight 224-pixel images, in training.
        _layer("encoder_step_base", "encoder_step", 8, 197, 768, 12, 64, 3072, layers=12, img=224, patch=16, cls=True),
        # Attention placed on its own, 448-pixel images at patch 14 (1025 tokens).
        dict(name="attn_step_long", kind="attn_step", batch=4, seq=1025, heads=16, head_dim=80),
        # LayerNorm placed on its own at ViT-5B width.
        dict(name="norm_step_5b", kind="norm_step", rows=8 * 257, cols=3072),
        # The MLP of one ViT-Huge image (257 rows): serving a single request.
        dict(name="mlp_fwd_one_image", kind="mlp_fwd", rows=257, hidden=1280, mlp=5120),
        # Backward of the QKV projection placed on its own at ViT-3B width.
        dict(name="qkv_bwd_3b", kind="qkv_bwd", rows=8 * 257, hidden=2304, heads=18, head_dim=128),
    ]


# ------------------------------------------------------------------ drawn cases

_MAX_FLOPS, _MAX_BYTES = 4.0e12, 6.0e9


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A width between lo and hi: a multiple of 64 mostly, of 8 now and then."""
    q = 64 if rng.random() < 0.8 else 8
    return max(1, round(_logint(rng, lo, hi) / q)) * q


def _draw_once(rng):
    kind = rng.choice(["layer_step", "layer_step", "layer_step", "layer_fwd", "parallel_step", "encoder_step",
                       "attn_step", "norm_step", "mlp_fwd", "qkv_bwd"])
    seq = _logint(rng, 50, 1025)
    batch = _logint(rng, 1, max(1, 8224 // seq))
    head_dim = rng.choice([64, 80, 128])
    if kind == "norm_step":
        return dict(kind=kind, rows=_logint(rng, 50, 8224), cols=_width(rng, 192, 6144))
    if kind == "attn_step":
        return dict(kind=kind, batch=batch, seq=seq, heads=_logint(rng, 1, 48), head_dim=head_dim)
    if kind == "mlp_fwd":
        hidden = _width(rng, 192, 6144)
        return dict(kind=kind, rows=_logint(rng, 50, 8224), hidden=hidden, mlp=_width(rng, 768, 4 * hidden))
    if kind == "qkv_bwd":
        heads = _logint(rng, 1, 48)
        return dict(kind=kind, rows=_logint(rng, 50, 8224), hidden=_width(rng, 192, 6144), heads=heads,
                    head_dim=head_dim)
    if kind == "encoder_step":
        heads = _logint(rng, 3, 16)
        hidden = heads * head_dim
        patch = rng.choice([14, 16, 32])
        side = rng.choice([4, 7, 12, 14, 16])
        cls = rng.random() < 0.5
        return _layer("", kind, _logint(rng, 1, 16), side * side + int(cls), hidden, heads, head_dim, 4 * hidden,
                      layers=rng.randint(2, 12), img=side * patch, patch=patch, cls=cls)
    hidden = _width(rng, 192, 6144)
    heads = max(1, min(48, round(hidden / head_dim / rng.choice([1, 1, 1, 2, 8]))))
    mlp = _width(rng, 768, 4 * hidden) if rng.random() < 0.5 else 4 * hidden
    case = _layer("", kind, batch, seq, hidden, heads, head_dim, mlp)
    if kind == "layer_step":
        case["micro"] = rng.choice([1, 1, 2])
    return case


def draw(rng):
    while True:
        case = _draw_once(rng)
        case.pop("name", None)
        w = work(case)
        if w["flops"] <= _MAX_FLOPS and w["bytes"] <= _MAX_BYTES:
            return case


# ------------------------------------------------------------------ inputs

class _Rand:
    """Seeded normal draws on the GPU, rounded once to bf16."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def __call__(self, shape, std=1.0, mean=0.0):
        t = torch.randn(shape, generator=self.g, dtype=F32, device="cuda")
        return t.mul_(std).add_(mean).to(BF)


def _cfg(case):
    return dict(batch=case["batch"], seq=case["seq"], hidden=case["hidden"], heads=case["heads"],
                head_dim=case["head_dim"], mlp=case["mlp"], ln_eps=EPS)


def _params(rnd, shapes):
    # LayerNorm scales about one, every other weight and bias about zero
    scales = ("ln1_g", "ln2_g", "ln_g", "qn_g", "kn_g")
    return {n: rnd(s, 0.02, 1.0 if n in scales else 0.0) for n, s in shapes.items()}


def _empty(shape, dtype=BF):
    return torch.empty(shape, dtype=dtype, device="cuda")


def _grads(shapes):
    return {n: _empty(s, F32) for n, s in shapes.items()}


def _flat_grads(shapes):
    """One layer's gradients as views of one flat buffer, as a program that
    reduces a layer's gradients with one collective keeps them."""
    flat = _empty((sum(math.prod(s) for s in shapes.values()),), F32)
    views, o = {}, 0
    for n, s in shapes.items():
        views[n] = flat[o:o + math.prod(s)].view(s)
        o += math.prod(s)
    return flat, views


def _inputs(case, seed):
    """The random inputs of a case, the same for the library and for exact()."""
    rnd = _Rand(seed)
    kind = case["kind"]
    if kind == "norm_step":
        rc = (case["rows"], case["cols"])
        return dict(x=rnd(rc), gamma=rnd(rc[1:], 0.02, 1.0), beta=rnd(rc[1:], 0.02), dy=rnd(rc), dresid=rnd(rc))
    if kind == "attn_step":
        A, M = case["heads"] * case["head_dim"], case["batch"] * case["seq"]
        return dict(qkv=rnd((M, 3 * A)), do=rnd((M, A)))
    if kind == "mlp_fwd":
        M, H, F = case["rows"], case["hidden"], case["mlp"]
        return dict(y2=rnd((M, H)), w_1=rnd((F, H), 0.02), b_1=rnd((F,), 0.02), w_2=rnd((H, F), 0.02),
                    b_2=rnd((H,), 0.02), resid=rnd((M, H)))
    if kind == "qkv_bwd":
        M, H, A3 = case["rows"], case["hidden"], 3 * case["heads"] * case["head_dim"]
        return dict(dqkv=rnd((M, A3)), w_qkv=rnd((A3, H), 0.02), y1=rnd((M, H)))
    cfg = _cfg(case)
    M, H = cfg["batch"] * cfg["seq"], cfg["hidden"]
    if kind == "encoder_step":
        n_in = 3 * case["patch"] ** 2
        w_pe = rnd((H, B.patch_kp(3, case["patch"])), 0.02)
        w_pe[:, n_in:] = 0
        return dict(images=rnd((cfg["batch"], 3, case["img"], case["img"])), w_pe=w_pe, b_pe=rnd((H,), 0.02),
                    pos=rnd((cfg["seq"], H), 0.02), cls=rnd((H,), 0.02) if case["cls"] else None,
                    layers=[_params(rnd, B.param_shapes(cfg)) for _ in range(case["layers"])],
                    lnf_g=rnd((H,), 0.02, 1.0), lnf_b=rnd((H,), 0.02), dout=rnd((M, H)))
    shapes = B.parallel_param_shapes(cfg) if kind == "parallel_step" else B.param_shapes(cfg)
    inp = dict(params=_params(rnd, shapes))
    inp["x"] = [rnd((M, H)) for _ in range(case.get("micro", 1))]
    if kind != "layer_fwd":
        inp["dout"] = [rnd((M, H)) for _ in range(case.get("micro", 1))]
    return inp


def prepare(case, seed):
    st = dict(case=case, **_inputs(case, seed))
    kind = case["kind"]
    u8 = torch.uint8
    if kind == "norm_step":
        R, C = case["rows"], case["cols"]
        st.update(y=_empty((R, C)), mean=_empty((R,), F32), rstd=_empty((R,), F32), dx=_empty((R, C)),
                  dgamma=_empty((C,), F32), dbeta=_empty((C,), F32),
                  ws=_empty((B.ln_bwd_workspace_bytes(R, C),), u8))
    elif kind == "attn_step":
        Bn, S, h, d = (case[k] for k in ("batch", "seq", "heads", "head_dim"))
        st.update(o=_empty((Bn * S, h * d)), lse=_empty((Bn, h, S), F32), dqkv=_empty((Bn * S, 3 * h * d)),
                  ws=_empty((B.attn_bwd_workspace_bytes(Bn, S, h, d),), u8))
    elif kind == "mlp_fwd":
        M, H, F = case["rows"], case["hidden"], case["mlp"]
        need = max(B.linear_workspace_bytes(M, F, H), B.linear_workspace_bytes(M, H, F))
        st.update(u=_empty((M, F)), g=_empty((M, F)), out=_empty((M, H)), ws=_empty((need,), u8) if need else None)
    elif kind == "qkv_bwd":
        M, H, A3 = case["rows"], case["hidden"], 3 * case["heads"] * case["head_dim"]
        need = max(B.linear_workspace_bytes(M, H, A3), B.linear_bwd_weight_workspace_bytes(M, A3, H))
        st.update(dy1=_empty((M, H)), dw=_empty((A3, H), F32), db=_empty((A3,), F32),
                  ws=_empty((need,), u8) if need else None)
    else:
        cfg = st["cfg"] = _cfg(case)
        M, H = cfg["batch"] * cfg["seq"], cfg["hidden"]
        if kind == "encoder_step":
            n = case["layers"]
            shp = (cfg["batch"], 3, case["img"], case["img"])
            kp, N = B.patch_kp(3, case["patch"]), (case["img"] // case["patch"]) ** 2
            need = B.patch_embed_workspace_bytes(*shp[:2], *shp[2:], case["patch"], H, case["cls"])
            pe = {"w_pe": (H, kp), "b_pe": (H,), "pos": (cfg["seq"], H)}
            if case["cls"]:
                pe["cls"] = (H,)
            flat, views = zip(*[_flat_grads(B.param_shapes(cfg)) for _ in range(n)])
            st.update(x0=_empty((M, H)), patches=_empty((cfg["batch"] * N, kp)), out=_empty((M, H)),
                      saved=_empty((B.stack_saved_bytes(cfg, n),), u8), dx0=_empty((M, H)),
                      grads=list(views), flat_grads=list(flat),
                      lnf_grads=(_empty((H,), F32), _empty((H,), F32)), pe_grads=_grads(pe),
                      ws=_empty((B.stack_workspace_bytes(cfg, n),), u8),
                      pe_ws=_empty((need,), u8) if need else None)
        elif kind == "parallel_step":
            shapes = B.parallel_param_shapes(cfg)
            grads = _grads({k: s for k, s in shapes.items() if k not in _QK})
            # the QK-norm gradients live in one flat buffer
            st["qk_grads"] = _empty((4, cfg["head_dim"]), F32)
            grads.update({k: st["qk_grads"][i] for i, k in enumerate(_QK)})
            st.update(out=_empty((M, H)), dx=_empty((M, H)), grads=grads,
                      saved=_empty((B.parallel_saved_layout(cfg)["total"],), u8),
                      ws=_empty((B.parallel_workspace_bytes(cfg),), u8))
        else:
            n = case.get("micro", 1)
            st.update(out=[_empty((M, H)) for _ in range(n)], saved=_empty((B.saved_layout(cfg)["total"],), u8),
                      ws=_empty((B.layer_workspace_bytes(cfg),), u8))
            if kind == "layer_step":
                st.update(dx=[_empty((M, H)) for _ in range(n)], grads=_grads(B.param_shapes(cfg)))
    return st


_QK = ("qn_g", "qn_b", "kn_g", "kn_b")


# ------------------------------------------------------------------ one pass

def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "layer_step":
        for i, (x, dout) in enumerate(zip(st["x"], st["dout"])):
            B.encoder_layer_fwd(st["cfg"], st["params"], x, out=st["out"][i], saved=st["saved"], ws=st["ws"])
            B.encoder_layer_bwd(st["cfg"], st["params"], x, st["saved"], dout, grads=st["grads"], dx=st["dx"][i],
                                accumulate=i > 0, ws=st["ws"])
        return dict(out=st["out"], dx=st["dx"], grads=st["grads"])
    if kind == "layer_fwd":
        B.encoder_layer_fwd(st["cfg"], st["params"], st["x"][0], out=st["out"][0], saved=st["saved"], ws=st["ws"])
        return dict(out=st["out"])
    if kind == "parallel_step":
        x, dout = st["x"][0], st["dout"][0]
        B.encoder_parallel_fwd(st["cfg"], st["params"], x, out=st["out"], saved=st["saved"])
        B.encoder_parallel_bwd(st["cfg"], st["params"], x, st["saved"], dout, grads=st["grads"], dx=st["dx"],
                               ws=st["ws"])
        grads = {n: g for n, g in st["grads"].items() if n not in _QK}
        return dict(out=st["out"], dx=st["dx"], grads=grads, qk_grads=st["qk_grads"])
    if kind == "encoder_step":
        B.enc_patch_embed_fwd(st["images"], case["patch"], st["w_pe"], st["b_pe"], st["pos"], cls=st["cls"],
                              patches=st["patches"], x0=st["x0"], ws=st["pe_ws"])
        B.encoder_stack_fwd(st["cfg"], st["layers"], st["lnf_g"], st["lnf_b"], st["x0"], out=st["out"],
                            saved=st["saved"])
        B.encoder_stack_bwd(st["cfg"], st["layers"], st["lnf_g"], st["x0"], st["saved"], st["dout"],
                            grads=st["grads"], lnf_grads=st["lnf_grads"], dx0=st["dx0"], ws=st["ws"])
        B.enc_patch_embed_bwd(tuple(st["images"].shape), case["patch"], st["dx0"], st["patches"], case["cls"],
                              grads=st["pe_grads"], ws=st["pe_ws"])
        return dict(out=st["out"], grads=st["flat_grads"], lnf_grads=list(st["lnf_grads"]), pe_grads=st["pe_grads"])
    if kind == "attn_step":
        shape = tuple(case[k] for k in ("batch", "seq", "heads", "head_dim"))
        B.enc_attn_fwd(*shape, st["qkv"], o=st["o"], lse=st["lse"])
        B.enc_attn_bwd(*shape, st["qkv"], st["o"], st["lse"], st["do"], dqkv=st["dqkv"], ws=st["ws"])
        return dict(o=st["o"], lse=st["lse"], dqkv=st["dqkv"])
    if kind == "norm_step":
        B.enc_ln_fwd(st["x"], st["gamma"], st["beta"], EPS, y=st["y"], mean=st["mean"], rstd=st["rstd"])
        B.enc_ln_bwd(st["dy"], st["x"], st["mean"], st["rstd"], st["gamma"], dresid=st["dresid"], dx=st["dx"],
                     dgamma=st["dgamma"], dbeta=st["dbeta"], ws=st["ws"])
        return {k: st[k] for k in ("y", "mean", "rstd", "dx", "dgamma", "dbeta")}
    if kind == "mlp_fwd":
        B.enc_mlp_up_fwd(st["y2"], st["w_1"], st["b_1"], u=st["u"], g=st["g"], ws=st["ws"])
        B.enc_mlp_down_fwd(st["g"], st["w_2"], st["b_2"], st["resid"], out=st["out"], ws=st["ws"])
        return {k: st[k] for k in ("u", "g", "out")}
    B.enc_qkv_bwd_data(st["dqkv"], st["w_qkv"], dy1=st["dy1"], ws=st["ws"])
    B.enc_qkv_bwd_weight(st["dqkv"], st["y1"], st["dw"], st["db"], ws=st["ws"])
    return {k: st[k] for k in ("dy1", "dw", "db")}


# ------------------------------------------------------------------ work

def _layer_work(case):
    """(forward flops, parameters, rows, hidden) of one layer on one micro-batch."""
    M, H, A, F = case["batch"] * case["seq"], case["hidden"], case["heads"] * case["head_dim"], case["mlp"]
    flops = 2 * M * (4 * H * A + 2 * H * F) + 4 * M * case["seq"] * A
    return flops, 4 * H * A + 2 * H * F + 3 * A + F + 6 * H, M, H


def work(case):
    """Inputs read once (bf16), outputs written once (bf16, fp32 gradients);
    what a forward saves for its backward is not counted.  The backward's
    products are twice the forward's."""
    kind = case["kind"]
    if kind == "norm_step":
        R, C = case["rows"], case["cols"]
        return dict(bytes=2 * R * C * 5 + 8 * R + 12 * C, flops=20 * R * C)
    if kind == "attn_step":
        M, A, S = case["batch"] * case["seq"], case["heads"] * case["head_dim"], case["seq"]
        return dict(bytes=2 * M * A * 8 + 4 * M * case["heads"], flops=12 * M * S * A)
    if kind == "mlp_fwd":
        M, H, F = case["rows"], case["hidden"], case["mlp"]
        return dict(bytes=2 * (3 * M * H + 2 * M * F + 2 * H * F + H + F), flops=4 * M * H * F)
    if kind == "qkv_bwd":
        M, H, A3 = case["rows"], case["hidden"], 3 * case["heads"] * case["head_dim"]
        return dict(bytes=2 * (M * A3 + 2 * M * H + A3 * H) + 4 * (A3 * H + A3), flops=4 * M * H * A3)
    flops, params, M, H = _layer_work(case)
    if kind == "layer_fwd":
        return dict(bytes=2 * (params + 2 * M * H), flops=flops)
    if kind == "encoder_step":
        n, px = case["layers"], 3 * case["patch"] ** 2
        pe = 2 * M * px * H
        return dict(bytes=6 * (n * params + px * H + 2 * case["seq"] * H) + 2 * (M * px + 2 * M * H),
                    flops=3 * n * flops + 2 * pe)
    n = case.get("micro", 1)
    return dict(bytes=6 * params + 2 * n * 4 * M * H, flops=3 * n * flops)


def tolerance(case):
    # About four times the largest error against the 64-bit values over the
    # listed and some drawn cases: 9.4e-3 (gradients of a ViT-22B layer), 3.7e-3,
    # 6.9e-3, 1.3e-2 (twelve layers), 2.4e-3, and bf16 rounding alone (1.7e-3 to
    # 1.9e-3) for the kinds whose outputs round once.
    return {"rel": {"layer_step": 3e-2, "layer_fwd": 1.5e-2, "parallel_step": 2.5e-2, "encoder_step": 4e-2,
                    "attn_step": 1e-2, "norm_step": 7e-3, "mlp_fwd": 8e-3, "qkv_bwd": 7e-3}[case["kind"]]}


# ------------------------------------------------------------------ 64-bit values

def _ln(x, g, b):
    mean = x.mean(1, keepdim=True)
    rstd = (((x - mean) ** 2).mean(1, keepdim=True) + EPS).rsqrt()
    return (x - mean) * rstd * g + b, mean, rstd


def _ln_bwd(dy, x, mean, rstd, g):
    xh, gh = (x - mean) * rstd, dy * g
    dx = rstd * (gh - gh.mean(1, keepdim=True) - xh * (gh * xh).mean(1, keepdim=True))
    return dx, (dy * xh).sum(0), dy.sum(0)


def _gelu(u):
    return 0.5 * u * (1 + torch.erf(u / math.sqrt(2)))


def _gelu_grad(u):
    return 0.5 * (1 + torch.erf(u / math.sqrt(2))) + u * torch.exp(-0.5 * u * u) / math.sqrt(2 * math.pi)


def _heads(t, case):
    return t.view(case["batch"], case["seq"], case["heads"], case["head_dim"]).transpose(1, 2).contiguous()


def _rows(t):
    b, h, s, d = t.shape
    return t.transpose(1, 2).reshape(b * s, h * d)


def _attn(qkv, case):
    q, k, v = (_heads(t, case) for t in qkv.chunk(3, 1))
    s = q @ k.transpose(2, 3).contiguous() / math.sqrt(case["head_dim"])
    lse = torch.logsumexp(s, -1)
    return _rows(torch.exp(s - lse[..., None]) @ v), lse


def _attn_bwd(qkv, do, case):
    q, k, v = (_heads(t, case) for t in qkv.chunk(3, 1))
    do, c = _heads(do, case), 1 / math.sqrt(case["head_dim"])
    p = torch.softmax(q @ k.transpose(2, 3).contiguous() * c, -1)
    dp = do @ v.transpose(2, 3).contiguous()
    ds = p * (dp - (dp * p).sum(-1, keepdim=True)) * c
    tr = lambda t: t.transpose(2, 3).contiguous()  # noqa: E731
    return torch.cat([_rows(ds @ k), _rows(tr(ds) @ q), _rows(tr(p) @ do)], 1)


def _fwd(case, p, x):
    y1, m1, r1 = _ln(x, p["ln1_g"], p["ln1_b"])
    qkv = y1 @ p["w_qkv"].T + p["b_qkv"]
    o, _ = _attn(qkv, case)
    h = x + o @ p["w_o"].T + p["b_o"]
    y2, m2, r2 = _ln(h, p["ln2_g"], p["ln2_b"])
    u = y2 @ p["w_1"].T + p["b_1"]
    g = _gelu(u)
    return h + g @ p["w_2"].T + p["b_2"], (y1, m1, r1, qkv, o, h, y2, m2, r2, u, g)


def _bwd(case, p, x, saved, dout):
    y1, m1, r1, qkv, o, h, y2, m2, r2, u, g = saved
    gr = dict(w_2=dout.T @ g, b_2=dout.sum(0))
    du = (dout @ p["w_2"]) * _gelu_grad(u)
    gr.update(w_1=du.T @ y2, b_1=du.sum(0))
    dh, gr["ln2_g"], gr["ln2_b"] = _ln_bwd(du @ p["w_1"], h, m2, r2, p["ln2_g"])
    dh = dh + dout
    gr.update(w_o=dh.T @ o, b_o=dh.sum(0))
    dqkv = _attn_bwd(qkv, dh @ p["w_o"], case)
    gr.update(w_qkv=dqkv.T @ y1, b_qkv=dqkv.sum(0))
    dx, gr["ln1_g"], gr["ln1_b"] = _ln_bwd(dqkv @ p["w_qkv"], x, m1, r1, p["ln1_g"])
    return dx + dh, {n: gr[n] for n in B.PARAM_ORDER}


def _qk_norm(qkv, case, p):
    A, d = case["heads"] * case["head_dim"], case["head_dim"]
    q, k, v = qkv.chunk(3, 1)
    qn, qm, qr = _ln(q.reshape(-1, d), p["qn_g"], p["qn_b"])
    kn, km, kr = _ln(k.reshape(-1, d), p["kn_g"], p["kn_b"])
    return torch.cat([qn.view(-1, A), kn.view(-1, A), v], 1), (qm, qr, km, kr)


def _parallel(case, p, x, dout):
    A, d = case["heads"] * case["head_dim"], case["head_dim"]
    y, m, r = _ln(x, p["ln_g"], p["ln_b"])
    qkv = y @ p["w_qkv"].T
    qkvn, (qm, qr, km, kr) = _qk_norm(qkv, case, p)
    o, _ = _attn(qkvn, case)
    u = y @ p["w_1"].T + p["b_1"]
    g = _gelu(u)
    out = x + o @ p["w_o"].T + p["b_o"] + g @ p["w_2"].T + p["b_2"]
    gr = dict(w_2=dout.T @ g, b_2=dout.sum(0), w_o=dout.T @ o, b_o=dout.sum(0))
    du = (dout @ p["w_2"]) * _gelu_grad(u)
    gr.update(w_1=du.T @ y, b_1=du.sum(0))
    dn = _attn_bwd(qkvn, dout @ p["w_o"], case)
    dq, qg, qb = _ln_bwd(dn[:, :A].reshape(-1, d), qkv[:, :A].reshape(-1, d), qm, qr, p["qn_g"])
    dk, kg, kb = _ln_bwd(dn[:, A:2 * A].reshape(-1, d), qkv[:, A:2 * A].reshape(-1, d), km, kr, p["kn_g"])
    dqkv = torch.cat([dq.view(-1, A), dk.view(-1, A), dn[:, 2 * A:]], 1)
    gr["w_qkv"] = dqkv.T @ y
    dx, gr["ln_g"], gr["ln_b"] = _ln_bwd(dqkv @ p["w_qkv"] + du @ p["w_1"], x, m, r, p["ln_g"])
    shapes = B.parallel_param_shapes(_cfg(case))
    return dict(out=out, dx=dx + dout, grads={n: gr[n] for n in shapes if n not in _QK},
                qk_grads=torch.stack([qg, qb, kg, kb]))


def _encoder(case, inp):
    Bn, S, H, P = case["batch"], case["seq"], case["hidden"], case["patch"]
    gw = case["img"] // P
    px = inp["images"].view(Bn, 3, gw, P, gw, P).permute(0, 2, 4, 1, 3, 5).reshape(Bn * gw * gw, -1)
    n_in = px.shape[1]
    x = (px @ inp["w_pe"][:, :n_in].T + inp["b_pe"]).view(Bn, gw * gw, H)
    if case["cls"]:
        x = torch.cat([inp["cls"].expand(Bn, 1, H), x], 1)
    x = (x + inp["pos"]).reshape(Bn * S, H)
    xs, saves = [], []
    for p in inp["layers"]:
        xs.append(x)
        x, s = _fwd(case, p, x)
        saves.append(s)
    out, m, r = _ln(x, inp["lnf_g"], inp["lnf_b"])
    dx, dg, db = _ln_bwd(inp["dout"], x, m, r, inp["lnf_g"])
    grads = []
    for p, xi, s in zip(reversed(inp["layers"]), reversed(xs), reversed(saves)):
        dx, g = _bwd(case, p, xi, s, dx)
        grads.insert(0, torch.cat([g[n].reshape(-1) for n in B.param_shapes(_cfg(case))]))
    d = dx.view(Bn, S, H)
    tok = d[:, 1:] if case["cls"] else d
    tok = tok.reshape(-1, H)
    w = torch.zeros(H, inp["w_pe"].shape[1], dtype=F64, device=tok.device)
    w[:, :n_in] = tok.T @ px
    pe = dict(w_pe=w, b_pe=tok.sum(0), pos=d.sum(0))
    if case["cls"]:
        pe["cls"] = d[:, 0].sum(0)
    return dict(out=out, grads=grads, lnf_grads=[dg, db], pe_grads=pe)


def _f64(v):
    if isinstance(v, torch.Tensor):
        return v.to(F64)
    if isinstance(v, dict):
        return {k: _f64(x) for k, x in v.items()}
    if isinstance(v, list):
        return [_f64(x) for x in v]
    return v


def exact(case, seed):
    inp = _f64(_inputs(case, seed))
    kind = case["kind"]
    if kind in ("layer_step", "layer_fwd"):
        p, outs, dxs, grads = inp["params"], [], [], None
        for i, x in enumerate(inp["x"]):
            out, saved = _fwd(case, p, x)
            outs.append(out)
            if kind == "layer_fwd":
                return dict(out=outs)
            dx, g = _bwd(case, p, x, saved, inp["dout"][i])
            del saved
            dxs.append(dx)
            grads = g if grads is None else {n: grads[n] + g[n] for n in g}
        return dict(out=outs, dx=dxs, grads=grads)
    if kind == "parallel_step":
        return _parallel(case, inp["params"], inp["x"][0], inp["dout"][0])
    if kind == "encoder_step":
        return _encoder(case, inp)
    if kind == "attn_step":
        o, lse = _attn(inp["qkv"], case)
        return dict(o=o, lse=lse, dqkv=_attn_bwd(inp["qkv"], inp["do"], case))
    if kind == "norm_step":
        y, m, r = _ln(inp["x"], inp["gamma"], inp["beta"])
        dx, dg, db = _ln_bwd(inp["dy"], inp["x"], m, r, inp["gamma"])
        return dict(y=y, mean=m[:, 0], rstd=r[:, 0], dx=dx + inp["dresid"], dgamma=dg, dbeta=db)
    if kind == "mlp_fwd":
        u = inp["y2"] @ inp["w_1"].T + inp["b_1"]
        g = _gelu(u)
        return dict(u=u, g=g, out=inp["resid"] + g @ inp["w_2"].T + inp["b_2"])
    return dict(dy1=inp["dqkv"] @ inp["w_qkv"], dw=inp["dqkv"].T @ inp["y1"], db=inp["dqkv"].sum(0))
