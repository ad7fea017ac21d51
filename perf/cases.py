"""The work that a user of the token mixer has it do, as cases that can be timed and compared.

Three kinds of call, through the public binding, with every buffer owned by the caller and kept between calls as a
program that runs a UNet would keep it:

  fwd     out = mixer(q, k, v).  layout "heads": contiguous [B, H, N, d] tensors (linfusion_attn_fwd_ex);
          "tokens": views of the UNet's token-major [B, N, H*d] activations (linfusion_attn_fwd_strided).
  mlp     the mixer fed by the two-branch MLPs: the five branch results are column blocks of one projection
          [B, N, 5*H*d] (linfusion_attn_fwd_mlp_strided).
  train   one step of a distillation run through the layer: the forward call, then the backward call, which takes the
          state that the forward call left in its workspace; returns out, dq, dk, dv.

q, k, v, dout and the linear branches are N(0, 1), the second branches' Linear results N(0.5, 1.5^2), the affine
vectors N(1, 0.25^2) and N(0, 0.5^2): what normalised activations through trained projections look like, and the draw
that this repository's workloads use.
"""
import math

import torch

import paper_2409_02097_amd as lf

EPS = 1e-6
LN_EPS, SLOPE = 1e-5, 0.01
TORCH_DTYPE = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
CODE = {"f32": lf.DTYPE_F32, "f16": lf.DTYPE_F16, "bf16": lf.DTYPE_BF16}
ITEMSIZE = {"f32": 4, "f16": 2, "bf16": 2}


def _case(name, kind, layout, B, H, N, d, dtype):
    return {"name": name, "kind": kind, "layout": layout, "B": B, "H": H, "N": N, "d": d, "dtype": dtype}


def listed():
    return [
        # SD-v1.5 at 512 px, a classifier-free-guidance pair: the innermost level (16 x 16 tokens of 8 x 160 channels)
        # and the outermost (64 x 64 of 8 x 40).  Such a call runs hundreds of times per image; latency is all of it.
        _case("sd15_512_d160_f16", "fwd", "heads", 2, 8, 16 * 16, 160, "f16"),
        _case("sd15_512_f16", "fwd", "heads", 2, 8, 64 * 64, 40, "f16"),
        # SD-v2.1 at 768 px in the layout its projections write
        _case("sd21_768_tokens_f16", "fwd", "tokens", 2, 5, 96 * 96, 64, "f16"),
        # SD-XL at 2048 px in the type it is run in, and in fp32 as it is run where 16 bits overflow
        _case("sdxl_2048_bf16", "fwd", "heads", 2, 10, 128 * 128, 64, "bf16"),
        _case("sdxl_2048_f32", "fwd", "heads", 2, 10, 128 * 128, 64, "f32"),
        # SD-v1.5's outermost level on an image of odd size (211 x 173 latent tokens: no whole tile, no whole split)
        _case("sd15_ragged_tokens_bf16", "fwd", "tokens", 2, 8, 211 * 173, 40, "bf16"),
        # the 16384 x 8192 image: 2048 x 1024 latent tokens at the outermost level, 512 x 256 at the innermost
        _case("sd15_16k_f16", "fwd", "heads", 1, 8, 2048 * 1024, 40, "f16"),
        _case("sd15_16k_d160_tokens_bf16", "fwd", "tokens", 1, 8, 512 * 256, 160, "bf16"),
        # the layer as the paper builds it, queries and keys from the two-branch MLPs, at SD-XL's size
        _case("mlp_sdxl_2048_bf16", "mlp", "tokens", 2, 10, 128 * 128, 64, "bf16"),
        # distillation at 512 px: 96 images over 8 GPUs.  Outermost level in bf16, innermost in fp16, and the
        # outermost in fp32 (training without mixed precision)
        _case("train_sd15_512_bf16", "train", "tokens", 12, 8, 64 * 64, 40, "bf16"),
        _case("train_sd15_512_d160_f16", "train", "heads", 12, 8, 16 * 16, 160, "f16"),
        _case("train_sd15_512_f32", "train", "heads", 12, 8, 64 * 64, 40, "f32"),
    ]


NARROW = (8, 16, 24, 32, 40, 40, 40, 48, 56, 64, 64, 64)
WIDE = (80, 80, 96, 128, 160, 160)


def draw(rng):
    kind = rng.choice(("fwd", "fwd", "fwd", "fwd", "mlp", "train", "train"))
    dtype = rng.choice(("f16", "f16", "bf16", "bf16", "f32")) if kind != "mlp" else rng.choice(("f16", "bf16"))
    if dtype == "f32":
        widths = NARROW
    elif kind == "train" and dtype == "bf16":
        widths = NARROW + (80, 80)
    else:
        widths = NARROW + WIDE
    d = rng.choice(widths)
    H = rng.choice((4, 5, 8, 8, 8, 10, 10, 16, 20))
    B = rng.choice((1, 2, 4, 6, 12)) if kind == "train" else rng.choice((1, 1, 2, 2, 3, 4))
    # tokens: from 8 x 8 latents up to what keeps the call below the largest listed one
    most = {"fwd": 400e6 if dtype != "f32" else 60e6, "mlp": 60e6,
            "train": 30e6 if d <= 80 and dtype != "f32" else 12e6}[kind]
    top = max(128.0, most / (B * H * d))
    N = int(math.exp(rng.uniform(math.log(64), math.log(top))))
    N = max(1, N - N % 32 if rng.random() < 0.4 else N)
    layout = "tokens" if kind == "mlp" else rng.choice(("heads", "tokens"))
    return {"kind": kind, "layout": layout, "B": B, "H": H, "N": N, "d": d, "dtype": dtype}


def _dims(case):
    return case["B"], case["H"], case["N"], case["d"], case["dtype"]


def _normal(shape, gen, dtype):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(TORCH_DTYPE[dtype])


def _tensor(case, gen):
    """One tensor of the case as a [B, H, N, d] view of its storage."""
    B, H, N, d, dtype = _dims(case)
    if case["layout"] == "heads":
        return _normal((B, H, N, d), gen, dtype)
    return _normal((B, N, H * d), gen, dtype).view(B, N, H, d).permute(0, 2, 1, 3)


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    B, H, N, d, dtype = _dims(case)
    if case["kind"] == "mlp":
        C = H * d
        x = torch.randn((B, N, 5 * C), generator=gen, device="cuda", dtype=torch.float32)   # a_q, t_q, a_k, t_k, v
        for i in (1, 3):
            x[..., i * C:(i + 1) * C].mul_(1.5).add_(0.5)
        vec = lambda scale, shift: torch.randn(C, generator=gen, device="cuda") * scale + shift
        return {"x": x.to(TORCH_DTYPE[dtype]), "gamma_q": vec(0.25, 1.0), "beta_q": vec(0.5, 0.0),
                "gamma_k": vec(0.25, 1.0), "beta_k": vec(0.5, 0.0)}
    names = ("q", "k", "v", "dout") if case["kind"] == "train" else ("q", "k", "v")
    return {name: _tensor(case, gen) for name in names}


def _bytes(n):
    return torch.empty(n, dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    B, H, N, d, dtype = _dims(case)
    state = dict(_inputs(case, seed), kind=case["kind"], layout=case["layout"], H=H)
    code = CODE[dtype]
    if case["kind"] == "mlp":
        C = H * d
        state["branches"] = [state["x"][..., i * C:(i + 1) * C] for i in range(5)]
        state["out"] = torch.empty((B, N, C), dtype=TORCH_DTYPE[dtype], device="cuda")
        state["workspace"] = _bytes(lf.linfusion_attn_mlp_workspace_bytes(B, H, N, d, code))
        return state
    state["out"] = torch.empty_like(state["q"])
    state["workspace"] = _bytes(lf.linfusion_attn_workspace_bytes(B, H, N, d, code))
    if case["kind"] == "train":
        for name, like in (("dq", "q"), ("dk", "k"), ("dv", "v")):
            state[name] = torch.empty_like(state[like])
        state["bwd_workspace"] = _bytes(lf.linfusion_attn_bwd_workspace_bytes(B, H, N, d, code))
        at = lf.linfusion_attn_workspace_state_offset(B, H, N, d, code)
        size = 4 * B * H * (d * d + d)
        state["saved"] = state["workspace"][at:at + size].view(torch.float32)
    return state


def run(state):
    s = state
    if s["kind"] == "mlp":
        a_q, t_q, a_k, t_k, v = s["branches"]
        lf.linfusion_attn_fwd_mlp_strided(a_q, t_q, a_k, t_k, v, s["out"], s["gamma_q"], s["beta_q"], s["gamma_k"],
                                          s["beta_k"], s["H"], eps=EPS, ln_eps=LN_EPS, slope=SLOPE,
                                          workspace=s["workspace"])
        return s["out"]
    heads = s["layout"] == "heads"
    forward = lf.linfusion_attn_fwd_ex if heads else lf.linfusion_attn_fwd_strided
    forward(s["q"], s["k"], s["v"], s["out"], eps=EPS, workspace=s["workspace"])
    if s["kind"] == "fwd":
        return s["out"]
    backward = lf.linfusion_attn_bwd if heads else lf.linfusion_attn_bwd_strided
    backward(s["q"], s["k"], s["v"], s["dout"], s["dq"], s["dk"], s["dv"], eps=EPS, workspace=s["bwd_workspace"],
             state=s["saved"])
    return {name: s[name] for name in ("out", "dq", "dk", "dv")}


def work(case):
    B, H, N, d, dtype = _dims(case)
    elements = B * H * N * d
    # tensors that come in or go out once; matrix products of 2 d operations per element: S and out forward;
    # S dout, dS, dS v and dS^T phi(k) backward
    tensors, products = {"fwd": (4, 2), "mlp": (6, 2), "train": (8, 6)}[case["kind"]]
    return {"bytes": tensors * elements * ITEMSIZE[dtype], "flops": products * 2 * d * elements}


def tolerance(case):
    # Relative error of one path against 64 bits, measured over the listed cases and draws: fp16 outputs 2.3e-4 to
    # 3e-4 and gradients up to 6e-4 (operands and results rounded once to 11 bits), bf16 1.7e-3 (the result's own
    # rounding to 8 bits), fp32 2e-7 to 4e-7 and gradients up to 2e-6 (cancelling sums).  Four times that.
    return {"f16": {"rel": 2.4e-3}, "bf16": {"rel": 6.8e-3}, "f32": {"rel": 1e-5}}[case["dtype"]]


def _phi(x):
    return torch.where(x > 0, x + 1, torch.exp(x))


def _mixer(q, k, v):
    r, p = _phi(q), _phi(k)
    return (r @ (p.transpose(-1, -2) @ v)) / (r @ p.sum(dim=-2).unsqueeze(-1) + EPS)


def exact(case, seed):
    """What run() returns, in 64 bits, one head at a time."""
    B, H, N, d, _ = _dims(case)
    x = _inputs(case, seed)
    wide = lambda t: t.to(torch.float64)
    if case["kind"] == "mlp":
        C = H * d
        a_q, t_q, a_k, t_k, v = (wide(x["x"][..., i * C:(i + 1) * C]) for i in range(5))
        formed = []
        for a, t, g, b in ((a_q, t_q, "gamma_q", "beta_q"), (a_k, t_k, "gamma_k", "beta_k")):
            y = torch.nn.functional.layer_norm(t, (C,), wide(x[g]), wide(x[b]), LN_EPS)
            formed.append(a + torch.nn.functional.leaky_relu(y, SLOPE))
        q, k, v = (t.view(B, N, H, d) for t in (*formed, v))
        out = torch.empty((B, N, H, d), dtype=torch.float64, device="cuda")
        for b in range(B):
            for h in range(H):
                out[b, :, h] = _mixer(q[b, :, h], k[b, :, h], v[b, :, h])
        return out.view(B, N, C)
    names = ("out", "dq", "dk", "dv") if case["kind"] == "train" else ("out",)
    got = {name: torch.empty((B, H, N, d), dtype=torch.float64, device="cuda") for name in names}
    for b in range(B):
        for h in range(H):
            q, k, v = (wide(x[name][b, h]) for name in ("q", "k", "v"))
            if case["kind"] == "train":
                leaves = [t.clone().requires_grad_() for t in (q, k, v)]
                out = _mixer(*leaves)
                grads = torch.autograd.grad(out, leaves, wide(x["dout"][b, h]))
                for name, value in zip(names, (out.detach(), *grads)):
                    got[name][b, h] = value
            else:
                got["out"][b, h] = _mixer(q, k, v)
    return got if case["kind"] == "train" else got["out"]
