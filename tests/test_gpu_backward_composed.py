"""GPU parity of the backward pass of fp16 at head widths above 80 (the d = 160 level of the SD-v1.5 UNet and the other
widths of the wide kernels) and of fp32 at every width, against the fp64 oracle's gradients, rule of tests/parity.py:
check_gradients."""
import pytest
import torch

import paper_2409_02097_amd as lf
from oracle import linattn_oracle as orc
from paper_2409_02097_amd import workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu


def _ws(B, H, N, d, code=lf.DTYPE_F16):
    n = lf.linfusion_attn_bwd_workspace_bytes(B, H, N, d, code)
    assert n > 0
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    ws.fill_(0xFF)
    return ws


def _run(q, k, v, g, fm=0, eps=1e-6, flags=0, state=None):
    B, H, N, d = q.shape
    outs = [torch.full_like(q, float("nan")).cuda() for _ in range(3)]
    code = lf.DTYPE_F32 if q.dtype == torch.float32 else lf.DTYPE_F16
    lf.linfusion_attn_bwd(q.cuda(), k.cuda(), v.cuda(), g.cuda(), *outs, fm, eps, flags, _ws(B, H, N, d, code), state=state)
    torch.cuda.synchronize()
    return outs


def _check(outs, q, k, v, g, fm, eps, normalize, what, dtype="f16"):
    qs, ks, vs, gs = (wl.stored_numpy(t) for t in (q, k, v, g))
    B, H = qs.shape[:2]
    worst = 0.0
    for b in range(B):
        for h in range(H):
            w = [orc.widen(x[b, h], dtype) for x in (qs, ks, vs, gs)]
            got = [parity.to_f64(t[b, h]) for t in outs]
            worst = max(worst, parity.check_gradients(got, *w, dtype, fm, eps, normalize, f"{what} b={b} h={h}"))
    return worst


SHAPES = [
    # SD-v1.5 at 512 px has (2, 8, 256 / 64, 160)
    (2, 8, 256, 160), (2, 8, 64, 160), (1, 2, 1, 160), (1, 3, 33, 160), (1, 1, 4099, 160), (1, 2, 700, 96),
    (2, 2, 333, 128), (1, 2, 1, 96), (1, 1, 20011, 160),
]


# short streams in one launch ("1": by length), and all by the launches of longer ones ("2")
by_both_routes = pytest.mark.parametrize("short", ["1", "2"])


@by_both_routes
@pytest.mark.parametrize("B,H,N,d", SHAPES)
def test_wide_backward_matches_oracle(B, H, N, d, short, monkeypatch, tuning):
    print(f"wide bwd B={B} H={H} N={N} d={d} short={short}", flush=True)
    monkeypatch.setenv("LINFUSION_BWDW_SHORT", short)
    q, k, v = wl.make_qkv(B, H, N, d, "f16", idx=90, device="cpu")
    g = wl.draw((B, H, N, d), wl.BASE_SEED + 90777, "f16", "cpu")
    outs = _run(q, k, v, g)
    worst = _check(outs, q, k, v, g, 0, 1e-6, True, f"wide bwd N={N} d={d}")
    print(f"  worst error / term scale {worst:.2e}", flush=True)
    again = _run(q, k, v, g)
    for a, b in zip(outs, again):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16)), "not run-to-run identical"


@by_both_routes
@pytest.mark.parametrize("fm,normalize", [(1, True), (2, True), (0, False), (1, False)])
def test_wide_backward_other_feature_maps_and_unnormalized(fm, normalize, short, monkeypatch, tuning):
    B, H, N, d = 1, 2, 300, 160
    print(f"wide bwd fm={fm} normalize={normalize} short={short}", flush=True)
    monkeypatch.setenv("LINFUSION_BWDW_SHORT", short)
    q, k, v = wl.make_qkv(B, H, N, d, "f16", idx=91, device="cpu")
    g = wl.draw((B, H, N, d), wl.BASE_SEED + 91777, "f16", "cpu")
    if fm == 2:
        q, k = q.abs(), k.abs()
    if not normalize:
        v, g = v * 0.02, g * 0.02      # keeps the un-normalized sums inside fp16's range
    outs = _run(q, k, v, g, fm, 1e-6, 0 if normalize else lf.FLAG_UNNORMALIZED)
    _check(outs, q, k, v, g, fm, 1e-6, normalize, f"wide bwd fm={fm} norm={normalize}")


@by_both_routes
@pytest.mark.parametrize("N,d", [(515, 160), (256, 160), (33, 128), (500, 96)])   # three launches; one, all rounds and a few
def test_wide_backward_with_the_forward_state_handed_in(N, d, short, monkeypatch, tuning):
    """A forward call leaves the fp32 state in its workspace; handing it to the backward call skips the first
    reduction and must not change a bit."""
    B, H = 2, 4
    print(f"wide bwd, state handed in, N={N} d={d} short={short}", flush=True)
    monkeypatch.setenv("LINFUSION_BWDW_SHORT", short)
    q, k, v = wl.make_qkv(B, H, N, d, "f16", idx=92, device="cpu")
    g = wl.draw((B, H, N, d), wl.BASE_SEED + 92777, "f16", "cpu")
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    fws = torch.empty(lf.linfusion_attn_workspace_bytes(B, H, N, d, lf.DTYPE_F16), dtype=torch.uint8, device="cuda")
    out = torch.empty_like(qd)
    lf.linfusion_attn_fwd_ex(qd, kd, vd, out, 0, 1e-6, 0, fws)
    off = lf.linfusion_attn_workspace_state_offset(B, H, N, d, lf.DTYPE_F16)
    state = fws[off:off + B * H * (d * d + d) * 4].view(torch.float32)
    with_state = _run(q, k, v, g, state=state)
    without = _run(q, k, v, g)
    for a, b in zip(with_state, without):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    _check(with_state, q, k, v, g, 0, 1e-6, True, "wide bwd with saved state")


@by_both_routes
def test_wide_backward_token_major_views(short, monkeypatch, tuning):
    B, H, N, d = 2, 4, 300, 160
    print(f"wide bwd token-major short={short}", flush=True)
    monkeypatch.setenv("LINFUSION_BWDW_SHORT", short)
    q, k, v = wl.make_qkv(B, H, N, d, "f16", idx=93, device="cpu")
    g = wl.draw((B, H, N, d), wl.BASE_SEED + 93777, "f16", "cpu")
    tm = lambda t: t.permute(0, 2, 1, 3).contiguous().cuda().permute(0, 2, 1, 3)   # [B, N, H, d] in memory
    outs = [tm(torch.full_like(q, float("nan"))) for _ in range(3)]
    lf.linfusion_attn_bwd_strided(tm(q), tm(k), tm(v), tm(g), *outs, 0, 1e-6, 0, _ws(B, H, N, d))
    torch.cuda.synchronize()
    dense = _run(q, k, v, g)
    for a, b in zip(outs, dense):
        assert torch.equal(a.contiguous().view(torch.int16), b.view(torch.int16)), "token-major differs from contiguous"


def test_wide_backward_rejects_bf16():
    x = torch.zeros(1, 1, 64, 160, dtype=torch.bfloat16, device="cuda")
    assert lf.linfusion_attn_bwd_workspace_bytes(1, 1, 64, 160, lf.DTYPE_BF16) == 0
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    assert lf.linfusion_attn_bwd(x, x, x, x, *[torch.empty_like(x) for _ in range(3)], 0, 1e-6, 0, ws, check=False) == -2


F32_SHAPES = [
    # SD-v1.5 at 256 px in fp32 is (2, 8, 1024, 40)
    (2, 8, 1024, 40), (1, 2, 1, 40), (2, 3, 33, 40), (1, 1, 4099, 64), (1, 2, 300, 8), (1, 2, 515, 24), (1, 2, 300, 16),
    (1, 2, 300, 32), (1, 1, 200, 48), (1, 1, 130, 56), (1, 2, 20011, 40),
]


@pytest.mark.parametrize("B,H,N,d", F32_SHAPES)
def test_fp32_backward_matches_oracle(B, H, N, d):
    print(f"fp32 bwd B={B} H={H} N={N} d={d}", flush=True)
    q, k, v = wl.make_qkv(B, H, N, d, "f32", idx=94, device="cpu")
    g = wl.draw((B, H, N, d), wl.BASE_SEED + 94777, "f32", "cpu")
    outs = _run(q, k, v, g)
    worst = _check(outs, q, k, v, g, 0, 1e-6, True, f"fp32 bwd N={N} d={d}", "f32")
    print(f"  worst error / term scale {worst:.2e}", flush=True)
    again = _run(q, k, v, g)
    for a, b in zip(outs, again):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32)), "not run-to-run identical"


@pytest.mark.parametrize("fm,normalize", [(1, True), (2, True), (0, False), (1, False)])
def test_fp32_backward_other_feature_maps_and_unnormalized(fm, normalize):
    B, H, N, d = 1, 2, 500, 40
    q, k, v = wl.make_qkv(B, H, N, d, "f32", idx=95, device="cpu")
    g = wl.draw((B, H, N, d), wl.BASE_SEED + 95777, "f32", "cpu")
    if fm == 2:
        q, k = q.abs(), k.abs()
    outs = _run(q, k, v, g, fm, 1e-6, 0 if normalize else lf.FLAG_UNNORMALIZED)
    _check(outs, q, k, v, g, fm, 1e-6, normalize, f"fp32 bwd fm={fm} norm={normalize}", "f32")


# narrow heads: a wave's one tile and several, one partial state, a few and the finished state
@pytest.mark.parametrize("d", [8, 16, 24])
@pytest.mark.parametrize("B,H,N", [(1, 1, 1), (12, 8, 300), (2, 3, 1100), (1, 1, 20011)])
def test_fp32_backward_of_narrow_heads(B, H, N, d):
    print(f"fp32 bwd, narrow, B={B} H={H} N={N} d={d}", flush=True)
    q, k, v = wl.make_qkv(B, H, N, d, "f32", idx=97, device="cpu")
    g = wl.draw((B, H, N, d), wl.BASE_SEED + 97777, "f32", "cpu")
    st = torch.full((B, H, d * d + d), float("nan"), dtype=torch.float32, device="cuda")
    fws = torch.empty(lf.linfusion_attn_workspace_bytes(B, H, N, d, lf.DTYPE_F32), dtype=torch.uint8, device="cuda")
    lf.linfusion_attn_state(k.cuda(), v.cuda(), st, 0, fws)
    for state in (None, st):
        _check(_run(q, k, v, g, state=state), q, k, v, g, 0, 1e-6, True, f"fp32 bwd, narrow, N={N} d={d}", "f32")


def test_fp32_backward_token_major_views_and_saved_state():
    B, H, N, d = 2, 4, 300, 40
    q, k, v = wl.make_qkv(B, H, N, d, "f32", idx=96, device="cpu")
    g = wl.draw((B, H, N, d), wl.BASE_SEED + 96777, "f32", "cpu")
    tm = lambda t: t.permute(0, 2, 1, 3).contiguous().cuda().permute(0, 2, 1, 3)   # [B, N, H, d] in memory
    outs = [tm(torch.full_like(q, float("nan"))) for _ in range(3)]
    lf.linfusion_attn_bwd_strided(tm(q), tm(k), tm(v), tm(g), *outs, 0, 1e-6, 0, _ws(B, H, N, d, lf.DTYPE_F32))
    torch.cuda.synchronize()
    dense = _run(q, k, v, g)
    for a, b in zip(outs, dense):
        assert torch.equal(a.contiguous().view(torch.int32), b.view(torch.int32)), "token-major differs from contiguous"
    st = torch.full((B, H, d * d + d), float("nan"), dtype=torch.float32, device="cuda")
    fws = torch.empty(lf.linfusion_attn_workspace_bytes(B, H, N, d, lf.DTYPE_F32), dtype=torch.uint8, device="cuda")
    lf.linfusion_attn_state(k.cuda(), v.cuda(), st, 0, fws)
    with_state = _run(q, k, v, g, state=st)
    _check(with_state, q, k, v, g, 0, 1e-6, True, "fp32 bwd with saved state", "f32")
