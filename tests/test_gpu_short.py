"""GPU parity of the one-launch forward call for short token streams at head widths above 80 (lf_short16.hpp)."""
import pytest
import torch

import paper_2409_02097_amd as lf
from paper_2409_02097_amd import workloads as wl
from tests import parity
from tests.test_gpu_partial_counts import _launches

pytestmark = pytest.mark.gpu


# rounds of 64 tokens (four on their way), query blocks of 16; 32 value channels per workgroup ("2") or half of the head's ("1")
@pytest.mark.parametrize("half", ["1", "2"])
@pytest.mark.parametrize("d,dtype", [(96, "f16"), (128, "bf16"), (160, "f16"), (160, "bf16")])
@pytest.mark.parametrize("N", [1, 16, 17, 64, 65, 255, 257, 512])
def test_short_streams_in_one_launch(N, d, dtype, half, monkeypatch, tuning):
    B, H = 2, 3
    print(f"short N={N} d={d} {dtype} half={half}", flush=True)
    monkeypatch.setenv("LINFUSION_WIDE_SHORT_HALF", half)
    code = wl.DTYPE_CODE[dtype]
    q, k, v = wl.make_qkv(B, H, N, d, dtype, idx=150, device="cpu")
    tm = lambda t: t.permute(0, 2, 1, 3).contiguous().cuda().permute(0, 2, 1, 3)
    need = lf.linfusion_attn_workspace_bytes(B, H, N, d, code)
    off = lf.linfusion_attn_workspace_state_offset(B, H, N, d, code)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    got = []
    for place in (lambda t: t.cuda(), tm):           # contiguous, and the token-major view of the same values
        qd, kd, vd = place(q), place(k), place(v)
        out = place(torch.full_like(q, float("nan")))
        call = lambda: lf.linfusion_attn_fwd_strided(qd, kd, vd, out, 0, 1e-6, 0, ws)
        call()
        torch.cuda.synchronize()
        got.append(out.contiguous())
    assert _launches(call) == 1
    parity.check_all(got[0], q, k, v, dtype, 0, 1e-6, True, f"short N={N} d={d} {dtype}")
    assert torch.equal(got[0].view(torch.int16), got[1].view(torch.int16)), "token-major differs from contiguous"
    # the state it leaves is the state-only call's, and the split path's up to the order of the sums
    left = lambda: ws[off:off + 4 * B * H * (d * d + d)].clone().view(torch.float32)
    state = left()
    lf.linfusion_attn_state(k.cuda(), v.cuda(), alone := torch.empty_like(state), 0, ws)
    # in place the query rows must be read before they are written: other launches, the same bits in output and state
    qd = q.cuda()
    lf.linfusion_attn_fwd_strided(qd, k.cuda(), v.cuda(), qd, 0, 1e-6, 0, ws)
    torch.cuda.synchronize()
    assert torch.equal(state, alone) and torch.equal(state, left())
    assert torch.equal(got[0].view(torch.int16), qd.view(torch.int16)), "in place differs from out of place"
    out = torch.full_like(qd, float("nan"))
    lf.linfusion_attn_fwd_strided(q.cuda(), k.cuda(), v.cuda(), out, 0, 1e-6, lf.FLAG_FORCE_SPLIT, ws)
    torch.cuda.synchronize()
    split = left()
    assert ((state - split).norm() <= 1e-6 * split.norm()).item()     # (random signs: 2^-24 sqrt(N) of the sums' terms)
    parity.check_all(out, q, k, v, dtype, 0, 1e-6, True, f"short, split path, N={N} d={d} {dtype}")


# one workgroup of the state reduction per head, or several; few heads, and more than the one launch's workgroups run at once
@pytest.mark.parametrize("keys", [0.0, -20.0])
@pytest.mark.parametrize("B,H,N,d,dtype", [(2, 8, 64, 160, "f16"), (6, 8, 65, 160, "bf16"), (20, 8, 128, 160, "f16"),
                                           (20, 8, 200, 128, "bf16"), (25, 8, 33, 96, "f16"), (40, 8, 100, 160, "bf16"),
                                           (2, 8, 400, 96, "f16")])
def test_the_state_alone_has_the_bits_of_the_calls(B, H, N, d, dtype, keys):
    """Also where keys far below zero make either kernel sum them a second time."""
    print(f"state alone {B}x{H}x{N}x{d} {dtype} keys {keys}", flush=True)
    code = wl.DTYPE_CODE[dtype]
    q, k, v = (t.cuda() for t in wl.make_qkv(B, H, N, d, dtype, idx=151))
    k = k + keys
    need = lf.linfusion_attn_workspace_bytes(B, H, N, d, code)
    off = lf.linfusion_attn_workspace_state_offset(B, H, N, d, code)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
    call = lambda: lf.linfusion_attn_fwd_ex(q, k, v, torch.empty_like(q), 0, 1e-6, 0, ws)
    assert _launches(call) == 1
    call()
    left = ws[off:off + 4 * B * H * (d * d + d)].clone().view(torch.float32)
    lf.linfusion_attn_state(k, v, alone := torch.full_like(left, float("nan")), 0, ws)
    torch.cuda.synchronize()
    assert torch.equal(left, alone)


@pytest.mark.parametrize("B,H,N,d,launches", [(2, 8, 256, 160, 1), (2, 8, 513, 160, 3), (50, 8, 128, 128, 1), (50, 8, 129, 128, 3),
                                                (50, 8, 256, 96, 3), (48, 8, 128, 96, 1), (50, 8, 128, 96, 3),
                                                (50, 8, 64, 96, 1), (50, 8, 65, 96, 3), (80, 8, 64, 96, 1), (81, 8, 64, 96, 3)])
def test_which_calls_are_short(B, H, N, d, launches):
    """512 tokens while all workgroups run at once, fewer for more heads (96 fp16 channels: no more than three rounds of
    them, or five of 64 tokens); the forced split path is never short."""
    x = torch.zeros(B, H, N, d, dtype=torch.float16, device="cuda")
    out = torch.empty_like(x)
    ws = torch.empty(lf.linfusion_attn_workspace_bytes(B, H, N, d, lf.DTYPE_F16), dtype=torch.uint8, device="cuda")
    assert _launches(lambda: lf.linfusion_attn_fwd_ex(x, x, x, out, 0, 1e-6, 0, ws)) == launches
    # ... and what the library says it runs
    plan = lf.linfusion_attn_plan(B, H, N, d, lf.DTYPE_F16)
    assert (plan["path"] == 3) == (launches == 1)
    assert lf.linfusion_attn_apply_kernel(B, H, N, d, lf.DTYPE_F16) == ("short16" if launches == 1 else "apply16_wave")
    assert lf.linfusion_attn_plan(B, H, N, d, lf.DTYPE_F16, lf.FLAG_FORCE_SPLIT)["path"] == 0
    assert _launches(lambda: lf.linfusion_attn_fwd_ex(x, x, x, out, 0, 1e-6, lf.FLAG_FORCE_SPLIT, ws)) >= 2


def _one_launch(q, k, v, dtype, fm=0, eps=1e-6, flags=0, what="", oracle_k=None):
    """The call, which must be the one launch, against the oracle."""
    B, H, N, d = q.shape
    code = wl.DTYPE_CODE[dtype]
    assert lf.linfusion_attn_plan(B, H, N, d, code, flags)["path"] == 3
    ws = torch.full((lf.linfusion_attn_workspace_bytes(B, H, N, d, code),), 0xFF, dtype=torch.uint8, device="cuda")
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    out = torch.full_like(qd, float("nan"))
    lf.linfusion_attn_fwd_ex(qd, kd, vd, out, fm, eps, flags, ws)
    torch.cuda.synchronize()
    what = f"{what} N={N} d={d} {dtype} eps={eps}"
    worst = parity.check_all(out, q, k if oracle_k is None else oracle_k, v, dtype, fm, eps, flags == 0, what)
    print(f"{what}: worst max-norm ratio {worst[0]:.2e}, rel L2 {worst[1]:.2e}", flush=True)


def _half(monkeypatch, half):
    monkeypatch.setenv("LINFUSION_WIDE_SHORT_HALF", half)


# fp16 keys whose exponentials leave fp16's normal range are summed a second time, relative to the largest key
@pytest.mark.parametrize("half", ["1", "2"])
@pytest.mark.parametrize("N", [17, 65, 257, 512])
@pytest.mark.parametrize("d", [96, 160])
@pytest.mark.parametrize("case", ["k-12", "k-20", "k-20_q-20", "some_tokens_k-25", "one_head_k-20", "k-70"])
def test_short_fp16_keys_far_below_zero(case, d, N, half, monkeypatch, tuning):
    _half(monkeypatch, half)
    q, k, v = wl.make_qkv(1, 3, N, d, "f32", idx=152, device="cpu")
    if case == "k-12":
        k = k - 12.0
    elif case in ("k-20", "k-20_q-20"):
        k = k - 20.0
    elif case == "some_tokens_k-25":
        k[:, :, ::2] -= 25.0
    elif case == "one_head_k-20":
        k[:, 1] -= 20.0
    else:
        k = k * 3.0 - 70.0
    if case == "k-20_q-20":
        q = q - 20.0
    for eps in (1e-6, 0.0):
        _one_launch(q.half(), k.half(), v.half(), "f16", eps=eps, what=f"short {case}")


# keys masked with the type's lowest value or -infinity count as nothing (phi = 0), among ordinary keys and small ones
@pytest.mark.parametrize("half", ["1", "2"])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("shift", [0.0, -20.0])
@pytest.mark.parametrize("lowest", [True, False])
@pytest.mark.parametrize("N,d", [(65, 96), (300, 160)])
def test_short_masked_keys_count_as_nothing(N, d, lowest, shift, dtype, half, monkeypatch, tuning):
    _half(monkeypatch, half)
    tt = wl.TORCH_DTYPE[dtype]
    q, k, v = (t.to(tt) for t in wl.make_qkv(2, 2, N, d, "f32", idx=153, device="cpu"))
    k = k + shift
    as_zero = k.clone()
    k[:, :, N // 2:] = torch.finfo(tt).min if lowest else float("-inf")
    as_zero[:, :, N // 2:] = -1e4
    _one_launch(q, k, v, dtype, what=f"short masked shift={shift}", oracle_k=as_zero)


@pytest.mark.parametrize("half", ["1", "2"])
@pytest.mark.parametrize("N,d,dtype", [(65, 96, "bf16"), (300, 160, "bf16"), (300, 160, "f16"), (65, 128, "f16")])
@pytest.mark.parametrize("case", ["q-20", "q-60", "some_rows_q-300", "q+3000", "q_near_the_top", "some_rows_q*1e30",
                                  "q*1e-20", "one_channel_up"])
def test_short_query_rows_of_any_magnitude(case, N, d, dtype, half, monkeypatch, tuning):
    if dtype == "f16" and case in ("some_rows_q*1e30", "q*1e-20"):
        pytest.skip("outside what fp16 storage holds")
    _half(monkeypatch, half)
    B, H = 1, 2
    q, k, v = wl.make_qkv(B, H, N, d, "f32", idx=154, device="cpu")
    if case == "q-20":
        q = q - 20.0
    elif case == "q-60":
        q = q * 3.0 - 60.0
    elif case == "some_rows_q-300":
        q[:, :, ::3] -= 300.0
    elif case == "q+3000":
        q = q * 500.0 + 3000.0
    elif case == "q_near_the_top":
        q = q * 2500.0 + 50000.0
    elif case == "some_rows_q*1e30":
        q[:, :, 1::2] *= 1e30
    elif case == "q*1e-20":
        q = q * 1e-20
    else:
        q = q - 30.0
        q[:, :, :, 7] += 25.0 + 10.0 * torch.rand(B, H, N)
    tt = wl.TORCH_DTYPE[dtype]
    q, k, v = q.to(tt), k.to(tt), v.to(tt)
    for eps in (1e-6, 0.0):
        _one_launch(q, k, v, dtype, eps=eps, what=f"short {case}")
    if case in ("q-20", "some_rows_q-300", "q+3000"):      # the un-normalized arm takes the row's factor out again
        vs = (v.float() * (1e-4 if case == "q+3000" else 0.01)).to(tt)
        _one_launch(q, k, vs, dtype, flags=lf.FLAG_UNNORMALIZED, what=f"short {case} unnormalized")


@pytest.mark.parametrize("half", ["1", "2"])
@pytest.mark.parametrize("N,d,dtype", [(17, 96, "f16"), (65, 160, "bf16"), (300, 160, "f16"), (512, 128, "bf16")])
@pytest.mark.parametrize("fm,normalize", [(1, True), (2, True), (0, False), (1, False), (2, False)])
def test_short_feature_maps_and_unnormalized(fm, normalize, N, d, dtype, half, monkeypatch, tuning):
    _half(monkeypatch, half)
    q, k, v = wl.make_qkv(1, 2, N, d, dtype, idx=155, device="cpu")
    if fm == 2:
        q, k = q.abs(), k.abs()
    if not normalize:
        v = v * 0.01          # keeps the un-normalized sums inside fp16's range
    _one_launch(q, k, v, dtype, fm, 1e-6, 0 if normalize else lf.FLAG_UNNORMALIZED, what=f"short fm={fm} norm={normalize}")
