"""GPU parity of the fp32 kernels at the sizes where their tiles and launches change: tiles of 16 tokens (apply and
gradients), of 32 (state reduction) and of 64 (its two token groups at d = 8 and 24), the apply kernel that changes
above d = 24, and partial states summed by their consumers or by a launch of their own."""
import pytest
import torch

import paper_2409_02097_amd as lf
from paper_2409_02097_amd import workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu


def _forward(q, k, v, out, ws):
    lf.linfusion_attn_fwd_strided(q, k, v, out, 0, 1e-6, 0, ws)
    torch.cuda.synchronize()


def _case(B, H, N, d, tokens, what):
    q, k, v = wl.make_qkv(B, H, N, d, "f32", idx=120, device="cpu")
    g = wl.draw((B, H, N, d), wl.BASE_SEED + 120777, "f32", "cpu")
    lay = (lambda t: t.permute(0, 2, 1, 3).contiguous().cuda().permute(0, 2, 1, 3)) if tokens else (lambda t: t.cuda())
    qd, kd, vd, gd = (lay(t) for t in (q, k, v, g))
    out, dq, dk, dv = (torch.full_like(qd, float("nan")) for _ in range(4))
    ws = torch.full((lf.linfusion_attn_workspace_bytes(B, H, N, d, lf.DTYPE_F32),), 0xFF, dtype=torch.uint8, device="cuda")
    bws = torch.full((lf.linfusion_attn_bwd_workspace_bytes(B, H, N, d, lf.DTYPE_F32),), 0xFF, dtype=torch.uint8,
                     device="cuda")
    _forward(qd, kd, vd, out, ws)
    parity.check_all(out, q, k, v, "f32", what=what)
    off = lf.linfusion_attn_workspace_state_offset(B, H, N, d, lf.DTYPE_F32)
    state = ws[off:off + B * H * (d * d + d) * 4].view(torch.float32)
    grads = []
    for st in (state, None):
        for t in (dq, dk, dv):
            t.fill_(float("nan"))
        lf.linfusion_attn_bwd_strided(qd, kd, vd, gd, dq, dk, dv, 0, 1e-6, 0, bws, state=st)
        torch.cuda.synchronize()
        grads.append([t.clone() for t in (dq, dk, dv)])
    for a, b in zip(*grads):
        assert torch.equal(a, b), f"{what}: another gradient when the forward's state is handed over"
    for b in range(B):
        for h in range(H):
            ins = [t[b, h].double().numpy() for t in (q, k, v, g)]
            parity.check_gradients([parity.to_f64(t[b, h]) for t in grads[0]], *ins, "f32", 0, 1e-6, True, what)


@pytest.mark.parametrize("d", [8, 16, 24, 32, 40, 56, 64])
@pytest.mark.parametrize("N", [1, 15, 17, 33, 63, 65, 129])
def test_edges_of_the_tiles(d, N):
    print(f"f32 edges d={d} N={N}", flush=True)
    _case(1, 3, N, d, tokens=bool(N % 2 == 1 and d > 24), what=f"f32 d={d} N={N}")


# (partials per head on 256 compute units: 5 of 6.6 KB -- summed by the consumer; 32 of 16.6 KB -- by combine_state;
# d = 24: always combine_state in the forward pass)
@pytest.mark.parametrize("B,H,N,d", [(12, 8, 333, 40), (2, 2, 9001, 64), (6, 8, 500, 24), (1, 8, 70001, 40)])
def test_partials_folded_or_combined(B, H, N, d):
    print(f"f32 partials B={B} H={H} N={N} d={d}", flush=True)
    _case(B, H, N, d, tokens=False, what=f"f32 {B}x{H}x{N}x{d}")


@pytest.mark.parametrize("d", [8, 24, 40, 64])
@pytest.mark.parametrize("fm,normalize", [(1, True), (2, True), (0, False), (2, False)])
def test_other_feature_maps(d, fm, normalize):
    B, H, N = 1, 2, 91
    q, k, v = wl.make_qkv(B, H, N, d, "f32", idx=121, device="cpu")
    if fm == 2:
        q, k = q.abs() + 0.1, k.abs() + 0.1
    out = torch.full_like(q, float("nan")).cuda()
    ws = torch.empty(lf.linfusion_attn_workspace_bytes(B, H, N, d, lf.DTYPE_F32), dtype=torch.uint8, device="cuda")
    lf.linfusion_attn_fwd_ex(q.cuda(), k.cuda(), v.cuda(), out, fm, 1e-6, 0 if normalize else lf.FLAG_UNNORMALIZED, ws)
    torch.cuda.synchronize()
    parity.check_all(out, q, k, v, "f32", fm, 1e-6, normalize, what=f"f32 fm={fm} norm={normalize} d={d}")


# the largest token stride that is accepted: 64-token tiles (d = 8 and 24) reach 63 * 2^26 floats behind their first row
@pytest.mark.parametrize("d", [8, 24, 40])
def test_rows_as_far_apart_as_accepted(d):
    N, row = 67, 4 * (2 ** 24 - 1)                 # 16.5 GiB from the first to the last token, of which 67 rows are used
    print(f"f32 rows {row} floats apart, d={d}", flush=True)
    q, k, v = wl.make_qkv(1, 1, N, d, "f32", idx=122, device="cpu")
    store = torch.empty((N - 1) * row + 2 * d, dtype=torch.float32, device="cuda")
    kd, vd = (store.as_strided((1, 1, N, d), (N * row, N * row, row, 1), at) for at in (0, d))
    kd.copy_(k)
    vd.copy_(v)
    out = torch.full((1, 1, N, d), float("nan"), device="cuda")
    ws = torch.empty(lf.linfusion_attn_workspace_bytes(1, 1, N, d, lf.DTYPE_F32), dtype=torch.uint8, device="cuda")
    _forward(q.cuda(), kd, vd, out, ws)
    parity.check_all(out, q, k, v, "f32", what=f"f32 far rows d={d}")
