"""GPU parity where the number of partial states per head decides the route: the narrow heads' apply kernel sums up to
eight partials itself, the backward pass above width 80 packs its operands from one partial, a few or many, and the
backward pass on row pieces takes as many workgroups as there is room for partials."""
import ctypes

import pytest
import torch

import paper_2409_02097_amd as lf
from oracle import linattn_oracle as orc
from paper_2409_02097_amd import workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu


def _scratch(n):
    assert n > 0
    return torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")


def _gradients_match(outs, ins, dtype, what):
    """First and last (batch, head) slice against the oracle's gradients, rule of tests/parity.py: check_gradients."""
    stored = [wl.stored_numpy(t) for t in ins]
    B, H = stored[0].shape[:2]
    for b, h in {(0, 0), (B - 1, H - 1)}:
        w = [orc.widen(x[b, h], dtype) for x in stored]
        parity.check_gradients([parity.to_f64(t[b, h]) for t in outs], *w, dtype, 0, 1e-6, True, f"{what} b={b} h={h}")


def _launches(call):
    """How many nodes the call records into a graph: its launches."""
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64.so" in line)   # the one torch runs on
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    count = ctypes.c_size_t(0)
    assert ctypes.CDLL(path).hipGraphGetNodes(ctypes.c_void_p(graph.raw_cuda_graph()), None, ctypes.byref(count)) == 0
    return count.value


# 64 to 20001 tokens: one partial, two to eight, more
@pytest.mark.parametrize("dtype,d", [("f16", 40), ("bf16", 64), ("f16", 8), ("bf16", 80), ("f32", 40), ("f32", 64)])
@pytest.mark.parametrize("N", [64, 129, 300, 700, 1000, 2100, 20001])
def test_narrow_partials_summed_by_the_apply_kernel(N, d, dtype, monkeypatch, tuning):
    B, H = 2, 3
    print(f"narrow partials N={N} d={d} {dtype}", flush=True)
    code = wl.DTYPE_CODE[dtype]
    q, k, v = (t.cuda() for t in wl.make_qkv(B, H, N, d, dtype, idx=140))
    ws = _scratch(lf.linfusion_attn_workspace_bytes(B, H, N, d, code))
    off = lf.linfusion_attn_workspace_state_offset(B, H, N, d, code)
    parts = lf.linfusion_attn_plan(B, H, N, d, code, lf.FLAG_FORCE_SPLIT)["reduce_wgs_per_head"]
    folded = parts <= 8 and parts * (d * d + d) * 4 <= 65536
    res = []
    for fold in ("1", "2"):                     # "2": a launch of its own sums them, whatever their number
        monkeypatch.setenv("LINFUSION_FOLD", fold)
        ws.fill_(0xFF)
        out = torch.full_like(q, float("nan"))
        call = lambda: lf.linfusion_attn_fwd_ex(q, k, v, out, 0, 1e-6, lf.FLAG_FORCE_SPLIT, ws)
        call()
        torch.cuda.synchronize()
        res.append((out, ws[off:off + B * H * (d * d + d) * 4].clone()))
        assert _launches(call) == (2 if folded and fold == "1" else 3)
    parity.check_all(res[0][0], q, k, v, dtype, what=f"narrow partials {N}x{d}")
    # the same order of additions: the same bits, in the output and in the state left in the workspace
    assert torch.equal(res[0][0].view(torch.uint8), res[1][0].view(torch.uint8))
    assert torch.equal(res[0][1], res[1][1])


# partials per head with 256 compute units: 1, 2, 4, 9, 32, as the launches of longer streams take them ("2"; by length the first three
# are one launch)
@pytest.mark.parametrize("short", ["1", "2"])
@pytest.mark.parametrize("B,H,N,d", [(1, 8, 64, 160), (12, 8, 256, 160), (1, 4, 100, 96), (1, 8, 777, 160), (1, 8, 2001, 96)])
@pytest.mark.parametrize("saved", [False, True])
def test_wide_backward_partials(B, H, N, d, saved, short, monkeypatch, tuning):
    print(f"wide backward partials B={B} H={H} N={N} d={d} saved={saved} short={short}", flush=True)
    monkeypatch.setenv("LINFUSION_BWDW_SHORT", short)
    q, k, v = wl.make_qkv(B, H, N, d, "f16", idx=141, device="cpu")
    g = wl.draw((B, H, N, d), wl.BASE_SEED + 14141, "f16", "cpu")
    dev = [t.cuda() for t in (q, k, v, g)]
    state = None
    if saved:
        state = torch.empty(B * H * (d * d + d), dtype=torch.float32, device="cuda")
        lf.linfusion_attn_state(dev[1], dev[2], state, 0, _scratch(lf.linfusion_attn_workspace_bytes(B, H, N, d, lf.DTYPE_F16)))
    outs = [torch.full_like(dev[0], float("nan")) for _ in range(3)]
    lf.linfusion_attn_bwd(*dev, *outs, 0, 1e-6, 0, _scratch(lf.linfusion_attn_bwd_workspace_bytes(B, H, N, d, lf.DTYPE_F16)),
                          state=state)
    torch.cuda.synchronize()
    _gradients_match(outs, (q, k, v, g), "f16", "wide backward partials")


# groups of eight and of four heads; one group and many; whole tiles and a last row alone
@pytest.mark.parametrize("B,H,N,d,dtype", [(12, 8, 70, 40, "bf16"), (12, 8, 70, 40, "f16"), (3, 8, 513, 8, "bf16"),
                                           (1, 12, 640, 32, "bf16"), (5, 16, 33, 24, "bf16")])
def test_row_piece_backward_of_many_heads(B, H, N, d, dtype, monkeypatch, tuning):
    print(f"row-piece backward B={B} H={H} N={N} d={d} {dtype}", flush=True)
    monkeypatch.setenv("LINFUSION_BWD_ROWS", "3")
    q, k, v = wl.make_qkv(B, H, N, d, dtype, idx=142, device="cpu")
    g = wl.draw((B, H, N, d), wl.BASE_SEED + 14242, dtype, "cpu")
    tm = lambda t: t.permute(0, 2, 1, 3).contiguous().cuda().permute(0, 2, 1, 3)   # [B, N, H, d] in memory
    dev = [tm(t) for t in (q, k, v, g)]
    outs = [torch.full((B, N, H, d), float("nan"), dtype=q.dtype, device="cuda").permute(0, 2, 1, 3) for _ in range(3)]
    lf.linfusion_attn_bwd_strided(*dev, *outs, 0, 1e-6, 0,
                                  _scratch(lf.linfusion_attn_bwd_workspace_bytes(B, H, N, d, wl.DTYPE_CODE[dtype])))
    torch.cuda.synchronize()
    assert all(torch.isfinite(o).all() for o in outs)
    _gradients_match([o.contiguous() for o in outs], (q, k, v, g), dtype, "row-piece backward")


# phi'(q) in fp32 in the merged row-piece kernel as in the separate one: the same dq to the bit (both W, every map)
@pytest.mark.parametrize("H,d,fm", [(8, 40, 0), (4, 40, 0), (8, 32, 0), (8, 24, 0), (12, 16, 0), (8, 8, 0), (8, 40, 1), (8, 40, 2)])
@pytest.mark.parametrize("flags", [0, lf.FLAG_UNNORMALIZED])
def test_row_piece_dq_is_the_separate_kernels(H, d, fm, flags, monkeypatch, tuning):
    B, N, dtype = 2, 1500, "bf16"
    print(f"row-piece dq H={H} d={d} fm={fm} flags={flags}", flush=True)
    q, k, v = wl.make_qkv(B, H, N, d, dtype, idx=143, device="cpu")
    if fm == 2:
        q, k = q.abs() + 0.1, k.abs() + 0.1
    g = wl.draw((B, H, N, d), wl.BASE_SEED + 14343, dtype, "cpu")
    tm = lambda t: t.permute(0, 2, 1, 3).contiguous().cuda().permute(0, 2, 1, 3)
    dev = [tm(t) for t in (q, k, v, g)]
    ws = _scratch(lf.linfusion_attn_bwd_workspace_bytes(B, H, N, d, wl.DTYPE_CODE[dtype]))
    monkeypatch.setenv("LINFUSION_BWD_ROWS", "3")
    got = []
    for merged in ("1", "2"):
        monkeypatch.setenv("LINFUSION_BWD_MERGED", merged)
        outs = [torch.full_like(dev[0], float("nan")) for _ in range(3)]
        lf.linfusion_attn_bwd_strided(*dev, *outs, fm, 1e-6, flags, ws)
        torch.cuda.synchronize()
        got.append(outs[0].contiguous().view(torch.int16))
    assert torch.equal(got[0], got[1]), f"{(got[0] != got[1]).sum().item()} of {got[0].numel()} values differ"
