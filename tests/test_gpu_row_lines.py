"""Which token-major calls go to the row-piece kernels: the line of every width, from both sides."""
import ctypes

import pytest
import torch

import paper_2409_02097_amd as lf
from paper_2409_02097_amd import workloads as wl
from tests import parity

pytestmark = pytest.mark.gpu

MB = 1 << 20


def _token_major(B, H, N, d, dtype, fill=None):
    t = torch.empty((B, N, H, d), dtype=wl.TORCH_DTYPE[dtype], device="cuda")
    t = t.normal_() if fill is None else t.fill_(fill)
    return t.permute(0, 2, 1, 3)


def _knob(monkeypatch, name, value):
    if value is None:
        monkeypatch.delenv(name, raising=False)
    else:
        monkeypatch.setenv(name, value)


# (H, d, type, MB of one tensor from which the row pieces are due: forward, backward)
# (one batch; groups of eight and of four heads, heads left over (forward only); 24 heads do not fill the chip one by one)
LINES = [(8, 16, "f16", 6, 6), (8, 32, "bf16", 28, 15), (8, 40, "f16", 13, 10), (4, 40, "bf16", 18, 15), (8, 48, "f16", 21, 12),
         (8, 48, "bf16", 21, 16), (8, 56, "f16", 25, 36), (4, 56, "bf16", 25, 75), (4, 80, "bf16", 62, 110),
         (4, 24, "f16", 10, 7), (24, 32, "f16", 14, 6), (12, 40, "bf16", 18, 15), (24, 40, "f16", 11, 7),
         (24, 48, "bf16", 17, 13), (24, 56, "f16", 19, 20), (24, 80, "f16", 40, 250), (8, 80, "f16", 62, 340),
         (5, 16, "bf16", 26, None), (10, 40, "f16", 60, None), (10, 48, "bf16", 60, None), (18, 8, "f16", 8, None),
         (18, 40, "bf16", 36, None)]


@pytest.mark.parametrize("above", [False, True])
@pytest.mark.parametrize("H,d,dtype,fwd_mb,bwd_mb", LINES)
def test_row_pieces_from_their_line_up(H, d, dtype, fwd_mb, bwd_mb, above, monkeypatch, tuning):
    """Just below its line a call gives the bits of the per-head kernels, from the line on those of the row pieces; where
    the two differ they do so by the order of the sums, and the forward result is the oracle's."""
    torch.manual_seed(d)
    code = wl.DTYPE_CODE[dtype]
    forced = "3" if above else "2"
    # forward
    N = -(-fwd_mb * MB // (2 * H * d)) - (0 if above else 1)
    print(f"line H={H} d={d} {dtype} N={N} above={above}", flush=True)
    q, k, v = (_token_major(1, H, N, d, dtype) for _ in range(3))
    ws = torch.empty(lf.linfusion_attn_workspace_bytes(1, H, N, d, code), dtype=torch.uint8, device="cuda")
    outs = []
    for mode in (None, forced):
        _knob(monkeypatch, "LINFUSION_HEAD_GROUPS", mode)
        outs.append(_token_major(1, H, N, d, dtype, float("nan")))
        lf.linfusion_attn_fwd_strided(q, k, v, outs[-1], 0, 1e-6, 0, ws)
    torch.cuda.synchronize()
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))
    parity.check_all(outs[0][:, :1].contiguous().cpu(), *(t[:, :1].contiguous().cpu() for t in (q, k, v)), dtype, 0, 1e-6, True,
                     f"line d={d}")
    if bwd_mb is None:
        return
    # backward
    N = -(-bwd_mb * MB // (2 * H * d)) - (0 if above else 1)
    q, k, v, g = (_token_major(1, H, N, d, dtype) for _ in range(4))
    ws = torch.empty(lf.linfusion_attn_bwd_workspace_bytes(1, H, N, d, code), dtype=torch.uint8, device="cuda")
    got = []
    for mode in (None, forced, "2"):
        _knob(monkeypatch, "LINFUSION_BWD_ROWS", mode)
        got.append([_token_major(1, H, N, d, dtype, float("nan")) for _ in range(3)])
        lf.linfusion_attn_bwd_strided(q, k, v, g, *got[-1], 0, 1e-6, 0, ws)
    torch.cuda.synchronize()
    ulp2 = 2.0 ** -7 if dtype == "bf16" else 2.0 ** -10      # two units in the last place of the 16-bit results
    for a, b, c in zip(*got):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
        assert (a.float() - c.float()).abs().max().item() <= ulp2 * c.float().abs().max().item()


class _KernelNode(ctypes.Structure):      # hipKernelNodeParams
    _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p), ("grid", ctypes.c_uint * 3),
                ("params", ctypes.c_void_p), ("lds", ctypes.c_uint)]


def _block_sizes(call):
    """Threads per workgroup of every kernel that the call records into a graph."""
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64.so" in line)   # the one torch runs on
    hip = ctypes.CDLL(path)
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        call()
    raw, count = ctypes.c_void_p(graph.raw_cuda_graph()), ctypes.c_size_t(0)
    assert hip.hipGraphGetNodes(raw, None, ctypes.byref(count)) == 0
    nodes = (ctypes.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(raw, nodes, ctypes.byref(count)) == 0
    sizes = []
    for node in nodes:
        p = _KernelNode()
        assert hip.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
        sizes.append(p.block[0])
    return sizes


# workgroups per head with four waves and with eight on 256 compute units: 24 and 12, 8 and 4, 24 and 11; 16 and 8, 20 and 10, 32 and 16
@pytest.mark.parametrize("B,H,N,d,waves", [(2, 20, 6072, 8, 4), (3, 20, 3542, 56, 4), (8, 5, 5509, 24, 4), (4, 8, 2000, 24, 8),
                                           (3, 16, 2500, 40, 8), (4, 8, 4000, 40, 8)])
def test_waves_of_the_token_major_apply(B, H, N, d, waves):
    """Eight where the workgroups of neighbouring heads then still share an XCD, and always on contiguous tensors; the
    results have the same bits."""
    print(f"apply waves {B}x{H}x{N}x{d}", flush=True)
    tm = [_token_major(B, H, N, d, "f16") for _ in range(3)]
    dense = [t.contiguous() for t in tm]
    ws = torch.empty(lf.linfusion_attn_workspace_bytes(B, H, N, d, lf.DTYPE_F16), dtype=torch.uint8, device="cuda")
    outs = []
    for ins, expect in ((tm, waves), (dense, 8)):
        outs.append(torch.full_like(ins[0], float("nan")))
        sizes = _block_sizes(lambda: lf.linfusion_attn_fwd_strided(*ins, outs[-1], 0, 1e-6, 0, ws))
        assert sizes[-1] == 64 * expect, sizes
        lf.linfusion_attn_fwd_strided(*ins, outs[-1], 0, 1e-6, 0, ws)
    torch.cuda.synchronize()
    assert torch.equal(outs[0].contiguous().view(torch.int16), outs[1].view(torch.int16))
