"""The one-launch kernel of short streams, several rounds of tokens between two barriers and one: the same sums in the same order."""
import pytest
import torch

import paper_2409_02097_amd as lf
from paper_2409_02097_amd import workloads as wl
from tests import parity
from tests.test_gpu_partial_counts import _launches

pytestmark = pytest.mark.gpu


# rounds of 64 tokens, four together at most (bf16 above 96 channels: two, fp16 of 160: one); keys at -20: fp16 sums them a second time
@pytest.mark.parametrize("keys", [0.0, -20.0])
@pytest.mark.parametrize("d,dtype", [(96, "bf16"), (96, "f16"), (128, "f16"), (160, "f16"), (160, "bf16")])
@pytest.mark.parametrize("N", [1, 63, 64, 65, 129, 192, 193, 256])
def test_rounds_together_and_one_by_one(N, d, dtype, keys, monkeypatch, tuning):
    """A head among few, whose workgroups have a CU each and leave others free, and the same head among more than run at once."""
    print(f"short rounds N={N} d={d} {dtype} keys={keys}", flush=True)
    monkeypatch.setenv("LINFUSION_WIDE_SHORT_HALF", "2")
    code, H = wl.DTYPE_CODE[dtype], 256 // (d // 32) + 1
    q, k, v = (t.cuda() for t in wl.make_qkv(1, H, N, d, dtype, idx=152))
    k = k + keys

    def run(heads):
        x = [t[:, :heads].contiguous() for t in (q, k, v)]
        out = torch.full_like(x[0], float("nan"))
        need = lf.linfusion_attn_workspace_bytes(1, heads, N, d, code)
        off = lf.linfusion_attn_workspace_state_offset(1, heads, N, d, code)
        ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
        call = lambda: lf.linfusion_attn_fwd_ex(*x, out, 0, 1e-6, 0, ws)
        assert _launches(call) == 1
        call()
        torch.cuda.synchronize()
        return out[:, :2].contiguous(), ws[off:off + 4 * 2 * (d * d + d)].clone()

    few, many = run(2), run(H)
    assert torch.equal(few[0].view(torch.int16), many[0].view(torch.int16)) and torch.equal(few[1], many[1])
    two = [t[:, :2].contiguous().cpu() for t in (q, k, v)]
    parity.check_all(few[0], *two, dtype, 0, 1e-6, True, f"short rounds N={N} d={d} {dtype}")
