"""elu(x) + 1 chosen by the sign bit: zeros of both signs, infinities and NaNs of both signs, in the bf16 kernels that do so."""
import pytest
import torch

import paper_2409_02097_amd as lf
from paper_2409_02097_amd import workloads as wl

pytestmark = pytest.mark.gpu


# the per-head kernels, the single launch, and the row-piece kernels on token-major views
@pytest.mark.parametrize("groups,layout,flags", [("2", "heads", lf.FLAG_FORCE_SPLIT), ("2", "heads", lf.FLAG_FORCE_FUSED),
                                                 ("3", "tokens", 0)])
@pytest.mark.parametrize("N,d", [(64, 40), (77, 64), (1000, 40)])
def test_values_at_the_edges(N, d, groups, layout, flags, monkeypatch, tuning):
    print(f"phi by sign N={N} d={d} {layout} groups={groups} flags={flags}", flush=True)
    monkeypatch.setenv("LINFUSION_HEAD_GROUPS", groups)
    B, H, dtype = 1, 8, "bf16"
    code = wl.DTYPE_CODE[dtype]
    q, k, v = wl.make_qkv(B, H, N, d, dtype, idx=153, device="cpu")
    inf, nan = float("inf"), float("nan")
    k[..., 0], k[..., 1], k[..., 2] = 0.0, -0.0, -inf
    k[0, 0, 3, 3], k[0, 0, 5, 4] = nan, nan                # (of head 0 alone)
    q[:, 1, 0], q[:, 1, 1] = 0.0, -0.0
    q[:, 1, 2, 0], q[:, 1, 3, d - 1], q[:, 1, 4, 1] = nan, nan, -inf
    for t, at in ((k, (0, 0, 3, 3)), (q, (0, 1, 3, d - 1))):   # (an assignment of -nan loses the sign)
        t.view(torch.int16)[at] = -64
        assert t.view(torch.int16)[at] < 0 and t[at].isnan()
    place = (lambda t: t.cuda()) if layout == "heads" else \
        (lambda t: t.permute(0, 2, 1, 3).contiguous().cuda().permute(0, 2, 1, 3))
    qd, kd, vd = place(q), place(k), place(v)
    assert kd[0, 0, 3, 3].view(torch.int16).item() == qd[0, 1, 3, d - 1].view(torch.int16).item() == -64
    out = place(torch.full_like(q, 7.0))
    ws = torch.full((lf.linfusion_attn_workspace_bytes(B, H, N, d, code),), 0xFF, dtype=torch.uint8, device="cuda")
    off = lf.linfusion_attn_workspace_state_offset(B, H, N, d, code)
    lf.linfusion_attn_fwd_strided(qd, kd, vd, out, 0, 1e-6, flags, ws)
    torch.cuda.synchronize()
    state = ws[off:off + 4 * B * H * (d * d + d)].clone().view(torch.float32).view(B * H, d * d + d).cpu().double()
    S, z = state[:, :d * d].view(B * H, d, d), state[:, d * d:]
    phi = lambda x: torch.where(x > 0, x + 1, torch.exp(x))
    p, vw = phi(k[0].double()), v[0].double()
    want, terms = p.transpose(1, 2) @ vw, p.abs().transpose(1, 2) @ vw.abs()
    assert S[0, 3:5].isnan().all() and z[0, 3:5].isnan().all()
    fine = [c for c in range(d) if c not in (3, 4)]
    for h in range(H):
        rows = fine if h == 0 else list(range(d))
        # phi(k) as two bf16 terms (2^-17), fp32 sums: 1e-5 of the sum of the terms' magnitudes
        assert ((S[h, rows] - want[h, rows]).abs() <= 1e-5 * terms[h, rows] + 1e-30).all()
        assert ((z[h, rows] - p[h].sum(0)[rows]).abs() <= 1e-5 * p[h].sum(0)[rows] + 1e-30).all()
    assert torch.equal(S[:, 0], S[:, 1]) and (S[:, 2] == 0).all() and (z[:, 2] == 0).all()
    got = out.contiguous().cpu()
    assert torch.equal(got[0, 1, 0].view(torch.int16), got[0, 1, 1].view(torch.int16))
    assert got[0, 0].isnan().all() and got[0, 1, 2:4].isnan().all()
    rest = [i for i in range(N) if i not in (2, 3)]
    r = phi(q[0, 1, rest].double())
    num, den = r @ want[1], r @ p[1].sum(0) + 1e-6
    err = (got[0, 1, rest].double() - num / den.unsqueeze(-1)).abs()
    # the output's half ulp (2^-9) and the operands' 16 bits over the sum of magnitudes
    assert (err <= 2.0 ** -8 * (num / den.unsqueeze(-1)).abs() + 1e-4 * (r @ terms[1]) / den.unsqueeze(-1)).all()
