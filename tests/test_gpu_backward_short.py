"""GPU parity of the one-launch backward pass of short fp16 streams above 80 channels (rounds of 64 tokens, two workgroups per
head) against the fp64 oracle's gradients, and the launches it replaces beside it."""
import pytest
import torch

import paper_2409_02097_amd as lf
from paper_2409_02097_amd import workloads as wl
from tests.test_gpu_backward_composed import _check, _run
from tests.test_gpu_partial_counts import _gradients_match, _launches

pytestmark = pytest.mark.gpu


def _inputs(B, H, N, d, idx):
    q, k, v = wl.make_qkv(B, H, N, d, "f16", idx=idx, device="cpu")
    return q, k, v, wl.draw((B, H, N, d), wl.BASE_SEED + 1000 * idx + 777, "f16", "cpu")


# one token, the edges of a round, odd and even numbers of rounds; 7 and 130 heads: workgroups that are no multiple of eight and
# more than run at once; 428 / 429 tokens of 4 heads: the last stream that takes the launch and the first that does not
@pytest.mark.parametrize("d", [96, 128, 160])
@pytest.mark.parametrize("B,H,N", [(1, 1, 1), (1, 3, 63), (1, 7, 64), (1, 2, 65), (2, 2, 191), (10, 13, 40), (1, 4, 428), (1, 4, 429)])
def test_short_backward_matches_oracle(B, H, N, d):
    print(f"short bwd B={B} H={H} N={N} d={d}", flush=True)
    q, k, v, g = _inputs(B, H, N, d, 190)
    outs = _run(q, k, v, g)
    _check(outs, q, k, v, g, 0, 1e-6, True, f"short bwd N={N} d={d}")
    for a, b in zip(outs, _run(q, k, v, g)):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16)), "not run-to-run identical"


@pytest.mark.parametrize("d", [96, 160])
@pytest.mark.parametrize("case", ["rows far below zero", "rows near the top", "equal keys far below zero", "relu", "identity"])
def test_short_backward_over_the_range_of_its_operands(case, d):
    """Query rows whose phi leaves fp16's normal range (scaled into it, and the scale taken out of the other factor), and the
    other feature maps: the oracle's gradients."""
    B, H, N = 1, 2, 150
    print(f"short bwd, {case}, d={d}", flush=True)
    q, k, v, g = _inputs(B, H, N, d, 191)
    fm, eps = 0, 1e-6
    if case == "rows far below zero":
        q[:, :, ::3] = q[:, :, ::3] * 0.25 - 14.0        # phi about 1e-6
        q[:, :, 1::3] -= 6.0
        eps = 0.0
    elif case == "rows near the top":
        q[:, :, ::5] = 60000.0
        q[:, :, 1::5] *= 100.0
    elif case == "equal keys far below zero":
        k -= 12.0
        eps = 0.0
    else:
        fm = 1 if case == "relu" else 2
        if fm == 2:
            q, k = q.abs(), k.abs()
    _check(_run(q, k, v, g, fm, eps), q, k, v, g, fm, eps, True, f"short bwd, {case}, d={d}")


# with 256 compute units: one and two rounds of workgroups, and 96 channels with three, four, five, eight and more, on both sides of the line
@pytest.mark.parametrize("heads,N,d,launches", [(128, 1100, 96, 1), (128, 1101, 96, 6), (129, 1100, 160, 1), (257, 1024, 96, 1), (257, 1025, 96, 6),
                                                (385, 384, 96, 1), (400, 385, 96, 6), (513, 768, 96, 1), (640, 769, 96, 6), (641, 320, 96, 1),
                                                (1024, 321, 96, 6), (1025, 192, 96, 1), (1025, 193, 96, 6), (400, 1100, 128, 1)])
def test_the_line_between_the_launches(heads, N, d, launches):
    print(f"short bwd line heads={heads} N={N} d={d}", flush=True)
    q, k, v, g = _inputs(1, heads, N, d, 195)
    dev = [t.cuda() for t in (q, k, v, g)]
    outs = [torch.full_like(dev[0], float("nan")) for _ in range(3)]
    scratch = lambda n: torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")
    state = torch.empty(heads * (d * d + d), dtype=torch.float32, device="cuda")
    lf.linfusion_attn_state(dev[1], dev[2], state, 0, scratch(lf.linfusion_attn_workspace_bytes(1, heads, N, d, lf.DTYPE_F16)))
    ws = scratch(lf.linfusion_attn_bwd_workspace_bytes(1, heads, N, d, lf.DTYPE_F16))
    call = lambda: lf.linfusion_attn_bwd(*dev, *outs, 0, 1e-6, 0, ws, state=state)
    count = _launches(call)
    # (six, seven where more partials are summed first)
    assert (count == 1 if launches == 1 else count >= launches), f"{count} launches"
    call()
    torch.cuda.synchronize()
    _gradients_match(outs, (q, k, v, g), "f16", "short bwd line")


# large gradients, and query rows whose largest phi lies far above the row's normalizer: the same inputs to the launches of longer streams
@pytest.mark.parametrize("short_tokens", ["256", "1"])
@pytest.mark.parametrize("d", [96, 160])
@pytest.mark.parametrize("case", ["dout 1e-4", "dout 1e3", "dout 4e3", "dout 4e3, wide queries", "largest dout 2e4", "one channel of 300", "one channel of 1000",
                                  "one channel of 100 above small ones", "relu, a channel without keys"])
def test_backward_stays_finite(case, d, short_tokens, monkeypatch, tuning):
    """Query row and g / den' are rounded to fp16 each: neither may leave its range where the gradients do not."""
    B, H, N = 1, 2, 256
    print(f"bwd stays finite, {case}, d={d} short_tokens={short_tokens}", flush=True)
    monkeypatch.setenv("LINFUSION_BWDW_SHORT_TOKENS", short_tokens)
    q, k, v, g = _inputs(B, H, N, d, 194)
    fm, eps = 0, 1e-6
    if case.startswith("dout"):
        g *= float(case.split()[1].rstrip(","))
        if "wide" in case:
            q *= 2.0
    elif case == "largest dout 2e4":
        g *= 2e4 / g.abs().max().float()
    elif case == "one channel of 300":
        q[:, :, ::7, 3] = 300.0
        g *= 256.0
    elif case == "one channel of 1000":
        q[:, :, ::7, 3] = 1000.0
        g *= 1024.0
    elif case == "one channel of 100 above small ones":
        q[:] = q * 0.25 - 14.0
        q[..., 0] = 100.0
        k[..., 0] = -9.0
        g *= 0.05
    else:
        fm = 1
        q[:, :, ::7, 3] = 500.0
        k[..., 3] = -1.0
        g *= 100.0
    _check(_run(q, k, v, g, fm, eps), q, k, v, g, fm, eps, True, f"bwd stays finite, {case}, d={d}")


@pytest.mark.parametrize("N", [64, 200])
def test_short_backward_beside_the_launches_it_replaces(N, monkeypatch, tuning):
    """Contiguous and token-major, the same values: bit for bit alike; the other launches round phi(q) unscaled and sum in
    another order, so theirs agree to that (two units in the last place of the largest gradient)."""
    B, H, d = 2, 4, 128
    q, k, v, g = _inputs(B, H, N, d, 192)
    one = _run(q, k, v, g)
    tm = lambda t: t.permute(0, 2, 1, 3).contiguous().cuda().permute(0, 2, 1, 3)   # [B, N, H, d] in memory
    views = [tm(torch.full_like(q, float("nan"))) for _ in range(3)]
    ws = torch.empty(lf.linfusion_attn_bwd_workspace_bytes(B, H, N, d, lf.DTYPE_F16), dtype=torch.uint8, device="cuda")
    lf.linfusion_attn_bwd_strided(tm(q), tm(k), tm(v), tm(g), *views, 0, 1e-6, 0, ws)
    monkeypatch.setenv("LINFUSION_BWDW_SHORT_TOKENS", "1")
    for a, b, c in zip(one, views, _run(q, k, v, g)):
        assert torch.equal(a.view(torch.int16), b.contiguous().view(torch.int16)), "token-major differs from contiguous"
        assert (a.float() - c.float()).abs().max().item() <= 2.0 ** -10 * c.float().abs().max().item()


def test_short_backward_gives_nan_for_nan():
    """A query that is not a number reaches its own dq and, through the state gradient, every dk and dv of its head; other heads
    stay clear of it."""
    B, H, N, d = 1, 2, 100, 160
    q, k, v, g = _inputs(B, H, N, d, 193)
    clean = _run(q, k, v, g)
    q[0, 0, 70, 5] = float("nan")
    dq, dk, dv = _run(q, k, v, g)
    assert bool(torch.isnan(dq[0, 0, 70]).all()) and bool(torch.isnan(dk[0, 0]).all()) and bool(torch.isnan(dv[0, 0]).all())
    for a, b in zip((dq, dk, dv), clean):
        assert torch.equal(a[0, 1].view(torch.int16), b[0, 1].view(torch.int16))
    rest = torch.arange(N, device="cuda") != 70
    assert torch.equal(dq[0, 0, rest].view(torch.int16), clean[0][0, 0, rest].view(torch.int16))
