"""The norm backward of small activations (gradient sums beside dx in one launch) and of those beyond (two launches), around the row
groups', batches' and column groups' edges and the limits between the two, rows of more than 6144 elements (512 threads each), and with dx
written over its inputs."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2510_27257_amd as stp
from paper_2510_27257_amd.synth import Workload


@pytest.fixture(scope="module")
def ctx():
    c = stp.Context(0)
    c.ensure_workspace([stp.make_desc(Workload("n", 8192, 1, 64, 8192, 1032, 1))])
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("norm", ["ln", "rms"])
@pytest.mark.parametrize("T,h", [(1, 8), (3, 264), (5, 40), (257, 1032), (512, 264), (513, 264), (704, 1032), (705, 1032), (896, 520), (897, 520), (1023, 2048), (1024, 2056), (1024, 4096), (1025, 1024), (600, 4104), (37, 6152), (1026, 8192)])
@pytest.mark.parametrize("rsum,over", [(True, None), (False, None), (True, "dy"), (True, "d_resid")])
def test_against_64_bits(ctx, T, h, norm, dtype, rsum, over):
    td, code = (torch.float32, stp.F32) if dtype == "f32" else (torch.bfloat16, stp.BF16)
    g = torch.Generator(device="cuda").manual_seed(T * h)
    x, dy, dr = (torch.randn((T, h), generator=g, device="cuda").to(td) for _ in range(3))
    gain = (1.0 + 0.1 * torch.randn(h, generator=g, device="cuda")).to(td)
    X, D, R, G = (v.double() for v in (x, dy, dr, gain))
    mean = X.mean(1, keepdim=True) if norm == "ln" else torch.zeros((T, 1), dtype=torch.float64, device="cuda")
    rstd = (((X - mean) ** 2).mean(1, keepdim=True) + 1e-5).rsqrt()
    stats = torch.cat([mean, rstd], 1).float()
    mean, rstd = stats[:, :1].double(), stats[:, 1:].double()
    xh, gd = (X - mean) * rstd, D * G
    ref = rstd * (gd - (gd.mean(1, keepdim=True) if norm == "ln" else 0.0) - xh * (gd * xh).mean(1, keepdim=True)) + R
    sums = torch.randn((3, h), generator=g, device="cuda")
    start = sums.double()
    dx = {"dy": dy, "d_resid": dr}.get(over, torch.empty_like(x))
    code_n = stp.NORM_LN if norm == "ln" else stp.NORM_RMS
    ctx.norm_backward(code, code_n, T, h, x, gain, stats, dy, dr, dx, sums[0], sums[1] if norm == "ln" else None,
                      d_resid_sum=sums[2] if rsum else None, d_resid_sum_scale=0.25)
    torch.cuda.synchronize()
    # dx: one rounding of the storage type (8 bits of significand: at most 2^-8 of a value) on top of 32-bit arithmetic (a few sums of
    # h terms); the terms may cancel, so the error is taken against what goes in
    scale = float((R.norm() ** 2 + (rstd * gd).norm() ** 2) ** 0.5)
    assert float((dx.double() - ref).norm()) < (2.0 ** -8 if dtype == "bf16" else 2.0 ** -20) * 1.05 * scale
    n = T // 64 + 64          # terms added one to the next
    for k, term in enumerate([D * xh, D if norm == "ln" else None, R * 0.25 if rsum else None]):
        want = start[k] + (term.sum(0) if term is not None else 0.0)
        bound = n * 2.0 ** -23 * ((term.abs().sum(0) if term is not None else 0.0) + start[k].abs())
        assert bool(((sums[k].double() - want).abs() <= bound).all()), f"sum {k}"
