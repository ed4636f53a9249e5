"""Infinities and NaN in the kernels that sum columns beside rows and in the SwiGLU products' epilogues: they reach what depends on them, in the
form that arithmetic gives, and nothing else (not past a ragged end, where a last row or column stands in for what is not there)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2510_27257_amd as stp
from paper_2510_27257_amd.synth import Workload
from harness import LayerOnDevice

INF, NAN = float("inf"), float("nan")


@pytest.fixture(scope="module")
def ctx():
    c = stp.Context(0)
    c.ensure_workspace([stp.make_desc(Workload("n", 8192, 1, 64, 8192, 1032, 1))])
    yield c
    torch.cuda.synchronize()
    c.close()


def same_kind(got, ref):
    """NaN where the reference has one, the same infinities, finite elsewhere"""
    got, ref = got.double(), ref.double()
    return bool(((got.isnan() == ref.isnan()) & (got.isinf() == ref.isinf()) & (~ref.isinf() | (got == ref))).all())


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("T,N", [(130, 72), (500, 264), (2050, 72)])
def test_column_sum(ctx, T, N, dtype):
    td, code = (torch.float32, stp.F32) if dtype == "f32" else (torch.bfloat16, stp.BF16)
    x = torch.randn((T, N), generator=torch.Generator(device="cuda").manual_seed(T), device="cuda").to(td)
    x[T - 1, 3], x[0, 5], x[T // 2, N - 1], x[7, 8], x[9, 8] = INF, -INF, NAN, INF, -INF
    out = torch.zeros(N, device="cuda")
    ctx.colsum(code, T, N, x, 0.5, out)
    torch.cuda.synchronize()
    assert same_kind(out, 0.5 * x.double().sum(0))


# one launch, two launches, rows of 512 threads
@pytest.mark.parametrize("T,h", [(37, 264), (500, 264), (1030, 264), (9, 6152)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("norm", ["ln", "rms"])
def test_norm_backward(ctx, T, h, dtype, norm):
    td, code = (torch.float32, stp.F32) if dtype == "f32" else (torch.bfloat16, stp.BF16)
    g = torch.Generator(device="cuda").manual_seed(T * h)
    x, dy, dr = (torch.randn((T, h), generator=g, device="cuda").to(td) for _ in range(3))
    gain = torch.ones(h, device="cuda", dtype=td)
    stats = torch.rand((T, 2), generator=g, device="cuda") + 0.5
    if norm == "rms":
        stats[:, 0] = 0.0
    dy[T - 1, 2], dr[0, 11], x[3, h - 1], dr[T - 1, h - 2] = INF, -INF, NAN, NAN
    X, D, R = x.double(), dy.double(), dr.double()
    mean, rstd = stats[:, :1].double(), stats[:, 1:].double()
    xh = (X - mean) * rstd
    ref = rstd * (D - (D.mean(1, keepdim=True) if norm == "ln" else 0.0) - xh * (D * xh).mean(1, keepdim=True)) + R
    sums, dx = torch.zeros((3, h), device="cuda"), torch.empty_like(x)
    ctx.norm_backward(code, stp.NORM_LN if norm == "ln" else stp.NORM_RMS, T, h, x, gain, stats, dy, dr, dx, sums[0], sums[1] if norm == "ln" else None,
                      d_resid_sum=sums[2], d_resid_sum_scale=0.25)
    torch.cuda.synchronize()
    assert same_kind(dx, ref)
    for got, term in ((sums[0], D * xh), (sums[1], D if norm == "ln" else 0.0 * R.nan_to_num()), (sums[2], 0.25 * R)):
        assert same_kind(got, term.sum(0))


# together (ragged rows, columns and contractions), apart
@pytest.mark.parametrize("T,h,f", [(1096, 520, 1096), (264, 264, 264)])
def test_swiglu_unit(ctx, T, h, f):
    wl = Workload("mlp", h, 1, 64, f, T, 2, norm="rms", act="swiglu", has_bias=False)
    lay = LayerOnDevice(ctx, wl, seed=1)
    g = torch.Generator(device="cuda").manual_seed(T)
    x, dy = (torch.randn((T, h), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    y, dz = lay.new_act(), lay.new_act()
    ctx.forward_unit(lay.desc, stp.PRE_MLP, lay.w, lay.stash[0], x_in=x)
    # whole rows that are not finite: the last of the activations, the first of the gradient; an infinite up activation by its weight
    lay.field("Z_LN").view(T, h)[T - 1] = NAN
    lay.w_dev["w_up"][0, f - 1] = INF
    dy[0] = NAN
    ctx.forward_unit(lay.desc, stp.MLP, lay.w, lay.stash[0], x_resid=x, y_out=y)
    ctx.backward_input_unit(lay.desc, stp.MLP, lay.w, lay.stash[0], dy=dy, dx=dz)
    torch.cuda.synchronize()
    w = {k: v.double() for k, v in lay.w_dev.items()}
    z, gate, up, act, dg, du = (lay.field(k).view(T, -1) for k in ("Z_LN", "H", "HU", "G", "DH", "DHU"))
    assert same_kind(gate, z.double() @ w["w_fc1"]) and same_kind(up, z.double() @ w["w_up"])
    G, U = gate.double(), up.double()
    sig = torch.sigmoid(G)
    assert same_kind(act, G * sig * U)
    d = dy.double() @ w["w_fc2"].T
    assert same_kind(du, d * G * sig) and same_kind(dg, d * U * sig * (1.0 + G * (1.0 - sig)))
    assert same_kind(dz, dg.double() @ w["w_fc1"].T + du.double() @ w["w_up"].T)
