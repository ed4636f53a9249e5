"""The SwiGLU MLP's GEMMs with the activation in the epilogue, at sizes around their tiles' edges, against fp32 products of the same
bf16 operands.  Rounding to bf16 moves a value with significand m by up to 2^-8 / m of itself, uniformly: 2^-7 / sqrt(12) / m, 2^-9.3 of the
2-norm over many values; sums differ by a few 1e-6."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2510_27257_amd as stp
from paper_2510_27257_amd import synth
from paper_2510_27257_amd.synth import Workload
from harness import LayerOnDevice, to_dev

ROUND = 2.0 ** -9 * 1.01


@pytest.fixture(scope="module")
def ctx():
    c = stp.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def off(got, ref):
    return float((got.float() - ref).norm() / ref.norm())


# tokens, hidden, ffn: one row beyond whole tiles, contractions that end inside a K-tile in either product, less than one K-tile, outputs
# that the contraction-splitting kernel takes (the first two), with and without a gate bias
@pytest.mark.parametrize("T,h,f,bias", [(264, 640, 712, False), (8, 520, 1032, True), (1096, 520, 1096, True), (1032, 1032, 2056, False),
                                        (3000, 1032, 2744, False), (640, 64, 4104, False), (2048, 2048, 40, True), (776, 56, 4168, False),
                                        (4096, 5120, 3456, False), (520, 4096, 13064, False)])      # the last: apart
def test_mlp_unit_forward_and_input_gradient(ctx, T, h, f, bias):
    wl = Workload("mlp", h, 1, 64, f, T, 2, norm="rms", act="swiglu", has_bias=bias)
    lay = LayerOnDevice(ctx, wl, seed=1)
    x, dy = (to_dev(synth.make_activation(wl, 1, k), "bf16") for k in ("x", "dy"))
    w = {k: v.float() for k, v in lay.w_dev.items()}
    y, dz = lay.new_act(), lay.new_act()
    ctx.forward_unit(lay.desc, stp.PRE_MLP, lay.w, lay.stash[0], x_in=x)
    ctx.forward_unit(lay.desc, stp.MLP, lay.w, lay.stash[0], x_resid=x, y_out=y)
    ctx.backward_input_unit(lay.desc, stp.MLP, lay.w, lay.stash[0], dy=dy, dx=dz)
    torch.cuda.synchronize()
    z, gate, up, act, dg, du = (lay.field(k).reshape(T, -1).float() for k in ("Z_LN", "H", "HU", "G", "DH", "DHU"))
    assert off(gate, z @ w["w_fc1"] + (w["b_fc1"] if bias else 0.0)) < ROUND
    assert off(up, z @ w["w_up"]) < ROUND
    sig = torch.sigmoid(gate)
    assert off(act, gate * sig * up) < ROUND                                      # of the stored activations
    d = dy.float() @ w["w_fc2"].T
    assert off(du, d * gate * sig) < ROUND
    assert off(dg, d * up * sig * (1.0 + gate * (1.0 - sig))) < ROUND
    assert off(dz, dg @ w["w_fc1"].T + du @ w["w_up"].T) < ROUND
    # the projections apart store the same bits: which way they are launched is a question of time alone
    args = lambda b, c, bias: stp.GemmArgs(dtype=stp.BF16, M=T, N=f, K=h, A=zb.data_ptr(), lda=h, B=b.data_ptr(), ldb=f, C=c.data_ptr(), ldc=f,
                                           bias=bias, bias_scale=1.0, resid_scale=1.0)
    zb = lay.field("Z_LN")
    g1, u1, a1 = (torch.empty((T, f), dtype=torch.bfloat16, device="cuda") for _ in range(3))
    ctx.gemm(args(lay.w_dev["w_fc1"], g1, lay.w_dev["b_fc1"].data_ptr() if bias else None))
    ctx.gemm(args(lay.w_dev["w_up"], u1, None))
    ctx.swiglu_forward(stp.BF16, T * f, g1, u1, a1)
    torch.cuda.synchronize()
    for one, field in ((g1, "H"), (u1, "HU"), (a1, "G")):
        assert torch.equal(one, lay.field(field).view(T, f))
