"""The rotary embedding where the units apply it (the QKV product's epilogue, the ends of the attention backward kernels) against one
evaluated in 64 bits, at sizes around tiles' and chunks' edges and over several sequences."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2510_27257_amd as stp
from paper_2510_27257_amd import synth
from paper_2510_27257_amd.synth import Workload
from harness import LayerOnDevice, to_dev

# 2-norm of the rounding of many values to bf16 against theirs: errors uniform in half a unit either way are 2^-7 / sqrt(12) / m of a value
# with significand m in [1, 2), 2^-9.3 over all of them
ROUND = 2.0 ** -9 * 1.01


@pytest.fixture(scope="module")
def ctx():
    c = stp.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def off(got, ref):
    return float((got.double() - ref).norm() / ref.norm())


def rotate(x, seq, d, rot_heads, sign):
    """x: [T, heads * d] in 64 bits; the first rot_heads heads are rotated by their row's position."""
    T = x.shape[0]
    v = x.view(T, -1, d).clone()
    pos = (torch.arange(T, device=x.device) % seq).double()
    ang = pos[:, None] * 10000.0 ** (-2.0 * torch.arange(d // 2, device=x.device).double() / d)
    sn, cs = sign * ang.sin()[:, None], ang.cos()[:, None]
    a, b = v[:, :rot_heads, :d // 2].clone(), v[:, :rot_heads, d // 2:].clone()
    v[:, :rot_heads, :d // 2], v[:, :rot_heads, d // 2:] = a * cs - b * sn, b * cs + a * sn
    return v.view(T, -1)


# heads, kv heads, head dimension, sequence, sequences, hidden: the contraction-splitting kernel's shapes (rotated by a kernel of their own),
# sequences shorter than a strip, positions that start again inside one, half-empty tiles, long positions.  (The tiles that the rule picks here
# are 128 x 128, 128 x 256 and 256 x 256; the bitwise test of hinted blocks runs the others.)
@pytest.mark.parametrize("n,nk,d,seq,mbsz,hidden", [(2, 1, 128, 264, 1, 640), (6, 2, 64, 1000, 3, 1032), (9, 3, 64, 24, 170, 520), (5, 1, 128, 1096, 1, 264),
                                                    (10, 10, 128, 4096, 1, 5120), (14, 2, 128, 2056, 1, 128), (16, 16, 64, 520, 8, 1024),
                                                    (4, 4, 128, 8, 300, 72), (3, 3, 64, 6144, 1, 2048), (1, 1, 64, 5000, 1, 512)])
@pytest.mark.parametrize("bias", [False, True])
def test_attention_unit(ctx, n, nk, d, seq, mbsz, hidden, bias):
    wl = Workload("rope", hidden, n, d, 64, seq, 4, norm="rms", act="swiglu", rope=True, has_bias=bias, kv_heads=nk)
    lay = LayerOnDevice(ctx, wl, seed=2, mbsz=mbsz)
    T, a = seq * mbsz, n * d
    g = torch.Generator(device="cuda").manual_seed(seq + hidden)
    x, dy = (torch.randn((T, hidden), generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    y, dx = lay.new_act(), lay.new_act()
    ctx.forward_unit(lay.desc, stp.PRE_ATTN, lay.w, lay.stash[0], x_in=x)
    ctx.forward_unit(lay.desc, stp.ATTN, lay.w, lay.stash[0], x_resid=x, y_out=y)
    torch.cuda.synchronize()
    w = lay.w_dev["w_qkv"].double()
    qkv = lay.field("X_LN").view(T, hidden).double() @ w + (lay.w_dev["b_qkv"].double() if bias else 0.0)
    # one rounding, two where a kernel of its own rotates the stored product; a few 1e-6 of sums and angles
    one_kernel = -(-T // 64) * -(-w.shape[1] // 64) > 256 or hidden < 256
    got = lay.field("QKV").view(T, -1)
    assert off(got, rotate(qkv, seq, d, n + nk, 1.0)) < ROUND * (1.0 if one_kernel else 1.5)
    # backward: the call without the rotation, rotated back here, against the unit's
    ctx.backward_input_unit(lay.desc, stp.ATTN, lay.w, lay.stash[0], dy=dy, dx=dx)
    torch.cuda.synchronize()
    unit = lay.field("DQKV").view(T, -1).clone()
    plain = torch.empty_like(unit)
    ctx.attention_backward(lay.desc, lay.field("QKV"), lay.field("CTX"), lay.field("LSE"), lay.field("DCTX"), torch.empty_like(lay.field("DELTA")), plain)
    torch.cuda.synchronize()
    back = rotate(plain.double(), seq, d, n + nk, -1.0)
    for lo, hi in ((0, a), (a, a + nk * d)):                 # both sides rounded once from the same sums
        assert off(unit[:, lo:hi], back[:, lo:hi]) < 1.5 * ROUND
    assert torch.equal(unit[:, a + nk * d:], plain[:, a + nk * d:])


# the first two: products of the contraction-splitting kernel, rotated by the kernel of its own; then both head dimensions in the epilogue
@pytest.mark.parametrize("n,nk,d,seq,mbsz,hidden", [(1, 1, 64, 5000, 1, 512), (1, 1, 128, 2560, 1, 264), (6, 2, 64, 4096, 1, 640), (4, 4, 128, 4104, 2, 520)])
def test_angles(ctx, n, nk, d, seq, mbsz, hidden):
    """Both routes of the forward pass and the stand-alone call, either way, on pairs (1, 0): what comes out is the sine and the cosine.  A value near zero
    is stored to a fraction of 2^-8 of itself, so an angle that is off by more than the 1e-6 of the hardware's sine shows there."""
    wl = Workload("rope", hidden, n, d, 64, seq, 4, norm="rms", act="swiglu", rope=True, has_bias=False, kv_heads=nk)
    lay = LayerOnDevice(ctx, wl, seed=2, mbsz=mbsz)
    T, width = seq * mbsz, (n + 2 * nk) * d
    lay.field("X_LN").view(T, hidden).zero_()[:, 0] = 1.0
    pairs = torch.zeros(n + 2 * nk, d, device="cuda")
    pairs[:, :d // 2] = 1.0
    lay.w_dev["w_qkv"].zero_()[0] = pairs.flatten()
    ones = pairs.flatten().to(torch.bfloat16).expand(T, width).contiguous()
    x, y = lay.new_act().zero_(), lay.new_act()
    ctx.forward_unit(lay.desc, stp.ATTN, lay.w, lay.stash[0], x_resid=x, y_out=y)
    alone, back = ones.clone(), ones.clone()
    ctx.rope(lay.desc, alone)
    ctx.rope(lay.desc, back, inverse=True)
    torch.cuda.synchronize()
    for got, sign in ((lay.field("QKV").view(T, width), 1.0), (alone, 1.0), (back, -1.0)):
        ref = rotate(ones.double(), seq, d, n + nk, sign)
        worst = float(((got.double() - ref).abs() - 2.0 ** -8 * ref.abs()).max())
        assert worst < 4e-6, worst
