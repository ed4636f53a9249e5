"""Every workgroup tile of the launch that forms a unit's weight gradients together, with a whole and a partly empty last K-tile:
the launch is taken (the library's own choice is asked), and its bits are those of one launch per product."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2510_27257_amd as stp
from paper_2510_27257_amd import binding as B
from paper_2510_27257_amd.synth import Workload


@pytest.fixture(scope="module")
def ctx():
    c = stp.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("seq", [512, 1000])
@pytest.mark.parametrize("tile,hidden,ffn", [((128, 128), 1032, 1032), ((128, 256), 1032, 1168), ((256, 128), 1968, 2664), ((256, 256), 1032, 2392)])
def test_set_tile(ctx, tile, hidden, ffn, seq):
    desc = stp.make_desc(Workload("w", hidden, 2, 64, ffn, seq, 1, norm="rms", act="swiglu", has_bias=False))
    ctx.ensure_workspace([desc])
    mem = torch.empty(ctx.stash_bytes(desc), dtype=torch.uint8, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(hidden + ffn + seq)

    def field(name, width):
        off, nbytes = ctx.stash_field(desc, name)
        t = mem[off:off + nbytes].view(torch.bfloat16).view(seq, width)
        t.copy_(torch.randn((seq, width), generator=g, device="cuda"))
        return t

    dy = torch.randn((seq, hidden), generator=g, device="cuda").to(torch.bfloat16)
    zln = field("Z_LN", hidden)
    products = {"w_fc2": (field("G", ffn), dy), "w_fc1": (zln, field("DH", ffn)), "w_up": (zln, field("DHU", ffn))}
    start = {k: torch.randn((x.shape[1], y.shape[1]), generator=g, device="cuda") for k, (x, y) in products.items()}
    together, apart = ({k: v.clone() for k, v in start.items()} for _ in range(2))

    def args(k, acc):
        x, y = products[k]
        return stp.GemmArgs(dtype=stp.BF16, M=x.shape[1], N=y.shape[1], K=seq, A=x.data_ptr(), lda=x.shape[1], a_trans=1, B=y.data_ptr(),
                            ldb=y.shape[1], b_trans=0, C=acc[k].data_ptr(), ldc=y.shape[1], c_f32_accum=1, bias_scale=1.0, resid_scale=1.0)

    three = (stp.GemmArgs * 3)(*[args(k, together) for k in products])
    choice = stp.lib().stp_wgrad_set_tile(C.byref(three), 3)
    assert (choice >> 16, choice & 0xffff) == tile
    ctx.backward_weight_unit(desc, B.MLP, B.Stash(base=mem.data_ptr(), bytes=mem.numel()), dy, B.WGrads(**{k: v.data_ptr() for k, v in together.items()}))
    for k in products:
        ctx.gemm(args(k, apart))
    torch.cuda.synchronize()
    for k in products:
        assert torch.equal(together[k], apart[k]), k
        assert not torch.equal(together[k], start[k])
