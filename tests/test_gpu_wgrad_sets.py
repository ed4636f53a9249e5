"""The weight gradients of a unit, several products in one launch: ragged tile edges, a partly empty last K-tile, absent
accumulators, and one accumulator for two products (which then have to add to it one after the other)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2510_27257_amd as stp
from paper_2510_27257_amd import binding as B
from paper_2510_27257_amd.synth import Workload
from harness import rel_err, to_host


@pytest.fixture(scope="module")
def ctx():
    c = stp.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


# widths that leave partial tiles of every size; 1000 and 264 tokens are no multiples of a K-tile, 512 is
@pytest.mark.parametrize("hidden,ffn,heads,seq", [(2056, 1544, 9, 1000), (1032, 2744, 6, 264), (3072, 1664, 8, 512)])
@pytest.mark.parametrize("case", ["mlp", "attn", "mlp_without_fc1", "mlp_shared_accumulator"])
def test_weight_unit(ctx, hidden, ffn, heads, seq, case):
    wl = Workload("w", hidden, heads, 128, ffn, seq, 1, norm="rms", act="swiglu", has_bias=False)
    desc = stp.make_desc(wl)
    ctx.ensure_workspace([desc])
    mem = torch.empty(ctx.stash_bytes(desc), dtype=torch.uint8, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(hidden + seq)

    def field(name, width):
        off, nbytes = ctx.stash_field(desc, name)
        t = mem[off:off + nbytes].view(torch.bfloat16).view(seq, width)
        t.copy_(torch.randn((seq, width), generator=g, device="cuda"))
        return t.float()

    a, q = heads * 128, 3 * heads * 128
    dy = torch.randn((seq, hidden), generator=g, device="cuda").to(torch.bfloat16)
    if case == "attn":
        products = {"w_o": (field("CTX", a), dy.float()), "w_qkv": (field("X_LN", hidden), field("DQKV", q))}
    else:
        zln = field("Z_LN", hidden)
        products = {"w_fc2": (field("G", ffn), dy.float()), "w_fc1": (zln, field("DH", ffn)), "w_up": (zln, field("DHU", ffn))}
    if case == "mlp_without_fc1":
        del products["w_fc1"]
    out = {k: torch.full((x.shape[1], y.shape[1]), 0.5, device="cuda") for k, (x, y) in products.items()}
    ref = {k: 0.5 + x.double().t() @ y.double() for k, (x, y) in products.items()}
    if case == "mlp_shared_accumulator":
        out["w_up"] = out["w_fc1"]
        ref["w_fc1"] = ref["w_up"] = ref["w_fc1"] + ref["w_up"] - 0.5
    ctx.backward_weight_unit(desc, B.ATTN if case == "attn" else B.MLP, B.Stash(base=mem.data_ptr(), bytes=mem.numel()), dy,
                             B.WGrads(**{k: v.data_ptr() for k, v in out.items()}))
    torch.cuda.synchronize()
    for k in out:
        assert rel_err(to_host(out[k]), to_host(ref[k])) < 1e-5      # fp32 sums of exact bf16 products
