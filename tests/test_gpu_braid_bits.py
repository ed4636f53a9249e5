"""A step's bits do not depend on what runs beside it: layers whose attention is cut into chunks and whose products are beyond
the contraction-splitting kernel's range, serialized (attention and weight gradients each alone on the GPU, the weight gradients
of a unit in one launch), braided, and braided with a different tile for every product."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2510_27257_amd as stp
from paper_2510_27257_amd import tune
from paper_2510_27257_amd.stage import StageOnDevice, stage_sequence
from paper_2510_27257_amd.synth import Workload


@pytest.fixture(scope="module")
def ctx():
    c = stp.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


LAYERS = {
    # the vision-encoder layer: one chunk a block; four or eight waves a workgroup is a close call
    "bidirectional_d64": Workload("v", 1024, 16, 64, 4096, 1024, 1, causal=False, has_bias=True),
    # several chunks in all three attention kernels, grouped heads, tokens no multiple of a tile
    "grouped_d128": Workload("g", 1032, 8, 128, 2064, 1104, 4, norm="rms", act="swiglu", rope=True, has_bias=False, kv_heads=2),
    # the same with rotated heads of dimension 64: every tile of the QKV product's rotating kernel, contractions that end inside a K-tile
    "rotated_d64": Workload("r", 1032, 16, 64, 2064, 1104, 4, norm="rms", act="swiglu", rope=True, has_bias=False, kv_heads=4),
    # many key blocks of one long group
    "one_kv_head": Workload("k", 520, 5, 128, 1096, 3072, 8, norm="rms", act="swiglu", rope=True, has_bias=False, kv_heads=1),
}


@pytest.mark.parametrize("name", list(LAYERS))
def test_braided_and_hinted_equal_serialized_bitwise(ctx, name):
    wl = LAYERS[name]
    shapes = list(tune.layer_gemm_shapes(wl).values())
    if name in ("grouped_d128", "rotated_d64"):      # every product takes a tile, so the hints below apply to all twelve
        assert all(-(-M // 64) * -(-N // 64) > 256 for M, N, *_ in shapes)
    stg = StageOnDevice(ctx, [wl], 3, seed=5, tuned_tiles=False)
    stg.load_inputs()
    ctx.gemm_tile_hints_clear()

    def run(streams):
        ctx.braid_reset()
        stg.zero_grads()
        for step in stage_sequence(1, 3):
            ctx.braid_step(stg.stage, step, *streams)
        torch.cuda.synchronize()
        return [t.clone() for t in [*stg.act, *stg.grad, *stg.tail_act.values(), *stg.stash_mem]] + [g.clone() for g in stg.g_dev[0].values()]

    s0 = torch.cuda.current_stream()
    serial = run((s0, s0, s0))
    streams = tuple(torch.cuda.Stream() for _ in range(3))
    try:
        for shift in range(-1, len(tune.TILES)):
            if shift >= 0:
                for i, (M, N, K, at, bt) in enumerate(shapes):
                    ctx.gemm_tile_hint(M, N, K, at, bt, *tune.TILES[(i + shift) % len(tune.TILES)])
            for i, (a, b) in enumerate(zip(serial, run(streams))):
                assert torch.equal(a, b), f"{name}, hints {shift}: tensor {i} differs from the serialized order"
    finally:
        ctx.gemm_tile_hints_clear()
