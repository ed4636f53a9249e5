"""The braided block on the GPU: same bits as the serialized order, parity with the oracle over a
multi-layer, multi-microbatch stage sequence, boundary callbacks, W-before-B rejection."""
import ctypes as C

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2510_27257_amd as stp
from paper_2510_27257_amd import synth
from paper_2510_27257_amd.binding import Op, OP_F, OP_B, OP_W, OP_BW, PRE_ATTN, ATTN, PRE_MLP, MLP
from paper_2510_27257_amd.stage import StageOnDevice, stage_sequence, braid, forward_ops, backward_ops
from paper_2510_27257_amd.synth import Workload
from oracle import stp_oracle as O
from harness import TOL, oracle_cfg, oracle_layer_pass, rel_err, to_host, to_dev


def to_dev_like(x, wl):
    return to_dev(x, wl.dtype)


@pytest.fixture(scope="module")
def ctx():
    c = stp.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def run_sequence(ctx, stg, streams):
    ctx.braid_reset()
    stg.zero_grads()
    for step in stage_sequence(len(stg.layers), stg.n_mb):
        ctx.braid_step(stg.stage, step, *streams)
    torch.cuda.synchronize()


def snapshot(stg):
    out = [t.clone() for t in stg.act] + [t.clone() for t in stg.grad] + [t.clone() for t in stg.tail_act.values()]
    for gd in stg.g_dev:
        out += [gd[k].clone() for k in sorted(gd)]
    return out


STAGES = {
    "tiny_fp32_x2": ([synth.WORKLOADS["tiny"]] * 2, 4),
    "gpt_bf16_x2": ([Workload("g", 512, 2, 128, 1024, 264, 8)] * 2, 5),
    "llama_bf16_x1": ([Workload("l", 384, 3, 64, 520, 136, 4, norm="rms", act="swiglu", rope=True, has_bias=False)], 4),
}


@pytest.mark.parametrize("name", list(STAGES))
def test_braided_equals_serialized_bitwise_and_matches_oracle(ctx, name):
    layers, n_mb = STAGES[name]
    stg = StageOnDevice(ctx, layers, n_mb, seed=2)
    stg.load_inputs()
    s0 = torch.cuda.current_stream()
    run_sequence(ctx, stg, (s0, s0, s0))
    serial = snapshot(stg)
    sF, sB, sW = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
    for rep in range(4):
        run_sequence(ctx, stg, (sF, sB, sW))
        for a, b in zip(serial, snapshot(stg)):
            assert torch.equal(a, b), f"{name}: braided run {rep} differs from the serialized order"
    # oracle: chain the layers with identity at the AR points, accumulate weight grads over microbatches
    L = len(layers)
    tol = TOL[layers[0].dtype]
    g_ref = [dict() for _ in range(L)]
    for mb in range(n_mb):
        xs = [synth.make_activation(layers[0], 2, f"x.mb{mb}").astype(np.float64)]
        stashes = []
        for l in range(L):
            cfg, W = oracle_cfg(layers[l]), {k: v.astype(np.float64) for k, v in stg.w_host[l].items()}
            st = {}
            O.forward_unit(cfg, O.PRE_ATTN, W, st, x_in=xs[-1])
            xa = O.forward_unit(cfg, O.ATTN, W, st, x_resid=xs[-1])
            O.forward_unit(cfg, O.PRE_MLP, W, st, x_in=xa)
            xs.append(O.forward_unit(cfg, O.MLP, W, st, x_resid=xa))
            stashes.append(st)
        assert rel_err(to_host(stg.act_slot(L, mb)), xs[-1]) < tol
        dy = synth.make_activation(layers[-1], 2, f"dy.mb{mb}").astype(np.float64)
        for l in reversed(range(L)):
            cfg, W = oracle_cfg(layers[l]), {k: v.astype(np.float64) for k, v in stg.w_host[l].items()}
            st = stashes[l]
            dz = O.backward_input_unit(cfg, O.MLP, W, st, dy)
            dxa = O.backward_input_unit(cfg, O.PRE_MLP, W, st, dz, d_resid=dy, grads=g_ref[l])
            dxl = O.backward_input_unit(cfg, O.ATTN, W, st, dxa)
            dx = O.backward_input_unit(cfg, O.PRE_ATTN, W, st, dxl, d_resid=dxa, grads=g_ref[l])
            O.backward_weight_unit(cfg, O.MLP, st, dy, g_ref[l])
            O.backward_weight_unit(cfg, O.ATTN, st, dxa, g_ref[l])
            dy = dx
        assert rel_err(to_host(stg.grad_slot(0, mb)), dy) < tol
    for l in range(L):
        for k, r in g_ref[l].items():
            assert rel_err(to_host(stg.g_dev[l][k]), r) < tol, (l, k)


@pytest.mark.parametrize("name", ["gpt_bf16_x2", "llama_bf16_x1"])
def test_repeated_blocks_overlap_only_where_data_allows(ctx, name):
    """The same block, F of the last microbatch braided with the full backward of microbatch 0, issued eight times
    in a row without a synchronisation: a block's streams wait for the previous block only where they read or
    overwrite its data (here the backward stream overwrites what the previous block's weight-gradient stream
    reads), so blocks overlap at their edges.  Outputs, stashes and the eight-fold accumulated weight gradients
    must equal the serialized run's bit for bit."""
    from paper_2510_27257_amd.binding import OP_BW
    from paper_2510_27257_amd.stage import backward_ops, braid, forward_ops
    layers, n_mb = STAGES[name]
    L = len(layers)
    stg = StageOnDevice(ctx, layers, n_mb, seed=7)
    stg.load_inputs()
    s0 = torch.cuda.current_stream()
    block = braid(forward_ops(L, n_mb - 1), backward_ops(L, 0, OP_BW))

    def run(streams):
        torch.cuda.synchronize()
        ctx.braid_reset()
        stg.zero_grads()
        ctx.braid_step(stg.stage, forward_ops(L, 0), s0, s0, s0)
        torch.cuda.synchronize()
        for _ in range(8):
            ctx.braid_step(stg.stage, block, *streams)
        torch.cuda.synchronize()
        return snapshot(stg) + [m.clone() for m in stg.stash_mem]

    serial = run((s0, s0, s0))
    streams = tuple(torch.cuda.Stream() for _ in range(3))
    for rep in range(3):
        for u, v in zip(serial, run(streams)):
            assert torch.equal(u, v), f"{name}: run {rep} of overlapping blocks differs from the serialized order"


def test_tile_hints_change_the_time_of_a_block_never_its_bits(ctx):
    """stp_gemm_tile_hint: a preference for every GEMM shape of the stage's layers, a different tile each, applies
    to the launches of concurrent streams only; the braided run still equals the serialized one bit for bit
    (every element of a product is summed over K in the same order whatever the tile).  Bad tiles are statuses."""
    from paper_2510_27257_amd import tune
    layers, n_mb = STAGES["gpt_bf16_x2"]
    stg = StageOnDevice(ctx, layers, n_mb, seed=2, tuned_tiles=False)
    stg.load_inputs()
    s0 = torch.cuda.current_stream()
    ctx.gemm_tile_hints_clear()
    run_sequence(ctx, stg, (s0, s0, s0))
    serial = snapshot(stg)
    streams = tuple(torch.cuda.Stream() for _ in range(3))
    try:
        for i, (M, N, K, at, bt) in enumerate(tune.layer_gemm_shapes(layers[0]).values()):
            ctx.gemm_tile_hint(M, N, K, at, bt, *tune.TILES[i % len(tune.TILES)])
        run_sequence(ctx, stg, streams)
        for u, v in zip(serial, snapshot(stg)):
            assert torch.equal(u, v)
        for bad in [(64, 128), (128, 0), (192, 128), (256, 512)]:
            with pytest.raises(stp.StpError) as e:
                ctx.gemm_tile_hint(512, 512, 512, 0, 0, *bad)
            assert e.value.status == 1
        with pytest.raises(stp.StpError) as e:
            ctx.gemm_tile_hint(512, 512, 512, 1, 0, 192, 256)      # the 192-row tile needs a k-contiguous A
        assert e.value.status == 1
        with pytest.raises(stp.StpError) as e:
            ctx.gemm_tile_hint(0, 512, 512, 0, 0, 128, 128)
        assert e.value.status == 2
        ctx.gemm_tile_hint(512, 512, 512, 0, 0, 192, 256)
        ctx.gemm_tile_hint(512, 512, 512, 0, 0, 0, 0)              # forgotten again
    finally:
        ctx.gemm_tile_hints_clear()


def test_streams_may_change_between_steps_without_a_synchronisation(ctx):
    """A step joins the previous one whichever streams that one ran on: alternating between three streams, another
    set of three and a single stream from step to step, with no synchronisation in between, gives the serialized
    run's bits."""
    layers, n_mb = STAGES["gpt_bf16_x2"]
    stg = StageOnDevice(ctx, layers, n_mb, seed=2)
    stg.load_inputs()
    s0 = torch.cuda.current_stream()
    run_sequence(ctx, stg, (s0, s0, s0))
    serial = snapshot(stg)
    a = tuple(torch.cuda.Stream() for _ in range(3))
    b = tuple(torch.cuda.Stream() for _ in range(3))
    c = torch.cuda.Stream()
    choices = [a, (c, c, c), b, (s0, s0, s0), (b[2], b[0], a[1])]
    for rep in range(2):
        torch.cuda.synchronize()
        ctx.braid_reset()
        stg.zero_grads()
        torch.cuda.synchronize()
        for i, step in enumerate(stage_sequence(len(stg.layers), stg.n_mb)):
            ctx.braid_step(stg.stage, step, *choices[(i + rep) % len(choices)])
        torch.cuda.synchronize()
        for u, v in zip(serial, snapshot(stg)):
            assert torch.equal(u, v), f"run {rep} with changing streams differs from the serialized order"


def test_boundary_callback_sees_every_all_reduce_point(ctx):
    stg = StageOnDevice(ctx, [synth.WORKLOADS["tiny"]] * 2, 2, seed=1)
    stg.load_inputs()
    seen = []

    @stp.BOUNDARY_FN
    def cb(user, which, buf, nbytes, layer, mb, stream):
        seen.append((which, layer, mb, nbytes))

    s = torch.cuda.current_stream()
    ctx.braid_reset()
    ctx.braid_step(stg.stage, forward_ops(2, 0), s, s, s, cb=cb)
    ctx.braid_step(stg.stage, braid(forward_ops(2, 1), backward_ops(2, 0, OP_BW)), s, s, s, cb=cb)
    torch.cuda.synchronize()
    nbytes = 128 * 256 * 4
    assert seen[:4] == [(0, 0, 0, nbytes), (1, 0, 0, nbytes), (0, 1, 0, nbytes), (1, 1, 0, nbytes)]
    second = seen[4:]
    assert second == [(0, 0, 1, nbytes), (2, 1, 0, nbytes), (1, 0, 1, nbytes), (3, 1, 0, nbytes),
                      (0, 1, 1, nbytes), (2, 0, 0, nbytes), (1, 1, 1, nbytes), (3, 0, 0, nbytes)]


def test_weight_unit_before_its_backward_is_rejected(ctx):
    stg = StageOnDevice(ctx, [synth.WORKLOADS["tiny"]], 2, seed=1)
    stg.load_inputs()
    s = torch.cuda.current_stream()
    ctx.braid_reset()
    ctx.braid_step(stg.stage, forward_ops(1, 0), s, s, s)
    with pytest.raises(stp.StpError) as e:
        ctx.braid_step(stg.stage, [Op(OP_W, MLP, 0, 0)], s, s, s)
    assert e.value.status == 5
    ctx.braid_step(stg.stage, backward_ops(1, 0, OP_B), s, s, s)
    ctx.braid_step(stg.stage, [Op(OP_W, MLP, 0, 0), Op(OP_W, ATTN, 0, 0)], s, s, s)   # now legal
    ctx.braid_reset()
    with pytest.raises(stp.StpError):
        ctx.braid_step(stg.stage, [Op(OP_W, MLP, 0, 0)], s, s, s)
    torch.cuda.synchronize()


def test_heterogeneous_stage_with_chain_break(ctx):
    """A stage holding two independent chains (ViT-style bidirectional layers, then LM layers of another
    width): slot 2 is the LM chain's own input, the ViT chain's output goes to layer 1's tail slot."""
    vit = Workload("v", 128, 2, 64, 264, 72, 1, causal=False)
    lm = Workload("m", 256, 2, 128, 520, 136, 8)
    layers = [vit, vit, lm, lm]
    n_mb = 3
    stg = StageOnDevice(ctx, layers, n_mb, seed=5, chain_break=[0, 0, 1, 0, 0])
    # chain inputs / upstream gradients: ViT chain slot 0 (in), tail of layer 1 (out); LM chain slots 2 (in), 4 (out)
    for mb in range(n_mb):
        stg.act_slot(0, mb).copy_(to_dev_like(synth.make_activation(vit, 5, f"vx.mb{mb}"), vit))
        stg.act_slot(2, mb).copy_(to_dev_like(synth.make_activation(lm, 5, f"lx.mb{mb}"), lm))
        stg.grad_slot(4, mb).copy_(to_dev_like(synth.make_activation(lm, 5, f"ldy.mb{mb}"), lm))
    s0 = torch.cuda.current_stream()
    sF, sB, sW = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
    # LM chain only (layers 2..3): F(mb) then braided with BW of the previous microbatch
    def lm_f(mb):
        return [Op(OP_F, u, l, mb) for l in (2, 3) for u in (PRE_ATTN, ATTN, PRE_MLP, MLP)]
    def lm_b(mb):
        return [Op(OP_BW, u, l, mb) for l in (3, 2) for u in (MLP, PRE_MLP, ATTN, PRE_ATTN)]
    def vit_f(mb):
        return [Op(OP_F, u, l, mb) for l in (0, 1) for u in (PRE_ATTN, ATTN, PRE_MLP, MLP)]
    results = []
    for streams in ((s0, s0, s0), (sF, sB, sW)):
        ctx.braid_reset()
        stg.zero_grads()
        ctx.braid_step(stg.stage, vit_f(0) + lm_f(0), *streams)          # two chains in one forward list
        ctx.braid_step(stg.stage, braid(vit_f(1) + lm_f(1), lm_b(0)), *streams)
        ctx.braid_step(stg.stage, braid(vit_f(2) + lm_f(2), lm_b(1)), *streams)
        ctx.braid_step(stg.stage, lm_b(2), *streams)
        torch.cuda.synchronize()
        results.append(snapshot(stg))
    for a, b in zip(*results):
        assert torch.equal(a, b)
    # oracle for the LM chain of microbatch 1 and the ViT chain of microbatch 2
    tol = TOL["bf16"]
    def chain(ls, idx, x):
        for l in idx:
            cfg, W = oracle_cfg(ls[l]), {k: v.astype(np.float64) for k, v in stg.w_host[l].items()}
            st = {}
            O.forward_unit(cfg, O.PRE_ATTN, W, st, x_in=x)
            xa = O.forward_unit(cfg, O.ATTN, W, st, x_resid=x)
            O.forward_unit(cfg, O.PRE_MLP, W, st, x_in=xa)
            x = O.forward_unit(cfg, O.MLP, W, st, x_resid=xa)
        return x
    ref_lm = chain(layers, (2, 3), synth.make_activation(lm, 5, "lx.mb1").astype(np.float64))
    assert rel_err(to_host(stg.act_slot(4, 1)), ref_lm) < tol
    ref_vit = chain(layers, (0, 1), synth.make_activation(vit, 5, "vx.mb2").astype(np.float64))
    assert rel_err(to_host(stg.chain_out(1, 2)), ref_vit) < tol


# ---- op-list variants ---------------------------------------------------------------------------------------
def run_steps(ctx, stg, steps, streams):
    ctx.braid_reset()
    stg.zero_grads()
    for step in steps:
        ctx.braid_step(stg.stage, step, *streams)
    torch.cuda.synchronize()


@pytest.mark.parametrize("name", ["gpt_bf16_x2", "llama_bf16_x1"])
def test_warmup_depth_changes_the_order_not_the_result(ctx, name):
    """Memory-efficient (one forward in flight before the first backward) and throughput-efficient warm-up
    (Appendix A) issue the same units; every microbatch's weight gradients are added in the same order."""
    layers, _ = STAGES[name]
    n_mb = 8
    stg = StageOnDevice(ctx, layers, n_mb, seed=4)
    stg.load_inputs()
    streams = (torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream())
    run_steps(ctx, stg, stage_sequence(len(layers), n_mb, warmup=1), streams)
    ref = snapshot(stg)
    for k in (2, 4):
        run_steps(ctx, stg, stage_sequence(len(layers), n_mb, warmup=k), streams)
        for a, b in zip(ref, snapshot(stg)):
            assert torch.equal(a, b), (name, k)


def test_two_chunk_patterns_give_the_same_bits_and_match_the_oracle(ctx):
    """Section 4.1: pairing forward and backward units of the same chunk (pattern 2) or of different chunks
    (pattern 1) on a device that holds a short wide chunk and a long narrow one."""
    from paper_2510_27257_amd.stage import two_chunk_sequence
    vit = Workload("v", 256, 4, 64, 512, 200, 1, causal=False)
    lm = Workload("g", 512, 2, 128, 1024, 264, 8)
    layers, cb, n_mb = [vit, vit, vit, lm], [0, 0, 0, 1, 0], 4
    stg = StageOnDevice(ctx, layers, n_mb, seed=6, chain_break=cb)
    stg.load_inputs()
    s0 = torch.cuda.current_stream()
    streams = (torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream())
    run_steps(ctx, stg, two_chunk_sequence(4, 3, n_mb, 2), (s0, s0, s0))
    ref = snapshot(stg)
    for pattern in (2, 1):
        run_steps(ctx, stg, two_chunk_sequence(4, 3, n_mb, pattern), streams)
        for a, b in zip(ref, snapshot(stg)):
            assert torch.equal(a, b), pattern
    # oracle, chunk by chunk (identity at the AR points)
    for (first, last), tag in zip(stg.chains(), ("c0.", "c1.")):
        g_ref = {l: dict() for l in range(first, last + 1)}
        for mb in range(n_mb):
            x = synth.make_activation(layers[first], 6, f"{tag}x.mb{mb}").astype(np.float64)
            dy = synth.make_activation(layers[last], 6, f"{tag}dy.mb{mb}").astype(np.float64)
            xs, sts = [x], []
            for l in range(first, last + 1):
                cfg, W = oracle_cfg(layers[l]), {k: v.astype(np.float64) for k, v in stg.w_host[l].items()}
                st = {}
                O.forward_unit(cfg, O.PRE_ATTN, W, st, x_in=xs[-1])
                xa = O.forward_unit(cfg, O.ATTN, W, st, x_resid=xs[-1])
                O.forward_unit(cfg, O.PRE_MLP, W, st, x_in=xa)
                xs.append(O.forward_unit(cfg, O.MLP, W, st, x_resid=xa))
                sts.append(st)
            tol = TOL[layers[first].dtype]
            assert rel_err(to_host(stg.chain_output(last, mb)), xs[-1]) < tol
            for l in reversed(range(first, last + 1)):
                cfg, W = oracle_cfg(layers[l]), {k: v.astype(np.float64) for k, v in stg.w_host[l].items()}
                st = sts[l - first]
                dz = O.backward_input_unit(cfg, O.MLP, W, st, dy)
                dxa = O.backward_input_unit(cfg, O.PRE_MLP, W, st, dz, d_resid=dy, grads=g_ref[l])
                dxl = O.backward_input_unit(cfg, O.ATTN, W, st, dxa)
                dx = O.backward_input_unit(cfg, O.PRE_ATTN, W, st, dxl, d_resid=dxa, grads=g_ref[l])
                O.backward_weight_unit(cfg, O.MLP, st, dy, g_ref[l])
                O.backward_weight_unit(cfg, O.ATTN, st, dxa, g_ref[l])
                dy = dx
            assert rel_err(to_host(stg.grad_slot(first, mb)), dy) < tol
        for l in range(first, last + 1):
            for k, r in g_ref[l].items():
                assert rel_err(to_host(stg.g_dev[l][k]), r) < TOL[layers[l].dtype], (l, k)


@pytest.mark.parametrize("p,m,d", [(2, 6, 0), (2, 6, 1), (3, 9, 1)])
def test_generated_device_program_runs_and_matches_the_two_chunk_sequence(ctx, p, m, d):
    """A device's program from the schedule generator (Section 4.2), replayed block by block on a two-chunk stage:
    same activation gradients bit for bit as the plain two-chunk sequence, weight gradients equal up to the
    order in which the microbatches are added, and the outputs and input gradients of sampled microbatches equal
    to the oracle's."""
    from paper_2510_27257_amd import schedule as S
    from paper_2510_27257_amd.stage import two_chunk_sequence
    lm = Workload("g", 256, 2, 64, 512, 136, 4)
    layers, cb = [lm, lm, lm], [0, 0, 1, 0]
    stg = StageOnDevice(ctx, layers, m, seed=8, chain_break=cb)
    stg.load_inputs()
    streams = (torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream())
    run_steps(ctx, stg, two_chunk_sequence(3, 2, m, 2), streams)
    ref_grads = [t.clone() for t in stg.grad]
    ref_w = [{k: v.clone() for k, v in gd.items()} for gd in stg.g_dev]
    progs = S.build(p, m)
    S.simulate(p, progs, S.Times(1.0, 1.4, 0.8, 0.3))
    run_steps(ctx, stg, S.braid_steps(progs[d], 3, 2), streams)
    for a, b in zip(ref_grads, stg.grad):
        assert torch.equal(a, b)
    for l in range(3):
        for k, r in ref_w[l].items():
            got = stg.g_dev[l][k]
            assert float((got - r).abs().max()) <= 1e-5 * float(r.abs().max()) + 1e-12, (l, k)
    # and against the oracle directly: the first and the last microbatch of either chunk, forward output and input
    # gradient, through every layer of the chunk (identity at the AR points)
    for ci, (first, last) in enumerate(stg.chains()):
        for mb in (0, m - 1):
            x = synth.make_activation(layers[first], 8, f"c{ci}.x.mb{mb}").astype(np.float64)
            dy = synth.make_activation(layers[last], 8, f"c{ci}.dy.mb{mb}").astype(np.float64)
            sts = []
            for l in range(first, last + 1):
                cfg, W = oracle_cfg(layers[l]), {k: v.astype(np.float64) for k, v in stg.w_host[l].items()}
                st = {}
                O.forward_unit(cfg, O.PRE_ATTN, W, st, x_in=x)
                xa = O.forward_unit(cfg, O.ATTN, W, st, x_resid=x)
                O.forward_unit(cfg, O.PRE_MLP, W, st, x_in=xa)
                x = O.forward_unit(cfg, O.MLP, W, st, x_resid=xa)
                sts.append(st)
            assert rel_err(to_host(stg.chain_output(last, mb)), x) < TOL[lm.dtype], (ci, mb)
            for l in reversed(range(first, last + 1)):
                cfg, W = oracle_cfg(layers[l]), {k: v.astype(np.float64) for k, v in stg.w_host[l].items()}
                st = sts[l - first]
                dz = O.backward_input_unit(cfg, O.MLP, W, st, dy)
                dxa = O.backward_input_unit(cfg, O.PRE_MLP, W, st, dz, d_resid=dy)
                dxl = O.backward_input_unit(cfg, O.ATTN, W, st, dxa)
                dy = O.backward_input_unit(cfg, O.PRE_ATTN, W, st, dxl, d_resid=dxa)
            assert rel_err(to_host(stg.grad_slot(first, mb)), dy) < TOL[lm.dtype], (ci, mb)


def test_streams_without_work_come_after_the_step_before_last_too(ctx):
    """Three blocks of forward passes leave the other two streams without work.  What the caller puts on these then finds the first
    block's output whole (a spinning kernel holds the first block back until all of it is enqueued)."""
    layers, n_mb = STAGES["gpt_bf16_x2"]
    L = len(layers)
    stg = StageOnDevice(ctx, layers, n_mb, seed=4)
    stg.load_inputs()
    s0 = torch.cuda.current_stream()
    ctx.braid_reset()
    ctx.braid_step(stg.stage, forward_ops(L, 0), s0, s0, s0)
    torch.cuda.synchronize()
    first = stg.act_slot(L, 0)
    want, got = first.clone(), [torch.empty_like(first) for _ in range(2)]
    streams = tuple(torch.cuda.Stream() for _ in range(3))
    for step in range(2):      # (the change of streams joins them all: the steps that matter come behind two of their own)
        ctx.braid_step(stg.stage, forward_ops(L, 4), *streams)
    torch.cuda.synchronize()
    first.fill_(float("nan"))
    torch.cuda.synchronize()
    with torch.cuda.stream(streams[0]):
        torch.cuda._sleep(20_000_000)
    for mb in range(3):
        ctx.braid_step(stg.stage, forward_ops(L, mb), *streams)
    for s, out in zip(streams[1:], got):
        with torch.cuda.stream(s):
            out.copy_(first)
    torch.cuda.synchronize()
    for out in got:
        assert torch.equal(out, want)


@pytest.mark.parametrize("mode", ["global", "thread_local", "relaxed"])
def test_steps_run_while_another_stream_is_being_captured(ctx, mode):
    """Steps on three streams of their own, with weight-gradient units put off behind their B units, between the beginning and the end of
    a capture on a fourth: both are whole afterwards."""
    layers, n_mb = STAGES["gpt_bf16_x2"]
    stg = StageOnDevice(ctx, layers, n_mb, seed=2)
    stg.load_inputs()
    s0 = torch.cuda.current_stream()
    streams = tuple(torch.cuda.Stream() for _ in range(3))
    run_sequence(ctx, stg, (s0, s0, s0))
    want = snapshot(stg)
    run_sequence(ctx, stg, streams)                     # events and kernel attributes are made here
    ctx.braid_reset()
    stg.zero_grads()
    x = torch.ones(1 << 16, device="cuda")
    x.mul_(1.0)
    torch.cuda.synchronize()
    with torch.cuda.stream(streams[1]):
        torch.cuda._sleep(2_000_000)                    # so that B units are pending when their W units are looked at
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream(), capture_error_mode=mode):
        x.mul_(2.0)
        for step in stage_sequence(len(stg.layers), stg.n_mb):
            ctx.braid_step(stg.stage, step, *streams)
        x.add_(1.0)
    torch.cuda.synchronize()
    for a, b in zip(want, snapshot(stg)):
        assert torch.equal(a, b)
    for value in (3.0, 7.0, 15.0):
        graph.replay()
        torch.cuda.synchronize()
        assert bool((x == value).all())


@pytest.mark.parametrize("name", ["gpt_bf16_x2", "llama_bf16_x1"])
def test_streams_shared_by_two_kinds_of_work_give_the_serialized_bits(ctx, name):
    """Two streams for the three kinds of work, each way; the stage's sequence, the same block again and again, and another choice at every step."""
    layers, n_mb = STAGES[name]
    L = len(layers)
    stg = StageOnDevice(ctx, layers, n_mb, seed=9)
    stg.load_inputs()
    s0, a, b = torch.cuda.current_stream(), torch.cuda.Stream(), torch.cuda.Stream()
    block = braid(forward_ops(L, n_mb - 1), backward_ops(L, 0, OP_BW))

    def run(choices, steps, first=()):
        ctx.braid_reset()
        stg.zero_grads()
        for step in first:
            ctx.braid_step(stg.stage, step, s0, s0, s0)
        torch.cuda.synchronize()
        for i, step in enumerate(steps):
            ctx.braid_step(stg.stage, step, *choices[i % len(choices)])
        torch.cuda.synchronize()
        return snapshot(stg) + [m.clone() for m in stg.stash_mem]

    triples = [(a, a, b), (a, b, a), (a, b, b)]
    for steps, first in ((stage_sequence(L, n_mb), ()), ([block] * 8, (forward_ops(L, 0),))):
        serial = run([(s0, s0, s0)], steps, first)
        for choices in [[t] for t in triples] + [triples, [(b, a, b), (a, a, a), (a, b, a)]]:
            for u, v in zip(serial, run(choices, steps, first)):
                assert torch.equal(u, v), f"{name}: {[[a, b].index(s) for t in choices for s in t]} differs from the serialized order"
