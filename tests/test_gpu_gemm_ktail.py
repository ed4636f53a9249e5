"""The bf16 GEMM at contraction lengths that are not a multiple of the 64-deep K-tile: the last tile is partly empty.
What lies past K in memory (the padding of the rows, the rows after the last one) is NaN and must not reach a result."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2510_27257_amd as stp
from harness import rel_err, to_host


@pytest.fixture(scope="module")
def ctx():
    c = stp.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def operand(g, rows, K, std, k_outer):
    """[rows, K] bf16 stored with a NaN surround; returns (storage, leading dimension, values as fp32)."""
    x = (torch.randn((rows, K), generator=g, device="cuda") * std).to(torch.bfloat16)
    if k_outer:
        store = torch.full((K + 32, rows + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
        store[:K, :rows] = x.t()
    else:
        store = torch.full((rows + 1, K + 8), float("nan"), dtype=torch.bfloat16, device="cuda")
        store[:rows, :K] = x
    return store, store.stride(0), x.float()


# (8, 8): one tile and one K-tile, mostly empty; then shapes that take each of the workgroup tiles
@pytest.mark.parametrize("a_trans,b_trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(8, 8, 8), (8, 8, 40), (136, 264, 72), (264, 136, 120), (520, 776, 152), (1032, 2744, 1000), (3000, 1032, 328),
                                   (6144, 2048, 1048), (6144, 4096, 88)])
def test_k_tail(ctx, M, N, K, a_trans, b_trans):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, lda, a = operand(g, M, K, 1.0, a_trans)
    B, ldb, b = operand(g, N, K, 0.05, not b_trans)
    ref = a @ b.t()
    base = dict(dtype=stp.BF16, M=M, N=N, K=K, A=A.data_ptr(), lda=lda, a_trans=a_trans, B=B.data_ptr(), ldb=ldb, b_trans=b_trans, ldc=N,
                bias_scale=1.0, resid_scale=1.0)
    C = torch.zeros((M, N), dtype=torch.bfloat16, device="cuda")
    ctx.gemm(stp.GemmArgs(**base, C=C.data_ptr()))
    acc = torch.ones((M, N), dtype=torch.float32, device="cuda")
    ctx.gemm(stp.GemmArgs(**base, C=acc.data_ptr(), c_f32_accum=1))
    torch.cuda.synchronize()
    assert rel_err(to_host(C), to_host(ref)) < 4e-3
    assert rel_err(to_host(acc), to_host(ref) + 1.0) < 1e-5


# every workgroup tile, fewer K-tiles than its rings hold, as many, and more, with and without a half-empty last one; also
# just more tiles of 128 x 128 than compute units (another ring length)
@pytest.mark.parametrize("tile,a_trans,b_trans", [(t, a, b) for t in [(256, 256), (192, 256), (128, 256), (256, 128), (128, 128)] for a in (0, 1)
                                                  for b in (0, 1) if not (a and t[0] == 192)])     # 192 rows: k-contiguous A only
@pytest.mark.parametrize("M,N,K", [(264, 520, 32), (264, 520, 64), (264, 520, 128), (264, 520, 192), (264, 520, 224), (264, 520, 256), (264, 520, 544),
                                   (2056, 2056, 352)])
def test_rings(ctx, M, N, K, tile, a_trans, b_trans):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, lda, a = operand(g, M, K, 1.0, a_trans)
    B, ldb, b = operand(g, N, K, 0.05, not b_trans)
    ref = a @ b.t()
    out = torch.full((M, N), float("nan"), device="cuda", dtype=torch.bfloat16)
    ctx.gemm(stp.GemmArgs(dtype=stp.BF16, M=M, N=N, K=K, A=A.data_ptr(), lda=lda, a_trans=a_trans, B=B.data_ptr(), ldb=ldb, b_trans=b_trans,
                          C=out.data_ptr(), ldc=N, bias_scale=1.0, resid_scale=1.0, tile_m=tile[0], tile_n=tile[1]))
    torch.cuda.synchronize()
    assert rel_err(to_host(out), to_host(ref)) < 6e-3      # as above: the bf16 rounding of an fp32 sum


# K <= 128 takes shorter rings on the 128 x 128 tile: the bits of the 256 x 256 tile, with a half-empty last K-tile and without, with
# every epilogue
@pytest.mark.parametrize("a_trans,b_trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("K", [32, 64, 96, 128])
def test_short_contraction_bits(ctx, K, a_trans, b_trans):
    M, N = 392, 264
    g = torch.Generator(device="cuda").manual_seed(K)
    A, lda, _ = operand(g, M, K, 1.0, a_trans)
    B, ldb, _ = operand(g, N, K, 0.05, not b_trans)
    R = torch.randn((M, N), generator=g, device="cuda").to(torch.bfloat16)
    bias = torch.randn(N, generator=g, device="cuda").to(torch.bfloat16)
    base = dict(dtype=stp.BF16, M=M, N=N, K=K, A=A.data_ptr(), lda=lda, a_trans=a_trans, B=B.data_ptr(), ldb=ldb, b_trans=b_trans, ldc=N,
                bias_scale=0.5, resid_scale=0.25)
    got = []
    for tile in (128, 256):
        C, C2, D, E = (torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda") for _ in range(4))
        acc = torch.ones((M, N), device="cuda")
        t = dict(tile_m=tile, tile_n=tile)
        ctx.gemm(stp.GemmArgs(**base | t, C=C.data_ptr(), bias=bias.data_ptr(), resid=R.data_ptr(), ldr=N))
        ctx.gemm(stp.GemmArgs(**base | t, C=D.data_ptr(), epilogue=1, C2=C2.data_ptr(), ld2=N))
        ctx.gemm(stp.GemmArgs(**base | t, C=E.data_ptr(), epilogue=2, aux=R.data_ptr(), ld2=N))
        ctx.gemm(stp.GemmArgs(**base | t, C=acc.data_ptr(), c_f32_accum=1))
        got.append((C, D, C2, E, acc))
    torch.cuda.synchronize()
    for x, y in zip(*got):
        assert torch.equal(x, y)
