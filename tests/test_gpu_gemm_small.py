"""The bf16 GEMM of small outputs (at most 256 tiles of 64 x 64, K >= 256), whose contraction is split over the four waves of a
workgroup: edges of the tile, waves with unequal or single K-tiles, a partly empty last K-tile, every epilogue."""
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


# K = 256: one 64-deep K-tile per wave; 264: one of eight elements more; 320: a wave has two; 1024 x 1024: exactly 256 tiles
@pytest.mark.parametrize("a_trans,b_trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(8, 8, 256), (64, 64, 264), (72, 136, 320), (200, 264, 456), (136, 72, 1000), (384, 1032, 3000), (1024, 1024, 1056)])
def test_small_output(ctx, M, N, K, a_trans, b_trans):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = torch.randn((M, K), generator=g, device="cuda").to(torch.bfloat16)
    b = (torch.randn((K, N), generator=g, device="cuda") * 0.05).to(torch.bfloat16)
    A = a.t().contiguous() if a_trans else a
    B = b.t().contiguous() if b_trans else b
    R = torch.randn((M, N), generator=g, device="cuda").to(torch.bfloat16)
    bias = torch.randn(N, generator=g, device="cuda").to(torch.bfloat16)
    ref = a.double() @ b.double()
    C, C2 = torch.zeros_like(R), torch.zeros_like(R)
    base = dict(dtype=stp.BF16, M=M, N=N, K=K, A=A.data_ptr(), lda=A.stride(0), a_trans=a_trans, B=B.data_ptr(), ldb=B.stride(0), b_trans=b_trans,
                ldc=N, bias_scale=1.0, resid_scale=1.0)
    # the bounds of the larger tiles' epilogue tests: a bf16 result of an fp32 sum (2^-9 relative), twice rounded for GELU
    ctx.gemm(stp.GemmArgs(**base | dict(bias_scale=0.5, resid_scale=0.25), C=C.data_ptr(), bias=bias.data_ptr(), resid=R.data_ptr(), ldr=N))
    torch.cuda.synchronize()
    assert rel_err(to_host(C), to_host(ref + 0.5 * bias.double() + 0.25 * R.double())) < 6e-3
    ctx.gemm(stp.GemmArgs(**base, C=C.data_ptr(), epilogue=1, C2=C2.data_ptr(), ld2=N))
    torch.cuda.synchronize()
    assert rel_err(to_host(C), to_host(ref)) < 6e-3
    assert rel_err(to_host(C2), to_host(torch.nn.functional.gelu(ref))) < 6e-3
    x = R.double().requires_grad_()
    torch.nn.functional.gelu(x).sum().backward()
    ctx.gemm(stp.GemmArgs(**base, C=C.data_ptr(), epilogue=2, aux=R.data_ptr(), ld2=N))
    torch.cuda.synchronize()
    assert rel_err(to_host(C), to_host(ref * x.grad)) < 6e-3
    acc = torch.full((M, N), 0.5, device="cuda")
    for _ in range(2):
        ctx.gemm(stp.GemmArgs(**base, C=acc.data_ptr(), c_f32_accum=1))
    torch.cuda.synchronize()
    assert rel_err(to_host(acc), to_host(0.5 + 2 * ref)) < 1e-5
