"""The register-staged bf16 GEMM, which takes operands that span 2 GiB or more: small matrices in rows so far apart that one of
them does, in every layout, with whole, partly empty and several K-tiles, ragged tiles, every epilogue."""
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


@pytest.fixture(scope="module")
def space():
    return torch.empty(1200 << 20, dtype=torch.bfloat16, device="cuda")      # 2.3 GiB, mostly never touched


@pytest.mark.parametrize("wide", ["A", "B"])
@pytest.mark.parametrize("a_trans,b_trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(136, 264, 72), (264, 136, 200), (128, 128, 64)])
def test_wide_pitch(ctx, space, M, N, K, a_trans, b_trans, wide):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)

    def operand(rows, cols, std, far):
        x = (torch.randn((rows, cols), generator=g, device="cuda") * std).to(torch.bfloat16)
        if not far:
            return x, x.stride(0), x
        ld = (space.numel() - cols) // (rows - 1) // 8 * 8
        assert ((rows - 1) * ld + cols) * 2 >= 1 << 31
        view = torch.as_strided(space, (rows, cols), (ld, 1))
        view.copy_(x)
        return view, ld, x

    A, lda, a = operand(*((K, M) if a_trans else (M, K)), 1.0, wide == "A")
    B, ldb, b = operand(*((N, K) if b_trans else (K, N)), 0.05, wide == "B")
    ref = (a.t() if a_trans else a).double() @ (b.t() if b_trans else b).double()
    R = torch.randn((M, N), generator=g, device="cuda").to(torch.bfloat16)
    bias = torch.randn(N, generator=g, device="cuda").to(torch.bfloat16)
    out, out2 = torch.zeros_like(R), torch.zeros_like(R)
    base = dict(dtype=stp.BF16, M=M, N=N, K=K, A=A.data_ptr(), lda=lda, a_trans=a_trans, B=B.data_ptr(), ldb=ldb, b_trans=b_trans, ldc=N,
                bias_scale=0.5, resid_scale=0.25)

    def check(t, r, bound=6e-3):      # a bf16 result of an fp32 sum (2^-9 relative), twice rounded for GELU
        torch.cuda.synchronize()
        assert rel_err(to_host(t), to_host(r)) < bound

    ctx.gemm(stp.GemmArgs(**base, C=out.data_ptr(), bias=bias.data_ptr(), resid=R.data_ptr(), ldr=N))
    check(out, ref + 0.5 * bias.double() + 0.25 * R.double())
    ctx.gemm(stp.GemmArgs(**base, C=out.data_ptr(), epilogue=1, C2=out2.data_ptr(), ld2=N))
    check(out, ref)
    check(out2, torch.nn.functional.gelu(ref))
    x = R.double().requires_grad_()
    torch.nn.functional.gelu(x).sum().backward()
    ctx.gemm(stp.GemmArgs(**base, C=out.data_ptr(), epilogue=2, aux=R.data_ptr(), ld2=N))
    check(out, ref * x.grad)
    acc = torch.full((M, N), 0.5, device="cuda")
    ctx.gemm(stp.GemmArgs(**base, C=acc.data_ptr(), c_f32_accum=1))
    check(acc, 0.5 + ref, 1e-5)
