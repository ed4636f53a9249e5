"""The fp32 GEMM at the edges of its tiles: all three workgroup tiles, ragged rows, columns and contraction lengths
(K = 8 leaves half of the only 16-deep chunk empty, K = 136 gives the contraction-splitting waves unequal shares)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2510_27257_amd as stp
from harness import rel_err, to_dev, to_host


@pytest.fixture(scope="module")
def ctx():
    c = stp.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("a_trans,b_trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(8, 40, 8), (136, 256, 136), (1000, 840, 72), (1032, 776, 264), (2056, 1800, 40), (2048, 1536, 144)])
def test_gemm_f32(ctx, M, N, K, a_trans, b_trans):
    rng = np.random.default_rng(M + N + K)
    A, B = rng.standard_normal((M, K), dtype=np.float32), rng.standard_normal((K, N), dtype=np.float32)
    R, bias = rng.standard_normal((M, N), dtype=np.float32), rng.standard_normal(N, dtype=np.float32)
    Ad = to_dev(np.ascontiguousarray(A.T) if a_trans else A, "f32")
    Bd = to_dev(np.ascontiguousarray(B.T) if b_trans else B, "f32")
    Rd, bd = to_dev(R, "f32"), to_dev(bias, "f32")
    Cd = torch.full((M, N), 7.0, dtype=torch.float32, device="cuda")
    base = dict(dtype=stp.F32, M=M, N=N, K=K, A=Ad.data_ptr(), lda=M if a_trans else K, a_trans=a_trans, B=Bd.data_ptr(),
                ldb=K if b_trans else N, b_trans=b_trans, C=Cd.data_ptr(), ldc=N, bias_scale=1.0, resid_scale=1.0)
    AB = A.astype(np.float64) @ B.astype(np.float64)
    # a sum of K products of unit variance has standard deviation sqrt(K); its rounding error grows like
    # sqrt(K) * 2^-24 of that: well below 2e-6 of the largest of M * N such values
    ctx.gemm(stp.GemmArgs(**base))
    torch.cuda.synchronize()
    assert rel_err(to_host(Cd), AB) < 2e-6
    ctx.gemm(stp.GemmArgs(**base | dict(bias=bd.data_ptr(), bias_scale=0.5, resid=Rd.data_ptr(), ldr=N, resid_scale=0.25)))
    torch.cuda.synchronize()
    assert rel_err(to_host(Cd), AB + 0.5 * bias + 0.25 * R) < 2e-6
    before = Cd.clone()
    ctx.gemm(stp.GemmArgs(**base | dict(c_f32_accum=1)))
    torch.cuda.synchronize()
    assert rel_err(to_host(Cd), to_host(before) + AB) < 2e-6


# head dimensions at and between the kernels' 32-column blocks; sequences below, at and past a 32-row block and with more
# blocks than waves; groups; several sequences whose length is not a multiple of 8
@pytest.mark.parametrize("seq,mbsz,n,d,causal,nk", [(8, 1, 1, 8, True, 0), (32, 1, 2, 40, False, 0), (33, 8, 2, 96, True, 1), (200, 1, 2, 128, True, 1),
                                                    (164, 2, 3, 72, False, 0), (328, 1, 3, 64, True, 1), (296, 1, 1, 24, False, 0)])
def test_attention_f32(ctx, seq, mbsz, n, d, causal, nk):
    import test_gpu_kernels
    test_gpu_kernels.test_attention_forward_backward(ctx, "f32", seq, mbsz, n, d, causal, nk)


# contractions that are not split: 32 x 32 wave tiles as 2 x 2, 1 x 4 and 4 x 1, ragged in both directions, every epilogue
@pytest.mark.parametrize("a_trans,b_trans", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("M,N,K", [(1000, 840, 72), (2056, 1800, 8), (24, 16440, 40), (16440, 24, 16), (32840, 40, 128)])
def test_gemm_f32_short_contraction(ctx, M, N, K, a_trans, b_trans):
    rng = np.random.default_rng(M + N + K)
    A, B = rng.standard_normal((M, K), dtype=np.float32), rng.standard_normal((K, N), dtype=np.float32) / np.float32(np.sqrt(K))
    R, bias = rng.standard_normal((M, N), dtype=np.float32), rng.standard_normal(N, dtype=np.float32)
    Ad = to_dev(np.ascontiguousarray(A.T) if a_trans else A, "f32")
    Bd = to_dev(np.ascontiguousarray(B.T) if b_trans else B, "f32")
    Rd, bd = to_dev(R, "f32"), to_dev(bias, "f32")
    C, C2 = torch.full((M, N), 7.0, device="cuda"), torch.full((M, N), 7.0, device="cuda")
    base = dict(dtype=stp.F32, M=M, N=N, K=K, A=Ad.data_ptr(), lda=M if a_trans else K, a_trans=a_trans, B=Bd.data_ptr(),
                ldb=K if b_trans else N, b_trans=b_trans, C=C.data_ptr(), ldc=N, bias_scale=1.0, resid_scale=1.0)
    AB = torch.from_numpy(A.astype(np.float64) @ B.astype(np.float64))

    def check(t, ref):        # the bound of the sums above; GELU and its derivative are within a few units in the last place
        torch.cuda.synchronize()
        assert rel_err(to_host(t), np.asarray(ref)) < 2e-6

    ctx.gemm(stp.GemmArgs(**base | dict(bias=bd.data_ptr(), bias_scale=0.5, resid=Rd.data_ptr(), ldr=N, resid_scale=0.25)))
    check(C, AB.numpy() + 0.5 * bias + 0.25 * R)
    ctx.gemm(stp.GemmArgs(**base, epilogue=1, C2=C2.data_ptr(), ld2=N))
    check(C, AB)
    check(C2, torch.nn.functional.gelu(AB))
    x = torch.from_numpy(R.astype(np.float64)).requires_grad_()
    torch.nn.functional.gelu(x).sum().backward()
    ctx.gemm(stp.GemmArgs(**base, epilogue=2, aux=Rd.data_ptr(), ld2=N))
    check(C, AB * x.grad)
    before = to_host(C)
    ctx.gemm(stp.GemmArgs(**base, c_f32_accum=1))
    check(C, before + AB.numpy())
