"""The column sum in one launch (up to 768 rows of fp32, 2048 of bf16 and of wide fp32) and in two, around the row-lanes', batches' and column groups' edges."""
import pytest
import torch

pytestmark = pytest.mark.gpu

import paper_2510_27257_amd as stp


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("N", [8, 64, 72, 1032, 8192])
@pytest.mark.parametrize("T", [1, 7, 128, 129, 768, 769, 1024, 1031, 2048, 2049])
def test_column_sum(T, N, dtype):
    ctx = stp.Context(0)
    g = torch.Generator(device="cuda").manual_seed(T * N)
    x = torch.randn((T, N), generator=g, device="cuda").to(torch.float32 if dtype == "f32" else torch.bfloat16)
    start = torch.randn(N, generator=g, device="cuda")
    out = start.clone()
    ctx.colsum_noalloc(stp.F32 if dtype == "f32" else stp.BF16, T, N, x, 0.125, out)
    torch.cuda.synchronize()
    ref = start.double() + 0.125 * x.double().sum(0)
    # a sum of n terms added one to the next is off by at most n 2^-24 of the sum of their magnitudes; here n is a row-lane's rows,
    # the exchanges, the waves (or 64-row patches) and the accumulator
    n = -(-T // 32) + 64
    bound = n * 2.0 ** -24 * (0.125 * x.double().abs().sum(0) + start.double().abs())
    assert bool(((out.double() - ref).abs() <= bound).all())
    ctx.close()
