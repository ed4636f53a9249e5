// bf16 MFMA GEMM, operand layout "mn": A row-contiguous, B row-contiguous
// (one translation unit per layout so that the four compile in parallel).
#include "gemm_bf16_impl.h"

int stp_launch_gemm_bf16_mn(stp_ctx *ctx, const stp_gemm_args *a, hipStream_t s) {
  return launch_layout<false, false>(ctx, a, s);
}

// The weight gradients of a unit in one launch where the chip is theirs alone: 13B shard, [3456 | 5120, 5120 | 3456] three times over
// 4096 tokens, 169 + 2 x 180 -> 430 us.  Beside other streams, which fill what a launch's last round leaves idle, one long launch is the
// worse one (blocks 0.3 - 5 % slower).
int stp_launch_gemm_bf16_wgrads(stp_ctx *ctx, const stp_gemm_args *a, int n, hipStream_t s) {
  TileChoice c;
  if (n > 1 && !(ctx && ctx->concurrent) && set_tile(ctx, a, n, &c))
    return a[0].K % DK ? launch_set_tile<true>(ctx, a, n, c, s) : launch_set_tile<false>(ctx, a, n, c, s);
  for (int i = 0; i < n; i++) {
    const int rc = stp_launch_gemm_bf16_mn(ctx, &a[i], s);
    if (rc != STP_OK) return rc;
  }
  return STP_OK;
}
