// bf16 MFMA GEMM, operand layout "mn": A row-contiguous, B row-contiguous
// (one translation unit per layout so that the four compile in parallel).
#include "gemm_bf16_impl.h"

int stp_launch_gemm_bf16_mn(stp_ctx *ctx, const stp_gemm_args *a, hipStream_t s) {
  return launch_layout<false, false>(ctx, a, s);
}

// The weight gradients of a unit in one launch where the chip is theirs alone: 13B shard, three products of 3456 x 5120 over
// 4096 tokens and two smaller ones, 85 us of a pass of 2400.  Beside other streams, which fill what a launch's last round leaves idle, one long launch is the
// worse one (blocks 0.3 - 5 % slower).  Outputs of the contraction-splitting kernel go together there too: blocks of 36 layers of hidden 128 - 1100 take 4 %
// longer (median) with a launch each.
int stp_launch_gemm_bf16_wgrads(stp_ctx *ctx, const stp_gemm_args *a, int n, hipStream_t s) {
  TileChoice c;
  if (wavek_set(a, n)) return a[0].K % 32 ? launch_wavek_set<true>(ctx, a, n, s) : launch_wavek_set<false>(ctx, a, n, s);
  if (n > 1 && !(ctx && ctx->concurrent) && set_tile(a, n, &c))
    return a[0].K % DK ? launch_set_tile<true>(ctx, a, n, c, s) : launch_set_tile<false>(ctx, a, n, c, s);
  for (int i = 0; i < n; i++) {
    const int rc = stp_launch_gemm_bf16_mn(ctx, &a[i], s);
    if (rc != STP_OK) return rc;
  }
  return STP_OK;
}

extern "C" int stp_wgrad_set_tile(const stp_gemm_args *a, int n) {
  TileChoice c;
  return a && n > 1 && n <= 3 && set_tile(a, n, &c) ? c.bm << 16 | c.bn : 0;
}
