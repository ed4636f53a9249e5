// bf16 GEMMs of a SwiGLU MLP.  What they save against the plain products with the activation as kernels of its own is traffic and
// launches: forward, the activation kernel's pass over three [T, f] tensors becomes one store, and the two projections share the tiles of
// their common operand; backward, the gradient of the product is neither written nor read, and the input gradient's two terms
// are added in the accumulators instead of through a rounded [T, h] tensor.  Measured (us, apart -> here): 13B shard, 4096 tokens, hidden
// 5120, f = 3456: forward 2 x 123.5 + 14.3 -> 250, gradient of the activations 120.4 + 24.5 -> 138, input gradient 2 x 134.7 -> 250; 3000
// tokens, 1032, 2744: 2 x 25.5 + 9.5 -> 56, 28.8 + 14.4 -> 41, 2 x 32.2 -> 58.6.  Bound as the plain products are, and at the end of
// a round by the epilogues, which move up to four [T, f] tensors while the matrix pipes wait.
#include "gemm_bf16_impl.h"

namespace {

template <int BM, int BN, int WAVES_M, int WAVES_N, int NSTA, int NSTB, bool B_KC, int EPI, bool KTAIL, int MM>
int launch_two(stp_ctx *ctx, const stp_gemm_args *a, const Epi &ep, const void *A2, const void *B2, hipStream_t s) {
  constexpr size_t smem = (size_t)(NSTA * BM + NSTB * BN) * DK * 2;
  static_assert(smem <= 160 * 1024 && smem >= (size_t)WAVES_M * WAVES_N * 32 * (BN / WAVES_N + 8) * sizeof(float), "LDS budget");
  auto kern = gemm_bf16_two_kernel<BM, BN, WAVES_M, WAVES_N, NSTA, NSTB, true, B_KC, EPI, KTAIL, MM>;
  static bool attr_set = false;
  if (!attr_set) {
    STP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    attr_set = true;
  }
  constexpr int COLS = MM == MM_PAIR ? BN / 2 : BN;      // columns of C in a tile
  const int tiles_m = (a->M + BM - 1) / BM, tiles_n = (a->N + COLS - 1) / COLS;
  const long ab = operand_bytes(true, a->M, a->K, a->lda), bb = operand_bytes(B_KC, a->N, a->K, a->ldb);
  hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(64 * WAVES_M * WAVES_N), smem, s, (const bf16_t *)a->A, (const bf16_t *)A2, a->lda, (int)ab,
                     (const bf16_t *)a->B, (const bf16_t *)B2, a->ldb, (int)bb, a->M, a->N, a->K, tiles_m, tiles_n, ep);
  STP_LAUNCH_CHECK(ctx);
  return STP_OK;
}

template <bool B_KC, int EPI, bool KTAIL, int MM>
int launch_two_tile(stp_ctx *ctx, const stp_gemm_args *a, TileChoice c, const Epi &ep, const void *A2, const void *B2, hipStream_t s) {
  constexpr int WM = MM == MM_PAIR ? 4 : 2, WN = 8 / WM;      // 128 columns: a wave's 64 are a block of each product
  if (c.bm == 192 && c.bn == 256) return launch_two<192, 256, 2, 4, 3, 2, B_KC, EPI, KTAIL, MM>(ctx, a, ep, A2, B2, s);
  if (c.bm == 128 && c.bn == 256) return launch_two<128, 256, 2, 4, 3, 3, B_KC, EPI, KTAIL, MM>(ctx, a, ep, A2, B2, s);
  if (c.bm == 256 && c.bn == 128) return launch_two<256, 128, WM, WN, 3, 3, B_KC, EPI, KTAIL, MM>(ctx, a, ep, A2, B2, s);
  if (c.bm == 128 && c.bn == 128) {
    const int cols = MM == MM_PAIR ? 64 : 128;
    if (a->K > 128 && ((a->M + 127) / 128) * ((a->N + cols - 1) / cols) <= 256)      // as for one product
      return launch_two<128, 128, WM, WN, 4, 4, B_KC, EPI, KTAIL, MM>(ctx, a, ep, A2, B2, s);
    return launch_two<128, 128, WM, WN, 3, 2, B_KC, EPI, KTAIL, MM>(ctx, a, ep, A2, B2, s);
  }
  return launch_two<256, 256, 2, 4, 3, 2, B_KC, EPI, KTAIL, MM>(ctx, a, ep, A2, B2, s);
}

inline bool addressable(const stp_gemm_args *a, bool b_kc) {
  return a->K > 0 && operand_bytes(true, a->M, a->K, a->lda) > 0 && operand_bytes(b_kc, a->N, a->K, a->ldb) > 0;
}

// Whether the two projections, alone on the GPU, take longer together than apart, activation kernel included: for few tokens and long
// contractions, where a tile of both is slower by more than one launch saves.  The MLP unit (us, together / apart): 520 tokens, f = 14336, hidden
// 4096 261 / 256, 7168 442 / 431; 1032 tokens, 5120, 8192 301 / 290.  Beyond 1152 tokens the estimates are close where it is said to
// pay, and it does not: [1544, 2 x 5120] K = 7168 345 / 373, [2568, 2 x 3456] 363 / 383.  Both ways store the same bits.
inline bool longer_together(const stp_gemm_args *a, TileChoice *c) {
  double together, one;
  *c = pick_tile(a->M, 2L * a->N, a->K, true, false, false, false, &together, true);
  pick_tile(a->M, a->N, a->K, true, false, false, false, &one);
  return a->M <= 1152 && together > 2.0 * one + 1.33e-6 * (double)a->M * a->N;      // the kernel moves three tensors at 4.5 TB/s
}

}  // namespace

// tile (bm << 16 | bn) of the projections' launch alone on the GPU, 0 where they are launched apart; host only, no part of the interface
extern "C" int stp_swiglu_pair_tile(int M, int N, int K) {
  stp_gemm_args a = {};
  a.M = M; a.N = N; a.K = K;
  TileChoice c;
  return wavek_shape(M, N, K) || longer_together(&a, &c) ? 0 : c.bm << 16 | c.bn;
}

int stp_launch_gemm_bf16_swiglu(stp_ctx *ctx, const stp_gemm_args *a, const void *B2, void *up, void *act, hipStream_t s) {
  // products small enough for the contraction-splitting kernel stay apart
  if (!addressable(a, false) || wavek_shape(a->M, a->N, a->K)) return STP_EUNSUPPORTED;
  TileChoice c;
  if (!ctx->concurrent && !a->tile_m && longer_together(a, &c)) return STP_EUNSUPPORTED;
  Epi ep = make_epi(a);
  ep.C2 = (bf16_t *)up;
  ep.C3 = (bf16_t *)act;
  ep.ld2 = a->ldc;
  c = tile_for(ctx, a, true, false, false, 2L * a->N, a->K, true);
  return a->K % DK ? launch_two_tile<false, EPI_SWIGLU_FWD, true, MM_PAIR>(ctx, a, c, ep, nullptr, B2, s)
                   : launch_two_tile<false, EPI_SWIGLU_FWD, false, MM_PAIR>(ctx, a, c, ep, nullptr, B2, s);
}

int stp_launch_gemm_bf16_swiglu_bwd(stp_ctx *ctx, const stp_gemm_args *a, const void *gate, const void *up, void *dup, hipStream_t s) {
  Epi ep = make_epi(a);
  ep.C2 = (bf16_t *)dup;
  ep.aux = (const bf16_t *)gate;
  ep.aux2 = (const bf16_t *)up;
  ep.ld2 = a->ldc;
  return launch_tile<true, true, EPI_SWIGLU_BWD>(ctx, a, ep, s);
}

int stp_launch_gemm_bf16_sum(stp_ctx *ctx, const stp_gemm_args *a, const void *A2, const void *B2, hipStream_t s) {
  if (!addressable(a, true)) return STP_EUNSUPPORTED;
  const Epi ep = make_epi(a);
  if (wavek_shape(a->M, a->N, 2L * a->K))
    return a->K % 64 ? launch_wavek<64, true, true, EPI_STORE, true, MM_SUM>(ctx, a, ep, s, A2, B2)
                     : launch_wavek<64, true, true, EPI_STORE, false, MM_SUM>(ctx, a, ep, s, A2, B2);
  const TileChoice c = tile_for(ctx, a, true, true, false, a->N, 2L * a->K);
  return a->K % DK ? launch_two_tile<true, EPI_STORE, true, MM_SUM>(ctx, a, c, ep, A2, B2, s)
                   : launch_two_tile<true, EPI_STORE, false, MM_SUM>(ctx, a, c, ep, A2, B2, s);
}
