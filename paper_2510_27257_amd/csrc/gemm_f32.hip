// fp32 GEMM of the fp32 configuration on the fp32 matrix instruction v_mfma_f32_32x32x2_f32 (true fp32 products
// and sums, no reduced-precision mode; twice the rate of scalar FMAs).
//
// What bounds it: the layers of this configuration are small (tens to hundreds of rows, K up to about a thousand),
// so a call is a chain of load latencies and of dependent products, not bytes or flops.  Hence
//   * the contraction is split over the waves of a workgroup (KS waves per output tile, added up through LDS in a
//     fixed order) and the tile is small, so that a [128, 1024] output still occupies 128 compute units and the
//     longest chain of a wave is K / KS deep;
//   * no LDS for the operands: the waves of a workgroup share nothing but the tile, the matrices sit in L2, and a
//     lane fetches exactly what its matrix instructions consume.  The order of the contraction index is free as long
//     as A and B agree, so a 16-deep chunk gives the lane halves 8 consecutive k each: two 16-byte loads of an operand
//     that is contiguous in k, 8 loads of 32 consecutive elements of one that is contiguous in its rows.  The next
//     chunk's loads are in flight under the current chunk's matrix instructions.
// Measured on a training pass of two microbatches over an unsharded layer of hidden 256 / FFN 1024, 128 tokens (24 of
// these GEMMs): 1841 us with 64 x 64 LDS tiles and scalar FMAs (80 us a GEMM: at most 32 workgroups, K one 16-deep step
// after the other), 554 us now.
#include "common.h"

namespace {
struct EpiF {
  float *C; int ldc; int accum;
  const float *bias; float bias_scale;
  const float *resid; int ldr; float resid_scale;
  int mode; float *C2; const float *aux; int ld2;
};

// The 8 values a lane feeds to a chunk's 8 matrix instructions for one 32-row block of an operand: row `row`,
// k = k0 + 8 * (lane / 32) .. +7 (all real or all past the end: K is a multiple of 8).
template <bool KC>
__device__ __forceinline__ void load_chunk(float (&f)[8], const float *__restrict__ p, size_t ld, int row, int k, bool ok) {
  if (KC) {
    const float *q = p + (size_t)row * ld + (ok ? k : 0);
    const float4 u = *reinterpret_cast<const float4 *>(q), v = *reinterpret_cast<const float4 *>(q + 4);
    f[0] = u.x; f[1] = u.y; f[2] = u.z; f[3] = u.w; f[4] = v.x; f[5] = v.y; f[6] = v.z; f[7] = v.w;
  } else {
    const float *q = p + (size_t)(ok ? k : 0) * ld + row;
#pragma unroll
    for (int i = 0; i < 8; i++) f[i] = q[(size_t)i * ld];
  }
#pragma unroll
  for (int i = 0; i < 8; i++) f[i] = ok ? f[i] : 0.f;
}

// The weight gradients of a unit that take 32 x 32 tiles, in one launch: two or three of these short kernels one after the other are mostly
// starts and ends.
struct F32Problem { const float *A, *B; float *C; int lda, ldb, ldc, M, N, tiles_n, first; };
struct F32Set { int n, K, tiles; F32Problem p[3]; };
// the workgroup's product of the set and its tile there
__device__ __forceinline__ void pick_problem(const F32Set &set, const float *&A, int &lda, const float *&B, int &ldb, int &M, int &N, int &K, EpiF &ep, int &tm, int &tn) {
  const int pid = blockIdx.x, i = set.n > 2 && pid >= set.p[2].first ? 2 : pid >= set.p[1].first ? 1 : 0;
  const F32Problem &q = set.p[i];
  A = q.A; lda = q.lda; B = q.B; ldb = q.ldb; M = q.M; N = q.N; K = set.K;
  ep = EpiF{};      // known here, so the epilogue is the short one
  ep.C = q.C; ep.ldc = q.ldc; ep.accum = 1;
  tm = (pid - q.first) / q.tiles_n;
  tn = (pid - q.first) % q.tiles_n;
}

// WT: a wave's tile is (32 WT)^2; WM x WN such tiles make the workgroup's tile; KS waves share each of them.
// Set: nothing, or the set that the product is taken from (first, so that its start comes with the first cache line of the arguments).  (One kernel for both: as a function called by two, the plain products' epilogues were
// scheduled differently, [520, 2744] K = 1032 with a row-contiguous A 62.4 -> 67.9 us, [4096, 4096] K = 512 with a transposed B 196 -> 204.)
template <int WT, int WM, int WN, int KS, bool A_KC, bool B_KC, typename... Set>
__global__ __launch_bounds__(64 * WM * WN * KS) void gemm_f32_kernel(Set... set, const float *__restrict__ A, int lda,
                                                                     const float *__restrict__ B, int ldb, int M, int N, int K, EpiF ep) {
  constexpr int TM = 32 * WT * WM, TN = 32 * WT * WN, NTH = 64 * WM * WN * KS;
  constexpr int RP = TN + 4;                          // pitch of a staged row
  extern __shared__ __attribute__((aligned(16))) float red[];   // [KS][TM][RP]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 31, lg = lane >> 5;
  const int ks = wave % KS, wt = wave / KS, wm = wt / WN, wn = wt % WN;
  int tm = blockIdx.y, tn = blockIdx.x;
  if constexpr (sizeof...(Set) > 0) {
    const float *a, *b;
    pick_problem(set..., a, lda, b, ldb, M, N, K, ep, tm, tn);
    A = a;
    B = b;
  }
  const int m0 = tm * TM, n0 = tn * TN;
  int ra[WT], rb[WT];                                 // this lane's operand rows; past the end: the last row, never stored
#pragma unroll
  for (int i = 0; i < WT; i++) {
    ra[i] = min(m0 + (wm * WT + i) * 32 + lr, M - 1);
    rb[i] = min(n0 + (wn * WT + i) * 32 + lr, N - 1);
  }
  f32x16_t acc[WT][WT];
#pragma unroll
  for (int i = 0; i < WT; i++)
#pragma unroll
    for (int j = 0; j < WT; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;
  const int nch = (K + 15) / 16;
  float fa[2][WT][8], fb[2][WT][8];
  auto fetch = [&](int c, float (&a)[WT][8], float (&b)[WT][8]) {
    const int k = 16 * c + 8 * lg;
    const bool ok = k < K;
#pragma unroll
    for (int i = 0; i < WT; i++) {
      load_chunk<A_KC>(a[i], A, lda, ra[i], k, ok);
      load_chunk<B_KC>(b[i], B, ldb, rb[i], k, ok);
    }
  };
  auto mac = [&](const float (&a)[WT][8], const float (&b)[WT][8]) {
#pragma unroll
    for (int e = 0; e < 8; e++)
#pragma unroll
      for (int i = 0; i < WT; i++)
#pragma unroll
        for (int j = 0; j < WT; j++) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][e], b[j][e], acc[i][j], 0, 0, 0);
  };
  // chunks ks, ks + KS, ... in pairs, so that the two register sets are named at compile time; a chunk past the end is all zeros
  if (ks < nch) fetch(ks, fa[0], fb[0]);
  for (int c = ks; c < nch; c += 2 * KS) {
    if (c + KS < nch) fetch(c + KS, fa[1], fb[1]);
    mac(fa[0], fb[0]);
    if (c + KS >= nch) break;
    if (c + 2 * KS < nch) fetch(c + 2 * KS, fa[0], fb[0]);
    mac(fa[1], fb[1]);
  }
  // accumulator v of lane l: row 8 * (v / 4) + 4 * (l / 32) + v % 4, column l % 32
  if constexpr (KS == 1) {                             // nothing to add up: straight from the registers, 32 neighbouring columns per store
#pragma unroll
    for (int i = 0; i < WT; i++)
#pragma unroll
      for (int j = 0; j < WT; j++) {
        const int col = n0 + (wn * WT + j) * 32 + lr;
        if (col >= N) continue;
        const float bias = ep.bias ? ep.bias[col] * ep.bias_scale : 0.f;
        const int row0 = m0 + (wm * WT + i) * 32 + 4 * lg;
        float other[16];                               // the old sum or the GELU' argument (never both), read together
        if (ep.accum || ep.mode == 2) {
          const float *p = ep.accum ? ep.C : ep.aux;
          const int ld = ep.accum ? ep.ldc : ep.ld2;
#pragma unroll
          for (int v = 0; v < 16; v++) other[v] = p[(size_t)min(row0 + 8 * (v >> 2) + (v & 3), M - 1) * ld + col];
        }
#pragma unroll
        for (int v = 0; v < 16; v++) {
          const int row = row0 + 8 * (v >> 2) + (v & 3);
          if (row >= M) continue;
          float val = acc[i][j][v] + bias;
          if (ep.resid) val += ep.resid[(size_t)row * ep.ldr + col] * ep.resid_scale;
          if (ep.mode == 2) val *= gelu_grad_f(other[v]);
          if (ep.accum) val += other[v];
          ep.C[(size_t)row * ep.ldc + col] = val;
          if (ep.mode == 1) ep.C2[(size_t)row * ep.ld2 + col] = gelu_f(val);
        }
      }
    return;
  }
#pragma unroll
  for (int i = 0; i < WT; i++)
#pragma unroll
    for (int j = 0; j < WT; j++)
#pragma unroll
      for (int v = 0; v < 16; v++)
        red[(size_t)(ks * TM + (wm * WT + i) * 32 + 8 * (v >> 2) + 4 * lg + (v & 3)) * RP + (wn * WT + j) * 32 + lr] = acc[i][j][v];
  __syncthreads();
  // the KS partial tiles in order, then the epilogue, two neighbouring columns per thread
  for (int q = tid; q < TM * TN / 2; q += NTH) {
    const int r = q / (TN / 2), c = (q % (TN / 2)) * 2;
    const int row = m0 + r, col = n0 + c;
    float2 s = make_float2(0.f, 0.f);
#pragma unroll
    for (int k = 0; k < KS; k++) {
      const float2 p = *reinterpret_cast<const float2 *>(red + (size_t)(k * TM + r) * RP + c);
      s.x += p.x; s.y += p.y;
    }
    if (row >= M || col >= N) continue;               // N is even
    float val[2] = {s.x, s.y};
#pragma unroll
    for (int e = 0; e < 2; e++) {
      if (ep.bias) val[e] += ep.bias[col + e] * ep.bias_scale;
      if (ep.resid) val[e] += ep.resid[(size_t)row * ep.ldr + col + e] * ep.resid_scale;
      if (ep.mode == 2) val[e] *= gelu_grad_f(ep.aux[(size_t)row * ep.ld2 + col + e]);
    }
    float2 *cp = reinterpret_cast<float2 *>(ep.C + (size_t)row * ep.ldc + col);
    if (ep.accum) { const float2 old = *cp; val[0] += old.x; val[1] += old.y; }
    *cp = make_float2(val[0], val[1]);
    if (ep.mode == 1) {
      ep.C2[(size_t)row * ep.ld2 + col] = gelu_f(val[0]);
      ep.C2[(size_t)row * ep.ld2 + col + 1] = gelu_f(val[1]);
    }
  }
}

template <int WT, int WM, int WN, int KS, bool A_KC, bool B_KC>
int launch_f32(stp_ctx *ctx, const stp_gemm_args *a, const EpiF &ep, hipStream_t s) {
  constexpr int TM = 32 * WT * WM, TN = 32 * WT * WN;
  constexpr size_t smem = KS == 1 ? 0 : (size_t)KS * TM * (TN + 4) * sizeof(float);
  static_assert(smem <= 160 * 1024, "LDS budget");
  auto kern = gemm_f32_kernel<WT, WM, WN, KS, A_KC, B_KC>;
  static bool attr_set = false;
  if (smem > 64 * 1024 && !attr_set) {
    STP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    attr_set = true;
  }
  hipLaunchKernelGGL(kern, dim3((a->N + TN - 1) / TN, (a->M + TM - 1) / TM), dim3(64 * WM * WN * KS), smem, s, (const float *)a->A,
                     a->lda, (const float *)a->B, a->ldb, a->M, a->N, a->K, ep);
  STP_LAUNCH_CHECK(ctx);
  return STP_OK;
}

// Tile: the largest of the three that still gives most of the 256 compute units a workgroup (a larger wave tile
// reads fewer operand bytes per product: 32 B per clock and compute unit at 32 x 32, half of that at 64 x 64), and that is not
// mostly past the end of a narrow output.
// Short contractions of outputs large enough to fill the chip are bound by the output, not by a chain: there the contraction is
// not split, nothing passes through LDS and 32 x 32 tiles store from the registers.  us, split / not (scalar FMAs on LDS tiles before
// either): [4096, 4096] K = 8: 33 / 20 (20), added to C 53 / 28 (28), K = 64: 49 / 43 (51); [65536, 32] K = 128: 37 / 14 (31).  Past
// K = 80 the chain counts again ([1024, 1024] K = 96: 7.8 / 8.5), for narrow outputs of very many tiles past 128.
inline long f32_tiles(const stp_gemm_args *a, long t) { return ((a->M + t - 1) / t) * ((a->N + t - 1) / t); }
inline bool f32_unsplit(const stp_gemm_args *a) { return a->K <= 80 || (a->K <= 128 && (a->M <= 64 || a->N <= 64) && f32_tiles(a, 64) >= 512); }
// whether the product takes the 32 x 32 tile of eight waves (the last choice below)
inline bool f32_small(const stp_gemm_args *a) {
  if (f32_unsplit(a) && ((f32_tiles(a, 64) >= 192 && a->M > 32 && a->N > 32) || (f32_tiles(a, 32) >= 512 && (a->M <= 32 || a->N <= 32)))) return false;
  return !(f32_tiles(a, 128) >= 192 && a->M > 64 && a->N > 64) && !(f32_tiles(a, 64) >= 192 && a->M > 32 && a->N > 32);
}
template <bool A_KC, bool B_KC>
int launch_f32_layout(stp_ctx *ctx, const stp_gemm_args *a, const EpiF &ep, hipStream_t s) {
  auto tiles = [&](long t) { return f32_tiles(a, t); };
  if (f32_unsplit(a)) {
    if (tiles(64) >= 192 && a->M > 32 && a->N > 32) return launch_f32<1, 2, 2, 1, A_KC, B_KC>(ctx, a, ep, s);
    if (tiles(32) >= 512 && a->M <= 32) return launch_f32<1, 1, 4, 1, A_KC, B_KC>(ctx, a, ep, s);
    if (tiles(32) >= 512 && a->N <= 32) return launch_f32<1, 4, 1, 1, A_KC, B_KC>(ctx, a, ep, s);
  }
  if (tiles(128) >= 192 && a->M > 64 && a->N > 64) return launch_f32<2, 2, 2, 2, A_KC, B_KC>(ctx, a, ep, s);
  if (tiles(64) >= 192 && a->M > 32 && a->N > 32) return launch_f32<2, 1, 1, 4, A_KC, B_KC>(ctx, a, ep, s);
  return launch_f32<1, 1, 1, 8, A_KC, B_KC>(ctx, a, ep, s);
}
}  // namespace

int stp_launch_gemm_f32(stp_ctx *ctx, const stp_gemm_args *a, hipStream_t s) {
  EpiF ep;
  ep.C = (float *)a->C; ep.ldc = a->ldc; ep.accum = a->c_f32_accum;
  ep.bias = (const float *)a->bias; ep.bias_scale = a->bias_scale;
  ep.resid = (const float *)a->resid; ep.ldr = a->ldr; ep.resid_scale = a->resid_scale;
  ep.mode = a->epilogue; ep.C2 = (float *)a->C2; ep.aux = (const float *)a->aux; ep.ld2 = a->ld2;
  const bool a_kc = !a->a_trans, b_kc = a->b_trans != 0;
  if (a_kc && b_kc) return launch_f32_layout<true, true>(ctx, a, ep, s);
  if (a_kc) return launch_f32_layout<true, false>(ctx, a, ep, s);
  if (b_kc) return launch_f32_layout<false, true>(ctx, a, ep, s);
  return launch_f32_layout<false, false>(ctx, a, ep, s);
}

int stp_launch_gemm_f32_wgrads(stp_ctx *ctx, const stp_gemm_args *a, int n, hipStream_t s) {
  bool set = n > 1 && !stp_accumulators_overlap(a, n);
  for (int i = 0; i < n; i++) set = set && a[i].K > 0 && f32_small(&a[i]);
  if (!set) {
    for (int i = 0; i < n; i++) {
      const int rc = stp_launch_gemm_f32(ctx, &a[i], s);
      if (rc != STP_OK) return rc;
    }
    return STP_OK;
  }
  F32Set f = {};
  f.n = n;
  f.K = a[0].K;
  for (int i = 0; i < n; i++) {
    f.p[i] = {(const float *)a[i].A, (const float *)a[i].B, (float *)a[i].C, a[i].lda, a[i].ldb, a[i].ldc, a[i].M, a[i].N, (a[i].N + 31) / 32, f.tiles};
    f.tiles += (int)f32_tiles(&a[i], 32);
  }
  hipLaunchKernelGGL((gemm_f32_kernel<1, 1, 1, 8, false, false, F32Set>), dim3(f.tiles), dim3(512), (size_t)8 * 32 * 36 * sizeof(float), s, f, nullptr, 0, nullptr, 0, 0, 0, 0,
                     EpiF{});
  STP_LAUNCH_CHECK(ctx);
  return STP_OK;
}
