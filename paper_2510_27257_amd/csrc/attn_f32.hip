// Attention forward / backward of the fp32 configuration on the fp32 matrix instruction v_mfma_f32_32x32x2_f32
// (true fp32 products and sums; any head dimension that is a multiple of 8, up to 128).
//
// A workgroup owns 32 queries of one head (forward, dQ) or 32 keys of one key / value head (dK, dV); its waves
// share out the 32-row blocks of the other index (for dK / dV: the pairs of a query head of the group and a query
// block) and their results are merged through LDS in wave order, so every sum has a fixed order.
// Scores are formed transposed in the forward and dQ (S^T = K Q^T: a lane's accumulator column is one query, the
// softmax statistics are per-lane scalars) and straight for dK / dV (the column is one key).  Either way the
// accumulator is the B operand of the following product as it stands: with the pair of contraction indices
// (8 j + r, 8 j + 4 + r) given to the two lane halves, its register 4 j + r is the value instruction 4 j + r wants.
// Operands come straight from L2, as in the fp32 GEMM: 8 consecutive floats per lane where the contraction runs along
// the row, one float per lane (32 lanes contiguous) where it runs across rows.
//
// What bounds it: latency.  At 128 tokens and 4 heads of 64 there are 16 workgroups, and a wave works through one or
// two 32 x 32 blocks (32 + 32 matrix instructions of 64 clocks each in the forward).  One wave per row with a
// cross-lane reduction per score was a chain of 128 such reductions: forward / dQ / dK dV 91 / 56 / 46 us against
// 10 / 11 / 16 us.  So few workgroups take row dot, dQ and dK / dV in one launch: 27.0 -> 14.3 us (see one_launch).
#include "attn_f32_rows.h"
#include <type_traits>

int stp_launch_rowdot(stp_ctx *ctx, const stp_layer_desc *d, const void *a, const void *b, float *delta, hipStream_t s);

namespace {

constexpr int RB = 32;      // rows (queries or keys) of a workgroup and of a step

__device__ __forceinline__ f32x16_t mfma_f32(float a, float b, f32x16_t c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

// 8 values of a row for contraction chunk c (16 deep): index 16 c + 8 (lane / 32) .. +7, zero past d (a multiple of 8)
__device__ __forceinline__ void row_chunk(float (&f)[8], const float *__restrict__ row, int c, int lg, int d) {
  const int k = 16 * c + 8 * lg;
  const bool ok = k < d;
  const float *q = row + (ok ? k : 0);
  const float4 u = *reinterpret_cast<const float4 *>(q), v = *reinterpret_cast<const float4 *>(q + 4);
  f[0] = u.x; f[1] = u.y; f[2] = u.z; f[3] = u.w; f[4] = v.x; f[5] = v.y; f[6] = v.z; f[7] = v.w;
#pragma unroll
  for (int i = 0; i < 8; i++) f[i] = ok ? f[i] : 0.f;
}
__device__ __forceinline__ void zero(f32x16_t &a) {
#pragma unroll
  for (int v = 0; v < 16; v++) a[v] = 0.f;
}
// row of accumulator register v within its 32 x 32 block
__device__ __forceinline__ int acc_row(int v, int lg) { return 8 * (v >> 2) + 4 * lg + (v & 3); }

// acc^T[column][.] += X^T p over 32 rows of X: instruction v takes rows acc_row(v, 0) and acc_row(v, 1); rows past the
// end are read from the last one (their p is zero), columns past d land in accumulator rows that are never stored
template <int DB>
__device__ __forceinline__ void add_rows(f32x16_t (&acc)[DB], const float *__restrict__ x, size_t ld, int row0, int last, const f32x16_t &p,
                                         int lr, int lg, int d) {
#pragma unroll
  for (int v = 0; v < 16; v++) {
    const float *r = x + (size_t)min(row0 + acc_row(v, lg), last) * ld;
#pragma unroll
    for (int i = 0; i < DB; i++) acc[i] = mfma_f32(r[min(32 * i + lr, d - 1)], p[v], acc[i]);
  }
}

// Rows that take no part in a column (the causal mask, the end of the sequence) have p = 0 in add_rows, but the matrix instruction
// multiplies them all the same, and 0 * inf or 0 * NaN makes a sum NaN that should not see them.  Looking at every operand takes
// the kernel a quarter longer; the accumulators show it too, so they are looked at once, after the last block (0 - 5 % of the
// shortest sequences' time): if one of the workgroup's is not finite (merge_waves says so), its rows are computed one by one
// instead (attn_f32_rows.h).
template <int DB> __device__ __forceinline__ float zero_or_nan(const f32x16_t (&acc)[DB]) {
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < DB; i++)
#pragma unroll
    for (int v = 0; v < 16; v++) s[v & 7] = fmaf(acc[i][v], 0.f, s[v & 7]);
  return ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
}

// The waves' accumulators to LDS, then their sum in wave order with a factor per wave and column, four consecutive
// columns of one row at a time: put(row 0..31, first of four columns, values).  False, and nothing put, if a lane of the workgroup
// brings a `nan` that is not zero.
template <int DB, int NW, typename Factor, typename Put>
__device__ __forceinline__ bool merge_waves(const f32x16_t (&acc)[DB], float nan, float *red, int wave, int lane, int d, Factor factor, Put put) {
  int *flags = reinterpret_cast<int *>(red + NW * (DB * 1024 + 64));
#pragma unroll
  for (int i = 0; i < DB; i++)
#pragma unroll
    for (int v = 0; v < 16; v++) red[((wave * DB + i) * 16 + v) * 64 + lane] = acc[i][v];
  const bool bad = __builtin_amdgcn_ballot_w64(nan != 0.f) != 0;
  if (lane == 0) flags[wave] = bad;
  __syncthreads();
  int any = 0;
#pragma unroll
  for (int w = 0; w < NW; w++) any |= flags[w];
  if (__builtin_amdgcn_readfirstlane(any)) return false;
  for (int q = wave; q < 4 * DB; q += NW) {        // group q: block q / 4, registers 4 (q % 4) .. +3
    const int col = 32 * (q >> 2) + 8 * (q & 3) + 4 * (lane >> 5);
    float s[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; w++) {
      const float fw = factor(w);
#pragma unroll
      for (int r = 0; r < 4; r++) s[r] += red[(w * DB * 16 + 4 * q + r) * 64 + lane] * fw;
    }
    if (col < d) put(lane & 31, col, make_float4(s[0], s[1], s[2], s[3]));
  }
  return true;
}

// A launch has a workgroup for every (32-row block, head and sequence) pair, up to tens of millions: block-fastest numbers over a
// two-dimensional grid, whose second dimension is 1 up to 2^20 of them (a dimension alone holds 2^32 threads, or 65535 workgroups).
struct Work { int block, pair; };
__device__ __forceinline__ Work work_of(int nblk) {
  const unsigned id = blockIdx.y * gridDim.x + blockIdx.x;
  return {(int)(id % nblk), (int)(id / nblk)};
}
dim3 work_grid(int nblk, size_t pairs) {
  const size_t total = nblk * pairs, x = total < (1u << 20) ? total : (1u << 20);
  return dim3((unsigned)x, (unsigned)((total + x - 1) / x));
}

template <int DB, int NW>
__global__ __launch_bounds__(64 * NW) void attn_fwd_f32_kernel(const float *__restrict__ qkv, float *__restrict__ out, float *__restrict__ lse,
                                                               int seq, int n, int nk, int pairs, int d, int causal, float scale) {
  extern __shared__ __attribute__((aligned(16))) float red[];      // [NW][DB * 16][64], then m [NW][32], l [NW][32], flags [NW]
  float *red_m = red + NW * DB * 1024, *red_l = red_m + NW * 32;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 31, lg = lane >> 5;
  const int nblk = (seq + RB - 1) / RB;
  const Work w = work_of(nblk);
  if (w.pair >= pairs) return;
  const int q0 = (nblk - 1 - w.block) * RB;        // the late blocks, which see the most keys, first
  const int head = w.pair % n, b = w.pair / n;
  const int a = n * d;
  const size_t ld = (size_t)(n + 2 * nk) * d;
  const float *base = qkv + (size_t)b * seq * ld;
  const float *kp = base + a + (head / (n / nk)) * d, *vp = kp + nk * d;
  const int qg = q0 + lr;
  const float *qrow = base + (size_t)min(qg, seq - 1) * ld + head * d;
  float qf[2 * DB][8];
#pragma unroll
  for (int c = 0; c < 2 * DB; c++) row_chunk(qf[c], qrow, c, lg, d);
  f32x16_t o[DB];
#pragma unroll
  for (int i = 0; i < DB; i++) zero(o[i]);
  float m = -INFINITY, l = 0.f;
  const int kend = causal ? min(seq, q0 + RB) : seq;
  for (int k0 = wave * RB; k0 < kend; k0 += NW * RB) {
    const float *krow = kp + (size_t)min(k0 + lr, seq - 1) * ld;
    f32x16_t sc;
    zero(sc);
#pragma unroll
    for (int c = 0; c < 2 * DB; c++) {
      float kf[8];
      row_chunk(kf, krow, c, lg, d);
#pragma unroll
      for (int e = 0; e < 8; e++) sc = mfma_f32(kf[e], qf[c][e], sc);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int key = k0 + acc_row(v, lg);
      sc[v] = (key >= seq || (causal && key > qg)) ? -INFINITY : sc[v] * scale;
      mx = fmaxf(mx, sc[v]);
    }
    mx = fmaxf(mx, other_half(mx));
    const float mn = fmaxf(m, mx);                 // finite: key k0 is admissible for every query of the block
    const float corr = expf(m - mn);
    float rs = 0.f;
#pragma unroll
    for (int v = 0; v < 16; v++) { sc[v] = expf(sc[v] - mn); rs += sc[v]; }
    l = l * corr + rs + other_half(rs);
    m = mn;
#pragma unroll
    for (int i = 0; i < DB; i++)
#pragma unroll
      for (int v = 0; v < 16; v++) o[i][v] *= corr;
    add_rows<DB>(o, vp, ld, k0, seq - 1, sc, lr, lg, d);
  }
  if (lg == 0) { red_m[wave * 32 + lr] = m; red_l[wave * 32 + lr] = l; }
  __syncthreads();
  float M = -INFINITY, L = 0.f;
#pragma unroll
  for (int w = 0; w < NW; w++) M = fmaxf(M, red_m[w * 32 + lr]);
#pragma unroll
  for (int w = 0; w < NW; w++) L += red_l[w * 32 + lr] * expf(red_m[w * 32 + lr] - M);     // a wave without keys: exp(-inf) = 0
  const float inv = 1.0f / L;
  if (!merge_waves<DB, NW>(o, zero_or_nan(o), red, wave, lane, d, [&](int w) { return expf(red_m[w * 32 + lr] - M) * inv; },
                           [&](int r, int col, float4 s) {
                             if (q0 + r < seq) *reinterpret_cast<float4 *>(out + ((size_t)b * seq + q0 + r) * a + head * d + col) = s;
                           })) {
    for (int i = q0 + wave; i < min(q0 + RB, seq); i += NW) attn_fwd_row(qkv, out, lse, b, head, i, seq, n, nk, d, causal, scale);
    return;
  }
  if (wave == 0 && lg == 0 && qg < seq) lse[((size_t)b * n + head) * seq + qg] = M + logf(L);
}

// delta = rowsum(dO o O) of a row from the half of its columns that a lane holds as chunks, in the order of the row dot kernels:
// 8 columns one after the other, then pairwise.  (Columns past d are zero and add nothing.)
template <int DB>
__device__ __forceinline__ float row_delta(const float (&gf)[2 * DB][8], const float *__restrict__ orow, int lg, int d) {
  float t[2 * DB];
#pragma unroll
  for (int c = 0; c < 2 * DB; c++) {
    float of[8], s = 0.f;
    row_chunk(of, orow, c, lg, d);
#pragma unroll
    for (int e = 0; e < 8; e++) s += gf[c][e] * of[e];
    t[c] = s + other_half(s);
  }
#pragma unroll
  for (int h = 1; h < 2 * DB; h *= 2)
#pragma unroll
    for (int c = 0; c < 2 * DB; c += 2 * h) t[c] += t[c + h];
  return t[0];
}

// FROM_OUT: delta is formed from the attention output `out`, and written where it is read otherwise
template <int DB, int NW, bool FROM_OUT>
__device__ __forceinline__ void attn_bwd_dq_f32_block(Work w, const float *__restrict__ qkv, const float *__restrict__ lse,
                                                      const float *__restrict__ dout, const float *__restrict__ out, float *__restrict__ delta,
                                                      float *__restrict__ dqkv, int seq, int n, int nk, int d, int causal, float scale, float *red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 31, lg = lane >> 5;
  const int nblk = (seq + RB - 1) / RB;
  const int q0 = (nblk - 1 - w.block) * RB;
  const int head = w.pair % n, b = w.pair / n;
  const int a = n * d;
  const size_t ld = (size_t)(n + 2 * nk) * d;
  const float *base = qkv + (size_t)b * seq * ld;
  const float *kp = base + a + (head / (n / nk)) * d, *vp = kp + nk * d;
  const int qg = q0 + lr, qc = min(qg, seq - 1);
  const float *qrow = base + (size_t)qc * ld + head * d, *grow = dout + ((size_t)b * seq + qc) * a + head * d;
  const float L = lse[((size_t)b * n + head) * seq + qc];
  float qf[2 * DB][8], gf[2 * DB][8];
#pragma unroll
  for (int c = 0; c < 2 * DB; c++) { row_chunk(qf[c], qrow, c, lg, d); row_chunk(gf[c], grow, c, lg, d); }
  const float D = FROM_OUT ? row_delta<DB>(gf, out + ((size_t)b * seq + qc) * a + head * d, lg, d) : delta[((size_t)b * n + head) * seq + qc];
  f32x16_t dq[DB];
#pragma unroll
  for (int i = 0; i < DB; i++) zero(dq[i]);
  const int kend = causal ? min(seq, q0 + RB) : seq;
  for (int k0 = wave * RB; k0 < kend; k0 += NW * RB) {
    const size_t off = (size_t)min(k0 + lr, seq - 1) * ld;
    f32x16_t sc, dp;
    zero(sc);
    zero(dp);
#pragma unroll
    for (int c = 0; c < 2 * DB; c++) {
      float kf[8], vf[8];
      row_chunk(kf, kp + off, c, lg, d);
      row_chunk(vf, vp + off, c, lg, d);
#pragma unroll
      for (int e = 0; e < 8; e++) { sc = mfma_f32(kf[e], qf[c][e], sc); dp = mfma_f32(vf[e], gf[c][e], dp); }
    }
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int key = k0 + acc_row(v, lg);
      sc[v] = (key >= seq || (causal && key > qg)) ? 0.f : expf(sc[v] * scale - L) * (dp[v] - D) * scale;
    }
    add_rows<DB>(dq, kp, ld, k0, seq - 1, sc, lr, lg, d);
  }
  if (!merge_waves<DB, NW>(dq, zero_or_nan(dq), red, wave, lane, d, [](int) { return 1.0f; },
                           [&](int r, int col, float4 s) {
                             if (q0 + r < seq) *reinterpret_cast<float4 *>(dqkv + ((size_t)b * seq + q0 + r) * ld + head * d + col) = s;
                           }))
    for (int i = q0 + wave; i < min(q0 + RB, seq); i += NW)
      attn_bwd_dq_row(qkv, lse, dout, FROM_OUT ? out : nullptr, delta, dqkv, b, head, i, seq, n, nk, d, causal, scale);
  // (last: loads behind a store wait for it)
  if (FROM_OUT && wave == 0 && lg == 0 && qg < seq) delta[((size_t)b * n + head) * seq + qg] = D;
}

// sums over the query heads of the key / value head's group
template <int DB, int NW, bool FROM_OUT>
__device__ __forceinline__ void attn_bwd_dkv_f32_block(Work w, const float *__restrict__ qkv, const float *__restrict__ lse,
                                                       const float *__restrict__ dout, const float *__restrict__ out, const float *__restrict__ delta,
                                                       float *__restrict__ dqkv, int seq, int n, int nk, int d, int causal, float scale, float *red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lr = lane & 31, lg = lane >> 5;
  const int k0 = w.block * RB;                               // the early blocks, which most queries see, first
  const int kh = w.pair % nk, b = w.pair / nk;
  const int a = n * d, group = n / nk;
  const size_t ld = (size_t)(n + 2 * nk) * d;
  const float *base = qkv + (size_t)b * seq * ld;
  const int key = k0 + lr;
  const float *krow = base + (size_t)min(key, seq - 1) * ld + a + kh * d, *vrow = krow + nk * d;
  float kf[2 * DB][8], vf[2 * DB][8];
#pragma unroll
  for (int c = 0; c < 2 * DB; c++) { row_chunk(kf[c], krow, c, lg, d); row_chunk(vf[c], vrow, c, lg, d); }
  f32x16_t dk[DB], dv[DB];
#pragma unroll
  for (int i = 0; i < DB; i++) { zero(dk[i]); zero(dv[i]); }
  const int first = causal ? k0 / RB : 0, nblk = (seq + RB - 1) / RB - first;
  for (int u = wave; u < group * nblk; u += NW) {
    const int head = kh * group + u / nblk, q0 = (first + u % nblk) * RB;
    const float *qp = base + head * d, *gp = dout + (size_t)b * seq * a + head * d;
    const size_t row = min(q0 + lr, seq - 1);
    const float *Lr = lse + ((size_t)b * n + head) * seq;
    [[maybe_unused]] const float *Dr = FROM_OUT ? nullptr : delta + ((size_t)b * n + head) * seq;
    float Lrow = 0.f, Drow = 0.f;                            // FROM_OUT: of this lane's query
    if constexpr (FROM_OUT) {
      float gf[2 * DB][8];
#pragma unroll
      for (int c = 0; c < 2 * DB; c++) row_chunk(gf[c], gp + row * a, c, lg, d);
      Lrow = Lr[row];
      Drow = row_delta<DB>(gf, out + ((size_t)b * seq + row) * a + head * d, lg, d);
    }
    f32x16_t p, ds;
    zero(p);
    zero(ds);
#pragma unroll
    for (int c = 0; c < 2 * DB; c++) {
      float qf[8], gf[8];
      row_chunk(qf, qp + row * ld, c, lg, d);
      row_chunk(gf, gp + row * a, c, lg, d);
#pragma unroll
      for (int e = 0; e < 8; e++) { p = mfma_f32(qf[e], kf[c][e], p); ds = mfma_f32(gf[e], vf[c][e], ds); }
    }
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int i = q0 + acc_row(v, lg), ic = min(i, seq - 1);
      const float Li = FROM_OUT ? __shfl(Lrow, acc_row(v, lg)) : Lr[ic], Di = FROM_OUT ? __shfl(Drow, acc_row(v, lg)) : Dr[ic];
      const bool masked = i >= seq || (causal && key > i);
      const float e = masked ? 0.f : expf(p[v] * scale - Li);
      ds[v] = masked ? 0.f : e * (ds[v] - Di) * scale;
      p[v] = e;
    }
    add_rows<DB>(dv, gp, a, q0, seq - 1, p, lr, lg, d);
    add_rows<DB>(dk, qp, ld, q0, seq - 1, ds, lr, lg, d);
  }
  float *dkp = dqkv + (size_t)b * seq * ld + a + kh * d, *dvp = dkp + nk * d;
  if (!merge_waves<DB, NW>(dk, zero_or_nan(dk) + zero_or_nan(dv), red, wave, lane, d, [](int) { return 1.0f; },
                           [&](int r, int col, float4 s) { if (k0 + r < seq) *reinterpret_cast<float4 *>(dkp + (size_t)(k0 + r) * ld + col) = s; })) {
    for (int j = k0 + wave; j < min(k0 + RB, seq); j += NW)
      attn_bwd_dkv_row(qkv, lse, dout, FROM_OUT ? out : nullptr, delta, dqkv, b, kh, j, seq, n, nk, d, causal, scale);
    return;
  }
  __syncthreads();
  merge_waves<DB, NW>(dv, 0.f, red, wave, lane, d, [](int) { return 1.0f; },
                      [&](int r, int col, float4 s) { if (k0 + r < seq) *reinterpret_cast<float4 *>(dvp + (size_t)(k0 + r) * ld + col) = s; });
}

template <int DB, int NW>
__global__ __launch_bounds__(64 * NW) void attn_bwd_dq_f32_kernel(const float *__restrict__ qkv, const float *__restrict__ lse,
                                                                  const float *__restrict__ dout, float *__restrict__ delta,
                                                                  float *__restrict__ dqkv, int seq, int n, int nk, int pairs, int d, int causal,
                                                                  float scale) {
  extern __shared__ __attribute__((aligned(16))) float red[];
  const Work w = work_of((seq + RB - 1) / RB);
  if (w.pair < pairs) attn_bwd_dq_f32_block<DB, NW, false>(w, qkv, lse, dout, nullptr, delta, dqkv, seq, n, nk, d, causal, scale, red);
}
template <int DB, int NW>
__global__ __launch_bounds__(64 * NW) void attn_bwd_dkv_f32_kernel(const float *__restrict__ qkv, const float *__restrict__ lse,
                                                                   const float *__restrict__ dout, const float *__restrict__ delta,
                                                                   float *__restrict__ dqkv, int seq, int n, int nk, int pairs, int d, int causal,
                                                                   float scale) {
  extern __shared__ __attribute__((aligned(16))) float red[];
  const Work w = work_of((seq + RB - 1) / RB);
  if (w.pair < pairs) attn_bwd_dkv_f32_block<DB, NW, false>(w, qkv, lse, dout, nullptr, delta, dqkv, seq, n, nk, d, causal, scale, red);
}
// Row dot, dK / dV and dQ in one launch, for so few workgroups that they are all resident at once: see one_launch.
// nblk * pairs_kv workgroups for dK / dV, then nblk * pairs for dQ.
template <int DB, int NW>
__global__ __launch_bounds__(64 * NW) void attn_bwd_f32_kernel(const float *__restrict__ qkv, const float *__restrict__ lse,
                                                               const float *__restrict__ dout, const float *__restrict__ out,
                                                               float *__restrict__ delta, float *__restrict__ dqkv, int seq, int n, int nk,
                                                               int pairs_kv, int d, int causal, float scale) {
  extern __shared__ __attribute__((aligned(16))) float red[];
  const int nblk = (seq + RB - 1) / RB, first_dq = nblk * pairs_kv, id = blockIdx.x;
  if (id < first_dq) {
    attn_bwd_dkv_f32_block<DB, NW, true>({id % nblk, id / nblk}, qkv, lse, dout, out, nullptr, dqkv, seq, n, nk, d, causal, scale, red);
  } else {
    const int i = id - first_dq;
    attn_bwd_dq_f32_block<DB, NW, true>({i % nblk, i / nblk}, qkv, lse, dout, out, delta, dqkv, seq, n, nk, d, causal, scale, red);
  }
}

// The same for sequences of a few rows, a wave per row: a block of 32 would be mostly empty.
__global__ __launch_bounds__(256) void attn_fwd_rows_kernel(const float *__restrict__ qkv, float *__restrict__ out, float *__restrict__ lse, int seq,
                                                            int mbsz, int n, int nk, int d, int causal, float scale) {
  const size_t w = blockIdx.x * (size_t)4 + (threadIdx.x >> 6);
  if (w >= (size_t)mbsz * n * seq) return;
  attn_fwd_row(qkv, out, lse, w / ((size_t)seq * n), (w / seq) % n, w % seq, seq, n, nk, d, causal, scale);
}
__global__ __launch_bounds__(256) void attn_bwd_dq_rows_kernel(const float *__restrict__ qkv, const float *__restrict__ lse,
                                                               const float *__restrict__ dout, const float *__restrict__ delta,
                                                               float *__restrict__ dqkv, int seq, int mbsz, int n, int nk, int d, int causal,
                                                               float scale) {
  const size_t w = blockIdx.x * (size_t)4 + (threadIdx.x >> 6);
  if (w >= (size_t)mbsz * n * seq) return;
  attn_bwd_dq_row(qkv, lse, dout, nullptr, delta, dqkv, w / ((size_t)seq * n), (w / seq) % n, w % seq, seq, n, nk, d, causal, scale);
}
__global__ __launch_bounds__(256) void attn_bwd_dkv_rows_kernel(const float *__restrict__ qkv, const float *__restrict__ lse,
                                                                const float *__restrict__ dout, const float *__restrict__ delta,
                                                                float *__restrict__ dqkv, int seq, int mbsz, int n, int nk, int d, int causal,
                                                                float scale) {
  const size_t w = blockIdx.x * (size_t)4 + (threadIdx.x >> 6);
  if (w >= (size_t)mbsz * nk * seq) return;
  attn_bwd_dkv_row(qkv, lse, dout, nullptr, delta, dqkv, w / ((size_t)seq * nk), (w / seq) % nk, w % seq, seq, n, nk, d, causal, scale);
}

// Waves per workgroup: 8 (4 at head dimensions above 64, whose merge area is twice as large), 1 or 2 where there are only so many
// 32-row blocks to share out: a workgroup whose other waves have none holds a compute unit's registers and LDS for nothing (4096
// sequences of 32 rows of dimension 64, forward / backward: 182 / 316 us with 8 waves, 41 / 115 with one; 64 rows 378 / 722, 116 / 448).
template <int NW, int DB> constexpr size_t lds_of = (size_t)NW * (DB * 1024 + 65) * sizeof(float);
template <int DB, typename Launch>
int with_waves(int blocks, Launch launch) {
  constexpr int MOST = DB <= 2 ? 8 : 4;
  if (blocks <= 1) return launch(std::integral_constant<int, 1>{});
  if (blocks <= 2) return launch(std::integral_constant<int, 2>{});
  return launch(std::integral_constant<int, MOST>{});
}

struct Shape { int seq, mbsz, n, nk, d, causal, nblk; size_t pairs, pairs_kv; float scale; };

// Up to how many rows a sequence is better off with a wave per row (kind 0 forward, 1 dQ, 2 dK / dV).  With few rows in all both
// are a chain of latencies: the row's, one reduction per key (dK / dV: per query of each head of the group), against that of a
// block or, where a wave has several of them, of its blocks; with many, what counts is how much of a block is empty.  Measured over
// 1 .. 64 rows, 8 .. 4096 (head, sequence) pairs, dimensions 8 .. 128, groups of 1, 4 and 8.  Forward + backward, rows / blocks in us:
// 8 pairs of 8 rows of 64: 17 / 30; of 128: 19 / 52; of 24 rows of 64: 33 / 32; 4096 pairs of 4 rows of 64: 36 / 91, 12 rows: 148 / 108.
bool short_rows(const Shape &h, int kind) {
  static const int few[3][3] = {{8, 12, 16}, {8, 16, 40}, {24, 32, 64}}, many[3][3] = {{4, 4, 8}, {4, 4, 12}, {4, 8, 16}};
  const int w = h.d <= 32 ? 0 : h.d <= 64 ? 1 : 2;
  if (h.pairs * h.seq > 4096) return h.seq <= many[kind][w];
  if (kind < 2) return h.seq <= few[kind][w];
  const int group = h.n / h.nk, waves = w == 2 ? 4 : 8;
  return (long)h.seq * group <= (long)few[2][w] * ((h.nblk * group + waves - 1) / waves);
}

template <int DB>
int launch_fwd(stp_ctx *ctx, const Shape &h, const float *qkv, float *out, float *lse, hipStream_t s) {
  return with_waves<DB>(h.nblk, [&](auto nw) -> int {
    constexpr int NW = decltype(nw)::value;
    auto kern = attn_fwd_f32_kernel<DB, NW>;
    static bool attr_set = false;
    if (!attr_set) {
      STP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_of<NW, DB>));
      attr_set = true;
    }
    hipLaunchKernelGGL(kern, work_grid(h.nblk, h.pairs), dim3(64 * NW), (lds_of<NW, DB>), s, qkv, out, lse, h.seq, h.n, h.nk, (int)h.pairs, h.d, h.causal,
                       h.scale);
    STP_LAUNCH_CHECK(ctx);
    return STP_OK;
  });
}
template <int DB>
int launch_dq(stp_ctx *ctx, const Shape &h, const float *qkv, const float *lse, const float *dout, float *delta, float *dqkv, hipStream_t s) {
  return with_waves<DB>(h.nblk, [&](auto nw) -> int {
    constexpr int NW = decltype(nw)::value;
    auto kern = attn_bwd_dq_f32_kernel<DB, NW>;
    static bool attr_set = false;
    if (!attr_set) {
      STP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_of<NW, DB>));
      attr_set = true;
    }
    hipLaunchKernelGGL(kern, work_grid(h.nblk, h.pairs), dim3(64 * NW), (lds_of<NW, DB>), s, qkv, lse, dout, delta, dqkv, h.seq, h.n, h.nk, (int)h.pairs,
                       h.d, h.causal, h.scale);
    STP_LAUNCH_CHECK(ctx);
    return STP_OK;
  });
}
template <int DB>
int launch_dkv(stp_ctx *ctx, const Shape &h, const float *qkv, const float *lse, const float *dout, const float *delta, float *dqkv, hipStream_t s) {
  return with_waves<DB>(h.nblk * (h.n / h.nk), [&](auto nw) -> int {
    constexpr int NW = decltype(nw)::value;
    auto kern = attn_bwd_dkv_f32_kernel<DB, NW>;
    static bool attr_set = false;
    if (!attr_set) {
      STP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_of<NW, DB>));
      attr_set = true;
    }
    hipLaunchKernelGGL(kern, work_grid(h.nblk, h.pairs_kv), dim3(64 * NW), (lds_of<NW, DB>), s, qkv, lse, dout, delta, dqkv, h.seq, h.n, h.nk,
                       (int)h.pairs_kv, h.d, h.causal, h.scale);
    STP_LAUNCH_CHECK(ctx);
    return STP_OK;
  });
}

// Up to 256 workgroups in all, one for a compute unit, the backward pass is a chain of latencies, and one launch has one of them where
// row dot, dQ and dK / dV have three: 4 heads of 64, 128 rows 27.0 -> 14.3 us; 4 heads of 32 on 2, 200 rows 37.0 -> 23.9; 8 heads of 128,
// 256 rows 97.8 -> 52.4.  More of them fill the chip with either body, and delta formed once more by every key block would cost what the
// launch saves.  The bits are the same either way.
bool one_launch(const Shape &h) {
  auto waves = [](long blocks) { return blocks <= 2 ? blocks : 3; };       // as with_waves groups them
  return !short_rows(h, 1) && !short_rows(h, 2) && h.nblk * (h.pairs + h.pairs_kv) <= STP_CUS && waves(h.nblk) == waves((long)h.nblk * (h.n / h.nk));
}
template <int DB>
int launch_bwd(stp_ctx *ctx, const Shape &h, const float *qkv, const float *lse, const float *dout, const float *out, float *delta, float *dqkv,
               hipStream_t s) {
  return with_waves<DB>(h.nblk, [&](auto nw) -> int {
    constexpr int NW = decltype(nw)::value;
    auto kern = attn_bwd_f32_kernel<DB, NW>;
    static bool attr_set = false;
    if (!attr_set) {
      STP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_of<NW, DB>));
      attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(h.nblk * (h.pairs + h.pairs_kv))), dim3(64 * NW), (lds_of<NW, DB>), s, qkv, lse, dout, out, delta, dqkv,
                       h.seq, h.n, h.nk, (int)h.pairs_kv, h.d, h.causal, h.scale);
    STP_LAUNCH_CHECK(ctx);
    return STP_OK;
  });
}

Shape shape_of(const stp_layer_desc *d) {
  const int nk = stp_kv_heads(d);
  return {d->seq, d->mbsz, d->heads_local, nk, d->head_dim, d->causal, (d->seq + RB - 1) / RB, (size_t)d->heads_local * d->mbsz, (size_t)nk * d->mbsz,
          1.0f / sqrtf((float)d->head_dim)};
}

}  // namespace

extern "C" int stp_attn_bwd_f32_launches(const stp_layer_desc *d) { return one_launch(shape_of(d)) ? 1 : 3; }

int stp_launch_attn_fwd_f32(stp_ctx *ctx, const stp_layer_desc *d, const void *qkv, void *out, float *lse, hipStream_t s) {
  const float *x = (const float *)qkv;
  float *o = (float *)out;
  const Shape h = shape_of(d);
  if (short_rows(h, 0)) {
    hipLaunchKernelGGL(attn_fwd_rows_kernel, dim3((h.pairs * h.seq + 3) / 4), dim3(256), 0, s, x, o, lse, h.seq, h.mbsz, h.n, h.nk, h.d, h.causal, h.scale);
    STP_LAUNCH_CHECK(ctx);
    return STP_OK;
  }
  return h.d <= 32 ? launch_fwd<1>(ctx, h, x, o, lse, s) : h.d <= 64 ? launch_fwd<2>(ctx, h, x, o, lse, s) : launch_fwd<4>(ctx, h, x, o, lse, s);
}

int stp_launch_attn_bwd_f32(stp_ctx *ctx, const stp_layer_desc *d, const void *qkv, const void *out, const float *lse, const void *dout,
                            float *delta, void *dqkv, hipStream_t s) {
  const float *x = (const float *)qkv, *g = (const float *)dout;
  float *dx = (float *)dqkv;
  const Shape h = shape_of(d);
  // (gradients written over the output are fine behind the row dot, not where other workgroups still read it)
  const size_t row = (size_t)h.mbsz * h.seq * h.d * sizeof(float), out_end = (size_t)out + row * h.n, dx_end = (size_t)dqkv + row * (h.n + 2 * h.nk);
  if (one_launch(h) && ((size_t)out >= dx_end || (size_t)dqkv >= out_end)) {
    const float *o = (const float *)out;
    return h.d <= 32 ? launch_bwd<1>(ctx, h, x, lse, g, o, delta, dx, s) : h.d <= 64 ? launch_bwd<2>(ctx, h, x, lse, g, o, delta, dx, s)
                                                                                   : launch_bwd<4>(ctx, h, x, lse, g, o, delta, dx, s);
  }
  int rc = stp_launch_rowdot(ctx, d, dout, out, delta, s);
  if (rc != STP_OK) return rc;
  if (short_rows(h, 1)) {
    hipLaunchKernelGGL(attn_bwd_dq_rows_kernel, dim3((h.pairs * h.seq + 3) / 4), dim3(256), 0, s, x, lse, g, delta, dx, h.seq, h.mbsz, h.n, h.nk, h.d,
                       h.causal, h.scale);
    STP_LAUNCH_CHECK(ctx);
  } else {
    rc = h.d <= 32 ? launch_dq<1>(ctx, h, x, lse, g, delta, dx, s) : h.d <= 64 ? launch_dq<2>(ctx, h, x, lse, g, delta, dx, s)
                                                                           : launch_dq<4>(ctx, h, x, lse, g, delta, dx, s);
    if (rc != STP_OK) return rc;
  }
  if (short_rows(h, 2)) {
    hipLaunchKernelGGL(attn_bwd_dkv_rows_kernel, dim3((h.pairs_kv * h.seq + 3) / 4), dim3(256), 0, s, x, lse, g, delta, dx, h.seq, h.mbsz, h.n, h.nk, h.d,
                       h.causal, h.scale);
    STP_LAUNCH_CHECK(ctx);
    return STP_OK;
  }
  return h.d <= 32 ? launch_dkv<1>(ctx, h, x, lse, g, delta, dx, s) : h.d <= 64 ? launch_dkv<2>(ctx, h, x, lse, g, delta, dx, s)
                                                                         : launch_dkv<4>(ctx, h, x, lse, g, delta, dx, s);
}
