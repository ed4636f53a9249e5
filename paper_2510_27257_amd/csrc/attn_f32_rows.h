// fp32 attention, one row by one 64-lane wave: lanes split the head dimension (d <= 128) and every query-key dot product is a
// wave reduction, one key (query) after the other, only those that the row takes part with.  The block kernels of attn_f32.hip
// fall back to it where an operand is not finite.
// Grouped-query attention: nk key / value heads, query head i uses key / value head i / (n / nk); a row of qkv is
// [n Q heads | nk K heads | nk V heads].
#pragma once
#include "common.h"

// delta = rowsum(dO o O) of a row, as the row dot kernels form it
__device__ __forceinline__ float row_dot_out(const float *__restrict__ g, const float *__restrict__ o, int d) {
  const int col = (threadIdx.x & 63) * 8;
  float s = 0.f;
  if (col < d) {
    float u[8], v[8];
    Vec8<float>::load(g + col, u);
    Vec8<float>::load(o + col, v);
#pragma unroll
    for (int i = 0; i < 8; i++) s += u[i] * v[i];
  }
  return wave_sum(s);
}

// query row i of head `head` of sequence b
__device__ __forceinline__ void attn_fwd_row(const float *__restrict__ qkv, float *__restrict__ out, float *__restrict__ lse, int b, int head,
                                             int i, int seq, int n, int nk, int d, int causal, float scale) {
  const int lane = threadIdx.x & 63;
  const int a = n * d, ak = nk * d;
  const size_t ld = (size_t)a + 2 * ak;
  const float *base = qkv + (size_t)b * seq * ld;
  const bool h0 = lane < d, h1 = lane + 64 < d;
  const float *qp = base + (size_t)i * ld + head * d;
  float q0 = h0 ? qp[lane] : 0.f, q1 = h1 ? qp[lane + 64] : 0.f;
  const int jend = causal ? i + 1 : seq;
  float m = -INFINITY, l = 0.f, o0 = 0.f, o1 = 0.f;
  for (int j = 0; j < jend; j++) {
    const float *kp = base + (size_t)j * ld + a + (head / (n / nk)) * d;
    const float *vp = kp + ak;
    float part = (h0 ? q0 * kp[lane] : 0.f) + (h1 ? q1 * kp[lane + 64] : 0.f);
    float sc = wave_sum(part) * scale;
    float mn = fmaxf(m, sc);
    float corr = expf(m - mn), p = expf(sc - mn);
    l = l * corr + p;
    o0 = o0 * corr + (h0 ? p * vp[lane] : 0.f);
    o1 = o1 * corr + (h1 ? p * vp[lane + 64] : 0.f);
    m = mn;
  }
  float *op = out + ((size_t)b * seq + i) * a + head * d;
  if (h0) op[lane] = o0 / l;
  if (h1) op[lane + 64] = o1 / l;
  if (lane == 0) lse[((size_t)b * n + head) * seq + i] = m + logf(l);
}

// delta from the output `out`, or, without it, from memory
__device__ __forceinline__ void attn_bwd_dq_row(const float *__restrict__ qkv, const float *__restrict__ lse, const float *__restrict__ dout,
                                                const float *__restrict__ out, const float *__restrict__ delta, float *__restrict__ dqkv, int b,
                                                int head, int i, int seq, int n, int nk, int d, int causal, float scale) {
  const int lane = threadIdx.x & 63;
  const int a = n * d, ak = nk * d;
  const size_t ld = (size_t)a + 2 * ak;
  const float *base = qkv + (size_t)b * seq * ld;
  const bool h0 = lane < d, h1 = lane + 64 < d;
  const float *qp = base + (size_t)i * ld + head * d;
  const float *dop = dout + ((size_t)b * seq + i) * a + head * d;
  float q0 = h0 ? qp[lane] : 0.f, q1 = h1 ? qp[lane + 64] : 0.f;
  float g0 = h0 ? dop[lane] : 0.f, g1 = h1 ? dop[lane + 64] : 0.f;
  const float L = lse[((size_t)b * n + head) * seq + i];
  const float D = out ? row_dot_out(dop, out + ((size_t)b * seq + i) * a + head * d, d) : delta[((size_t)b * n + head) * seq + i];
  const int jend = causal ? i + 1 : seq;
  float dq0 = 0.f, dq1 = 0.f;
  for (int j = 0; j < jend; j++) {
    const float *kp = base + (size_t)j * ld + a + (head / (n / nk)) * d;
    const float *vp = kp + ak;
    float k0 = h0 ? kp[lane] : 0.f, k1 = h1 ? kp[lane + 64] : 0.f;
    float v0 = h0 ? vp[lane] : 0.f, v1 = h1 ? vp[lane + 64] : 0.f;
    float sc = wave_sum(q0 * k0 + q1 * k1) * scale;
    float dp = wave_sum(g0 * v0 + g1 * v1);
    float ds = expf(sc - L) * (dp - D) * scale;
    dq0 += ds * k0;
    dq1 += ds * k1;
  }
  float *dqp = dqkv + ((size_t)b * seq + i) * ld + head * d;
  if (h0) dqp[lane] = dq0;
  if (h1) dqp[lane + 64] = dq1;
}

// key row j of key / value head kh; sums over the query heads of its group in a fixed order
__device__ __forceinline__ void attn_bwd_dkv_row(const float *__restrict__ qkv, const float *__restrict__ lse, const float *__restrict__ dout,
                                                 const float *__restrict__ out, const float *__restrict__ delta, float *__restrict__ dqkv, int b,
                                                 int kh, int j, int seq, int n, int nk, int d, int causal, float scale) {
  const int lane = threadIdx.x & 63;
  const int a = n * d, ak = nk * d, group = n / nk;
  const size_t ld = (size_t)a + 2 * ak;
  const float *base = qkv + (size_t)b * seq * ld;
  const bool h0 = lane < d, h1 = lane + 64 < d;
  const float *kp = base + (size_t)j * ld + a + kh * d;
  const float *vp = kp + ak;
  float k0 = h0 ? kp[lane] : 0.f, k1 = h1 ? kp[lane + 64] : 0.f;
  float v0 = h0 ? vp[lane] : 0.f, v1 = h1 ? vp[lane + 64] : 0.f;
  float dk0 = 0.f, dk1 = 0.f, dv0 = 0.f, dv1 = 0.f;
  for (int g = 0; g < group; g++) {
    const int head = kh * group + g;
    const float *Lr = lse + ((size_t)b * n + head) * seq, *Dr = out ? nullptr : delta + ((size_t)b * n + head) * seq;
    for (int i = causal ? j : 0; i < seq; i++) {
      const float *qp = base + (size_t)i * ld + head * d;
      const float *dop = dout + ((size_t)b * seq + i) * a + head * d;
      float q0 = h0 ? qp[lane] : 0.f, q1 = h1 ? qp[lane + 64] : 0.f;
      float g0 = h0 ? dop[lane] : 0.f, g1 = h1 ? dop[lane + 64] : 0.f;
      float sc = wave_sum(q0 * k0 + q1 * k1) * scale;
      float dp = wave_sum(g0 * v0 + g1 * v1);
      const float D = out ? row_dot_out(dop, out + ((size_t)b * seq + i) * a + head * d, d) : Dr[i];
      float p = expf(sc - Lr[i]);
      float ds = p * (dp - D) * scale;
      dv0 += p * g0; dv1 += p * g1;
      dk0 += ds * q0; dk1 += ds * q1;
    }
  }
  float *dkp = dqkv + ((size_t)b * seq + j) * ld + a + kh * d;
  float *dvp = dkp + ak;
  if (h0) { dkp[lane] = dk0; dvp[lane] = dv0; }
  if (h1) { dkp[lane + 64] = dk1; dvp[lane + 64] = dv1; }
}
