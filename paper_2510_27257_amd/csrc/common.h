// Internal helpers shared by the HIP translation units of libstp.so.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include "stp.h"

typedef __bf16 bf16_t;
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef short s16x8_t __attribute__((ext_vector_type(8)));

#define STP_MAX_LAYER_EVENTS 4096

constexpr int STP_CUS = 256;      // compute units of the chip

// Work plan of a chunked attention kernel (forward, dq, dkv).  A workgroup owns one chunk of up to chunk_steps
// steps of one block (a query block, or a key block for dkv); `order` lists the (block, chunk) pairs, longest
// first, and the grid is (heads, n_items) so that the dispatcher, which hands out workgroups in grid order,
// starts the long ones first and fills the tail of the launch with the short ones.  item = block | chunk << 12.
// n_items = 0 (more pairs than the table holds): the grid is blocks x max_chunks x heads and a workgroup
// reads its pair from its grid position.
#define STP_ATTN_ORDER_CAP 1024
struct stp_attn_order { uint16_t item[STP_ATTN_ORDER_CAP]; };
struct stp_attn_plan {
  int key[8];          // what the plan was made for (cache tag)
  int chunk_steps, max_chunks, n_items;
  int halves;          // 2 = eight waves share a step's keys (dkv: queries), 1 = four waves take all of them
  int between;         // backward: dK / dV with the exponentials among the MFMAs
  stp_attn_order order;
};
#define STP_ATTN_PLAN_CACHE 12

// see rope_sincos.  Kernels read it from their arguments four or eight floats at a time.
struct alignas(16) stp_rope_tab { float hi[64], lo[64]; };

// What the streams of the braid steps are known to be ordered behind.  Slot = index of the first of the three streams with that
// handle.  Every slot is marked at the end of a step (by an event; the last two marks are kept); a mark remembers which steps of
// the other slots its stream was ordered behind when it was made, so that a wait for it also stands for those.
struct stp_joins {
  struct Mark { long step, known[3]; } mark[3][2];     // [slot][older, latest]; step 0: none
  long known[3][3];                                    // [slot][other slot]: the other's last step that the slot's stream is ordered behind
  long now;                                            // number of the step
  // the waits of slot i where it has to come after step need[j] of slot j: wait(j, which mark); the later ones
  // first, since they may stand for the earlier ones.  latest: where a wait is needed at all, for the other's latest mark.
  template <typename F> int join(int i, const long need[3], bool latest, F wait) {
    for (long back = 1; back <= 2; back++)
      for (int j = 0; j < 3; j++) {
        const long step = need[j] < mark[j][1].step ? need[j] : mark[j][1].step;
        if (j == i || need[j] != now - back || known[i][j] >= step) continue;
        const int which = !latest && mark[j][0].step >= step ? 0 : 1;
        const int rc = wait(j, which);
        if (rc != STP_OK) return rc;
        behind(i, j, mark[j][which].step, mark[j][which].known);
      }
    return STP_OK;
  }
  // slot i is ordered behind `step` of slot j, whose stream was behind `of` then
  void behind(int i, int j, long step, const long of[3]) {
    for (int k = 0; k < 3; k++)
      if (of[k] > known[i][k]) known[i][k] = of[k];
    if (step > known[i][j]) known[i][j] = step;
  }
  void make_mark(int i) {
    mark[i][0] = mark[i][1];
    mark[i][1].step = now;
    for (int k = 0; k < 3; k++) mark[i][1].known[k] = known[i][k];
  }
  void drop_marks() {
    for (int i = 0; i < 3; i++) mark[i][0].step = mark[i][1].step = 0;
  }
};

// What a step works on: its forward microbatch (-1: none) and, per microbatch, whether it holds B / W work.
struct stp_step_work { int f_mb; const uint8_t *b, *w; };

// The joins of one step with the steps before.  Data of a (layer, microbatch) is written by that microbatch's F units (forward
// stream), read and extended by its B units (backward stream), read by its W units (weight-gradient stream);
// gradient accumulators and workspace lanes belong to one stream each.  So, of the last step, a stream waits
// only for   F: the B / W streams if they worked on the microbatch this step's F overwrites;
//            B: the F stream if it produced one of this step's backward microbatches, the W stream if it read one;
//            W: the B stream if it produced what this step's W units read (and the F stream likewise).
// All streams are ordered behind the whole of the step before last, which bounds the skew to one block; those without
// work in this step too, since a caller may rely on it for work of its own there.
struct stp_step_joins {
  stp_joins &J;
  int slot_of[3];            // slots of the forward, backward and weight-gradient streams
  long need[3][3] = {};      // [slot][other slot]: the step of the other that the slot has to come after; 0: none
  bool w_joined = true;

  void needs(int mbs, const stp_step_work &cur, const stp_step_work &last) {
    const long now = J.now;
    auto after = [&](int i, int j, long step) {
      long &n = need[slot_of[i]][slot_of[j]];
      if (step > n) n = step;
    };
    for (int i = 0; i < 3; i++)
      for (int j = 0; j < 3; j++) after(i, j, now - 2);
    if (cur.f_mb >= 0 && last.b[cur.f_mb]) after(0, 1, now - 1);
    if (cur.f_mb >= 0 && last.w[cur.f_mb]) after(0, 2, now - 1);
    for (int m = 0; m < mbs; m++) {
      if (cur.b[m] && m == last.f_mb) after(1, 0, now - 1);
      if (cur.b[m] && last.w[m]) after(1, 2, now - 1);
      if (cur.w[m] && last.b[m]) after(2, 1, now - 1);
      if (cur.w[m] && m == last.f_mb) after(2, 0, now - 1);
    }
  }
  // the waits at the start of the step: wait(i, j, which mark), slot i for slot j.  A weight-gradient stream of its own that has work
  // joins behind its first wait for a B unit of this step, which may stand for its other waits.  A slot without work waits for
  // the last step's marks: its work in the next step has to come after those in any case and then finds the wait made (two ViT layers 1726 us
  // a pass, 1749 with waits for the marks before them; the fp32 layer of 128 tokens, which the host bounds, about 350 either way, 335 where
  // streams without work make no waits).
  template <typename F> int begin(const bool has[3], F wait) {
    bool busy[3] = {};
    for (int i = 0; i < 3; i++) busy[slot_of[i]] = busy[slot_of[i]] || has[i];
    w_joined = slot_of[2] != 2 || !has[2];
    for (int i = 0; i < 3; i++) {
      if (slot_of[i] != i || !(w_joined || i < 2)) continue;
      const int rc = J.join(i, need[i], !busy[i], [&](int j, int which) { return wait(i, j, which); });
      if (rc != STP_OK) return rc;
    }
    return STP_OK;
  }
  // before a W unit is enqueued, behind the wait for its B unit if that is one of this step on another stream
  template <typename F> int before_w(bool behind_b, F wait) {
    // the B stream has made this step's waits, so behind its event are the steps before and what those waits stand for
    if (behind_b) J.behind(slot_of[2], slot_of[1], J.now - 1, J.known[slot_of[1]]);
    if (w_joined) return STP_OK;
    w_joined = true;
    return J.join(2, need[2], false, [&](int j, int which) { return wait(2, j, which); });
  }
};

#define STP_TILE_HINTS 96
struct stp_ctx {
  int device;
  char err[512];
  char *ws;          // caller-supplied workspace (device)
  size_t ws_bytes;
  stp_joins joins;                  // between the braid steps
  hipEvent_t mark_ev[3][2];         // events of its marks
  hipStream_t step_stream[3];       // streams of the last step
  int last_f_mb, last_mbs;          // the last step's forward microbatch; extent of the tables below
  uint8_t *last_b, *last_w;         // [last_mbs]: whether it held B / W work of a microbatch
  int have_step_events;
  hipEvent_t *ev_pool;     // events recorded after B ops, waited on by their W ops
  int ev_pool_size;
  // which B units have been issued since the last reset: bitmap over (layer, mb, unit)
  uint8_t *b_done;
  size_t b_done_size;
  int b_layers, b_mbs;
  // events that order the copy stream of the activation offload against its producer / consumer streams
  // (a stream wait refers to the record that precedes it, so the ring may wrap)
  hipEvent_t ev_copy[16];
  int ev_copy_made, ev_copy_next;
  // set by stp_braid_step while it issues a step on distinct streams: kernels launched then share the GPU
  // with the other streams' kernels, which changes the best GEMM tile
  int concurrent;
  // Tile preferences of the bf16 GEMM for launches issued while stp_braid_step runs on concurrent streams
  // (stp_gemm_tile_hint): what is fastest there depends on the kernels of the other streams, which no model of
  // the GEMM alone sees, so a caller may measure and say.
  struct { int32_t M, N, K, layout, tile_m, tile_n; } tile_hint[STP_TILE_HINTS];
  int n_tile_hints;
  // plans of the attention kernels for the shapes seen so far (making one simulates the dispatch)
  stp_attn_plan attn_plan[STP_ATTN_PLAN_CACHE];
  int attn_plan_n, attn_plan_next;
  // rotary frequencies of the last head dimension and base
  stp_rope_tab rope_tab;
  int rope_dim;
  float rope_base;
};

static inline int stp_fail(stp_ctx *ctx, int status, const char *fmt, const char *a = "", long b = 0, long c = 0) {
  if (ctx) snprintf(ctx->err, sizeof(ctx->err), fmt, a, b, c);
  return status;
}

#define STP_HIP(ctx, call)                                                                 \
  do {                                                                                     \
    hipError_t e_ = (call);                                                                \
    if (e_ != hipSuccess) {                                                                \
      if (ctx) snprintf((ctx)->err, sizeof((ctx)->err), "%s failed: %s (%s:%d)", #call,    \
                        hipGetErrorString(e_), __FILE__, __LINE__);                        \
      return STP_EHIP;                                                                     \
    }                                                                                      \
  } while (0)

#define STP_LAUNCH_CHECK(ctx) STP_HIP(ctx, hipGetLastError())

static inline bool stp_aligned16(const void *p) { return (((uintptr_t)p) & 15u) == 0; }
static inline size_t stp_align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
static inline size_t stp_elem_size(int dtype) { return dtype == STP_BF16 ? 2 : 4; }

// ---- device-side 8-element vector access, math in fp32 -----------------------------
template <typename T> struct Vec8;
template <> struct Vec8<float> {
  static __device__ __forceinline__ void load(const float *p, float (&v)[8]) {
    float4 a = *reinterpret_cast<const float4 *>(p);
    float4 b = *reinterpret_cast<const float4 *>(p + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  }
  static __device__ __forceinline__ void store(float *p, const float (&v)[8]) {
    *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4 *>(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
  }
};
template <> struct Vec8<bf16_t> {
  static __device__ __forceinline__ void load(const bf16_t *p, float (&v)[8]) {
    uint4 u = *reinterpret_cast<const uint4 *>(p);
    uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; i++) {
      v[2 * i] = __uint_as_float(w[i] << 16);
      v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
  static __device__ __forceinline__ void store(bf16_t *p, const float (&v)[8]) {
    bf16x8_t o;
#pragma unroll
    for (int i = 0; i < 8; i++) o[i] = (bf16_t)v[i];
    *reinterpret_cast<bf16x8_t *>(p) = o;
  }
};

template <typename T> __device__ __forceinline__ float to_f32(T x) { return (float)x; }
template <typename T> __device__ __forceinline__ T from_f32(float x) { return (T)x; }

// The value lane (l ^ 32) holds, without the LDS round trip of a shuffle: v_permlane32_swap exchanges the
// upper half of one register with the lower half of another.  (Inline assembly: the builtin form was
// seen to return the same register for both results.  The no-ops cover the wait states between a
// vector write and the lane permute, which the compiler cannot insert inside assembly.)
__device__ __forceinline__ float other_half(float v) {
  float a = v, b = v;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32_e32 %0, %1\n\ts_nop 1" : "+v"(a), "+v"(b));
  // a = [v.lo | v.lo], b = [v.hi | v.hi]: lanes below 32 want b, the others a
  return (threadIdx.x & 32) ? a : b;
}

// Sum / maximum over the 64 lanes of a wave, the result in every lane.  Within a row of 16 lanes by cross-lane
// operand modifiers (quad permutes, then the half-row and row mirrors: no LDS round trips as a shuffle has),
// then the four rows through scalar registers, (r0 + r1) + (r2 + r3).
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_f32(float v, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_f32<0xB1>(v);    // quad_perm [1,0,3,2]
  v += dpp_f32<0x4E>(v);    // quad_perm [2,3,0,1]
  v += dpp_f32<0x141>(v);   // row_half_mirror
  v += dpp_f32<0x140>(v);   // row_mirror
  return (lane_f32(v, 0) + lane_f32(v, 16)) + (lane_f32(v, 32) + lane_f32(v, 48));
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_f32<0xB1>(v));
  v = fmaxf(v, dpp_f32<0x4E>(v));
  v = fmaxf(v, dpp_f32<0x141>(v));
  v = fmaxf(v, dpp_f32<0x140>(v));
  return fmaxf(fmaxf(lane_f32(v, 0), lane_f32(v, 16)), fmaxf(lane_f32(v, 32), lane_f32(v, 48)));
}

// exact GELU x*Phi(x) and its derivative Phi(x) + x*phi(x)
__device__ __forceinline__ float gelu_f(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad_f(float x) {
  float Phi = 0.5f * (1.0f + erff(x * 0.70710678118654752f));
  float phi = 0.3989422804014327f * __expf(-0.5f * x * x);
  return Phi + x * phi;
}
// The same two for bf16 storage, where the rounding of the result (2^-9) hides an absolute error of 1e-7: the
// normal distribution function from the rational-times-exponential approximation of erfc (Abramowitz & Stegun
// 7.1.26, |error| < 1.5e-7 in erf), branch-free: 0.5 erfc(|x|/sqrt 2) = 0.5 t (a1 + t (a2 + ... )) exp(-x^2/2),
// t = 1 / (1 + p |x| / sqrt 2); the lower tail is taken directly (no cancellation), the upper as 1 - tail.
// `e` returns exp(-x^2/2), which the derivative needs as well.
__device__ __forceinline__ float normal_cdf_fast(float x, float &e) {
  const float ax = fabsf(x) * 0.70710678118654752f;
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, ax, 1.0f));
  float p = fmaf(t, 1.061405429f, -1.453152027f);
  p = fmaf(t, p, 1.421413741f);
  p = fmaf(t, p, -0.284496736f);
  p = fmaf(t, p, 0.254829592f);
  e = __builtin_amdgcn_exp2f(ax * ax * -1.4426950408889634f);
  const float q = 0.5f * p * t * e;
  return x < 0.f ? q : 1.0f - q;
}
template <typename T> __device__ __forceinline__ float gelu_t(float x) {
  if constexpr (sizeof(T) == 4) return gelu_f(x);
  float e;
  return x * normal_cdf_fast(x, e);
}
template <typename T> __device__ __forceinline__ float gelu_grad_t(float x) {
  if constexpr (sizeof(T) == 4) return gelu_grad_f(x);
  float e;
  const float Phi = normal_cdf_fast(x, e);
  return fmaf(x * 0.3989422804014327f, e, Phi);
}
__device__ __forceinline__ float sigmoid_f(float x) { return 1.0f / (1.0f + __expf(-x)); }

// SwiGLU of a gate and an up activation, and its gradients
__device__ __forceinline__ float swiglu_f(float g, float u) { return g * sigmoid_f(g) * u; }
__device__ __forceinline__ void swiglu_grad(float g, float u, float d, float &dg, float &du) {
  const float sg = sigmoid_f(g);
  du = d * g * sg;
  dg = d * u * sg * (1.0f + g * (1.0f - sg));
}

// Rotary embedding for bf16 storage: the frequencies of the pairs (i, i + d/2) in revolutions per token as a float and what it leaves of
// the 64-bit value, so that the angle's fraction is right to 1e-7 at any position (a rounded product of position and
// frequency is off by 2e-4 at 4096), and the hardware's sine and cosine of revolutions (1e-6, against 2e-3 of a bf16 result).
__device__ __forceinline__ void rope_sincos(float pos, float hi, float lo, float &sn, float &cs) {
  const float p = pos * hi, rest = fmaf(pos, lo, fmaf(pos, hi, -p));
  const float turns = __builtin_amdgcn_fractf(p) + rest;
  sn = __builtin_amdgcn_sinf(turns);
  cs = __builtin_amdgcn_cosf(turns);
}

// ---- kernel launchers implemented in the .hip files ---------------------------------
int stp_launch_gemm_bf16(stp_ctx *ctx, const stp_gemm_args *a, hipStream_t s);
// n <= 3 products C += A^T B in fp32 with one contraction length, as one launch where that is shorter
int stp_launch_gemm_bf16_wgrads(stp_ctx *ctx, const stp_gemm_args *a, int n, hipStream_t s);
// tile (bm << 16 | bn) of that launch, 0 where the products are launched apart; host only, no part of the interface (tests check routes)
extern "C" int stp_wgrad_set_tile(const stp_gemm_args *a, int n);
// Further host functions for tests of routes and waits, no part of the interface either: the tile of the SwiGLU projections' launch (0: apart); the
// workgroups of the bf16 attention forward (0: four waves, 1: eight, matrix and vector phases apart, 2: eight, in phase); the wave halves of the attention
// backward's workgroups, and whether dK / dV have the exponentials among the MFMAs; the launches of the fp32 attention backward (1 or 3); the waits of a
// sequence of braid steps.
extern "C" int stp_swiglu_pair_tile(int M, int N, int K);
extern "C" int stp_attn_fwd_route(const stp_layer_desc *d);
extern "C" int stp_attn_bwd_halves(const stp_layer_desc *d);
extern "C" int stp_attn_bwd_between(const stp_layer_desc *d);
extern "C" int stp_attn_bwd_f32_launches(const stp_layer_desc *d);
extern "C" int stp_braid_plan_joins(int n_steps, int mbs, const int32_t *f_mb, const uint8_t *b, const uint8_t *w, const uint8_t *through, const int32_t *slot_of,
                                    int64_t *waits, int cap);
// The products of a SwiGLU MLP with the activation in the epilogue or both operands in one contraction.  `g` describes one of the two
// products; STP_EUNSUPPORTED where the operands are beyond the direct-to-LDS kernels or the first takes longer so (the caller then launches them apart).
//   up: C = A B (+ bias), up = A B2, act = SiLU(C) * up
int stp_launch_gemm_bf16_swiglu(stp_ctx *ctx, const stp_gemm_args *g, const void *B2, void *up, void *act, hipStream_t s);
//   C, dup = gradients of gate and up activation from their values and the product's sums
int stp_launch_gemm_bf16_swiglu_bwd(stp_ctx *ctx, const stp_gemm_args *g, const void *gate, const void *up, void *dup, hipStream_t s);
//   C = A B^T + A2 B2^T
int stp_launch_gemm_bf16_sum(stp_ctx *ctx, const stp_gemm_args *g, const void *A2, const void *B2, hipStream_t s);
int stp_launch_gemm_f32(stp_ctx *ctx, const stp_gemm_args *a, hipStream_t s);
// as stp_launch_gemm_bf16_wgrads
int stp_launch_gemm_f32_wgrads(stp_ctx *ctx, const stp_gemm_args *a, int n, hipStream_t s);
// whether two of n fp32 outputs share memory (those are added to one after the other)
static inline bool stp_accumulators_overlap(const stp_gemm_args *a, int n) {
  for (int i = 0; i < n; i++)
    for (int j = 0; j < i; j++) {
      const float *c = (const float *)a[i].C, *d = (const float *)a[j].C;
      if (c < d + (size_t)(a[j].M - 1) * a[j].ldc + a[j].N && d < c + (size_t)(a[i].M - 1) * a[i].ldc + a[i].N) return true;
    }
  return false;
}
int stp_launch_attn_fwd_bf16(stp_ctx *ctx, const stp_layer_desc *d, const void *qkv, void *out, float *lse, float *ws,
                             size_t ws_bytes, hipStream_t s);
int stp_launch_attn_bwd_bf16(stp_ctx *ctx, const stp_layer_desc *d, const void *qkv, const void *out, const float *lse,
                             const void *dout, float *delta, void *dqkv, float *ws, size_t ws_bytes, bool rope, hipStream_t s);
// the frequencies of a layer's rotary embedding
const stp_rope_tab &stp_rope_tab_for(stp_ctx *ctx, const stp_layer_desc *d);
// QKV = A B (+ bias) with the rotary embedding of the Q and K heads applied; STP_EUNSUPPORTED as above
int stp_launch_gemm_bf16_rope(stp_ctx *ctx, const stp_gemm_args *g, const stp_layer_desc *d, hipStream_t s);
// grouped-query attention: key / value heads of a rank and the width of its QKV activation
static inline int stp_kv_heads(const stp_layer_desc *d) { return d->kv_heads_local > 0 ? d->kv_heads_local : d->heads_local; }
static inline int stp_qkv_width(const stp_layer_desc *d) { return (d->heads_local + 2 * stp_kv_heads(d)) * d->head_dim; }

// Chunk lengths {dkv, dq} of the backward kernels, planned together because one launch runs both; steps_*[x] is the number of
// steps of block x.
// Returns the number of key or query halves that a workgroup's waves share: 2, or 1 where it has four waves.
int stp_attn_bwd_chunks(const stp_layer_desc *d, int nkv, const int *steps_kv, int nq, const int *steps_q, int chunk[2], int *between);
// fills in the work order of blocks cut into chunks of `chunk` steps
void stp_attn_plan_fill(stp_attn_plan *plan, int chunk, int nblocks, const int *steps);
// the context's (or, without one, the thread's) cache slot for a plan with this tag; *hit says whether it is filled
stp_attn_plan *stp_attn_plan_slot(stp_ctx *ctx, const int key[8], bool *hit);
// the plan's estimate of a workgroup's time in microseconds: `len` steps of a kernel of this kind
double stp_attn_item_cost(int kind, int head_dim, int len);
// the plan of one kernel for a layer shape (kind as above); bf16 shapes only
const stp_attn_plan *stp_attn_plan_for(stp_ctx *ctx, const stp_layer_desc *d, int kind);
const stp_attn_plan *stp_attn_bwd_plan_for(stp_ctx *ctx, const stp_layer_desc *d, int kind);

size_t stp_attn_fwd_ws_bytes(const stp_layer_desc *d);   // workspace the bf16 attention kernels need (chunk partials)
size_t stp_attn_bwd_ws_bytes(const stp_layer_desc *d);
int stp_launch_attn_fwd_f32(stp_ctx *ctx, const stp_layer_desc *d, const void *qkv, void *out, float *lse, hipStream_t s);
int stp_launch_attn_bwd_f32(stp_ctx *ctx, const stp_layer_desc *d, const void *qkv, const void *out, const float *lse,
                                const void *dout, float *delta, void *dqkv, hipStream_t s);
// byte offsets of all fields of a stash whose description has been checked
void stp_stash_offsets(const stp_layer_desc *d, size_t off[STP_ST_NFIELDS]);
// device address of the fixed scratch array of stp_colsum_noalloc on `device` (the current device); a lookup, no allocation
int stp_noalloc_init(stp_ctx *ctx, int device);
// Launch geometry that also sizes the workspace.  Norm backward: 256-thread row groups that stride over the rows,
// one partial per group.
static inline int stp_norm_bwd_blocks(int rows, int h) {
  (void)h;
  return rows < 512 ? rows : 512;
}
// Column sum: stage-1 patches of STP_COLSUM_ROWS rows, one partial row each
#define STP_COLSUM_ROWS 64
static inline int stp_colsum_slabs(int rows) { return (rows + STP_COLSUM_ROWS - 1) / STP_COLSUM_ROWS; }
// workspace lane: a third of the caller's workspace
static inline char *stp_ws_lane(stp_ctx *ctx, int lane, size_t *bytes) {
  size_t third = (ctx->ws_bytes / 3) & ~(size_t)255;
  *bytes = third;
  return ctx->ws ? ctx->ws + (size_t)lane * third : nullptr;
}
