// (included by the four per-layout translation units gemm_bf16_*.hip)
// bf16 GEMM on the CDNA4 matrix cores: C[M,N] = op(A) op(B), fp32 accumulate.
//
// Serves every dense contraction of the units (QKV, out-proj, FC1, FC2 in F; their
// transposed-weight forms in B; the token-contracting forms in W).
//
// Two kernels share the fragment scheme, the tile map and the epilogue:
//   * gemm_bf16_dma_kernel (further down): direct-to-LDS loads, rings of 64-deep K-tiles, the path of
//     every problem whose operands it can address;
//   * gemm_bf16_kernel: the fallback for operands of 2 GiB and more, described here.
//
// Fallback design (gfx950):
//   * one workgroup = WAVES_M x WAVES_N waves, block tile BM x BN x 64, each wave owns a
//     (BM/WAVES_M) x (BN/WAVES_N) sub-tile as a grid of 32x32 accumulators fed by v_mfma_f32_32x32x16_bf16;
//   * global -> registers -> LDS with two LDS stages: the loads of K-tile kt+1 are in
//     flight while the MFMAs of K-tile kt run, one barrier per K-tile;
//   * an operand whose contraction index is contiguous in memory sits in LDS as
//     [row][64 + 8] and is fetched with one 16-byte LDS read per fragment; an operand
//     whose contraction index is the OUTER index (B = W[in,out] in forward, both
//     operands of the weight-gradient GEMMs) is copied to LDS as it lies in memory,
//     [k][rows + 32], and fetched with the transposing LDS read (ds_read_b64_tr_b16):
//     a 16-lane group reads a 4(k) x 16(row) patch and every lane receives the four
//     k-consecutive values of its own row.  No register or memory transposes.
//   * LDS row pitches (144 B and rows*2+64 B) keep both fetch patterns bank-conflict free;
//   * the blockIdx -> tile map gives each XCD (blockIdx % 8) a contiguous band of tiles
//     walked in groups along M, so tiles resident on one XCD share their A / B panels
//     in that XCD's L2.
#pragma once
#include "common.h"
#include "lds_dma.h"
#include <utility>
#include <stdlib.h>
#include <math.h>

namespace {

constexpr int BK = 64;
constexpr int KPAD = 8;    // elements; pitch of a k-contiguous tile row = 72 el = 144 B
constexpr int XPAD = 32;   // elements; pitch of a row-contiguous tile = rows + 32

template <int ROWS, bool KC> struct TileGeom {
  static constexpr int pitch = KC ? (BK + KPAD) : (ROWS + XPAD);
  static constexpr int elems = KC ? ROWS * pitch : BK * pitch;
  static constexpr int chunks = ROWS * BK / 8;          // 16-byte chunks per tile
};

// Loads this thread's share of a ROWS x 64 operand tile from global memory into registers.
// KC: memory is [row][k] (ld = row pitch);  !KC: memory is [k][row].  Out-of-range chunks are
// read from the (always valid) first element; bit i of the returned mask says chunk i is real.
// The zero-fill happens when the registers are written to LDS, after the MFMAs of the current
// tile, so that all loads stay in flight together (no wait between them).
template <int ROWS, bool KC, int NTH, int NREG>
__device__ __forceinline__ unsigned tile_load(uint4 (&reg)[NREG], const bf16_t *__restrict__ base,
                                              int ld, int row0, int row_lim, int k0, int k_lim, int tid) {
  static_assert(NREG * NTH == TileGeom<ROWS, KC>::chunks, "register tile size");
  unsigned mask = 0;
#pragma unroll
  for (int i = 0; i < NREG; i++) {
    int q = tid + NTH * i;
    int r, k;
    if (KC) { r = q >> 3; k = (q & 7) * 8; }
    else { k = q / (ROWS / 8); r = (q % (ROWS / 8)) * 8; }
    const bool ok = (row0 + r < row_lim) && (k0 + k < k_lim);
    size_t off = KC ? (size_t)(row0 + r) * ld + (k0 + k) : (size_t)(k0 + k) * ld + (row0 + r);
    off = ok ? off : 0;
    mask |= ok ? (1u << i) : 0u;
    reg[i] = *reinterpret_cast<const uint4 *>(base + off);
  }
  return mask;
}

template <int ROWS, bool KC, int NTH, int NREG>
__device__ __forceinline__ void tile_store(const uint4 (&reg)[NREG], unsigned mask, bf16_t *lds, int tid) {
  constexpr int P = TileGeom<ROWS, KC>::pitch;
#pragma unroll
  for (int i = 0; i < NREG; i++) {
    int q = tid + NTH * i;
    int r, k;
    if (KC) { r = q >> 3; k = (q & 7) * 8; }
    else { k = q / (ROWS / 8); r = (q % (ROWS / 8)) * 8; }
    bf16_t *p = KC ? lds + r * P + k : lds + k * P + r;
    const bool ok = (mask >> i) & 1u;
    uint4 v;
    v.x = ok ? reg[i].x : 0u; v.y = ok ? reg[i].y : 0u; v.z = ok ? reg[i].z : 0u; v.w = ok ? reg[i].w : 0u;
    *reinterpret_cast<uint4 *>(p) = v;
  }
}

// MFMA operand fragment for the 32 rows starting at `row` and the 16 k-values starting at kk:
// lane l supplies row (l % 32), k = kk + 8*(l/32) .. +7.
template <int ROWS, bool KC>
__device__ __forceinline__ bf16x8_t frag_load(const bf16_t *lds, int row, int kk, int lane) {
  constexpr int P = TileGeom<ROWS, KC>::pitch;
  if (KC) {
    return *reinterpret_cast<const bf16x8_t *>(lds + (row + (lane & 31)) * P + kk + 8 * (lane >> 5));
  } else {
    // transposing read: the 16 lanes of a group point at rows k..k+3 (4 lanes each, 4 columns per lane)
    int k = kk + 8 * (lane >> 5) + ((lane & 15) >> 2);
    int c = row + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    const bf16_t *p = lds + k * P + c;
    typedef s16x4_t __attribute__((address_space(3))) * lds_ptr_t;
    s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p));
    s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p + 4 * P));
    s16x8_t v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8_t, v);
  }
}

struct Epi {
#ifdef STP_GEMM_TRACE
  long long *trace;   // measurement build only: 4 wall-clock stamps per workgroup
#endif
  void *C; int ldc; int c_f32_accum;
  const bf16_t *bias; float bias_scale;
  const bf16_t *resid; int ldr; float resid_scale;
  int mode; bf16_t *C2; const bf16_t *aux; int ld2;
  const bf16_t *aux2; bf16_t *C3;      // SwiGLU: up activation in (backward); its product out (forward); pitch ld2
  int rope_cols, rope_seq;
};
// of the kernels that rotate: the epilogue's description and the frequencies
struct EpiRope : Epi { stp_rope_tab tab; };
static_assert(alignof(EpiRope) >= 16, "store_rope reads the frequencies eight at a time");

// EPI_SWIGLU_BWD: C, C2 = gradients of gate and up activation from the sums, aux and aux2.  EPI_SWIGLU_FWD (kernels with paired B
// operands): C = gate, C2 = up, C3 = SiLU(gate) * up.
// EPI_ROPE64 / 128: columns below rope_cols are heads of that dimension, rotated by their row's position; a wave's two accumulators of a
// strip hold the two halves of 32 pairs.
enum { EPI_STORE = 0, EPI_GELU_DUAL = 1, EPI_GELU_BWD = 2, EPI_F32_ACCUM = 3, EPI_SWIGLU_BWD = 4, EPI_SWIGLU_FWD = 5, EPI_ROPE64 = 6, EPI_ROPE128 = 7 };

// What a tile of the direct-to-LDS kernel multiplies.  One product; the sum of two, A B + A2 B2, as one contraction twice as long; or
// two products of one A whose B tiles lie side by side: half of the tile's columns from B, half from B2, the same
// 32 columns of both in a wave's two accumulators.
enum { MM_ONE = 0, MM_SUM = 1, MM_PAIR = 2 };

// XCD-aware tile map: workgroups are dealt round-robin to the 8 XCDs, so XCD x (= blockIdx % 8) is given
// the contiguous band [x*total/8, (x+1)*total/8) of a tile order that walks groups of 4 tile-rows
// column by column: tiles resident on one XCD share their A / B panels in that XCD's L2.
__device__ __forceinline__ int xcd_order(int total) {
  const int base = total >> 3, rem = total & 7;
  const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
  return x * base + min(x, rem) + j;
}
__device__ __forceinline__ void tile_of(int pid, int tiles_m, int tiles_n, int &tm, int &tn) {
  constexpr int GROUP_M = 4;
  int group = pid / (GROUP_M * tiles_n);
  int first_m = group * GROUP_M;
  int gsize = min(tiles_m - first_m, GROUP_M);
  tm = first_m + (pid % (GROUP_M * tiles_n)) % gsize;
  tn = (pid % (GROUP_M * tiles_n)) / gsize;
}
__device__ __forceinline__ void map_tile(int tiles_m, int tiles_n, int &tm, int &tn) {
  tile_of(xcd_order(tiles_m * tiles_n), tiles_m, tiles_n, tm, tn);
}

// What the epilogue of 8 consecutive columns of one row reads from global memory: residual / aux in lo (8 bf16), the fp32
// accumulator in lo and hi.  Rows / columns past M / N are read from a clamped address and never stored.
struct EpiPre { uint4 lo, hi; };
template <int EPI>
__device__ __forceinline__ void epi_fetch(EpiPre &f, int row_, int col_, int M, int N, const Epi &ep) {
  const size_t row = (size_t)min(row_, M - 1);
  const int col = min(col_, N - 8);
  if (EPI == EPI_F32_ACCUM) {
    const uint4 *cp = reinterpret_cast<const uint4 *>(reinterpret_cast<const float *>(ep.C) + row * ep.ldc + col);
    f.lo = cp[0];
    f.hi = cp[1];
  } else if (EPI == EPI_GELU_BWD) {
    f.lo = *reinterpret_cast<const uint4 *>(ep.aux + row * ep.ld2 + col);
  } else if (EPI == EPI_SWIGLU_BWD) {
    f.lo = *reinterpret_cast<const uint4 *>(ep.aux + row * ep.ld2 + col);
    f.hi = *reinterpret_cast<const uint4 *>(ep.aux2 + row * ep.ld2 + col);
  } else if (ep.resid != nullptr) {
    f.lo = *reinterpret_cast<const uint4 *>(ep.resid + row * ep.ldr + col);
  }
}
__device__ __forceinline__ void epi_bias(float (&bias)[8], int col, int N, const Epi &ep) {
#pragma unroll
  for (int e = 0; e < 8; e++) bias[e] = 0.f;
  if (ep.bias != nullptr) {
    Vec8<bf16_t>::load(ep.bias + min(col, N - 8), bias);
#pragma unroll
    for (int e = 0; e < 8; e++) bias[e] *= ep.bias_scale;
  }
}
// val: the 8 sums; applies the epilogue and stores
template <int EPI>
__device__ __forceinline__ void epi_store(float (&val)[8], const float (&bias)[8], const EpiPre &f, int row, int col, int M, int N, const Epi &ep) {
#pragma unroll
  for (int e = 0; e < 8; e++) val[e] += bias[e];
  if (EPI == EPI_F32_ACCUM) {
    float old[8];
    old[0] = __builtin_bit_cast(float, f.lo.x); old[1] = __builtin_bit_cast(float, f.lo.y);
    old[2] = __builtin_bit_cast(float, f.lo.z); old[3] = __builtin_bit_cast(float, f.lo.w);
    old[4] = __builtin_bit_cast(float, f.hi.x); old[5] = __builtin_bit_cast(float, f.hi.y);
    old[6] = __builtin_bit_cast(float, f.hi.z); old[7] = __builtin_bit_cast(float, f.hi.w);
#pragma unroll
    for (int e = 0; e < 8; e++) old[e] += val[e];
    if (row < M && col < N) Vec8<float>::store(reinterpret_cast<float *>(ep.C) + (size_t)row * ep.ldc + col, old);
  } else if (EPI == EPI_SWIGLU_BWD) {
    const bf16x8_t g8 = __builtin_bit_cast(bf16x8_t, f.lo), u8 = __builtin_bit_cast(bf16x8_t, f.hi);
    float dg[8], du[8];
#pragma unroll
    for (int e = 0; e < 8; e++) swiglu_grad((float)g8[e], (float)u8[e], val[e], dg[e], du[e]);
    if (row < M && col < N) {
      Vec8<bf16_t>::store(reinterpret_cast<bf16_t *>(ep.C) + (size_t)row * ep.ldc + col, dg);
      Vec8<bf16_t>::store(ep.C2 + (size_t)row * ep.ld2 + col, du);
    }
  } else {
    if (EPI == EPI_GELU_BWD || ep.resid != nullptr) {
      const bf16x8_t h8 = __builtin_bit_cast(bf16x8_t, f.lo);
#pragma unroll
      for (int e = 0; e < 8; e++) {
        if (EPI == EPI_GELU_BWD) val[e] *= gelu_grad_t<bf16_t>((float)h8[e]);
        else val[e] += (float)h8[e] * ep.resid_scale;
      }
    }
    bf16x8_t o;
#pragma unroll
    for (int e = 0; e < 8; e++) o[e] = (bf16_t)val[e];
    if (row < M && col < N) {
      *reinterpret_cast<bf16x8_t *>(reinterpret_cast<bf16_t *>(ep.C) + (size_t)row * ep.ldc + col) = o;
      if (EPI == EPI_GELU_DUAL) {
        float gv[8];
#pragma unroll
        for (int e = 0; e < 8; e++) gv[e] = gelu_t<bf16_t>((float)o[e]);
        Vec8<bf16_t>::store(ep.C2 + (size_t)row * ep.ld2 + col, gv);
      }
    }
  }
}

// Epilogue.  Accumulator v of lane l is C[32*i + 8*(v/4) + 4*(l/32) + v%4][32*j + l%32].
// Each wave stages one 32 x WN strip at a time in its own LDS area (fp32, pitch WN + 8 keeps the two
// lane halves on different banks) and reads it back row-wise, 8 consecutive columns per lane, so
// that every global access of the epilogue (C, C2, residual, aux, bias) is a 16- or 32-byte vector.
// The staging area is private to the wave (LDS operations of a wave complete in order), so no barrier
// is needed.  What the epilogue reads from global memory (residual, aux, the fp32 accumulator) is
// fetched one strip ahead, all passes of a strip at once, so that its latency is paid once per tile
// and not once per pass.
// The caller guarantees that the operand stages in LDS are dead (barrier after the last K-tile).
template <int MI, int NI, int WN, int EPI>
__device__ __forceinline__ void store_tile(f32x16_t (&acc)[MI][NI], float *stage, int row_base, int col_base, int M, int N,
                                           const Epi &ep, int lane) {
  constexpr int SP = WN + 8;
  const int lr = lane & 31, lg = lane >> 5;
  constexpr int LPR = WN / 8;             // lanes per staged row
  constexpr int PASSES = 32 * LPR / 64;
  // pass p of a strip: staged row r_p, columns c_p .. c_p+7 (the same for every strip)
  int pr[PASSES], pc[PASSES];
  float bias[PASSES][8];
#pragma unroll
  for (int p = 0; p < PASSES; p++) {
    const int idx = p * 64 + lane;
    pr[p] = idx / LPR;
    pc[p] = col_base + (idx % LPR) * 8;
    epi_bias(bias[p], pc[p], N, ep);
  }
  // what strip i needs from global memory
  auto fetch = [&](int i, EpiPre (&f)[PASSES]) {
#pragma unroll
    for (int p = 0; p < PASSES; p++) epi_fetch<EPI>(f[p], row_base + i * 32 + pr[p], pc[p], M, N, ep);
  };
  auto strip = [&](int i, const EpiPre (&f)[PASSES]) {
#pragma unroll
    for (int j = 0; j < NI; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) stage[(8 * (v >> 2) + 4 * lg + (v & 3)) * SP + 32 * j + lr] = acc[i][j][v];
#pragma unroll
    for (int p = 0; p < PASSES; p++) {
      float val[8];
      Vec8<float>::load(stage + pr[p] * SP + (pc[p] - col_base), val);
      epi_store<EPI>(val, bias[p], f[p], row_base + i * 32 + pr[p], pc[p], M, N, ep);
    }
  };
  // strips alternate between two prefetch buffers
  EpiPre f0[PASSES], f1[PASSES];
  fetch(0, f0);
#pragma unroll
  for (int i = 0; i < MI; i += 2) {
    if (i + 1 < MI) fetch(i + 1, f1);
    strip(i, f0);
    if (i + 2 < MI) fetch(i + 2, f0);
    if (i + 1 < MI) strip(i + 1, f1);
  }
}

// The same for a wave whose two accumulators of a strip hold the same 32 columns of two products (EPI_SWIGLU_FWD): 8 columns of both
// per lane.
template <int MI, int EPI>
__device__ __forceinline__ void store_pairs(f32x16_t (&acc)[MI][2], float *stage, int row_base, int col_base, int M, int N, const Epi &ep, int lane) {
  static_assert(EPI == EPI_SWIGLU_FWD, "epilogue of two products");
  constexpr int SP = 64 + 8;
  const int lr = lane & 31, lg = lane >> 5, c = (lane & 3) * 8, col = col_base + c;
  float bias[8];
  epi_bias(bias, col, N, ep);
#pragma unroll
  for (int i = 0; i < MI; i++) {
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) stage[(8 * (v >> 2) + 4 * lg + (v & 3)) * SP + 32 * j + lr] = acc[i][j][v];
#pragma unroll
    for (int p = 0; p < 2; p++) {
      const int r = p * 16 + (lane >> 2), row = row_base + i * 32 + r;
      float g[8], u[8];
      Vec8<float>::load(stage + r * SP + c, g);
      Vec8<float>::load(stage + r * SP + 32 + c, u);
      bf16x8_t g8, u8, o8;
#pragma unroll
      for (int e = 0; e < 8; e++) {
        g8[e] = (bf16_t)(g[e] + bias[e]);
        u8[e] = (bf16_t)u[e];
        o8[e] = (bf16_t)swiglu_f((float)g8[e], (float)u8[e]);
      }
      if (row < M && col < N) {
        *reinterpret_cast<bf16x8_t *>(reinterpret_cast<bf16_t *>(ep.C) + (size_t)row * ep.ldc + col) = g8;
        *reinterpret_cast<bf16x8_t *>(ep.C2 + (size_t)row * ep.ld2 + col) = u8;
        *reinterpret_cast<bf16x8_t *>(ep.C3 + (size_t)row * ep.ld2 + col) = o8;
      }
    }
  }
}

// The same for two halves of rotary pairs, D/2 columns apart: 8 pairs per lane.  Sine and cosine are computed for the first pass of a
// strip and turned by 16 rows for the second (computed there too where a position starts again with the next sequence): as
// strips start at multiples of 32 rows in every tile, the bits do not depend on the tile.
template <int MI, int D>
__device__ __forceinline__ void store_rope(f32x16_t (&acc)[MI][2], float *stage, int row_base, int col_base, int M, int N, const EpiRope &ep, int lane) {
  constexpr int SP = 64 + 8;
  const int lr = lane & 31, lg = lane >> 5, c = (lane & 3) * 8, col = col_base + c;
  const bool rotate = col_base < ep.rope_cols;          // the same for the whole wave: its columns belong to one head
  float b0[8], b1[8];
  epi_bias(b0, col, N, ep);
  epi_bias(b1, col + D / 2, N, ep);
  float hi[8], lo[8], sn16[8], cs16[8];
  Vec8<float>::load(ep.tab.hi + col % D, hi);
  Vec8<float>::load(ep.tab.lo + col % D, lo);
#pragma unroll
  for (int e = 0; e < 8; e++) rope_sincos(16.f, hi[e], lo[e], sn16[e], cs16[e]);
#pragma unroll
  for (int i = 0; i < MI; i++) {
    int pos = (row_base + i * 32 + (lane >> 2)) % ep.rope_seq;
    float sn[8], cs[8];
    if (rotate) {
#pragma unroll
      for (int e = 0; e < 8; e++) rope_sincos((float)pos, hi[e], lo[e], sn[e], cs[e]);
    }
#pragma unroll
    for (int j = 0; j < 2; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) stage[(8 * (v >> 2) + 4 * lg + (v & 3)) * SP + 32 * j + lr] = acc[i][j][v];
#pragma unroll
    for (int p = 0; p < 2; p++) {
      const int r = p * 16 + (lane >> 2), row = row_base + i * 32 + r;
      float u[8], v[8];
      Vec8<float>::load(stage + r * SP + c, u);
      Vec8<float>::load(stage + r * SP + 32 + c, v);
      bf16x8_t o0, o1;
#pragma unroll
      for (int e = 0; e < 8; e++) {
        u[e] += b0[e];
        v[e] += b1[e];
        // spelt out: left to the compiler, the contraction of products and sums differs from tile to tile
        o0[e] = (bf16_t)(rotate ? fmaf(u[e], cs[e], -(v[e] * sn[e])) : u[e]);
        o1[e] = (bf16_t)(rotate ? fmaf(v[e], cs[e], u[e] * sn[e]) : v[e]);
      }
      if (row < M && col < N) {
        bf16_t *q = reinterpret_cast<bf16_t *>(ep.C) + (size_t)row * ep.ldc + col;
        *reinterpret_cast<bf16x8_t *>(q) = o0;
        *reinterpret_cast<bf16x8_t *>(q + D / 2) = o1;
      }
      if (rotate && p == 0) {
        pos += 16;
        if (__builtin_amdgcn_ballot_w64(pos >= ep.rope_seq) != 0) {
          pos %= ep.rope_seq;
#pragma unroll
          for (int e = 0; e < 8; e++) rope_sincos((float)pos, hi[e], lo[e], sn[e], cs[e]);
        } else {
#pragma unroll
          for (int e = 0; e < 8; e++) {
            const float s = sn[e];
            sn[e] = fmaf(s, cs16[e], cs[e] * sn16[e]);
            cs[e] = fmaf(cs[e], cs16[e], -(s * sn16[e]));
          }
        }
      }
    }
  }
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool A_KC, bool B_KC, int EPI>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_bf16_kernel(const bf16_t *__restrict__ A, int lda, const bf16_t *__restrict__ B,
                                                        int ldb, int M, int N, int K, int tiles_m, int tiles_n, Epi ep) {
  constexpr int NTH = 64 * WAVES_M * WAVES_N;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N, MI = WM / 32, NI = WN / 32;
  using GA = TileGeom<BM, A_KC>;
  using GB = TileGeom<BN, B_KC>;
  extern __shared__ __attribute__((aligned(16))) char smem_raw[];
  // stage s of A at s*STAGE, of B at s*STAGE + GA::elems (plain offsets from the LDS base keep the
  // accesses in the LDS address space; pointer tables would decay to flat addressing)
  constexpr int STAGE = GA::elems + GB::elems;
  bf16_t *const sbase = reinterpret_cast<bf16_t *>(smem_raw);

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;

  int tm, tn;
  map_tile(tiles_m, tiles_n, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;

  f32x16_t acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; i++)
#pragma unroll
    for (int j = 0; j < NI; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;

  uint4 ra[GA::chunks / NTH], rb[GB::chunks / NTH];
  const int KT = (K + BK - 1) / BK;
  unsigned ma = tile_load<BM, A_KC, NTH>(ra, A, lda, m0, M, 0, K, tid);
  unsigned mb = tile_load<BN, B_KC, NTH>(rb, B, ldb, n0, N, 0, K, tid);
  tile_store<BM, A_KC, NTH>(ra, ma, sbase, tid);
  tile_store<BN, B_KC, NTH>(rb, mb, sbase + GA::elems, tid);
  __syncthreads();

  for (int kt = 0; kt < KT; kt++) {
    const int cur = kt & 1;
    if (kt + 1 < KT) {
      ma = tile_load<BM, A_KC, NTH>(ra, A, lda, m0, M, (kt + 1) * BK, K, tid);
      mb = tile_load<BN, B_KC, NTH>(rb, B, ldb, n0, N, (kt + 1) * BK, K, tid);
    }
    const bf16_t *a_s = sbase + cur * STAGE, *b_s = sbase + cur * STAGE + GA::elems;
#pragma unroll
    for (int kk = 0; kk < BK; kk += 16) {
      bf16x8_t fa[MI], fb[NI];
#pragma unroll
      for (int i = 0; i < MI; i++) fa[i] = frag_load<BM, A_KC>(a_s, wm * WM + i * 32, kk, lane);
#pragma unroll
      for (int j = 0; j < NI; j++) fb[j] = frag_load<BN, B_KC>(b_s, wn * WN + j * 32, kk, lane);
#pragma unroll
      for (int i = 0; i < MI; i++)
#pragma unroll
        for (int j = 0; j < NI; j++)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i], fb[j], acc[i][j], 0, 0, 0);
    }
    if (kt + 1 < KT) {
      tile_store<BM, A_KC, NTH>(ra, ma, sbase + (cur ^ 1) * STAGE, tid);
      tile_store<BN, B_KC, NTH>(rb, mb, sbase + (cur ^ 1) * STAGE + GA::elems, tid);
    }
    __syncthreads();
  }

  store_tile<MI, NI, WN, EPI>(acc, reinterpret_cast<float *>(smem_raw) + wave * (32 * (WN + 8)), m0 + wm * WM, n0 + wn * WN, M, N,
                              ep, lane);
}


// =====================================================================================================
// Kernel with direct-to-LDS loads and rings of 64-deep K-tiles (the path every large GEMM takes).
//
// buffer_load_dwordx4 ... lds moves 16 bytes per lane from global memory straight into LDS (lane i of a
// wave instruction lands at M0 + 16*i): no staging registers, no ds_write, and the loads of one to three
// K-tiles stay in flight behind the MFMAs of the current one.  The buffer form (resource
// descriptor in SGPRs, one 32-bit byte offset per lane, the K position in a scalar offset) is used
// because the issue of a load with 64-bit per-lane addresses holds the SIMD's vector register ports
// long enough to stall the MFMAs of the other wave on that SIMD (measured: about 15 % of a K-tile).
// A wave instruction fills 1 KB of LDS contiguously, so padding is impossible; bank conflicts are
// avoided by permuting WHICH global chunk each lane fetches (an XOR swizzle applied on the global
// side and undone in the fragment address):
//   k-contiguous operand : tile [rows][64], 8 chunks per row; chunk c of row r sits in slot c ^ ((r>>1)&7)
//   row-contiguous operand: tile [64][rows], rows/8 chunks per k-row; chunk c of k-row k sits in slot
//                           c ^ (4*(k&3))   (read back with ds_read_b64_tr_b16); tiles of 64 rows, whose k-row is
//                           half of the 64 banks: c ^ (4*((k>>1)&1))
//
// Depth and rings.  What bounds the kernel besides the matrix pipes is what a compute unit takes in from L2.  A row of a
// 64-deep k-contiguous tile is a whole 128-byte line; with 32-deep tiles each request used half a line and the other half
// was fetched again one K-tile later.  A and B have rings of their own: A's is a stage longer where LDS has room for it
// but not for a third stage of both (256 x 256: 3 x 32 + 2 x 32 KB), and A's part of a K-tile is then loaded a whole
// K-tile ahead of B's.  Against one ring of four 32-deep tiles (us, 8192^3, both operands k-contiguous): 256 x 256 tile
// 867 -> 790, 128 x 256 1143 -> 886, 128 x 128 1276 -> 968; forward layout 854 / 991 / 1166 -> 799 / 882 / 972; weight gradient
// 862 / 927 / 1062 -> 796 / 908 / 1018.  [4096, 1792] K = 7168, k-contiguous: 127 -> 94; [3072, 640] K = 5120: 45 -> 34.  Two
// stages of both operands are worth less (256 x 256: 860, 128 x 256: 1097: the last loads have half a K-tile to arrive).
//
// Schedule.  Two waves per SIMD run freely (no phase lock); each wave software-pipelines its fragments:
// the LDS reads of the next 16-deep step are issued before the MFMAs of the current one, so LDS
// latency hides behind the wave's own MFMAs and the other wave on the SIMD fills what is left.  All
// fragment reads are inline assembly with explicit lgkmcnt waits: the compiler neither tracks the
// direct-to-LDS loads nor may it order LDS reads behind them (through builtins it would wait for
// vmcnt(0) before every transposing read).  One s_barrier per K-tile, between its last two steps:
//     s_waitcnt vmcnt(IN_FLIGHT) lgkmcnt(0) ; s_barrier
// after it tile kt+1 has landed for every wave, and no wave has a read of tile kt outstanding (the
// fragments of its last step are in registers), so its stages are refilled right there.
// Rows past M / N are fetched from a clamped (valid) address and never stored; each operand must span less than
// 2 GiB.  K is a multiple of 8; when it is not one of 64 (KTAIL) the last K-tile is partly empty: lanes whose 8-deep
// chunk lies past K fetch the tile's first chunk instead (in bounds, any value) and the fragments of that tile are
// zeroed in registers, both operands, where k >= K (a chunk of 8 is exactly a fragment's lane half).  Against the
// register-staged kernel, which such K took before: 37 - 45 -> 23 - 31 us for [3000, 1032] x [1032, 2744] and its backward
// forms.
// =====================================================================================================
constexpr int DK = 64;         // K-tile depth of the DMA kernel

template <int ROWS, bool KC, int NWAVES, int DEPTH = DK>
struct DmaOp {
  static_assert(DEPTH == 32 || DEPTH == 64, "K-tile depth");
  static_assert(ROWS % 16 == 0, "a tile is a whole number of 1 KB pieces per K-tile");
  static_assert(KC || (ROWS / 8) % 8 == 0, "the chunk permutation of a row-contiguous tile works on blocks of 8 or 16 chunks");
  static constexpr int PIECES = ROWS * DEPTH / 512;                      // 1 KB pieces (wave instructions) per K-tile
  static_assert(PIECES % NWAVES == 0, "every wave issues the same number of loads per K-tile, which the vmcnt waits rely on");
  static constexpr int NINST = PIECES / NWAVES;                          // loads per wave per K-tile
  static constexpr int bytes = ROWS * DEPTH * 2;
  static constexpr int CPR = KC ? DEPTH / 8 : ROWS / 8;                  // 16-byte chunks per tile row (k-contiguous) or k-row
  static constexpr int LDS_OPS_PER_FRAG = KC ? 1 : 2;
  // chunk permutation of row r (k-contiguous) or k-row r (row-contiguous)
  static __device__ __forceinline__ int swz(int r) {
    if (KC) return DEPTH == 32 ? (r >> 2) & 3 : (r >> 1) & 7;
    return CPR % 16 == 0 ? 4 * (r & 3) : 4 * ((r >> 1) & 1);
  }
  // piece that load j of wave `wave` fetches
  static __device__ __forceinline__ int piece(int j, int wave) { return wave + NWAVES * j; }
  // byte offset (from the operand base, K-tile 0) of the chunk that lane `lane` of this wave's j-th
  // instruction must fetch; a chunk at or past k_lim (within the K-tile) is replaced by one at its beginning
  static __device__ __forceinline__ unsigned chunk_offset(int j, int wave, int lane, int ld, int row0, int row_lim, int k_lim = DEPTH) {
    const int p = piece(j, wave) * 64 + lane;
    if (KC) {
      const int r = p / CPR;
      int c = (p % CPR) ^ swz(r);
      if (c * 8 >= k_lim) c = 0;
      const int row = min(row0 + r, row_lim - 1);
      return ((unsigned)row * (unsigned)ld + c * 8) * 2u;
    } else {
      int k = p / CPR;
      const int c = (p % CPR) ^ swz(k);
      if (k >= k_lim) k = 0;
      int col = row0 + c * 8;
      col = col < row_lim ? col : 0;
      return ((unsigned)k * (unsigned)ld + col) * 2u;
    }
  }
  // LDS byte offsets (within a tile) from which the fragments of rows row .. row + 32*NF - 1 are read:
  // k-contiguous: one address per 16-deep step (fragment i adds 32 rows as an immediate);
  // row-contiguous: one address per fragment (a step adds 16 k-rows as an immediate).
  // STRIDE: rows from one fragment to the next (row-contiguous)
  template <int NF, int STRIDE = 32>
  static __device__ __forceinline__ void frag_bases(unsigned (&ad)[KC ? DEPTH / 16 : NF], int row, int lane) {
    if (KC) {
      const int r = row + (lane & 31);
#pragma unroll
      for (int h = 0; h < DEPTH / 16; h++) {
        const int c = 2 * h + (lane >> 5);
        ad[h] = (r * CPR + (c ^ swz(r))) * 16;
      }
    } else {
      const int k = 8 * (lane >> 5) + ((lane & 15) >> 2);
#pragma unroll
      for (int i = 0; i < NF; i++) {
        const int col = row + STRIDE * i + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
        ad[i] = (k * CPR + ((col >> 3) ^ swz(k))) * 16 + (col & 7) * 2;
      }
    }
  }
  // issues the reads of the NF fragments of step H (k = 16*H .. 16*H+15) of the tile at LDS address `tile`
  template <int H, int NF, int... I>
  static __device__ __forceinline__ void frag_issue(u32x4_t (&f)[NF], const unsigned (&ad)[KC ? DEPTH / 16 : NF], unsigned tile,
                                                    std::integer_sequence<int, I...>) {
    if constexpr (KC) {
      const unsigned a = ad[H] + tile;
      ((f[I] = lds_read_b128<I * 32 * DEPTH * 2>(a)), ...);
    } else {
      ((f[I] = lds_read_tr16<H * 16 * CPR * 16, 4 * CPR * 16>(ad[I] + tile)), ...);
    }
  }
};

template <int BM, int BN, int WAVES_M, int WAVES_N, int NSTA, int NSTB, bool A_KC, bool B_KC, int EPI, bool KTAIL, int MM = MM_ONE, typename E = Epi>
__device__ __forceinline__ void gemm_dma_tile(const bf16_t *__restrict__ A, int lda, int a_bytes, const bf16_t *__restrict__ B, int ldb, int b_bytes,
                                              int M, int N, int K, int tm, int tn, const E &ep, const bf16_t *__restrict__ A2 = nullptr,
                                              const bf16_t *__restrict__ B2 = nullptr) {
  constexpr int NWAVES = WAVES_M * WAVES_N;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N, MI = WM / 32, NI = WN / 32;
  constexpr int NB = MM == MM_PAIR ? 2 : 1;     // B operands in the tile
  constexpr bool ROPE = EPI == EPI_ROPE64 || EPI == EPI_ROPE128;
  static_assert((MM != MM_PAIR && !ROPE) || (!B_KC && NI == 2), "a wave holds one 32-column block of each product, or of each half of a head");
  using OA = DmaOp<BM, A_KC, NWAVES, DK>;
  using OB = DmaOp<BN / NB, B_KC, NWAVES, DK>;
  constexpr int B_BYTES = NB * OB::bytes, B_NINST = NB * OB::NINST;
  constexpr int STEPS = DK / 16;
  static_assert(NSTA >= NSTB && NSTB >= 2, "the loads of a K-tile's B part go ahead of those of a later one's A part");
  constexpr int RING_B = NSTA * OA::bytes;      // LDS: ring of A, then ring of B
  constexpr int LOADS_PER_TILE = OA::NINST + B_NINST;
  constexpr int READS_PER_STEP = MI * OA::LDS_OPS_PER_FRAG + NI * OB::LDS_OPS_PER_FRAG;
  // lgkmcnt is a 4-bit counter: with 16 reads per step the wait for "the previous step's reads" also waits for
  // the first read of the step just issued (the reads of a wave complete in order)
  constexpr int READS_WAIT = READS_PER_STEP < 15 ? READS_PER_STEP : 15;
  static_assert(READS_PER_STEP <= 16, "one step's fragment reads must fit the lgkmcnt counter");
  extern __shared__ __attribute__((aligned(1024))) char smem_raw[];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#ifdef STP_GEMM_TRACE
  const long long tr0 = wall_clock64();
#endif
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);   // same value, known wave-uniform: LDS targets of the loads stay scalar
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  const int m0 = tm * BM, n0 = tn * (BN / NB);

  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(A), 0, a_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(B), 0, b_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t ra2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(MM == MM_SUM ? A2 : A), 0, a_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rb2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(MM == MM_ONE ? B : B2), 0, b_bytes, 0x00020000);
  unsigned offa[OA::NINST], offb[OB::NINST];
#pragma unroll
  for (int j = 0; j < OA::NINST; j++) offa[j] = OA::chunk_offset(j, wave, lane, lda, m0, M);
#pragma unroll
  for (int j = 0; j < OB::NINST; j++) offb[j] = OB::chunk_offset(j, wave, lane, ldb, n0, N);
  // the same for the last, partly empty K-tile
  const int k_rem = KTAIL ? K % DK : DK;
  unsigned taila[OA::NINST], tailb[OB::NINST];
#pragma unroll
  for (int j = 0; j < OA::NINST; j++) taila[j] = KTAIL ? OA::chunk_offset(j, wave, lane, lda, m0, M, k_rem) : offa[j];
#pragma unroll
  for (int j = 0; j < OB::NINST; j++) tailb[j] = KTAIL ? OB::chunk_offset(j, wave, lane, ldb, n0, N, k_rem) : offb[j];
  const unsigned stepa = (A_KC ? (unsigned)DK : (unsigned)DK * lda) * 2u;
  const unsigned stepb = (B_KC ? (unsigned)DK : (unsigned)DK * ldb) * 2u;

  unsigned ada[A_KC ? STEPS : MI], adb[B_KC ? STEPS : NI];
  OA::template frag_bases<MI>(ada, wm * WM, lane);
  // first column of the wave in the tile; at head dimension 128 its second block is the head's other half
  const int wcol = MM == MM_PAIR ? wn * 32 : EPI == EPI_ROPE128 ? (wn >> 1) * 128 + (wn & 1) * 32 : wn * WN;
  OB::template frag_bases<NI, EPI == EPI_ROPE128 ? 64 : 32>(adb, wcol, lane);
  if constexpr (MM == MM_PAIR) adb[1] = adb[0] + OB::bytes;      // the same columns of the other operand's tile
  const unsigned lds0 = (unsigned)(size_t)(const __attribute__((address_space(3))) char *)smem_raw;

  f32x16_t acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; i++)
#pragma unroll
    for (int j = 0; j < NI; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;

  const int KT1 = KTAIL ? K / DK + 1 : K / DK, KT = MM == MM_SUM ? 2 * KT1 : KT1;     // K-tiles of a product, of the tile
  // The direct-to-LDS loads form one stream of groups: group g (issued from K-tile g on) is B's part of tile g + NSTB, then
  // A's part of tile g + NSTA, the stages that tile g occupied.
  // Issuing a load holds the wave until the address unit takes it, so the loads are placed one at a time
  // between MFMAs (whose execution covers the hold) instead of in a burst behind the barrier, where the
  // eight waves would queue on the address FIFO with the matrix pipes idle.  The first LF loads of a group, B's, go into the
  // MFMA block that follows the barrier (the stages are free from there on), the rest into the next two.
#define STP_ISSUE(q, g, sta, stb)                                                                                \
  do {                                                                                                           \
    if ((q) < B_NINST) {                                                                                         \
      const int kt_ = min((g) + NSTB, KT - 1), q_ = (q) < B_NINST ? (q) : 0, j_ = q_ % OB::NINST;                \
      const bool second_ = MM == MM_PAIR ? q_ >= OB::NINST : MM == MM_SUM && kt_ >= KT1;                         \
      const int k_ = MM == MM_SUM && second_ ? kt_ - KT1 : kt_;                                                  \
      dma_load16(second_ ? rb2 : rb, smem_raw + RING_B + (stb) * B_BYTES + (q_ / OB::NINST) * OB::bytes + OB::piece(j_, wave_s) * 1024, \
                 KTAIL && k_ == KT1 - 1 ? tailb[j_] : offb[j_], k_ * stepb);                                     \
    } else {                                                                                                     \
      const int kt_ = min((g) + NSTA, KT - 1), j_ = (q) >= B_NINST ? (q) - B_NINST : 0;                          \
      const bool second_ = MM == MM_SUM && kt_ >= KT1;                                                           \
      const int k_ = second_ ? kt_ - KT1 : kt_;                                                                  \
      dma_load16(second_ ? ra2 : ra, smem_raw + (sta) * OA::bytes + OA::piece(j_, wave_s) * 1024,                \
                 KTAIL && k_ == KT1 - 1 ? taila[j_] : offa[j_], k_ * stepa);                                     \
    }                                                                                                            \
  } while (0)
  u32x4_t fa0[MI], fb0[NI], fa1[MI], fb1[NI];
  constexpr int LF = (LOADS_PER_TILE + 1) / 2, L0 = (LOADS_PER_TILE - LF + 1) / 2;
  // prologue: groups -NSTA .. -2 and the first LF loads of group -1 (a group's B part does not exist below -NSTB)
#pragma unroll
  for (int g = -NSTA; g < 0; g++)
#pragma unroll
    for (int q = g < -NSTB ? B_NINST : 0; q < (g < -1 ? LOADS_PER_TILE : LF); q++) STP_ISSUE(q, g, g + NSTA, g + NSTB);

  using SeqM = std::make_integer_sequence<int, MI>;
  using SeqN = std::make_integer_sequence<int, NI>;
#define STP_READ(H, FA, FB, sta, stb)                                                \
  do {                                                                               \
    OA::template frag_issue<H>(FA, ada, lds0 + (unsigned)(sta) * OA::bytes, SeqM{}); \
    OB::template frag_issue<H>(FB, adb, lds0 + RING_B + (unsigned)(stb) * B_BYTES, SeqN{}); \
    __builtin_amdgcn_sched_barrier(0);                                               \
  } while (0)
  // zeroes the fragments of step H of the last K-tile in the lanes whose k lies past K (after their lds_tie)
  auto mask_tail = [&](u32x4_t (&fa)[MI], u32x4_t (&fb)[NI], int H) {
    const unsigned keep = 16 * H + 8 * (lane >> 5) < k_rem ? ~0u : 0u;
#pragma unroll
    for (int i = 0; i < MI; i++) fa[i] &= keep;
#pragma unroll
    for (int j = 0; j < NI; j++) fb[j] &= keep;
  };
  // MI*NI MFMAs with loads Q0 .. Q0+NQ-1 of group g spread evenly between them
#define STP_MFMAS(H, FA, FB, Q0, NQ, g, sta, stb)                                   \
  do {                                                                               \
    lds_tie(FA);                                                                     \
    lds_tie(FB);                                                                     \
    if (KTAIL && (kt == KT - 1 || (MM == MM_SUM && kt == KT1 - 1))) mask_tail(FA, FB, H); \
    _Pragma("unroll") for (int i = 0; i < MI; i++)                                   \
      _Pragma("unroll") for (int j = 0; j < NI; j++) {                               \
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, FA[i]), __builtin_bit_cast(bf16x8_t, FB[j]), \
                                                            acc[i][j], 0, 0, 0);     \
        _Pragma("unroll") for (int r = 0; r < (NQ); r++)                             \
          if (i * NI + j == max(0, ((r + 1) * MI * NI) / ((NQ) + 1) - 1)) {          \
            __builtin_amdgcn_sched_barrier(0);                                       \
            STP_ISSUE((Q0) + r, g, sta, stb);                                        \
            __builtin_amdgcn_sched_barrier(0);                                       \
          }                                                                          \
      }                                                                              \
    __builtin_amdgcn_sched_barrier(0);                                               \
  } while (0)

  // loads that may still be on their way where K-tile kt+1 is needed: the groups behind the one with its B part and, if A
  // runs ahead, that group's own A part
  constexpr int IN_FLIGHT = (NSTB - 2) * LOADS_PER_TILE + (NSTA > NSTB ? OA::NINST : 0);
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(IN_FLIGHT + LF) : "memory");
#ifdef STP_GEMM_TRACE
  const long long tr1 = wall_clock64();
#endif
  STP_READ(0, fa0, fb0, 0, 0);

  int sa = 0, sb = 0;                    // kt % NSTA, kt % NSTB
  for (int kt = 0; kt < KT; kt++) {
    const int na = sa + 1 == NSTA ? 0 : sa + 1, nb = sb + 1 == NSTB ? 0 : sb + 1;
    STP_READ(1, fa1, fb1, sa, sb);
    lds_wait<READS_WAIT>();              // the reads of step 0 (issued one step ago) have returned
    STP_MFMAS(0, fa0, fb0, LF, L0, kt - 1, sa == 0 ? NSTA - 1 : sa - 1, sb == 0 ? NSTB - 1 : sb - 1);
    STP_READ(2, fa0, fb0, sa, sb);
    lds_wait<READS_WAIT>();
    STP_MFMAS(1, fa1, fb1, LF + L0, LOADS_PER_TILE - LF - L0, kt - 1, sa == 0 ? NSTA - 1 : sa - 1, sb == 0 ? NSTB - 1 : sb - 1);
    STP_READ(3, fa1, fb1, sa, sb);
    lds_wait<READS_WAIT>();
    STP_MFMAS(2, fa0, fb0, 0, 0, 0, 0, 0);
    // tile kt+1 has landed once at most IN_FLIGHT of this wave's loads remain on their way;
    // lgkmcnt(0): this wave's reads of tile kt are complete, so after the barrier its stages are free
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(IN_FLIGHT) : "memory");
    __builtin_amdgcn_sched_barrier(0);
    STP_READ(0, fa0, fb0, na, nb);   // past the last tile this reads a stale stage; never used
    lds_wait<READS_WAIT>();
    STP_MFMAS(3, fa1, fb1, 0, LF, kt, sa, sb);
    sa = na;
    sb = nb;
  }
#undef STP_READ
#undef STP_MFMAS
#undef STP_ISSUE
  // drain the (redundant) tail loads and reads before the stages are reused as epilogue staging
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
  lds_tie(fa0);
  lds_tie(fb0);
#ifdef STP_GEMM_TRACE
  const long long tr2 = wall_clock64();
#endif
  float *const stage = reinterpret_cast<float *>(smem_raw) + wave * (32 * (WN + 8));
  if constexpr (MM == MM_PAIR) store_pairs<MI, EPI>(acc, stage, m0 + wm * WM, n0 + wcol, M, N, ep, lane);
  else if constexpr (ROPE) store_rope<MI, EPI == EPI_ROPE128 ? 128 : 64>(acc, stage, m0 + wm * WM, n0 + wcol, M, N, ep, lane);
  else store_tile<MI, NI, WN, EPI>(acc, stage, m0 + wm * WM, n0 + wcol, M, N, ep, lane);
#ifdef STP_GEMM_TRACE
  if (ep.trace) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const long long tr3 = wall_clock64();
    if (tid == 0) {
      unsigned hw;
      asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(hw));
      long long *t = ep.trace + (size_t)blockIdx.x * 5;
      t[0] = tr0; t[1] = tr1; t[2] = tr2; t[3] = tr3; t[4] = hw;
    }
  }
#endif
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int NSTA, int NSTB, bool A_KC, bool B_KC, int EPI, bool KTAIL>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_bf16_dma_kernel(const bf16_t *__restrict__ A, int lda, int a_bytes,
                                                            const bf16_t *__restrict__ B, int ldb, int b_bytes, int M, int N, int K,
                                                            int tiles_m, int tiles_n, Epi ep) {
  int tm, tn;
  map_tile(tiles_m, tiles_n, tm, tn);
  gemm_dma_tile<BM, BN, WAVES_M, WAVES_N, NSTA, NSTB, A_KC, B_KC, EPI, KTAIL>(A, lda, a_bytes, B, ldb, b_bytes, M, N, K, tm, tn, ep);
}

// Two products in one kernel (the SwiGLU MLP's gate and up projections, and the two terms of its input gradient); the operands of a
// kind share pitch and extent.
template <int BM, int BN, int WAVES_M, int WAVES_N, int NSTA, int NSTB, bool A_KC, bool B_KC, int EPI, bool KTAIL, int MM>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_bf16_two_kernel(const bf16_t *__restrict__ A, const bf16_t *__restrict__ A2, int lda,
                                                            int a_bytes, const bf16_t *__restrict__ B, const bf16_t *__restrict__ B2, int ldb,
                                                            int b_bytes, int M, int N, int K, int tiles_m, int tiles_n, Epi ep) {
  int tm, tn;
  map_tile(tiles_m, tiles_n, tm, tn);
  gemm_dma_tile<BM, BN, WAVES_M, WAVES_N, NSTA, NSTB, A_KC, B_KC, EPI, KTAIL, MM>(A, lda, a_bytes, B, ldb, b_bytes, M, N, K, tm, tn, ep, A2, B2);
}

// QKV projection with the rotary embedding in the epilogue
template <int BM, int BN, int WAVES_M, int WAVES_N, int NSTA, int NSTB, int EPI, bool KTAIL>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_bf16_rope_kernel(const bf16_t *__restrict__ A, int lda, int a_bytes, const bf16_t *__restrict__ B,
                                                            int ldb, int b_bytes, int M, int N, int K, int tiles_m, int tiles_n, EpiRope ep) {
  int tm, tn;
  map_tile(tiles_m, tiles_n, tm, tn);
  gemm_dma_tile<BM, BN, WAVES_M, WAVES_N, NSTA, NSTB, true, false, EPI, KTAIL, MM_ONE, EpiRope>(A, lda, a_bytes, B, ldb, b_bytes, M, N, K, tm, tn, ep);
}

// Several products with one contraction length in one launch: the weight gradients of a unit.  Alone each of them ends in
// a round of workgroups that fills a part of the chip.
struct Problem { const bf16_t *A, *B; float *C; int lda, a_bytes, ldb, b_bytes, ldc, M, N, tiles_m, tiles_n, first; };
struct ProblemSet { int n, tiles; Problem p[3]; };
template <int BM, int BN, int WAVES_M, int WAVES_N, int NSTA, int NSTB, bool A_KC, bool B_KC, bool KTAIL>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N) void gemm_bf16_set_kernel(ProblemSet set, int K) {
  int pid = xcd_order(set.tiles);
  const int i = set.n > 2 && pid >= set.p[2].first ? 2 : pid >= set.p[1].first ? 1 : 0;
  const Problem &q = set.p[i];
  int tm, tn;
  tile_of(pid - q.first, q.tiles_m, q.tiles_n, tm, tn);
  Epi ep = {};
  ep.C = q.C;
  ep.ldc = q.ldc;
  gemm_dma_tile<BM, BN, WAVES_M, WAVES_N, NSTA, NSTB, A_KC, B_KC, EPI_F32_ACCUM, KTAIL>(q.A, q.lda, q.a_bytes, q.B, q.ldb, q.b_bytes, q.M, q.N, K,
                                                                                     tm, tn, ep);
}

// =====================================================================================================
// Few output tiles: a 64 x 64 tile whose contraction is shared out over the four waves of a workgroup.
//
// For outputs of so few 128 x 128 tiles that most of the 256 compute units would idle ([1024, 1024]: 64 tiles, each a
// chain of K / 32 K-tiles behind barriers).  Wave w takes the WK-deep K-tiles w, w + 4, ... of the whole tile through a
// ring of its own, so there is no barrier until the four partial sums are added (in wave order, through LDS); a
// fragment feeds two MFMAs instead of one, and four K-tiles advance at a time.  (The same tile as 2 x 2 waves with a
// barrier per 64-deep stage spent 350 clocks per 32-deep K-tile on barrier, LDS and load-issue latency one after the
// other, whatever the depth of the ring: 18.6 us for [1024, 1024] K = 4096 against 15.5.)
// Bound by what a compute unit takes in: 41 B per clock at K = 4096.  Rows of a k-contiguous operand are fetched 128 bytes
// at a time (WK = 64): with 64-byte pieces L2 delivers half as much per request and the same shape takes 18 us.  Without
// such an operand a row-contiguous tile has 128-byte rows anyway and 32-deep K-tiles, more of them in flight, are the
// faster (weight gradient [320, 784] K = 1824: 8.0 against 9.2 us).
// The sum over K is taken in another order than in the tiles above, so who takes this kernel is a question of the
// shape alone (never of other streams or tile preferences): see wavek_shape.
// =====================================================================================================
template <int WK, bool A_KC, bool B_KC, int EPI, bool KTAIL, int MM>
__device__ __forceinline__ void gemm_wavek_tile(const bf16_t *__restrict__ A, int lda, int a_bytes, const bf16_t *__restrict__ B, int ldb, int b_bytes,
                                                int M, int N, int K, int tm, int tn, const Epi &ep, const bf16_t *__restrict__ A2,
                                                const bf16_t *__restrict__ B2) {
  static_assert(MM == MM_ONE || MM == MM_SUM, "one output");
  constexpr int BM = 64, BN = 64, KS = 4, NSTG = 128 / WK, MI = 2, NI = 2;
  using OA = DmaOp<BM, A_KC, 1, WK>;
  using OB = DmaOp<BN, B_KC, 1, WK>;
  constexpr int STAGE_BYTES = OA::bytes + OB::bytes;
  constexpr int LOADS = OA::NINST + OB::NINST;                       // per K-tile
  constexpr int READS = MI * OA::LDS_OPS_PER_FRAG + NI * OB::LDS_OPS_PER_FRAG;   // per 16-deep step
  extern __shared__ __attribute__((aligned(1024))) char smem_raw[];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = tm * BM, n0 = tn * BN;
  const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(A), 0, a_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(B), 0, b_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t ra2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(MM == MM_SUM ? A2 : A), 0, a_bytes, 0x00020000);
  const __amdgpu_buffer_rsrc_t rb2 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(MM == MM_SUM ? B2 : B), 0, b_bytes, 0x00020000);
  const int k_rem = KTAIL ? K % WK : WK;
  unsigned offa[OA::NINST], offb[OB::NINST], taila[OA::NINST], tailb[OB::NINST];
#pragma unroll
  for (int j = 0; j < OA::NINST; j++) {
    offa[j] = OA::chunk_offset(j, 0, lane, lda, m0, M);
    taila[j] = KTAIL ? OA::chunk_offset(j, 0, lane, lda, m0, M, k_rem) : offa[j];
  }
#pragma unroll
  for (int j = 0; j < OB::NINST; j++) {
    offb[j] = OB::chunk_offset(j, 0, lane, ldb, n0, N);
    tailb[j] = KTAIL ? OB::chunk_offset(j, 0, lane, ldb, n0, N, k_rem) : offb[j];
  }
  const unsigned stepa = (A_KC ? (unsigned)WK : (unsigned)WK * lda) * 2u, stepb = (B_KC ? (unsigned)WK : (unsigned)WK * ldb) * 2u;
  unsigned ada[A_KC ? WK / 16 : MI], adb[B_KC ? WK / 16 : NI];
  OA::template frag_bases<MI>(ada, 0, lane);
  OB::template frag_bases<NI>(adb, 0, lane);
  char *const ring = smem_raw + wave * NSTG * STAGE_BYTES;
  const unsigned lds0 = (unsigned)(size_t)(const __attribute__((address_space(3))) char *)ring;

  f32x16_t acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; i++)
#pragma unroll
    for (int j = 0; j < NI; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) acc[i][j][v] = 0.f;

  const int KT1 = KTAIL ? K / WK + 1 : K / WK, KT = MM == MM_SUM ? 2 * KT1 : KT1;
  const int NT = (KT - wave + KS - 1) / KS;      // this wave's K-tiles: wave, wave + KS, ...
  auto issue = [&](int t) {
    const bool second = MM == MM_SUM && t * KS + wave >= KT1;
    const int kt = t * KS + wave - (second ? KT1 : 0);
    const bool last = KTAIL && kt == KT1 - 1;
    char *st = ring + (t % NSTG) * STAGE_BYTES;
#pragma unroll
    for (int q = 0; q < OA::NINST; q++) dma_load16(second ? ra2 : ra, st + q * 1024, last ? taila[q] : offa[q], kt * stepa);
#pragma unroll
    for (int q = 0; q < OB::NINST; q++) dma_load16(second ? rb2 : rb, st + OA::bytes + q * 1024, last ? tailb[q] : offb[q], kt * stepb);
    __builtin_amdgcn_sched_barrier(0);
  };
  using Seq2 = std::make_integer_sequence<int, 2>;
  u32x4_t fa[2][MI], fb[2][NI];                  // fragments of two consecutive 16-deep steps
#define STP_READ(H, t)                                                               \
  do {                                                                               \
    const unsigned t_ = lds0 + (unsigned)((t) % NSTG) * STAGE_BYTES;                 \
    OA::template frag_issue<H>(fa[(H) & 1], ada, t_, Seq2{});                        \
    OB::template frag_issue<H>(fb[(H) & 1], adb, t_ + OA::bytes, Seq2{});            \
    __builtin_amdgcn_sched_barrier(0);                                               \
  } while (0)
#define STP_MFMAS(H, t)                                                              \
  do {                                                                               \
    lds_tie(fa[(H) & 1]);                                                            \
    lds_tie(fb[(H) & 1]);                                                            \
    if (KTAIL && ((t) * KS + wave == KT - 1 || (MM == MM_SUM && (t) * KS + wave == KT1 - 1))) { \
      const unsigned keep = 16 * (H) + 8 * (lane >> 5) < k_rem ? ~0u : 0u;           \
      _Pragma("unroll") for (int i = 0; i < 2; i++) { fa[(H) & 1][i] &= keep; fb[(H) & 1][i] &= keep; } \
    }                                                                                \
    _Pragma("unroll") for (int i = 0; i < MI; i++)                                   \
      _Pragma("unroll") for (int j = 0; j < NI; j++)                                 \
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, fa[(H) & 1][i]),                \
                                                            __builtin_bit_cast(bf16x8_t, fb[(H) & 1][j]), acc[i][j], 0, 0, 0); \
    __builtin_amdgcn_sched_barrier(0);                                               \
  } while (0)
  // waits until at most n of this wave's K-tiles are still on their way
  auto wait_tiles = [&](int n) {
    if (n >= NSTG - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NSTG - 1) * LOADS) : "memory");
    else if (NSTG > 2 && n == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * LOADS) : "memory");
    else if (NSTG > 2 && n == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int t = 0; t < NSTG; t++)
    if (t < NT) issue(t);
  if (NT > 0) {
    wait_tiles(NT - 1);
    STP_READ(0, 0);
  }
  for (int t = 0; t < NT; t++) {
    STP_READ(1, t);
    lds_wait<READS>();
    STP_MFMAS(0, t);
    if constexpr (WK == 64) {
      STP_READ(2, t);
      lds_wait<READS>();
      STP_MFMAS(1, t);
      STP_READ(3, t);
      lds_wait<READS>();
      STP_MFMAS(2, t);
    }
    // this wave's reads of K-tile t are complete: its slot takes K-tile t + NSTG; K-tile t+1 has to land
    lds_wait<0>();
    __builtin_amdgcn_sched_barrier(0);
    if (t + NSTG < NT) issue(t + NSTG);
    wait_tiles(NT - 2 - t);
    if (t + 1 < NT) STP_READ(0, t + 1);
    STP_MFMAS(WK / 16 - 1, t);
  }
#undef STP_READ
#undef STP_MFMAS
  // ---- partial sums to LDS (pitch 72: the lane halves, 4 rows apart, use different banks), added in wave order
  constexpr int RP = BN + 8;
  float *red = reinterpret_cast<float *>(smem_raw);                  // [KS][64][RP]
  int pr[2], pc;
  EpiPre pre[2];
  float bias[8];
  pc = n0 + (tid & 7) * 8;
  epi_bias(bias, pc, N, ep);
#pragma unroll
  for (int p = 0; p < 2; p++) {
    pr[p] = p * 32 + (tid >> 3);
    epi_fetch<EPI>(pre[p], m0 + pr[p], pc, M, N, ep);
  }
  __syncthreads();                                                   // every wave is done with its ring
  const int lr = lane & 31, lg = lane >> 5;
#pragma unroll
  for (int i = 0; i < MI; i++)
#pragma unroll
    for (int j = 0; j < NI; j++)
#pragma unroll
      for (int v = 0; v < 16; v++) red[(wave * BM + i * 32 + 8 * (v >> 2) + 4 * lg + (v & 3)) * RP + 32 * j + lr] = acc[i][j][v];
  __syncthreads();
#pragma unroll
  for (int p = 0; p < 2; p++) {
    float val[8], part[8];
    Vec8<float>::load(red + pr[p] * RP + (tid & 7) * 8, val);
#pragma unroll
    for (int w = 1; w < KS; w++) {
      Vec8<float>::load(red + (w * BM + pr[p]) * RP + (tid & 7) * 8, part);
#pragma unroll
      for (int e = 0; e < 8; e++) val[e] += part[e];
    }
    epi_store<EPI>(val, bias, pre[p], m0 + pr[p], pc, M, N, ep);
  }
}

template <int WK, bool A_KC, bool B_KC, int EPI, bool KTAIL, int MM>
__global__ __launch_bounds__(256, 2) void gemm_bf16_wavek_kernel(const bf16_t *__restrict__ A, int lda, int a_bytes, const bf16_t *__restrict__ B,
                                                                 int ldb, int b_bytes, int M, int N, int K, int tiles_m, int tiles_n, Epi ep,
                                                                 const bf16_t *__restrict__ A2, const bf16_t *__restrict__ B2) {
  int tm, tn;
  map_tile(tiles_m, tiles_n, tm, tn);
  gemm_wavek_tile<WK, A_KC, B_KC, EPI, KTAIL, MM>(A, lda, a_bytes, B, ldb, b_bytes, M, N, K, tm, tn, ep, A2, B2);
}
// The weight gradients of a unit whose outputs are all this small, in one launch: each alone leaves compute units idle, and the second
// workgroup that fits one.
template <bool KTAIL>
__global__ __launch_bounds__(256, 2) void gemm_bf16_wavek_set_kernel(ProblemSet set, int K) {
  const int pid = xcd_order(set.tiles), i = set.n > 2 && pid >= set.p[2].first ? 2 : pid >= set.p[1].first ? 1 : 0;
  const Problem &q = set.p[i];
  int tm, tn;
  tile_of(pid - q.first, q.tiles_m, q.tiles_n, tm, tn);
  Epi ep = {};
  ep.C = q.C;
  ep.ldc = q.ldc;
  gemm_wavek_tile<32, false, false, EPI_F32_ACCUM, KTAIL, MM_ONE>(q.A, q.lda, q.a_bytes, q.B, q.ldb, q.b_bytes, q.M, q.N, K, tm, tn, ep, nullptr, nullptr);
}

// extent in bytes of a K x rows operand as the kernel addresses it; 0 if it does not fit a 31-bit offset
inline long operand_bytes(bool kc, long rows, long K, long ld) {
  long el = kc ? (rows - 1) * ld + K : (K - 1) * ld + rows;
  return el * 2 < 0x7fffffffL ? el * 2 : 0;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, int NSTA, int NSTB, bool A_KC, bool B_KC, int EPI, bool KTAIL>
int launch_dma(stp_ctx *ctx, const stp_gemm_args *a, const Epi &ep, hipStream_t s) {
  constexpr size_t smem = (size_t)(NSTA * BM + NSTB * BN) * DK * 2;
  static_assert(smem <= 160 * 1024 && smem >= (size_t)WAVES_M * WAVES_N * 32 * (BN / WAVES_N + 8) * sizeof(float), "LDS budget");
  auto kern = gemm_bf16_dma_kernel<BM, BN, WAVES_M, WAVES_N, NSTA, NSTB, A_KC, B_KC, EPI, KTAIL>;
  static bool attr_set = false;
  if (!attr_set) {
    STP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    attr_set = true;
  }
  const int tiles_m = (a->M + BM - 1) / BM, tiles_n = (a->N + BN - 1) / BN;
  const long ab = operand_bytes(A_KC, a->M, a->K, a->lda), bb = operand_bytes(B_KC, a->N, a->K, a->ldb);
  hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(64 * WAVES_M * WAVES_N), smem, s, (const bf16_t *)a->A, a->lda, (int)ab, (const bf16_t *)a->B,
                     a->ldb, (int)bb, a->M, a->N, a->K, tiles_m, tiles_n, ep);
  STP_LAUNCH_CHECK(ctx);
  return STP_OK;
}

template <int WK, bool A_KC, bool B_KC, int EPI, bool KTAIL, int MM = MM_ONE>
int launch_wavek(stp_ctx *ctx, const stp_gemm_args *a, const Epi &ep, hipStream_t s, const void *A2 = nullptr, const void *B2 = nullptr) {
  constexpr size_t smem = (size_t)4 * 128 * (64 + 64) * 2;               // four rings of K-tiles, 128 deep together
  static_assert(smem <= 160 * 1024 && smem >= (size_t)4 * 64 * (64 + 8) * sizeof(float), "LDS budget");
  auto kern = gemm_bf16_wavek_kernel<WK, A_KC, B_KC, EPI, KTAIL, MM>;
  static bool attr_set = false;
  if (!attr_set) {
    STP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    attr_set = true;
  }
  const int tiles_m = (a->M + 63) / 64, tiles_n = (a->N + 63) / 64;
  const long ab = operand_bytes(A_KC, a->M, a->K, a->lda), bb = operand_bytes(B_KC, a->N, a->K, a->ldb);
  hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(256), smem, s, (const bf16_t *)a->A, a->lda, (int)ab, (const bf16_t *)a->B, a->ldb,
                     (int)bb, a->M, a->N, a->K, tiles_m, tiles_n, ep, (const bf16_t *)A2, (const bf16_t *)B2);
  STP_LAUNCH_CHECK(ctx);
  return STP_OK;
}

template <int BM, int BN, int WAVES_M, int WAVES_N, bool A_KC, bool B_KC, int EPI>
int launch_cfg(stp_ctx *ctx, const stp_gemm_args *a, const Epi &ep, hipStream_t s) {
  using GA = TileGeom<BM, A_KC>;
  using GB = TileGeom<BN, B_KC>;
  constexpr size_t smem = (size_t)2 * (GA::elems + GB::elems) * sizeof(bf16_t);
  static_assert(smem <= 160 * 1024, "LDS budget");
  auto kern = gemm_bf16_kernel<BM, BN, WAVES_M, WAVES_N, A_KC, B_KC, EPI>;
  static bool attr_set = false;   // the attribute is per function; setting it twice is harmless
  if (!attr_set) {
    STP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    attr_set = true;
  }
  int tiles_m = (a->M + BM - 1) / BM, tiles_n = (a->N + BN - 1) / BN;
  hipLaunchKernelGGL(kern, dim3(tiles_m * tiles_n), dim3(64 * WAVES_M * WAVES_N), smem, s, (const bf16_t *)a->A, a->lda, (const bf16_t *)a->B,
                     a->ldb, a->M, a->N, a->K, tiles_m, tiles_n, ep);
  STP_LAUNCH_CHECK(ctx);
  return STP_OK;
}

// Tile choice.  A launch runs in rounds of as many workgroups as the 256 CUs hold at once (one per CU; two
// for the 128 x 128 tile, whose LDS and registers allow it), so a shape that leaves the last round
// nearly empty with big tiles can finish sooner with smaller, less efficient ones.  The estimate is
//   sum over rounds of (K/32 x t_ktile x (0.65 + 0.35 x fill^1.5) + t_fixed)
// with t_ktile the measured time of a 32-deep part of the contraction of a resident workgroup on a full chip
// (microseconds, from 8192^3 runs per operand layout), fill the fraction of the round's slots in use
// (a partly filled chip leaves each workgroup more L2 and fabric bandwidth) and t_fixed the prologue +
// epilogue of a tile: 4 us for a 256 x 256 tile of bf16, 20 where it is added to an fp32 accumulator (512 KB per tile, all tiles of a
// round at once: 134 MB; half of a tile's time at 4096 tokens, which is why the smaller tiles, whose workgroups overlap, win there: [5120,
// 3456] 200 -> 176 us).  Over 33 shapes of 256 .. 6144 tokens in three layouts the tile it picks is the fastest or within 1 %
// of it (three launches of 8 us: within 7 %).
// The 192 x 256 tile exists for 6144-token activations: 32 tile rows x (N / 256) columns fill the 256 CUs in
// whole rounds where the 256 x 256 tile leaves a quarter to a half of them idle; alone on the GPU it is the
// fastest tile for seven of the layer's eight token-major shapes (3-12 %).  When other streams run beside
// the GEMM (the braided block) those idle CUs are not idle and a GEMM spread over all of them only takes longer
// per tile: with `shared_gpu` the choice is made differently (first lines of pick_tile).
struct TileChoice { int bm, bn; };
struct TileCfg { int bm, bn, per_cu; double t_ktile[4]; };   // t_ktile index: 2 * a_kc + b_kc; 0 = layout not built
static const TileCfg kTiles[5] = {{256, 256, 1, {0.779, 0.766, 0.782, 0.760}},
                                   {192, 256, 1, {0.0, 0.0, 0.584, 0.583}},
                                   {128, 256, 1, {0.445, 0.440, 0.430, 0.432}},
                                   {256, 128, 1, {0.460, 0.440, 0.432, 0.434}},
                                   {128, 128, 2, {0.244, 0.240, 0.235, 0.235}}};
inline long tile_count(const TileCfg &c, long M, long N) { return ((M + c.bm - 1) / c.bm) * ((N + c.bn - 1) / c.bn); }
// time of a launch of so many tiles that has the GPU to itself
inline double launch_us(const TileCfg &c, long tiles, long K, int layout, bool accum) {
  const double kt = (double)((K + 31) / 32);
  const long slots = 256L * c.per_cu;
  const long full = tiles / slots, rem = tiles % slots;
  const double tk = kt * c.t_ktile[layout], t_fixed = 1.0 + (accum ? 19.0 : 3.0) * (c.bm * c.bn / 65536.0);
  double t = (double)full * c.per_cu * (tk + t_fixed);
  if (rem) {
    // a partial round of the two-per-CU tile runs one workgroup per CU if it fits the 256 CUs
    const bool paired = c.per_cu == 2 && rem > 256;
    const double fill = paired ? rem / 512.0 : (rem < 256 ? rem / 256.0 : 1.0);
    const double alone = accum && c.per_cu == 2 && !paired ? 3.0 : 0.0;      // no second workgroup works behind this one's epilogue
    t += (paired ? 2.0 : 1.0) * (tk * (0.65 + 0.35 * fill * sqrt(fill)) + t_fixed + alone);
  }
  return t;
}
// pair: two products side by side (MM_PAIR).  Tiles other than 256 x 256 take 6 % longer than the estimate for one product says (fitted to
// the five tiles at 607 shapes of 136 .. 6144 tokens, hidden 520 .. 7168, f 520 .. 14336: the tile it picks is on average 0.4 % behind the
// fastest one; with 15 % on the 128-wide tiles, the figure of one shape, 0.8 %, [136, 2 x 14336] K = 5120 106 us instead of 83).
inline TileChoice pick_tile(long M, long N, long K, bool a_kc, bool b_kc, bool accum, bool shared_gpu, double *us = nullptr, bool pair = false) {
  if (shared_gpu) {
    // Beside other streams' kernels the rounds of the estimate below mean nothing (what a round leaves idle the
    // other streams use), and what counts is the work a tile costs the compute units: the biggest tile, which
    // moves the fewest operand bytes per flop, as long as the launch still has enough workgroups to make progress
    // on its share of the machine.  Measured on nine workloads against the estimate below without the 192-row
    // tile: never more than 0.3 % behind, 1.5 - 7 % ahead on the shapes of the larger models.  A measured
    // preference (stp_gemm_tile_hint) overrides it shape by shape.
    const int opts[4][2] = {{256, 256}, {128, 256}, {256, 128}, {128, 128}};
    for (auto &o : opts)
      if (((M + o[0] - 1) / o[0]) * ((N + o[1] - 1) / o[1]) >= 96) return TileChoice{o[0], o[1]};
    return TileChoice{128, 128};
  }
  TileChoice best{256, 256};
  double best_t = 1e30;
  for (const TileCfg &c : kTiles) {
    if (c.t_ktile[2 * a_kc + b_kc] == 0.0) continue;
    const double t = launch_us(c, tile_count(c, M, N), K, 2 * a_kc + b_kc, accum) * (pair && c.bm * c.bn < 256 * 256 ? 1.06 : 1.0);
    if (t < best_t) { best_t = t; best = TileChoice{c.bm, c.bn}; }
  }
  if (us) *us = best_t;
  return best;
}

// Outputs of at most 256 tiles of 64 x 64 (one per compute unit) go to the contraction-splitting kernel, measured against
// the best of the larger tiles (us): [1024, 1024] with K = 256 / 1024 / 3072 / 4096: 5.3 -> 4.3, 9.1 -> 6.6, 19.4 -> 13.2,
// 24.4 -> 16.3; [1136, 512] K = 2816: 17.8 -> 10.3; [384, 1032] K = 3008 (weight gradient): 22.4 -> 13.0; [128, 2128] K = 480:
// 6.9 -> 5.0.  With more tiles a compute unit works through two of them and nothing is gained ([1080, 1344] K = 1792: 13.2 with the
// best tile), and it costs more compute-unit time, which counts beside other streams; below K = 256 the extra reduction
// outweighs the shorter chain.
inline bool wavek_shape(long M, long N, long K) { return ((M + 63) / 64) * ((N + 63) / 64) <= 256 && K >= 256; }

template <bool A_KC, bool B_KC, int EPI, bool KTAIL>
int launch_dma_tile(stp_ctx *ctx, const stp_gemm_args *a, TileChoice c, const Epi &ep, hipStream_t s) {
  if constexpr (A_KC) {
    // 192 rows: 6144 tokens are 32 such tiles, and 32 x (N / 256) fills the 256 compute units in whole rounds
    if (c.bm == 192 && c.bn == 256) return launch_dma<192, 256, 2, 4, 3, 2, A_KC, B_KC, EPI, KTAIL>(ctx, a, ep, s);
  }
  if (c.bm == 256 && c.bn == 128) return launch_dma<256, 128, 2, 4, 3, 3, A_KC, B_KC, EPI, KTAIL>(ctx, a, ep, s);
  if (c.bm == 128 && c.bn == 256) return launch_dma<128, 256, 2, 4, 3, 3, A_KC, B_KC, EPI, KTAIL>(ctx, a, ep, s);
  if (c.bm == 128 && c.bn == 128) {
    // up to one workgroup per compute unit: all of the LDS for loads in flight (a ring of two leaves 42 instead of 29 us for
    // [6144, 512] K = 4096); with more, two workgroups share it (8192^3: 968 against 1143 us).  One or two K-tiles
    // need no more than the shorter rings, which are sooner filled (with copies of the last K-tile: [1024, 1024] K = 64 4.4 -> 4.0 us,
    // [1024, 4096] K = 96 6.1 -> 5.8)
    if (a->K > 128 && ((a->M + 127) / 128) * ((a->N + 127) / 128) <= 256) return launch_dma<128, 128, 2, 4, 4, 4, A_KC, B_KC, EPI, KTAIL>(ctx, a, ep, s);
    return launch_dma<128, 128, 2, 4, 3, 2, A_KC, B_KC, EPI, KTAIL>(ctx, a, ep, s);
  }
  return launch_dma<256, 256, 2, 4, 3, 2, A_KC, B_KC, EPI, KTAIL>(ctx, a, ep, s);
}

// the tile of a launch of N columns and contraction length K in all; a->M, a->N, a->K: the product a preference is given for
inline TileChoice tile_for(stp_ctx *ctx, const stp_gemm_args *a, bool a_kc, bool b_kc, bool accum, long N, long K, bool pair = false) {
  if (a->tile_m) return TileChoice{a->tile_m, a->tile_n};
  if (ctx && ctx->concurrent)       // a measured preference for this shape beside other streams' kernels
    for (int i = 0; i < ctx->n_tile_hints; i++) {
      const auto &hnt = ctx->tile_hint[i];
      if (hnt.M == a->M && hnt.N == a->N && hnt.K == a->K && hnt.layout == 2 * (int)a_kc + (int)b_kc) return TileChoice{hnt.tile_m, hnt.tile_n};
    }
  return pick_tile(a->M, N, K, a_kc, b_kc, accum, ctx && ctx->concurrent, nullptr, pair);
}
inline Epi make_epi(const stp_gemm_args *a) {
  Epi ep = {};
#ifdef STP_GEMM_TRACE
  ep.trace = getenv("STP_TRACE_PTR") ? (long long *)strtoull(getenv("STP_TRACE_PTR"), nullptr, 0) : nullptr;
#endif
  ep.C = a->C; ep.ldc = a->ldc; ep.c_f32_accum = a->c_f32_accum;
  ep.bias = (const bf16_t *)a->bias; ep.bias_scale = a->bias_scale;
  ep.resid = (const bf16_t *)a->resid; ep.ldr = a->ldr; ep.resid_scale = a->resid_scale;
  ep.mode = a->epilogue; ep.C2 = (bf16_t *)a->C2; ep.aux = (const bf16_t *)a->aux; ep.ld2 = a->ld2;
  return ep;
}

template <bool A_KC, bool B_KC, int EPI>
int launch_tile(stp_ctx *ctx, const stp_gemm_args *a, const Epi &ep, hipStream_t s) {
  const bool dma_ok = a->K > 0 && operand_bytes(A_KC, a->M, a->K, a->lda) > 0 && operand_bytes(B_KC, a->N, a->K, a->ldb) > 0;
  if (!dma_ok) return launch_cfg<128, 128, 2, 2, A_KC, B_KC, EPI>(ctx, a, ep, s);
  if (!a->tile_m && wavek_shape(a->M, a->N, a->K)) {
    constexpr int WK = A_KC || B_KC ? 64 : 32;
    return a->K % WK ? launch_wavek<WK, A_KC, B_KC, EPI, true>(ctx, a, ep, s) : launch_wavek<WK, A_KC, B_KC, EPI, false>(ctx, a, ep, s);
  }
  const TileChoice c = tile_for(ctx, a, A_KC, B_KC, EPI == EPI_F32_ACCUM, a->N, a->K);
  return a->K % DK ? launch_dma_tile<A_KC, B_KC, EPI, true>(ctx, a, c, ep, s) : launch_dma_tile<A_KC, B_KC, EPI, false>(ctx, a, c, ep, s);
}

template <bool A_KC, bool B_KC>
int launch_layout(stp_ctx *ctx, const stp_gemm_args *a, hipStream_t s) {
  const Epi ep = make_epi(a);
  if (a->c_f32_accum) return launch_tile<A_KC, B_KC, EPI_F32_ACCUM>(ctx, a, ep, s);
  if (a->epilogue == 1) return launch_tile<A_KC, B_KC, EPI_GELU_DUAL>(ctx, a, ep, s);
  if (a->epilogue == 2) return launch_tile<A_KC, B_KC, EPI_GELU_BWD>(ctx, a, ep, s);
  return launch_tile<A_KC, B_KC, EPI_STORE>(ctx, a, ep, s);
}

// the set's problems in tiles of bm x bn
inline ProblemSet make_set(const stp_gemm_args *a, int n, int bm, int bn) {
  ProblemSet set;
  set.n = n;
  set.tiles = 0;
  for (int i = 0; i < n; i++) {
    const int tm = (a[i].M + bm - 1) / bm, tn = (a[i].N + bn - 1) / bn;
    set.p[i] = {(const bf16_t *)a[i].A, (const bf16_t *)a[i].B, (float *)a[i].C, a[i].lda, (int)operand_bytes(false, a[i].M, a[i].K, a[i].lda), a[i].ldb,
                (int)operand_bytes(false, a[i].N, a[i].K, a[i].ldb), a[i].ldc, a[i].M, a[i].N, tm, tn, set.tiles};
    set.tiles += tm * tn;
  }
  return set;
}
// all of them small enough for the contraction-splitting kernel
inline bool wavek_set(const stp_gemm_args *a, int n) {
  for (int i = 0; i < n; i++)
    if (a[i].K <= 0 || !operand_bytes(false, a[i].M, a[i].K, a[i].lda) || !operand_bytes(false, a[i].N, a[i].K, a[i].ldb) ||
        !wavek_shape(a[i].M, a[i].N, a[i].K)) return false;
  return n > 1 && !stp_accumulators_overlap(a, n);
}
template <bool KTAIL>
int launch_wavek_set(stp_ctx *ctx, const stp_gemm_args *a, int n, hipStream_t s) {
  constexpr size_t smem = (size_t)4 * 128 * (64 + 64) * 2;
  auto kern = gemm_bf16_wavek_set_kernel<KTAIL>;
  static bool attr_set = false;
  if (!attr_set) {
    STP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    attr_set = true;
  }
  const ProblemSet set = make_set(a, n, 64, 64);
  hipLaunchKernelGGL(kern, dim3(set.tiles), dim3(256), smem, s, set, a[0].K);
  STP_LAUNCH_CHECK(ctx);
  return STP_OK;
}

template <int BM, int BN, int NSTA, int NSTB, bool KTAIL>
int launch_set(stp_ctx *ctx, const stp_gemm_args *a, int n, hipStream_t s) {
  constexpr size_t smem = (size_t)(NSTA * BM + NSTB * BN) * DK * 2;
  auto kern = gemm_bf16_set_kernel<BM, BN, 2, 4, NSTA, NSTB, false, false, KTAIL>;
  static bool attr_set = false;
  if (!attr_set) {
    STP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    attr_set = true;
  }
  const ProblemSet set = make_set(a, n, BM, BN);
  hipLaunchKernelGGL(kern, dim3(set.tiles), dim3(512), smem, s, set, a[0].K);
  STP_LAUNCH_CHECK(ctx);
  return STP_OK;
}

// A set takes one launch where the estimate of its time is below the sum of the estimates of its products.
inline bool set_tile(const stp_gemm_args *a, int n, TileChoice *choice) {
  double apart = 0.0, together = 1e30;
  if (stp_accumulators_overlap(a, n)) return false;
  for (int i = 0; i < n; i++) {
    if (a[i].K <= 0 || !operand_bytes(false, a[i].M, a[i].K, a[i].lda) || !operand_bytes(false, a[i].N, a[i].K, a[i].ldb) ||
        wavek_shape(a[i].M, a[i].N, a[i].K)) return false;
    double t;
    pick_tile(a[i].M, a[i].N, a[i].K, false, false, true, false, &t);
    apart += t;
  }
  for (const TileCfg &c : kTiles) {
    if (c.t_ktile[0] == 0.0) continue;
    long tiles = 0;
    for (int i = 0; i < n; i++) tiles += tile_count(c, a[i].M, a[i].N);
    const double t = launch_us(c, tiles, a[0].K, 0, true);
    if (t < together) { together = t; *choice = TileChoice{c.bm, c.bn}; }
  }
  return together < 0.98 * apart;
}

template <bool KTAIL>
int launch_set_tile(stp_ctx *ctx, const stp_gemm_args *a, int n, TileChoice c, hipStream_t s) {
  if (c.bm == 256 && c.bn == 128) return launch_set<256, 128, 3, 3, KTAIL>(ctx, a, n, s);
  if (c.bm == 128 && c.bn == 256) return launch_set<128, 256, 3, 3, KTAIL>(ctx, a, n, s);
  if (c.bm == 128 && c.bn == 128) return launch_set<128, 128, 3, 2, KTAIL>(ctx, a, n, s);
  return launch_set<256, 256, 3, 2, KTAIL>(ctx, a, n, s);
}

}  // namespace
