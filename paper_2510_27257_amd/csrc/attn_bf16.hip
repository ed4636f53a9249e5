// Tiled attention forward for bf16 on the CDNA4 matrix cores ("Attention(.)" of Eq. 1:
// the attention core of one TP rank, no communication).
//
// Work decomposition.  A workgroup owns 128 query rows of one (sequence, head) and ONE CHUNK of up
// to `chunk_steps` * 128 keys (chosen per launch); chunks of the same query block are merged afterwards by a small combine kernel
// (fixed order, deterministic).  Cutting the key range into chunks turns the causal triangle into
// pieces of similar size instead of workgroups whose length varies 1..seq/128.  The chunk length and the
// order in which the (block, chunk) pairs are dispatched - longest first, so that the short remainders fill
// the end of the launch - come from a host-side plan that simulates the dispatch over the 256 compute units.
// Inside a workgroup 8 waves run as 4 query sub-tiles (32 rows) x 2 key halves: per 128-key step
// waves 0-3 (group A) take keys 0..63 and waves 4-7 (group B) keys 64..127; a SIMD holds one wave of
// each group.  The two halves are merged through LDS at the end.  At head dimension 64 many short blocks go to workgroups of
// four waves (HALVES = 1), which take every key themselves, 64 a step, as group A does: see four_wave_us.
//
// Grouped-query attention: query head i reads key / value head i / (n / nk); only the tile addresses change.
//
// Per wave the kernel works on the TRANSPOSED score tile, S^T = K Q^T: with the 32x32x16 MFMA the
// accumulator of lane l then holds column q = l % 32, i.e. every softmax statistic (running max,
// running sum, rescale factor) is a per-lane scalar and a row reduction is an in-lane loop plus one
// cross-half shuffle.  The probabilities are already in the register layout the next MFMA wants for
// its B operand (O^T += V^T P^T), so P never touches LDS.  V^T fragments come from the V tile as it
// lies in memory ([kv][d]) through the transposing LDS read.
//
// Schedule (head dimension 64 with eight waves: see qk_pv_exps).  A step of a wave is a matrix phase M(k) = { S(k+1) = K(k+1) Q^T ; O += V(k)^T P(k) } and
// a vector phase V(k) = { P(k) = online softmax of S(k) }, of about equal length.  In iteration k group
// A runs M(k) then V(k+1) and group B V(k) then M(k), so on every SIMD one wave feeds the matrix pipe
// while the other does the exponentials; there is one s_barrier per iteration, none between the phases.
// K and V tiles (128 keys x D) go global -> LDS directly (buffer_load ... lds), K and V each in a ring
// of two tiles.  Tile K(k+2) replaces K(k) and V(k+1) replaces V(k-1); both are issued at the top of
// iteration k, when every wave is done with the tiles they overwrite, and waited for (vmcnt(0) + the
// barrier) at the top of iteration k+1, where they are first used.  A direct-to-LDS wave instruction fills
// 1 KB contiguously, so rows cannot be padded; bank conflicts are avoided by an XOR permutation of
// the 16-byte chunks of a row, applied on the global side and undone in the fragment addresses:
//   K tile [key][D]: chunk c of row r in slot c ^ ((r / RPB) & (CPR-1))        (16-byte fragment reads)
//   V tile [key][D]: chunk c of row r in slot c ^ (4 * ((r & 3) / RPB))        (ds_read_b64_tr_b16 reads)
// with CPR = D/8 chunks per row and RPB = 128/D rows per 256 bytes.  Fragment reads are inline assembly
// with explicit waits, software-pipelined one group of MFMAs ahead.
#include "common.h"
#include "lds_dma.h"
#include <type_traits>
#include <vector>
#include <algorithm>
#include <queue>
#include <functional>
#include <cstring>

namespace {

constexpr int QB = 128;    // query rows per workgroup
constexpr int KSTEP = 128; // keys per step of the plan
constexpr float LN2 = 0.69314718055994531f;

struct AttnCost { double fixed, step; };

template <int D, int HALVES = 2> struct AttnGeom {
  static constexpr int KS = 64 * HALVES;         // keys per tile: 64 per wave
  static constexpr int RB = D * 2;               // bytes per tile row
  static constexpr int CPR = D / 8;              // 16-byte chunks per row
  static constexpr int RPB = 256 / RB;           // rows per 256 bytes (one pass over the 64 banks)
  static constexpr int RPI = 64 / CPR;           // tile rows covered by one direct-to-LDS wave instruction
  static constexpr int NLD = KS / RPI / (4 * HALVES);    // such instructions per wave per tile
  static constexpr int TILE = KS * RB;        // bytes of a K or V tile
  static constexpr int piece_floats = QB * D + 2 * QB;   // partial O, then m, then l
};

// number of 128-key steps a query block needs
__host__ __device__ inline int attn_steps(int qb, int seq, int causal) {
  int kv_end = causal ? (seq < qb * QB + QB ? seq : qb * QB + QB) : seq;
  return (kv_end + KSTEP - 1) / KSTEP;
}

// ---- fragment reads (results valid after lds_wait + lds_tie) ----
// K fragments of sub-block JB (32 keys), d-steps 4*SG .. 4*SG+3: A operand, lane supplies key row lr, d = 16 s + 8 lg ..
template <int D, int JB, int SG>
__device__ __forceinline__ void read_k(u32x4_t (&buf)[4], const unsigned (&kaddr)[D / 16], unsigned tile) {
  constexpr int OFF = JB * 32 * AttnGeom<D>::RB;
  buf[0] = lds_read_b128<OFF>(kaddr[4 * SG + 0] + tile);
  buf[1] = lds_read_b128<OFF>(kaddr[4 * SG + 1] + tile);
  buf[2] = lds_read_b128<OFF>(kaddr[4 * SG + 2] + tile);
  buf[3] = lds_read_b128<OFF>(kaddr[4 * SG + 3] + tile);
}
// V^T fragments of keys 32 JB + 16 T .. +15 for the D/32 blocks of 32 output columns
template <int D, int JB, int T>
__device__ __forceinline__ void read_v(u32x4_t (&buf)[4], const unsigned (&vaddr)[D / 32], unsigned tile) {
  constexpr int RB = AttnGeom<D>::RB, OFF = (32 * JB + 16 * T) * RB;
  buf[0] = lds_read_tr16<OFF, 8 * RB>(vaddr[0] + tile);
  buf[1] = lds_read_tr16<OFF, 8 * RB>(vaddr[1] + tile);
  if constexpr (D == 128) {
    buf[2] = lds_read_tr16<OFF, 8 * RB>(vaddr[2] + tile);
    buf[3] = lds_read_tr16<OFF, 8 * RB>(vaddr[3] + tile);
  }
}
template <int D, int SG>
__device__ __forceinline__ void mfma_qk(f32x16_t &sc, const u32x4_t (&buf)[4], const bf16x8_t (&qf)[D / 16]) {
#pragma unroll
  for (int i = 0; i < 4; i++)
    sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, buf[i]), qf[4 * SG + i], sc, 0, 0, 0);
}
template <int D>
__device__ __forceinline__ void mfma_pv(f32x16_t (&o)[D / 32], const u32x4_t (&buf)[4], bf16x8_t pf) {
#pragma unroll
  for (int db = 0; db < D / 32; db++)
    o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, buf[db]), pf, o[db], 0, 0, 0);
}

template <int D, int HALVES, bool IN_PHASE>
__global__ __launch_bounds__(256 * HALVES, 2) void attn_fwd_bf16_kernel(const bf16_t *__restrict__ qkv, float *__restrict__ part,
                                                            bf16_t *__restrict__ out, float *__restrict__ lse_out, int seq,
                                                            int n, int nk, int causal, int max_chunks, int chunk_steps, float scale_log2,
                                                            int n_items, stp_attn_order ord
#ifdef STP_ATTN_TRACE
                                                            , long long *trace
#endif
                                                            ) {
  using G = AttnGeom<D, HALVES>;
  static_assert(D == 64 || D == 128, "head dimension");
  static_assert(!IN_PHASE || (D == 64 && HALVES == 2), "qk_pv_exps forms S of head dimension 64");
#ifdef STP_ATTN_TRACE
  const long long tr0 = wall_clock64();
#endif
  constexpr int RB = G::RB, CPR = G::CPR, RPB = G::RPB, RPI = G::RPI, NLD = G::NLD, TILE = G::TILE, KS = G::KS;
  constexpr int KREADS = 4, VREADS = 2 * (D / 32);   // LDS operations of one fragment group
  extern __shared__ __attribute__((aligned(1024))) char smem_raw[];   // K ring [2][TILE], V ring [2][TILE]

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int lr = lane & 31, lg = lane >> 5;
  const int qsub = wave & 3;
  int half = wave >> 2;
  // opaque to the compiler: folded away, it rotates the main loop and needs 70 more registers (at D = 128 it spills)
  if (HALVES == 1) { half = 0; asm volatile("" : "+s"(half)); }
  const int nqb = (seq + QB - 1) / QB;
  // the workgroup's (query block, chunk): from the launch's work order (grid = heads x items), or, without
  // one, from a grid of blocks x chunks x heads with the late query blocks, which own the most chunks, first
  const int item = n_items ? ord.item[blockIdx.y] : 0;
  const int qb = n_items ? (item & 0xfff) : nqb - 1 - (int)blockIdx.x;
  const int chunk = n_items ? (item >> 12) : (int)blockIdx.y;
  const int bz = n_items ? blockIdx.x : blockIdx.z;
  const int head = bz % n, b = bz / n;
  const int nsteps = attn_steps(qb, seq, causal);
  if (chunk * chunk_steps >= nsteps) return;
  // the chunk in tiles of KS keys
  constexpr int TPS = KSTEP / KS;
  const int s_begin = chunk * chunk_steps * TPS;
  const int s_end = min(((causal ? min(seq, qb * QB + QB) : seq) + KS - 1) / KS, s_begin + chunk_steps * TPS);
  const int ns = s_end - s_begin;

  const int a = n * D;
  const int ld = (n + 2 * nk) * D;              // a qkv row: n Q heads, nk K heads, nk V heads
  const int kcol = a + (head / (n / nk)) * D, vcol = kcol + nk * D;   // this head's key / value head
  const bf16_t *bbase = qkv + (size_t)b * seq * ld;           // this sequence's [seq][3a] block
  const int q_wave0 = qb * QB + qsub * 32;
  const int qg = q_wave0 + lr;                  // this lane's query row
  const int q_ld = min(qg, seq - 1);            // clamp so that tail lanes read valid memory

  // Q fragments: B operand, lane supplies row q, k = d index 16*s + 8*lg .. +7
  bf16x8_t qf[D / 16];
#pragma unroll
  for (int s = 0; s < D / 16; s++)
    qf[s] = *reinterpret_cast<const bf16x8_t *>(bbase + (size_t)q_ld * ld + head * D + 16 * s + 8 * lg);

  // ---- direct-to-LDS loads of this wave: instruction I = wave * NLD + j covers tile rows I*RPI .. +RPI-1
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(bbase), 0, (int)min((size_t)seq * ld * 2, (size_t)0x7fffffff), 0x00020000);
  // lane's byte offset = min(row offset, last row's) + column offset; the row offset is this lane's row within the
  // wave's first instruction (a register) plus a wave-uniform part (step, instruction), so a load costs three
  // vector instructions and no multiplication, and its LDS target is computed on the scalar unit
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);     // same value, known to be wave-uniform
  const unsigned row_bytes = (unsigned)ld * 2u, max_rowoff = (unsigned)(seq - 1) * row_bytes;
  const unsigned ld_rowoff0 = (unsigned)(wave * NLD * RPI + lane / CPR) * row_bytes;
  unsigned ld_kcol[NLD], ld_vcol[NLD];          // byte offset within a qkv row of the chunk this lane fetches
#pragma unroll
  for (int j = 0; j < NLD; j++) {
    const int row = (wave * NLD + j) * RPI + lane / CPR, slot = lane % CPR;
    ld_kcol[j] = (unsigned)(kcol + (slot ^ ((row / RPB) & (CPR - 1))) * 8) * 2u;
    ld_vcol[j] = (unsigned)(vcol + (slot ^ (4 * ((row & 3) / RPB))) * 8) * 2u;
  }
  // load j (0 .. NLD-1) of the K or V tile of local step k, into ring slot k & 1; rows past the end of the
  // sequence read its last row
  auto issue_one = [&](int k, bool is_v, int j) {
    char *dst = smem_raw + (is_v ? 2 * TILE : 0) + (k & 1) * TILE + (wave_s * NLD + j) * 1024;
    const unsigned uni = (unsigned)((s_begin + k) * KS + j * RPI) * row_bytes;
    const unsigned rowoff = min(ld_rowoff0 + uni, max_rowoff);
    dma_load16(rs, dst, rowoff + (is_v ? ld_vcol[j] : ld_kcol[j]), 0);
  };
  auto issue_tile = [&](int k, bool is_v) {
#pragma unroll
    for (int j = 0; j < NLD; j++) issue_one(k, is_v, j);
  };

  // ---- fragment addresses within a tile (this wave's 64-key half)
  const unsigned lds0 = (unsigned)(size_t)(const __attribute__((address_space(3))) char *)smem_raw;
  unsigned kaddr[D / 16], vaddr[D / 32];
  {
    const int row = half * 64 + lr;
#pragma unroll
    for (int s = 0; s < D / 16; s++) kaddr[s] = lds0 + row * RB + (((2 * s + lg) ^ ((row / RPB) & (CPR - 1))) * 16);
    // lane reads 4 consecutive d of key kbase + 4 lg + (lane&15)/4 (and of that key + 8): the k-slot order of P^T
    const int key = half * 64 + 4 * lg + ((lane & 15) >> 2);
#pragma unroll
    for (int db = 0; db < D / 32; db++) {
      const int col = 32 * db + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      vaddr[db] = lds0 + 2 * TILE + key * RB + (((col >> 3) ^ (4 * ((key & 3) / RPB))) * 16) + (col & 7) * 2;
    }
  }

  f32x16_t o[D / 32];
#pragma unroll
  for (int i = 0; i < D / 32; i++)
#pragma unroll
    for (int v = 0; v < 16; v++) o[i][v] = 0.f;
  float m = -INFINITY, l = 0.f;
  f32x16_t sc0, sc1;                 // S^T of the step in flight: keys 0..31 and 32..63 of this wave's half
  bf16x8_t pf00, pf01, pf10, pf11;   // P^T of the step whose PV is pending: [sub-block][16-key half]
#pragma unroll
  for (int i = 0; i < 8; i++) { pf00[i] = (bf16_t)0.f; pf01[i] = (bf16_t)0.f; pf10[i] = (bf16_t)0.f; pf11[i] = (bf16_t)0.f; }

  // wave-uniform: does local step k hold a key this wave's queries may attend to?
  auto active = [&](int k) {
    const int kv0 = (s_begin + k) * KS + half * 64;
    return kv0 < seq && (!causal || kv0 <= q_wave0 + 31);
  };

#define STP_SB() __builtin_amdgcn_sched_barrier(0)
  // S(kn) = K(kn) Q^T
  auto qk_only = [&](int kn) {
    const unsigned kt = (kn & 1) * TILE;
    u32x4_t fa[4], fb[4];
#pragma unroll
    for (int v = 0; v < 16; v++) { sc0[v] = 0.f; sc1[v] = 0.f; }
    read_k<D, 0, 0>(fa, kaddr, kt);
    if constexpr (D == 128) {
      read_k<D, 0, 1>(fb, kaddr, kt); lds_wait<KREADS>(); lds_tie(fa); mfma_qk<D, 0>(sc0, fa, qf); STP_SB();
      read_k<D, 1, 0>(fa, kaddr, kt); lds_wait<KREADS>(); lds_tie(fb); mfma_qk<D, 1>(sc0, fb, qf); STP_SB();
      read_k<D, 1, 1>(fb, kaddr, kt); lds_wait<KREADS>(); lds_tie(fa); mfma_qk<D, 0>(sc1, fa, qf); STP_SB();
      lds_wait<0>(); lds_tie(fb); mfma_qk<D, 1>(sc1, fb, qf); STP_SB();
    } else {
      read_k<D, 1, 0>(fb, kaddr, kt); lds_wait<KREADS>(); lds_tie(fa); mfma_qk<D, 0>(sc0, fa, qf); STP_SB();
      lds_wait<0>(); lds_tie(fb); mfma_qk<D, 0>(sc1, fb, qf); STP_SB();
    }
  };
  // O^T += V(k)^T P^T
  auto pv_only = [&](int k) {
    const unsigned vt = (k & 1) * TILE;
    u32x4_t fa[4], fb[4];
    read_v<D, 0, 0>(fa, vaddr, vt);
    read_v<D, 0, 1>(fb, vaddr, vt); lds_wait<VREADS>(); lds_tie(fa); mfma_pv<D>(o, fa, pf00); STP_SB();
    read_v<D, 1, 0>(fa, vaddr, vt); lds_wait<VREADS>(); lds_tie(fb); mfma_pv<D>(o, fb, pf01); STP_SB();
    read_v<D, 1, 1>(fb, vaddr, vt); lds_wait<VREADS>(); lds_tie(fa); mfma_pv<D>(o, fa, pf10); STP_SB();
    lds_wait<0>(); lds_tie(fb); mfma_pv<D>(o, fb, pf11); STP_SB();
  };
  // both, as one software pipeline (the common case).  With `defer` the wave's direct-to-LDS loads of this
  // iteration (K(k+2) if ld_k, V(k+1) if ld_v) are issued one at a time behind the MFMA groups, whose
  // execution covers the time the address unit holds the wave, instead of in a burst before them.
  auto qk_pv = [&](int kn, int k, bool ld_k, bool ld_v) {
    const unsigned kt = (kn & 1) * TILE, vt = (k & 1) * TILE;
    u32x4_t fa[4], fb[4];
#pragma unroll
    for (int v = 0; v < 16; v++) { sc0[v] = 0.f; sc1[v] = 0.f; }
    // the 2 * NLD loads are spread over the first 2 * NLD of the 8 (D = 128) or 6 (D = 64) groups
#define STP_LD(g)                                                        \
    do {                                                                 \
      if ((g) < NLD) { if (ld_k) issue_one(k + 2, false, (g)); }         \
      else if ((g) < 2 * NLD) { if (ld_v) issue_one(k + 1, true, (g) - NLD); } \
      STP_SB();                                                          \
    } while (0)
    read_k<D, 0, 0>(fa, kaddr, kt);
    if constexpr (D == 128) {
      read_k<D, 0, 1>(fb, kaddr, kt); lds_wait<KREADS>(); lds_tie(fa); mfma_qk<D, 0>(sc0, fa, qf); STP_SB(); STP_LD(0);
      read_k<D, 1, 0>(fa, kaddr, kt); lds_wait<KREADS>(); lds_tie(fb); mfma_qk<D, 1>(sc0, fb, qf); STP_SB(); STP_LD(1);
      read_k<D, 1, 1>(fb, kaddr, kt); lds_wait<KREADS>(); lds_tie(fa); mfma_qk<D, 0>(sc1, fa, qf); STP_SB(); STP_LD(2);
      read_v<D, 0, 0>(fa, vaddr, vt); lds_wait<VREADS>(); lds_tie(fb); mfma_qk<D, 1>(sc1, fb, qf); STP_SB(); STP_LD(3);
      read_v<D, 0, 1>(fb, vaddr, vt); lds_wait<VREADS>(); lds_tie(fa); mfma_pv<D>(o, fa, pf00); STP_SB(); STP_LD(4);
      read_v<D, 1, 0>(fa, vaddr, vt); lds_wait<VREADS>(); lds_tie(fb); mfma_pv<D>(o, fb, pf01); STP_SB(); STP_LD(5);
      read_v<D, 1, 1>(fb, vaddr, vt); lds_wait<VREADS>(); lds_tie(fa); mfma_pv<D>(o, fa, pf10); STP_SB(); STP_LD(6);
      lds_wait<0>(); lds_tie(fb); mfma_pv<D>(o, fb, pf11); STP_SB(); STP_LD(7);
    } else {
      read_k<D, 1, 0>(fb, kaddr, kt); lds_wait<KREADS>(); lds_tie(fa); mfma_qk<D, 0>(sc0, fa, qf); STP_SB(); STP_LD(0);
      read_v<D, 0, 0>(fa, vaddr, vt); lds_wait<VREADS>(); lds_tie(fb); mfma_qk<D, 0>(sc1, fb, qf); STP_SB(); STP_LD(1);
      read_v<D, 0, 1>(fb, vaddr, vt); lds_wait<VREADS>(); lds_tie(fa); mfma_pv<D>(o, fa, pf00); STP_SB(); STP_LD(2);
      read_v<D, 1, 0>(fa, vaddr, vt); lds_wait<VREADS>(); lds_tie(fb); mfma_pv<D>(o, fb, pf01); STP_SB(); STP_LD(3);
      read_v<D, 1, 1>(fb, vaddr, vt); lds_wait<VREADS>(); lds_tie(fa); mfma_pv<D>(o, fa, pf10); STP_SB();
      lds_wait<0>(); lds_tie(fb); mfma_pv<D>(o, fb, pf11); STP_SB();
    }
#undef STP_LD
  };

  // P(k) = online softmax of S(k) in the log2 domain; accumulator v of lane l is key
  // kv0 + 32*jb + 8*(v/4) + 4*(l/32) + v%4, query l%32.
  // Raw scores are kept; the 1/sqrt(d) log2(e) factor is folded into the exponent's FMA.
  // Only a step that touches the causal diagonal or the end of the sequence needs the mask.
  auto first_key = [&](int k) { return (s_begin + k) * KS + half * 64; };
  auto touches_edge = [&](int k) { return (causal && first_key(k) + 63 > q_wave0) || first_key(k) + 64 > seq; };
  auto mask = [&](int kv0, f32x16_t &sc, int jb) {
#pragma unroll
    for (int v = 0; v < 16; v++) {
      const int kv = kv0 + 32 * jb + 8 * (v >> 2) + 4 * lg + (v & 3);
      sc[v] = ((causal && kv > qg) || kv >= seq) ? -INFINITY : sc[v];
    }
  };
  auto largest = [&](const f32x16_t &sc, float mx) {
#pragma unroll
    for (int v = 0; v < 16; v++) mx = fmaxf(mx, sc[v]);
    return mx;
  };
  // the reference of step k, whose largest score (of this lane's keys) is mx
  auto reference = [&](int k, float mx) {
    mx = fmaxf(mx, other_half(mx)) * scale_log2;      // scale > 0: max and scaling commute
    // Lazy rescaling: the reference m only moves when the block maximum exceeds it by more than 2^8,
    // so exponentials stay below 256 (harmless in fp32 / bf16) and the O rescale is skipped on almost
    // every block.  Softmax is invariant to the reference as long as l, O and P use the same one.
    // Over the first 512 keys of a chunk the reference follows the maximum: a row's largest probability is then the
    // exact 1 and not a rounded bf16, which a chunk of many keys would otherwise have for its first block's only.  Relative
    // error of the output against 64 bits, 16 heads of 64, 1024 keys: two chunks 2.28e-3, one chunk 2.31e-3, with this
    // 2.24e-3; 4 heads of 128, 2048 tokens, causal 2.05e-3, with this 2.00e-3.  Following it all the way takes 2 - 8 % longer.
    // A query row that has seen no admissible key keeps m = -inf.
    return (mx > m + (k * KS < 512 ? 0.0f : 8.0f)) ? mx : m;
  };
  // l and O to the new reference
  auto rescale = [&](float m_new) {
    if (__builtin_amdgcn_ballot_w64(m_new != m) != 0) {
      const float corr = __builtin_amdgcn_exp2f(m - (m_new == -INFINITY ? 0.f : m_new));
      l *= corr;
#pragma unroll
      for (int i = 0; i < D / 32; i++)
#pragma unroll
        for (int v = 0; v < 16; v++) o[i][v] *= corr;
      m = m_new;
    }
  };
  // k-slot i of lane-half g in the PV step (jb, t) is key 32*jb + 16*t + 8*(i/4) + 4*g + i%4: elements 8*t .. +7 of sc0 / sc1 (jb) are
  // the fragment of (jb, t).  Elements v0 .. v0 + c - 1 of sc: exponentials in place / their sum / their fragment p
  auto exps = [&](f32x16_t &sc, int v0, int c, float neg_ref) {
#pragma unroll
    for (int v = v0; v < v0 + c; v++) sc[v] = __builtin_amdgcn_exp2f(fmaf(sc[v], scale_log2, neg_ref));
  };
  auto sums = [&](const f32x16_t &sc, int v0, int c, float &rs) {
#pragma unroll
    for (int v = v0; v < v0 + c; v++) rs += sc[v];
  };
  auto pack = [&](const f32x16_t &sc, int v0, int c, bf16x8_t &p) {
#pragma unroll
    for (int v = v0; v < v0 + c; v++) p[v & 7] = (bf16_t)sc[v];
  };
  // Written so, with the mask beside the search for the maximum, and not built from the pieces above, the kernels whose phases stay apart are compiled
  // as before the others had them; otherwise four waves a workgroup lose 2 - 4 % here and there (16 heads, 8 x 392 tokens, no mask 16.0 / 16.4 us).
  auto softmax_impl = [&](int k, auto masked) {
    constexpr bool MASK = decltype(masked)::value;
    if constexpr (MASK) mask(first_key(k), sc0, 0);
    float mx = largest(sc0, -INFINITY);
    if constexpr (MASK) mask(first_key(k), sc1, 1);
    rescale(reference(k, largest(sc1, mx)));
    const float neg_ref = m == -INFINITY ? 0.f : -m;
    float rs = 0.f;
    auto exp_pack = [&](const f32x16_t &sc, bf16x8_t &p0, bf16x8_t &p1) {
#pragma unroll
      for (int v = 0; v < 16; v++) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sc[v], scale_log2, neg_ref));
        rs += p;
        if (v < 8) p0[v] = (bf16_t)p; else p1[v - 8] = (bf16_t)p;
      }
    };
    exp_pack(sc0, pf00, pf01);
    exp_pack(sc1, pf10, pf11);
    l += rs + other_half(rs);
  };
  auto softmax = [&](int k) {
    if (touches_edge(k)) softmax_impl(k, std::true_type{});
    else softmax_impl(k, std::false_type{});
  };

  // Head dimension 64, eight waves: S(k+1), then O += V(k)^T P(k) with the exponentials of step k+1 between its MFMAs, which take the
  // probabilities of the step before; both groups at once, so that neither ends a phase after the other.  Alone a wave takes M, then V,
  // as a chain of latencies, and with 16 MFMAs a step instead of 32 the other wave's phase does not cover them.  Measured (us): 16 heads, 1024
  // tokens, no mask 16.4 -> 15.4; 8 heads, 4096 tokens, causal 39.9 -> 36.6, 8192 104 -> 97; 4 heads, 12288 124 -> 114; a wave's M | V apart stay where
  // they are the faster: at dimension 128 (16384 tokens 277 us, in phase 290 - 309; group B half an iteration behind, 303) and for four waves, three
  // workgroups to a compute unit (16384 tokens 328, in phase 347).  Loads one at a time between the MFMA groups: 0 - 2 % slower than behind the barrier.
  auto qk_pv_exps = [&](int k) {
    constexpr int C = 4;               // scores per MFMA of O: the 8 of a fragment over its two MFMAs
    const unsigned kt = ((k + 1) & 1) * TILE, vt = (k & 1) * TILE;
    u32x4_t fa[4], fb[4];
#pragma unroll
    for (int v = 0; v < 16; v++) { sc0[v] = 0.f; sc1[v] = 0.f; }
    float rs = 0.f;
    // behind each MFMA of fragment P: the exponentials of C elements from V0 of S, and PRE, what is left to do with those before
#define STP_PV(buf, P, S, V0, PRE)                                                                                                 \
    do {                                                                                                                           \
      _Pragma("unroll") for (int db = 0; db < 2; db++) {                                                                           \
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, buf[db]), P, o[db], 0, 0, 0);                 \
        STP_SB();                                                                                                                  \
        exps(S, V0 + db * C, C, neg_ref);                                                                                          \
        PRE;                                                                                                                       \
        STP_SB();                                                                                                                  \
      }                                                                                                                            \
    } while (0)
    read_k<D, 0, 0>(fa, kaddr, kt);
    read_k<D, 1, 0>(fb, kaddr, kt); lds_wait<KREADS>(); lds_tie(fa); mfma_qk<D, 0>(sc0, fa, qf); STP_SB();
    read_v<D, 0, 0>(fa, vaddr, vt); lds_wait<VREADS>(); lds_tie(fb); mfma_qk<D, 0>(sc1, fb, qf); STP_SB();
    if (touches_edge(k + 1)) { mask(first_key(k + 1), sc0, 0); mask(first_key(k + 1), sc1, 1); }
    const float m_new = reference(k + 1, largest(sc1, largest(sc0, -INFINITY))), neg_ref = m_new == -INFINITY ? 0.f : -m_new;
    STP_SB();
    read_v<D, 0, 1>(fb, vaddr, vt); lds_wait<VREADS>(); lds_tie(fa);
    STP_PV(fa, pf00, sc0, 0, if (db > 0) sums(sc0, (db - 1) * C, C, rs));
    read_v<D, 1, 0>(fa, vaddr, vt); lds_wait<VREADS>(); lds_tie(fb);
    STP_PV(fb, pf01, sc0, 8, sums(sc0, 8 + (db - 1) * C, C, rs); pack(sc0, db * C, C, pf00));
    read_v<D, 1, 1>(fb, vaddr, vt); lds_wait<VREADS>(); lds_tie(fa);
    STP_PV(fa, pf10, sc1, 0, if (db > 0) sums(sc1, (db - 1) * C, C, rs); else sums(sc0, 16 - C, C, rs); pack(sc0, 8 + db * C, C, pf01));
    lds_wait<0>(); lds_tie(fb);
    STP_PV(fb, pf11, sc1, 8, sums(sc1, 8 + (db - 1) * C, C, rs); pack(sc1, db * C, C, pf10));
    sums(sc1, 16 - C, C, rs);
    pack(sc1, 8, 8, pf11);
    rescale(m_new);
    l += rs + other_half(rs);
#undef STP_PV
  };

  // ---- main loop.  Iteration k uses tiles K(k+1) and V(k).  At its top every wave's loads have landed
  // (vmcnt(0) + barrier) and every wave is done with K(k) and V(k-1), whose slots take K(k+2) and V(k+1).
  // Group A runs M(k) then V(k+1), group B V(k) then M(k): the matrix work of one wave of a SIMD
  // coincides with the vector work of the other without a barrier in between.
  const bool last_active = active(ns - 1);      // only the last step of a chunk can be masked out for a wave
  auto vector_phase = [&](int k) {
    if (k >= 0 && k < ns && (k < ns - 1 || last_active)) softmax(k);
  };
  issue_tile(0, false);
  issue_tile(0, true);
  if (ns > 1) {
    issue_tile(1, false);
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * NLD) : "memory");
  } else {
    asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(NLD) : "memory");
  }
#ifdef STP_ATTN_TRACE
  const long long tr1 = wall_clock64();
#endif
  for (int k = -1; k < ns; k++) {
    const bool do_qk = k + 1 < ns && (k + 1 < ns - 1 || last_active), do_pv = k >= 0 && (k < ns - 1 || last_active);
    const bool ld_k = k >= 0 && k + 2 < ns, ld_v = k >= 0 && k + 1 < ns;
    // group A starts with the matrix phase: its loads ride behind the MFMA groups
    const bool defer = !IN_PHASE && half == 0 && do_qk && do_pv;
    if (k >= 0) {
      STP_SB();
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
      STP_SB();
      if (!defer) {
        if (ld_k) issue_tile(k + 2, false);
        if (ld_v) issue_tile(k + 1, true);
      }
    }
    if constexpr (IN_PHASE) {
      if (do_qk && do_pv) {
        qk_pv_exps(k);
      } else {
        if (do_pv) pv_only(k);
        if (do_qk) {
          qk_only(k + 1);
          if (touches_edge(k + 1)) { mask(first_key(k + 1), sc0, 0); mask(first_key(k + 1), sc1, 1); }
          softmax_impl(k + 1, std::false_type{});
        }
      }
    } else {
      if (half == 1) vector_phase(k);
      if (do_qk && do_pv) qk_pv(k + 1, k, defer && ld_k, defer && ld_v);
      else if (do_qk) qk_only(k + 1);
      else if (do_pv) pv_only(k);
      if (half == 0) vector_phase(k + 1);
    }
  }
#undef STP_SB
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
#ifdef STP_ATTN_TRACE
  const long long tr2 = wall_clock64();
#endif

  // ---- merge the two key halves (upper half -> LDS -> lower half), then write this chunk's partial:
  // O (un-normalised, relative to m), m (log2 domain), l.
  float *red = reinterpret_cast<float *>(smem_raw);            // [4][D/2][64] accumulators, then [4][2][32] m, l
  float *red_ml = red + 4 * (D / 2) * 64;
  if (HALVES == 2) {
    if (half == 1) {
#pragma unroll
      for (int i = 0; i < D / 32; i++)
#pragma unroll
        for (int v = 0; v < 16; v++) red[(qsub * (D / 2) + i * 16 + v) * 64 + lane] = o[i][v];
      if (lg == 0) { red_ml[(qsub * 2 + 0) * 32 + lr] = m; red_ml[(qsub * 2 + 1) * 32 + lr] = l; }
    }
    __syncthreads();
  }
  if (half == 0) {
    float M = m, ea = 1.f, eb = 0.f;
    if (HALVES == 2) {
      const float m_b = red_ml[(qsub * 2 + 0) * 32 + lr], l_b = red_ml[(qsub * 2 + 1) * 32 + lr];
      M = fmaxf(m, m_b);
      const float m_ref = M == -INFINITY ? 0.f : M;
      ea = __builtin_amdgcn_exp2f(m - m_ref);
      eb = __builtin_amdgcn_exp2f(m_b - m_ref);
      l = l * ea + l_b * eb;
    }
    // the merged accumulator, formed where it is stored, so that the reads from LDS overlap the stores (merging all of it first: 63.5
    // against 61.4 us for 32 x 21 heads of 128, 176 tokens, 13.2 against 12.9 for 8 heads, 352 tokens)
    auto merged = [&](int i, int v) { return HALVES == 2 ? o[i][v] * ea + red[(qsub * (D / 2) + i * 16 + v) * 64 + lane] * eb : o[i][v]; };
    if (qg < seq && nsteps <= chunk_steps) {
      // the query block has this one chunk: its rows are final, so they go to the output (and the log-sum-exp)
      // directly and the combine kernel leaves them alone
      const float inv = 1.0f / l;
      bf16_t *op = out + ((size_t)b * seq + qg) * a + head * D;
      typedef bf16_t bf16x4_t __attribute__((ext_vector_type(4)));
#pragma unroll
      for (int i = 0; i < D / 32; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
          bf16x4_t w;
#pragma unroll
          for (int r = 0; r < 4; r++) {
            const int v = 4 * j + r;
            w[r] = (bf16_t)(merged(i, v) * inv);
          }
          *reinterpret_cast<bf16x4_t *>(op + 32 * i + 8 * j + 4 * lg) = w;
        }
      if (lg == 0) lse_out[((size_t)b * n + head) * seq + qg] = (M + log2f(l)) * LN2;
    } else if (qg < seq) {
      const size_t piece = (((size_t)b * n + head) * nqb + qb) * max_chunks + chunk;
      float *po = part + piece * G::piece_floats;
      const int qloc = qsub * 32 + lr;
#pragma unroll
      for (int i = 0; i < D / 32; i++)
#pragma unroll
        for (int j = 0; j < 4; j++) {
          f32x4_t w;
#pragma unroll
          for (int r = 0; r < 4; r++) {
            const int v = 4 * j + r;
            w[r] = merged(i, v);
          }
          *reinterpret_cast<f32x4_t *>(po + (size_t)qloc * D + 32 * i + 8 * j + 4 * lg) = w;
        }
      if (lg == 0) { po[QB * D + qloc] = M; po[QB * D + QB + qloc] = l; }
    }
  }
#ifdef STP_ATTN_TRACE
  if (trace) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const long long tr3 = wall_clock64();
    if (tid == 0) {
      unsigned hw, xcc;
      asm volatile("s_getreg_b32 %0, hwreg(HW_REG_HW_ID)" : "=s"(hw));
      asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcc));
      long long *t = trace + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * 8;
      t[0] = tr0; t[1] = tr1; t[2] = tr2; t[3] = tr3; t[4] = hw; t[5] = xcc; t[6] = ns; t[7] = 1;
    }
  }
#endif
}

// out[q, :] = sum_c O_c e^{m_c - M} / sum_c l_c e^{m_c - M}; lse = (M + log2 L) ln 2.  One thread per 8 columns of a query
// row, the loads of all its chunks in flight together (a wave per row, which went through the chunks one after the other:
// 7.9 against 4.4 us for 16 heads x 1024 rows of 64 in two chunks).
template <int D>
__global__ __launch_bounds__(256) void attn_fwd_combine_kernel(const float *__restrict__ part, bf16_t *__restrict__ out,
                                                               float *__restrict__ lse, int seq, int n, int mbsz, int causal,
                                                               int max_chunks, int chunk_steps, int q_first) {
  using G = AttnGeom<D>;
  constexpr int CPR = D / 8;
  const size_t idx = blockIdx.x * (size_t)256 + threadIdx.x;
  const int rows = seq - q_first;             // rows below q_first belong to one-chunk blocks, which the main kernel finished
  if (idx >= (size_t)mbsz * n * rows * CPR) return;
  const int c8 = (idx % CPR) * 8;
  const size_t w = idx / CPR;
  const int q = q_first + w % rows, head = (w / rows) % n, b = w / ((size_t)rows * n);
  const int nqb = (seq + QB - 1) / QB, qb = q / QB, qloc = q % QB;
  const int nch = (attn_steps(qb, seq, causal) + chunk_steps - 1) / chunk_steps;
  if (nch <= 1) return;
  const float *p0 = part + ((((size_t)b * n + head) * nqb + qb) * max_chunks) * G::piece_floats;
  float m[8], l[8], v[8][8];
#pragma unroll
  for (int c = 0; c < 8; c++) {               // a block has at most 8 chunks
    m[c] = -INFINITY;
    l[c] = 0.f;
#pragma unroll
    for (int e = 0; e < 8; e++) v[c][e] = 0.f;
    if (c < nch) {
      const float *pc = p0 + (size_t)c * G::piece_floats;
      m[c] = pc[QB * D + qloc];
      l[c] = pc[QB * D + QB + qloc];
      Vec8<float>::load(pc + (size_t)qloc * D + c8, v[c]);
    }
  }
  float M = -INFINITY;
#pragma unroll
  for (int c = 0; c < 8; c++) M = fmaxf(M, m[c]);
  float L = 0.f, acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < 8; c++) {
    const float e = __builtin_amdgcn_exp2f(m[c] - M);
    L += l[c] * e;
#pragma unroll
    for (int i = 0; i < 8; i++) acc[i] += v[c][i] * e;
  }
  const float inv = 1.0f / L;
#pragma unroll
  for (int i = 0; i < 8; i++) acc[i] *= inv;
  Vec8<bf16_t>::store(out + ((size_t)b * seq + q) * (n * D) + head * D + c8, acc);
  if (c8 == 0) lse[((size_t)b * n + head) * seq + q] = (M + log2f(L)) * LN2;
}

// the plan of the forward kernel for this shape (block x = query block x)
const stp_attn_plan *fwd_plan(stp_ctx *ctx, const stp_layer_desc *d);

template <int D, int HALVES, bool IN_PHASE>
int launch_fwd(stp_ctx *ctx, const stp_layer_desc *d, const void *qkv, void *out, float *lse, float *ws, size_t ws_bytes,
               hipStream_t s) {
  using G = AttnGeom<D, HALVES>;
  constexpr size_t smem = (size_t)4 * G::TILE;   // K ring and V ring of two tiles each
  static_assert(HALVES == 1 || smem >= (size_t)(4 * (D / 2) * 64 + 4 * 2 * 32) * sizeof(float), "merge area fits");
  static_assert(smem <= 160 * 1024, "LDS budget");
  auto kern = attn_fwd_bf16_kernel<D, HALVES, IN_PHASE>;
  static bool attr_set = false;
  if (!attr_set) {
    STP_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
    attr_set = true;
  }
  if ((size_t)d->seq * stp_qkv_width(d) * sizeof(bf16_t) > (size_t)0x7fffffff)
    return stp_fail(ctx, STP_ESHAPE, "attention forward: one sequence of QKV must span less than 2 GiB%s");
  const int nqb = (d->seq + QB - 1) / QB;
  const stp_attn_plan *plan = fwd_plan(ctx, d);
  const int chunk_steps = plan->chunk_steps, max_chunks = plan->max_chunks;
  const size_t need = (size_t)d->mbsz * d->heads_local * nqb * max_chunks * G::piece_floats * sizeof(float);
  if (!ws || ws_bytes < need)
    return stp_fail(ctx, STP_ENOSPACE, "attention forward: workspace lane too small%s (need %ld bytes)", "", (long)need);
  const dim3 grid = plan->n_items ? dim3(d->heads_local * d->mbsz, plan->n_items) : dim3(nqb, max_chunks, d->heads_local * d->mbsz);
  const dim3 block(256 * HALVES);
  float scale_log2 = 1.4426950408889634f / sqrtf((float)D);
  hipLaunchKernelGGL(kern, grid, block, smem, s, (const bf16_t *)qkv, ws, (bf16_t *)out, lse, d->seq, d->heads_local, stp_kv_heads(d), d->causal, max_chunks, chunk_steps,
                     scale_log2, plan->n_items, plan->order
#ifdef STP_ATTN_TRACE
                     , getenv("STP_TRACE_PTR") ? (long long *)strtoull(getenv("STP_TRACE_PTR"), nullptr, 0) : (long long *)nullptr
#endif
                     );
  STP_LAUNCH_CHECK(ctx);
  // query blocks with a single chunk were finished by the main kernel; with the causal mask they are the first ones
  int qb_first = 0;
  while (qb_first < nqb && attn_steps(qb_first, d->seq, d->causal) <= chunk_steps) qb_first++;
  if (qb_first < nqb) {
    const int q_first = qb_first * QB;
    const size_t r8 = (size_t)d->mbsz * d->heads_local * (d->seq - q_first) * (D / 8);
    hipLaunchKernelGGL(attn_fwd_combine_kernel<D>, dim3((r8 + 255) / 256), dim3(256), 0, s, ws, (bf16_t *)out, lse, d->seq,
                       d->heads_local, d->mbsz, d->causal, max_chunks, chunk_steps, q_first);
    STP_LAUNCH_CHECK(ctx);
  }
  return STP_OK;
}

// Head dimension 64, eight waves: two or three steps without a mask, of whose last the first wave half sees a part and the second nothing, keep M and V
// apart.  There the second half is through a step earlier, and its vector work fits beside the first half's matrix work; in phase both wait for the
// other's.  Measured (us, apart / in phase): 4 heads, 144 tokens 7.44 / 7.59; 8 x 8 heads, 152 tokens 7.71 / 8.08; 4 heads, 264 tokens 9.12 / 9.29; 80 shapes 1.3 % in the
// mean; but 8 heads, 192 tokens, a whole half, 7.39 / 7.07; 200 tokens, shared by the halves, 8.2 / 7.8; 392 tokens equal; with the mask 136 tokens 8.0 / 7.1.
// The bits are the same.
bool fwd_phases_apart(const stp_layer_desc *d) {
  const int last = d->seq % KSTEP;
  return !d->causal && d->seq > KSTEP && d->seq < 3 * KSTEP && last > 0 && last < KSTEP / 2;
}

}  // namespace

extern "C" int stp_attn_fwd_route(const stp_layer_desc *d) {
  return d->head_dim == 64 && fwd_plan(nullptr, d)->halves == 1 ? 0 : d->head_dim == 64 && !fwd_phases_apart(d) ? 2 : 1;
}

const stp_attn_plan *stp_attn_plan_for(stp_ctx *ctx, const stp_layer_desc *d, int kind) {
  return kind == 0 ? fwd_plan(ctx, d) : stp_attn_bwd_plan_for(ctx, d, kind);
}

size_t stp_attn_fwd_ws_bytes(const stp_layer_desc *d) {
  const int nqb = (d->seq + QB - 1) / QB;
  const int max_chunks = fwd_plan(nullptr, d)->max_chunks;
  return (size_t)d->mbsz * d->heads_local * nqb * max_chunks * (QB * d->head_dim + 2 * QB) * sizeof(float);
}

int stp_launch_attn_fwd_bf16(stp_ctx *ctx, const stp_layer_desc *d, const void *qkv, void *out, float *lse, float *ws,
                             size_t ws_bytes, hipStream_t s) {
  if (d->head_dim == 128) return launch_fwd<128, 2, false>(ctx, d, qkv, out, lse, ws, ws_bytes, s);
  if (d->head_dim == 64 && fwd_plan(ctx, d)->halves == 1) return launch_fwd<64, 1, false>(ctx, d, qkv, out, lse, ws, ws_bytes, s);
  if (d->head_dim == 64 && fwd_phases_apart(d)) return launch_fwd<64, 2, false>(ctx, d, qkv, out, lse, ws, ws_bytes, s);
  if (d->head_dim == 64) return launch_fwd<64, 2, true>(ctx, d, qkv, out, lse, ws, ws_bytes, s);
  return stp_fail(ctx, STP_ESHAPE, "bf16 attention needs head_dim 64 or 128%s");
}

// Cost of a workgroup of the chunked kernels in microseconds (0 forward, 1 dkv, 2 dq): start and end of a workgroup
// (first tiles, the merge of the wave halves, the partial result) and one step of its main loop, fitted to measured
// kernel times.  Head dimension 128: chunk lengths 8 .. 32 (16 .. 64 for dkv) at 4 and 10 heads, seq 4096 and 6144, causal,
// within 6 - 8 % (rms).  Head dimension 64: 256 .. 4096 tokens, 2 .. 32 heads, within 10 % (forward: with the exponentials among the MFMAs).
static AttnCost attn_cost(int kind, int head_dim) {
  static const AttnCost c128[3] = {{11.5, 1.75}, {12.0, 1.90}, {12.0, 2.65}}, c64[3] = {{5.0, 1.22}, {4.5, 1.20}, {4.5, 1.70}};
  return head_dim == 128 ? c128[kind] : c64[kind];
}
// The plan is made for the whole chip, also where other streams' kernels take a part of it: chunk lengths and the four-wave rule
// below decide in which order a row's keys are added up, and a layer's bits may not depend on what runs beside it.  A plan for 96
// compute units inside a braided block is 0 - 1 % faster there for the larger layers, 0.8 - 1.5 % slower for ViT layers.
constexpr int PLAN_CUS = STP_CUS;

namespace {

// One kind of work item of a launch: the steps of its blocks, each repeated for z (head, sequence) pairs, cut into chunks of c
// steps; partial: bytes of a chunk's partial result.
struct PlanPart {
  AttnCost cost;
  int nblocks, z, max_steps, c;
  const int *steps;
  size_t partial;
};

template <typename F>
void for_chunks(const PlanPart &p, F f) {
  for (int x = 0; x < p.nblocks; x++)
    for (int k = 0; k < p.steps[x]; k += p.c) f(p.cost.fixed + p.cost.step * std::min(p.c, p.steps[x] - k));
}

// The combine kernel of a launch with blocks of several chunks: a launch of its own (about 4 us) that reads the partials at
// about 3 TB/s.
double combine_us(const PlanPart &p) {
  if (p.max_steps <= p.c) return 0.0;
  size_t pieces = 0;
  for (int x = 0; x < p.nblocks; x++)
    if (p.steps[x] > p.c) pieces += (p.steps[x] + p.c - 1) / p.c;
  return 4.0 + (double)pieces * p.z * p.partial / 3e6;
}

// no schedule of these chunks over the chip is shorter
double plan_bound(const PlanPart *part, int n) {
  double sum = 0.0, longest = 0.0, combine = 0.0;
  for (int i = 0; i < n; i++) {
    double s = 0.0;
    for_chunks(part[i], [&](double t) { s += t; longest = std::max(longest, t); });
    sum += s * part[i].z;
    combine += combine_us(part[i]);
  }
  return std::max(longest, sum / PLAN_CUS) + combine;
}

// Time of a launch whose workgroups, longest first, each go to the compute unit that is free first (one workgroup each).
double plan_makespan(const PlanPart *part, int n) {
  // many (head, sequence) pairs: a smaller machine with proportionally fewer of them gives the same picture and keeps the
  // planning time bounded
  int zmin = part[0].z, zmax = part[0].z;
  for (int i = 1; i < n; i++) { zmin = std::min(zmin, part[i].z); zmax = std::max(zmax, part[i].z); }
  const int keep = std::max(1, std::min(zmin, 16 * zmin / zmax));       // of the zmin pairs of the part with the fewest
  const int cus = std::max(1, PLAN_CUS * keep / zmin);
  std::vector<std::pair<double, int>> items;
  double combine = 0.0;
  for (int i = 0; i < n; i++) {
    const int z = std::max(1, (int)((long)part[i].z * keep / zmin));
    for_chunks(part[i], [&](double t) { items.push_back({t, z}); });
    combine += combine_us(part[i]);
  }
  std::sort(items.begin(), items.end(), [](const std::pair<double, int> &u, const std::pair<double, int> &v) { return u.first > v.first; });
  std::priority_queue<double, std::vector<double>, std::greater<double>> cu;
  for (int i = 0; i < cus; i++) cu.push(0.0);
  double end = 0.0;
  for (auto &it : items)
    for (int z = 0; z < it.second; z++) {
      const double t = cu.top() + it.first;
      cu.pop();
      cu.push(t);
      end = std::max(end, t);
    }
  return end + combine;
}

// Chunk lengths (part[i].c) with the shortest simulated launch; returns its time.  Two kinds of item share a launch in the
// backward pass: the second's chunk is as long as the first's in time (or whole blocks).
// A block is never cut into more than 8 pieces (bounds the workspace and fits the table's 3 chunk bits).
double plan_chunks(PlanPart *part, int n) {
  auto least = [&](int i) { return std::max((part[i].max_steps + 7) / 8, std::min(part[i].max_steps, 4)); };
  struct Cand { double bound; int c[2]; };
  std::vector<Cand> cand;
  auto add = [&](int c0, int c1) {
    part[0].c = c0;
    if (n > 1) part[1].c = c1;
    cand.push_back({plan_bound(part, n), {c0, c1}});
  };
  const int lo = least(0), hi = std::max(lo, part[0].max_steps), stride = std::max(1, (hi - lo) / 40);
  auto first = [&](int c) {
    if (n == 1) { add(c, 0); return; }
    const double t = part[0].cost.fixed + part[0].cost.step * c;
    const int lo1 = least(1), hi1 = std::max(lo1, part[1].max_steps);
    const int c1 = std::max(lo1, std::min(hi1, (int)((t - part[1].cost.fixed) / part[1].cost.step)));
    add(c, c1);
    const int even = std::max(lo1, (part[1].max_steps + (part[1].max_steps + c1 - 1) / c1 - 1) / ((part[1].max_steps + c1 - 1) / c1));
    if (even != c1) add(c, even);
    if (hi1 != c1) add(c, hi1);
  };
  for (int c = lo; c < hi; c += stride) first(c);
  for (int j = 1; j <= 8; j++)                                       // equal pieces of the longest block
    if ((part[0].max_steps + j - 1) / j >= lo) first((part[0].max_steps + j - 1) / j);
  if (cand.empty()) first(hi);
  // the most promising first; the rest is simulated only while its bound leaves room for a gain of half a percent
  std::stable_sort(cand.begin(), cand.end(), [](const Cand &u, const Cand &v) { return u.bound < v.bound; });
  double best = 1e30;
  int bc[2] = {hi, n > 1 ? part[1].max_steps : 0}, tries = 0;
  for (auto &k : cand) {
    if (k.bound >= best * 0.995 || tries >= 24) break;
    part[0].c = k.c[0];
    if (n > 1) part[1].c = k.c[1];
    const double t = plan_makespan(part, n);
    tries++;
    if (t < best * 0.995) { best = t; bc[0] = k.c[0]; bc[1] = k.c[1]; }
  }
  part[0].c = bc[0];
  if (n > 1) part[1].c = bc[1];
  return best;
}

// the (block, chunk) pairs of a part, longest first; equal lengths keep the later blocks first
void plan_fill(const PlanPart &p, stp_attn_plan *plan) {
  plan->halves = 2;
  plan->between = 0;
  plan->chunk_steps = p.c;
  plan->max_chunks = (p.max_steps + p.c - 1) / p.c;
  struct Item { int len, block, chunk; };
  std::vector<Item> items;
  for (int x = p.nblocks - 1; x >= 0; x--)
    for (int k = 0; k * p.c < p.steps[x]; k++) items.push_back({std::min(p.c, p.steps[x] - k * p.c), x, k});
  std::stable_sort(items.begin(), items.end(), [](const Item &u, const Item &v) { return u.len > v.len; });
  plan->n_items = 0;
  if (items.size() <= STP_ATTN_ORDER_CAP && p.nblocks <= 4096 && plan->max_chunks <= 8) {
    plan->n_items = (int)items.size();
    for (size_t i = 0; i < items.size(); i++) plan->order.item[i] = (uint16_t)(items[i].block | (items[i].chunk << 12));
  }
}

// Head dimension 64, forward: four waves a workgroup, which take all the keys of a step in turn instead of sharing them with
// four others, have no halves to merge and sit three to a compute unit.  A workgroup with a compute unit of its own is slower
// that way (1.8 us a step), three together are faster (1.2 us a step of one of them): one chunk per block, and the longest
// block, the sum of all or what shares a compute unit bounds the launch.  Measured (us, eight waves / four): 2 x 16 heads, 4096 tokens 104 / 92;
// 14 heads on 2, 8 x 912 tokens, no mask 58 / 47; 8 heads, 16384 tokens 360 / 326; but 8 x 8 heads, 520 tokens 13.9 / 14.4; 8 heads, 5120 tokens, no
// mask 87 / 101; 6 heads on 3, 13568 tokens 198 / 223.  At head dimension 128 (two workgroups a compute unit) it is the slower one wherever there
// is work for the whole chip (281 / 308 at 16384 tokens).
double four_wave_us(const PlanPart &p, int seq) {
  double sum = 0.0;
  std::vector<double> len(p.steps, p.steps + p.nblocks);
  // their tiles are of 64 keys, half a step: 16 heads, 4 x 784 .. 824 tokens, causal 18.4 us, 888 20.4 (eight waves 19.0 and 19.1)
  if (seq % KSTEP && seq % KSTEP <= 64)
    for (int x = 0; x < p.nblocks; x++)
      if (p.steps[x] == (seq + KSTEP - 1) / KSTEP) len[x] -= 0.5;
  std::sort(len.begin(), len.end(), std::greater<double>());
  for (double x : len) sum += 2.0 + 1.2 * x;
  double t = std::max(6.0 + 1.8 * len[0], sum * p.z / PLAN_CUS);
  // longest first, a workgroup to the emptiest compute unit: the 257th is the second on one, the 513th the third, the 769th waits
  const double step[3] = {2.45, 3.25, 4.85};
  for (int r = 0; r < 3; r++) {
    const long x = (long)PLAN_CUS * (r + 1) / p.z;      // the block that it belongs to
    if (x < p.nblocks) t = std::max(t, 6.0 + step[r] * len[x]);
  }
  return t;
}

int max_of(const int *v, int n) { return *std::max_element(v, v + n); }

}  // namespace

double stp_attn_item_cost(int kind, int head_dim, int len) {
  const AttnCost c = attn_cost(kind, head_dim);
  return c.fixed + c.step * len;
}

stp_attn_plan *stp_attn_plan_slot(stp_ctx *ctx, const int key[8], bool *hit) {
  static thread_local stp_attn_plan scratch_of_kind[4];
  stp_attn_plan *p = &scratch_of_kind[(key[0] - 1) & 3];
  *hit = false;
  if (ctx) {
    for (int i = 0; i < ctx->attn_plan_n; i++)
      if (memcmp(ctx->attn_plan[i].key, key, 8 * sizeof(int)) == 0) { *hit = true; return &ctx->attn_plan[i]; }
    if (ctx->attn_plan_n < STP_ATTN_PLAN_CACHE) p = &ctx->attn_plan[ctx->attn_plan_n++];
    else { p = &ctx->attn_plan[ctx->attn_plan_next]; ctx->attn_plan_next = (ctx->attn_plan_next + 1) % STP_ATTN_PLAN_CACHE; }
  } else if (memcmp(p->key, key, 8 * sizeof(int)) == 0) {
    *hit = true;
    return p;
  }
  memcpy(p->key, key, 8 * sizeof(int));
  return p;
}

// The same for the backward kernels, two workgroups of four waves to a compute unit.  Alone on one a workgroup takes 5 + 2.0 (dq: 2.8) us a
// step, beside another 3 + 1.3 (1.85) of the unit's time: less than eight waves where blocks are short and many, since one workgroup's first
// tiles and results overlap the other's steps; long blocks gain nothing, and few of them leave waves idle.  Measured (us, row dot
// included, eight waves / four): 8 x 8 heads, 520 tokens, causal 32.3 / 28.9; 8 x 16 heads, 256 tokens 20.2 / 17.3; 16 x 16 heads, 512 tokens, no
// mask 114 / 95; 2 x 16 heads, 4096 tokens 290 / 290; 16 heads, 1024 tokens, no mask 27 / 36; 4 heads, 512 tokens 16.4 / 21.1.
struct FourWaveBwd { double longest, all; };      // the longest workgroup alone on its compute unit; all of them, shared out evenly
static FourWaveBwd four_wave_bwd_us(const PlanPart *p) {
  const double fixed = 3.0, step[2] = {1.3, 1.85}, fixed1 = 5.0, step1[2] = {2.0, 2.8};
  double sum = 0.0, longest = 0.0;
  for (int i = 0; i < 2; i++) {
    for (int x = 0; x < p[i].nblocks; x++) sum += p[i].z * (fixed + step[i] * p[i].steps[x]);
    longest = std::max(longest, fixed1 + step1[i] * p[i].max_steps);
  }
  return {longest, sum / PLAN_CUS};
}

// That bound is blind to a last round of few workgroups: of 691 shapes it would give to four waves (128 .. 8192 tokens, 2 .. 32 heads) they were slower
// than eight at 51, by up to 18 %, equal long blocks above all (6 heads, 6144 tokens, no mask 250 / 296; 10 heads, 4096 tokens 180 / 202; 6 x 8 heads on 4, 1024
// tokens 60 / 69).  So the launch is simulated too: longest first, each workgroup to the compute unit that has room first, two of a unit sharing
// its time.  With costs fitted for this choice none is more than 1.7 % slower, 567 stay, and on average they are where the bound alone had them.
static double four_wave_bwd_end(const PlanPart *p) {
  const double fixed = 2.2, step[2] = {1.15, 2.0}, fixed1 = 4.8, step1[2] = {1.5, 2.45};
  double sum = 0.0, longest = 0.0;
  for (int i = 0; i < 2; i++) {
    for (int x = 0; x < p[i].nblocks; x++) sum += p[i].z * (fixed + step[i] * p[i].steps[x]);
    longest = std::max(longest, fixed + step[i] * p[i].max_steps);
  }
  if (sum / PLAN_CUS > 16.0 * longest) return sum / PLAN_CUS;      // the last round is a small part of the whole (and this bounds the planning time)
  struct Work { double paired, alone; int count; };
  std::vector<Work> items;
  const int share = (p[0].z | p[1].z | PLAN_CUS) & -(p[0].z | p[1].z | PLAN_CUS);      // equal parts of the chip that get equal shares of each kind: one is simulated
  const int cus = PLAN_CUS / share;
  for (int i = 0; i < 2; i++)
    for (int x = 0; x < p[i].nblocks; x++) items.push_back({fixed + step[i] * p[i].steps[x], fixed1 + step1[i] * p[i].steps[x], p[i].z / share});
  std::sort(items.begin(), items.end(), [](const Work &u, const Work &v) { return u.paired > v.paired; });
  // two workgroups of a unit share its time, one alone goes at its own rate
  struct Unit { Work w[2]; double left[2], at; int n; };
  std::vector<Unit> cu(cus, Unit{{}, {}, 0.0, 0});
  size_t next = 0;
  auto start = [&](Unit &u) {
    u.w[u.n] = items[next];
    u.left[u.n++] = 1.0;
    if (--items[next].count == 0) next++;
  };
  for (int r = 0; r < 2; r++)
    for (Unit &u : cu)
      if (next < items.size()) start(u);
  auto rate = [](const Unit &u, int k) { return u.n == 1 ? 1.0 / u.w[k].alone : 0.5 / u.w[k].paired; };
  std::priority_queue<std::pair<double, int>, std::vector<std::pair<double, int>>, std::greater<std::pair<double, int>>> events;
  auto schedule = [&](int c) {
    const Unit &u = cu[c];
    if (!u.n) return;
    double first = u.left[0] / rate(u, 0);
    if (u.n == 2) first = std::min(first, u.left[1] / rate(u, 1));
    events.push({u.at + first, c});
  };
  for (int c = 0; c < cus; c++) schedule(c);
  double end = 0.0;
  while (!events.empty()) {
    const int c = events.top().second;
    end = events.top().first;
    events.pop();
    Unit &u = cu[c];
    const double dt = end - u.at, r[2] = {rate(u, 0), u.n == 2 ? rate(u, 1) : 0.0};
    u.at = end;
    int kept = 0;
    for (int k = 0; k < u.n; k++) {
      const double left = u.left[k] - dt * r[k];
      if (left > 1e-9) { u.w[kept] = u.w[k]; u.left[kept++] = left; }
    }
    u.n = kept;
    while (u.n < 2 && next < items.size()) start(u);
    schedule(c);
  }
  return end;
}

int stp_attn_bwd_chunks(const stp_layer_desc *d, int nkv, const int *steps_kv, int nq, const int *steps_q, int chunk[2], int *between) {
  const int nk = stp_kv_heads(d), D = d->head_dim;
  PlanPart part[2] = {{attn_cost(1, D), nkv, nk * d->mbsz, max_of(steps_kv, nkv), 0, steps_kv, (size_t)2 * 128 * D * sizeof(float)},
                      {attn_cost(2, D), nq, d->heads_local * d->mbsz, max_of(steps_q, nq), 0, steps_q, (size_t)128 * D * sizeof(float)}};
  const double t = plan_chunks(part, 2);
  const bool fits = nkv + d->heads_local / nk * nq <= STP_ATTN_ORDER_CAP;        // one launch for both kinds
  const FourWaveBwd us = four_wave_bwd_us(part);
  const bool four = D == 64 && fits && std::max(us.longest, us.all) < 0.97 * t && four_wave_bwd_end(part) < 1.01 * t;
  // dK / dV with the exponentials among the MFMAs (head dimension 64): always with eight waves.  With four, a compute unit's next workgroup comes when one
  // of dQ is through, and beside a denser one of dK / dV that is later (us, apart / among): 8 x 8 heads, 520 tokens, no mask 39.1 / 41.9; 12 heads, 4 x 1000 tokens, causal
  // 40.5 / 42.0.  So only where all are on the chip at once, two to a compute unit (90 drawn shapes: 3.6 % in the mean, none slower; but the causal ones that fill it
  // to the last place, 16 heads, 8 x 256 tokens 16.9 / 17.3, stay apart), or where the longest workgroup bounds the launch and not their sum (110 drawn shapes: 2 - 7 %;
  // 8 x 8 heads, 520 tokens, causal 26.5 / 25.4; 24 heads on 8, 10 x 168 tokens 25.3 / 24.6).  Among the rest 0.93 - 1.10x, 0.5 % in the mean.  The bits are the same.
  const long groups = (long)nkv * part[0].z + (long)nq * part[1].z;
  const bool one_round = groups < 2 * PLAN_CUS + (d->causal ? 0 : 1), by_longest = groups > 2 * PLAN_CUS && us.longest > 1.015 * us.all;
  *between = D == 64 && (!four || one_round || by_longest);
  chunk[0] = four ? part[0].max_steps : part[0].c;
  chunk[1] = four ? part[1].max_steps : part[1].c;
  return four ? 1 : 2;
}

void stp_attn_plan_fill(stp_attn_plan *plan, int chunk, int nblocks, const int *steps) {
  plan_fill(PlanPart{AttnCost{}, nblocks, 1, max_of(steps, nblocks), chunk, steps, 0}, plan);
}

namespace {

const stp_attn_plan *fwd_plan(stp_ctx *ctx, const stp_layer_desc *d) {
  const int nqb = (d->seq + QB - 1) / QB;
  const int key[8] = {1, d->seq, d->causal, d->heads_local, stp_kv_heads(d), d->mbsz, d->head_dim, nqb};
  bool hit;
  stp_attn_plan *plan = stp_attn_plan_slot(ctx, key, &hit);
  if (hit) return plan;
  std::vector<int> steps(nqb);
  for (int x = 0; x < nqb; x++) steps[x] = attn_steps(x, d->seq, d->causal);
  PlanPart part = {attn_cost(0, d->head_dim), nqb, d->heads_local * d->mbsz, max_of(steps.data(), nqb), 0, steps.data(),
                   (size_t)(QB * d->head_dim + 2 * QB) * sizeof(float)};
  const double t = plan_chunks(&part, 1);
  // Where equal long blocks are cut into several pieces the simulation is up to 12 % low (3 heads, 2 x 8856 tokens 195 us, four waves 173; 5 heads, 15160 tokens
  // 425 / 401; 7 heads on one, 7632 tokens 162 / 150): there eight waves have to be expected shorter by 3 % (with 4.6 % 5 heads on one, 2 x 3376 tokens 64 / 69).
  const double margin = !d->causal && part.c < part.max_steps ? 1.03 : 1.0;
  const bool four = d->head_dim == 64 && four_wave_us(part, d->seq) < margin * t;
  if (four) part.c = part.max_steps;
  plan_fill(part, plan);
  if (four) plan->halves = 1;
  return plan;
}

}  // namespace
