// Packed variable-length attention backward for gfx950 (bf16 MFMA, fp32 accumulate).
//
// Runs of clips of at most 256 tokens: one kernel (attn_bwd_fused_kernel, further down), one workgroup per
// (clip, head), but for small runs (bwd_one_pass).  Otherwise two passes, dQ and dK/dV, without atomics
// (device-wide fp32 atomics are executed at the memory side on this chip and were measured to bound the
// fused variant of long clips), so every output is written once and the result is bitwise reproducible;
// they run one after the other or, up to 1,024 rows, from one grid (bwd_order).  Both need
//   Delta[h,i] = sum_d dO[i,h,d] O[i,h,d],  lse2 = lse * log2(e), and two sentinel statistics (+inf, 0) for rows
//   past a clip's end, which the dQ pass forms itself where it runs first, else bwd_prepare before both.
//   bwd_dkdv    : one workgroup owns kBC key/value rows of one (clip, head); its four
//                 wavefronts own 32 of those rows each and keep their K and V rows, and
//                 their dK^T / dV^T accumulators, in registers.  The workgroup walks the
//                 clip's query rows in tiles of kBQ, staged (Q, dO, lse, Delta) through
//                 LDS, and per tile computes
//                     S  = Q K^T,  dP = dO V^T            (A = Q/dO rows, B = K/V registers)
//                     P  = exp(scale*S - lse),  dS = P o (dP - Delta)
//                     dV^T += dO^T P,  dK^T += Q^T dS     (A = transposing LDS reads, B = P/dS registers)
//   bwd_dq      : one workgroup owns a query tile (like the forward kernel) and streams
//                 the clip's K/V tiles through LDS:
//                     S^T = K Q^T,  dP^T = V dO^T          (A = K/V rows, B = Q/dO registers)
//                     dS^T = P^T o (dP^T - Delta)          (lse, Delta are per-lane scalars)
//                     dQ^T += K^T dS^T                     (A = transposing reads of the K tile)
//                 S and dP are recomputed here (7 GEMMs in total instead of 5).
#include <algorithm>
#include <atomic>
#include <type_traits>

#include "vfm_common.h"

namespace vfm {

constexpr int kBwdWaves = 4;
constexpr int kBwdBC = 128;  // key/value rows per workgroup (32 per wavefront)
constexpr int kBwdBQ = 64;   // query rows per inner step
constexpr float kLog2eB = 1.4426950408889634f;

// ---------------------------------------------------------------- prepare
constexpr int kPrepHeads = 4;   // heads per workgroup (grid.y = ceil(n_heads / kPrepHeads))

template <int D>
__global__ __launch_bounds__(256) void bwd_prepare_kernel(const u32x4* __restrict__ out,
                                                          const u32x4* __restrict__ dout,
                                                          const float* __restrict__ lse,
                                                          float* __restrict__ delta,
                                                          float* __restrict__ lse2,
                                                          float* __restrict__ sentinel, int total,
                                                          int n_heads, int tok0, int tok_end) {
  constexpr int kLanesPerRow = D / 8;
  constexpr int kTokPerBlock = 256 / kLanesPerRow;
  const int tok = tok0 + blockIdx.x * kTokPerBlock + threadIdx.x / kLanesPerRow;   // the run's query tokens
  const int chunk = threadIdx.x % kLanesPerRow;
  const bool valid = tok < tok_end;
  const int tk = valid ? tok : tok_end - 1;
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {   // statistics fetched for rows past a clip's end
    sentinel[0] = INFINITY;                    // lse2: P = exp2(s - inf) = 0
    sentinel[1] = 0.f;                         // Delta
  }
  // blockIdx.y picks a group of kPrepHeads heads: their rows of one token are contiguous, the
  // loads of a group are in flight together, and a small call still spreads over the chip
  const int h0 = blockIdx.y * kPrepHeads;
  u32x4 a[kPrepHeads], b[kPrepHeads];
#pragma unroll
  for (int i = 0; i < kPrepHeads; ++i) {
    const size_t row = (size_t)tk * n_heads + min(h0 + i, n_heads - 1);
    a[i] = out[row * kLanesPerRow + chunk];
    b[i] = dout[row * kLanesPerRow + chunk];
  }
#pragma unroll
  for (int i = 0; i < kPrepHeads; ++i) {
    const int h = h0 + i;
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s = __builtin_fmaf(__builtin_bit_cast(float, a[i][e] << 16), __builtin_bit_cast(float, b[i][e] << 16), s);
      s = __builtin_fmaf(__builtin_bit_cast(float, a[i][e] & 0xffff0000u),
                         __builtin_bit_cast(float, b[i][e] & 0xffff0000u), s);
    }
#pragma unroll
    for (int o = kLanesPerRow / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, kLanesPerRow);
    if (valid && chunk == 0 && h < n_heads) {
      delta[(size_t)h * total + tok] = s;
      lse2[(size_t)h * total + tok] = lse[(size_t)h * total + tok] * kLog2eB;   // log2 units
    }
  }
}

// ---------------------------------------------------------------- Delta for short key ranges
// Delta_i = sum_d dO_id O_id is taken from the bf16 `out` the call is given.  In a sequence
// with a handful of keys |O| is as large as |V|, dS_ij = P_ij (dP_ij - Delta_i) is small by
// cancellation, and the rounding of `out` (2^-9 relative) shows in dQ and dK: up to 13% of the
// tensor in a two-token clip, below 0.1% from 32 keys on.  For sequences with at most
// kShortKeys keys Delta is therefore recomputed here in its other form,
//     Delta_i = sum_j P_ij dP_ij,   P_ij = exp(scale q_i.k_j - lse_i),   dP_ij = dO_i.v_j,
// with fp32 sums of the bf16 operands (the two forms are the same quantity for the exact O).
// One wavefront per 32 query rows: the scores S^T = K Q^T and dP^T = V dO^T of all (at most 32)
// keys are one 32x32 MFMA tile each, operands straight from memory, so the kernel is one round of
// loads deep.  (One lane per query row walking the keys in a serial loop took 31 us of the smallest
// training step, 32 tokens x 2 heads; this takes 2.6 us.)  Launched only when the call has such
// a sequence, over the tiles of those sequences only.

// A product that is rounded by itself, not within a fused multiply-add: two kernels that sum such products
// in the same order get the same bits.
__device__ __forceinline__ float mul_alone(float a, float b) {
#pragma clang fp contract(off)
  return a * b;
}

template <int D, class Segs>
__global__ __launch_bounds__(64) void bwd_short_delta_kernel(
    const __bf16* __restrict__ q, const __bf16* __restrict__ k, const __bf16* __restrict__ v,
    const __bf16* __restrict__ dout, const float* __restrict__ lse, float* __restrict__ delta,
    const Segs segs, const TileIndex ti, int total, int n_heads, float scale_log2) {
  constexpr int KS = D / 16;
  int seq, t;
  locate_tile(ti, segs.n, blockIdx.x, seq, t);
  const int nk = segs.kv_len(seq);
  const int head = blockIdx.y;
  const int lane = threadIdx.x, c = lane & 31, g = lane >> 5;
  const int q_b = segs.q_start(seq) + segs.q_len(seq);
  const int i = segs.q_start(seq) + t * 32 + c;
  const int ir = min(i, q_b - 1);                        // rows and keys past the end: copies of the last one
  const size_t row_stride = (size_t)n_heads * D;
  const size_t qoff = (size_t)ir * row_stride + (size_t)head * D + 8 * g;
  const size_t koff = (size_t)(segs.kv_start(seq) + min(c, nk - 1)) * row_stride + (size_t)head * D + 8 * g;
  const float lse_i = lse[(size_t)head * total + ir] * kLog2eB;
  f32x16 s = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 dp = s;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    s = mfma32(*reinterpret_cast<const bf16x8*>(k + koff + ks * 16),
               *reinterpret_cast<const bf16x8*>(q + qoff + ks * 16), s);
    dp = mfma32(*reinterpret_cast<const bf16x8*>(v + koff + ks * 16),
                *reinterpret_cast<const bf16x8*>(dout + qoff + ks * 16), dp);
  }
  // summed in the order of the key's index bits, 0 to 4, as the one-pass kernel does over its lanes
  float y[4];                                            // keys 8 x .. 8 x + 7 of query i
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    float t[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      t[e] = 8 * x + 4 * g + e < nk ? mul_alone(fast_exp2(s[4 * x + e] * scale_log2 - lse_i), dp[4 * x + e]) : 0.f;
    y[x] = pair_sum((t[0] + t[1]) + (t[2] + t[3]));
  }
  const float acc = (y[0] + y[1]) + (y[2] + y[3]);
  if (i < q_b && g == 0) delta[(size_t)head * total + i] = acc;
}

// ---------------------------------------------------------------- dK, dV
// Software pipelined over query blocks of 32 rows so that a single wavefront per SIMD
// always has independent MFMA and VALU work: iteration b runs
//   phase A:  S(b+1), dP(b+1) MFMAs        |  P(b)  = exp2(S(b)*scale - lse2)        (VALU)
//   phase B:  dV^T += dO(b)^T P(b) MFMAs   |  dS(b) = P(b) o (dP(b) - Delta)         (VALU)
//   phase C:  dK^T += Q(b)^T dS(b) MFMAs   |  row-operand reads of block b+2, tile requests
// Q/dO tiles of 64 rows (two blocks) live in a ring of three LDS stages filled by direct
// global->LDS loads two tiles ahead; there is one workgroup barrier per tile.  (Not further
// ahead on purpose: a workgroup that runs ahead of the others of its head then waits for
// its own L2 misses while the ones behind it hit, which keeps the workgroups of an XCD on
// the same part of Q/dO; three tiles ahead was measured to quadruple the HBM fetches.)
// Query rows past the clip end need no mask: their lse2 is fetched from a +inf sentinel
// (so P = 0) and their Delta from a 0 sentinel.  Key rows past the clip end need none
// either: a lane's key only feeds that lane's own dK/dV row, which is never stored.
constexpr int kBwdRing = 3;
constexpr int kSgValuB = 0x002, kSgMfmaB = 0x008, kSgDsReadB = 0x100;

template <int D>
struct BwdCfg {
  static constexpr int kTileBytes = kBwdBQ * D * 2;                      // one Q or dO tile
  static constexpr int kStageBytes = 2 * kTileBytes;                     // Q, dO tiles of one stage
  static constexpr int kStatBytes = 4 * kBwdBQ * 4;                      // lse2, Delta (+ spare) of one stage
  // tiles first (two stages span exactly 64 KB at head_dim 128: immediate LDS offsets), statistics behind them
  static constexpr int kStatBase = kBwdRing * kStageBytes;
  // the workgroup's K rows on their way into registers: over the ring's last stage, which fills after the prologue;
  // V rows: behind the statistics
  static constexpr int kOwnK = 2 * kStageBytes;
  static constexpr int kOwnV = kStatBase + kBwdRing * kStatBytes;
  static constexpr int kLdsBytes = kOwnV + kBwdBC * D * 2;
  static_assert(kBwdBC * D * 2 <= kStageBytes && kOwnV % 1024 == 0, "K rows fit a stage");
  static constexpr int kChunksPerRow = D / 8;
  static constexpr int kLoadsPerWave = kBwdBQ * kChunksPerRow / (kBwdWaves * 64);  // per tile, per tensor
};

// Adds a wavefront's 32 x D fp32 tile (accumulator layout, see store_tile_rows) to rows of fp32 sums in memory.  Turned
// through 32*D*4 bytes of LDS (16-byte chunk x of row r kept at chunk x ^ (r mod chunks-per-row)), so that an instruction
// adds 64 neighbouring elements.  Straight from the accumulators, 4 bytes of each of 64 places, the additions took
// as long as the products of a small call (whole backward, before -> now: 9,000 x 100 and 4,000 x 300 keys, 16 heads
// 251 -> 131 us; 20,000 x 77, 8 heads 152 -> 87; 56,320 x 512, 32 heads 1,722 -> 1,650).
template <int D>
__device__ __forceinline__ void add_tile_rows(char* turn, const f32x16 (&acc)[D / 32], float mul, float* dst,
                                              size_t row_stride, int rows_valid) {
  constexpr int CPR = D / 4, RB = D * 4;
  const int lane = threadIdx.x & 63, c = lane & 31, g = lane >> 5;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      f32x4 a;
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = acc[db][q4 * 4 + e] * mul;
      *reinterpret_cast<f32x4*>(turn + c * RB + (((db * 8 + q4 * 2 + g) ^ (c & (CPR - 1))) << 4)) = a;
    }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  for (int r = 0; r < min(32, rows_valid); ++r)
#pragma unroll
    for (int x = 0; x < D; x += 64) {
      const int col = x + lane;
      const float w = *reinterpret_cast<const float*>(turn + r * RB + (((col >> 2) ^ (r & (CPR - 1))) << 4) + (col & 3) * 4);
      __hip_atomic_fetch_add(dst + (size_t)r * row_stride + col, w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// SPLIT: the sequence's query range is cut into q_split chunks, one workgroup each; partial
// dK/dV are added to zeroed fp32 accumulators (dkv32: dK, then dV) with fp32 atomics and
// converted afterwards.  Used when a few long key tiles would otherwise leave CUs idle.
// The work of one workgroup: key tile tk of sequence seq, one head (and, if SPLIT, one chunk of
// the sequence's queries).
template <int D, class Segs, bool SPLIT>
__device__ __forceinline__
void bwd_dkdv_unit(const __bf16* __restrict__ q, const __bf16* __restrict__ k,
                   const __bf16* __restrict__ v, const __bf16* __restrict__ dout,
                   const float* __restrict__ lse2, const float* __restrict__ delta,
                   const float* __restrict__ sentinel,   // [+inf, 0]
                   __bf16* __restrict__ dk, __bf16* __restrict__ dv, const Segs& segs,
                   int total, int n_heads, float scale, float scale_log2,
                   float* __restrict__ dkv32, size_t kv_elems, int q_split,
                   int head, int seq, int tk, int q_chunk) {
  using Cfg = BwdCfg<D>;
  constexpr int KS = D / 16;
  constexpr int DB = D / 32;
  constexpr int LPW = Cfg::kLoadsPerWave;
  constexpr int SB = Cfg::kStageBytes;
  constexpr int TB = Cfg::kTileBytes;
  constexpr int RB = D * 2;
  constexpr bool kAsm = D == 128;   // more than 256 registers (see mfma32_v)

  extern __shared__ __attribute__((aligned(16))) char smem[];

  // key rows [j0, j0 + kBwdBC) of the sequence's key/value range [.., kv_b); the queries it
  // walks are rows [seg_a, seg_b) of q, dout (the same range for self-attention)
  const int kv_b = segs.kv_start(seq) + segs.kv_len(seq);
  const int j0 = segs.kv_start(seq) + tk * kBwdBC;
  int qa = segs.q_start(seq), qb = qa + segs.q_len(seq);
  if constexpr (SPLIT) {   // this workgroup's share of the query tiles
    const int per = ((qb - qa + kBwdBQ - 1) / kBwdBQ + q_split - 1) / q_split * kBwdBQ;
    qa += q_chunk * per;
    qb = min(qb, qa + per);
    if (qa >= qb) return;  // nothing to add (the accumulators start at zero)
  }
  const int seg_a = qa, seg_b = qb;

  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  const int lane = tid & 63;
  const int c = lane & 31;
  const int g = lane >> 5;
  const size_t row_stride = (size_t)n_heads * D;
  const size_t head_off = (size_t)head * D;

  // ---- this wavefront's key/value rows as B operands (lane: row c, columns ks*16+8g..)
  const int jrow = j0 + wave * 32 + c;
  const bool jvalid = jrow < kv_b;
  if (seg_b == seg_a) {   // keys of a sequence without queries: zero gradients (cross-attention only)
    if (jvalid) {
      u32x2 z = {0u, 0u};
#pragma unroll
      for (int x = 0; x < D / 8; ++x) {
        *reinterpret_cast<u32x2*>(dk + (size_t)jrow * row_stride + head_off + 4 * g + 8 * x) = z;
        *reinterpret_cast<u32x2*>(dv + (size_t)jrow * row_stride + head_off + 4 * g + 8 * x) = z;
      }
    }
    return;
  }

  // ---- tile requests (direct global->LDS).  Lane L of wave instruction (x, wave) owns
  // LDS chunk P = (x*waves + wave)*64 + L of the tile (row P / chunks_per_row, physical
  // chunk P % chunks_per_row) and fetches the logical chunk the swizzle maps there.
  // Every wave also fetches 64 row statistics (4 bytes per lane): waves 0/2 lse2, waves
  // 1/3 Delta (2 and 3 into spare LDS, so that all waves have equally many loads in
  // flight).  Tiles are requested strictly in order; offsets advance by one tile.
  const uint32_t row_bytes = (uint32_t)row_stride * 2u;
  const uint32_t last_row_off = (uint32_t)(seg_b - 1) * row_bytes;
  const __bf16* qbase = q + head_off;
  const __bf16* dobase = dout + head_off;
  uint32_t st_rowoff[LPW], st_colb[LPW];
#pragma unroll
  for (int x = 0; x < LPW; ++x) {
    const int p = (x * kBwdWaves + wave) * 64 + lane;
    const int r = p / Cfg::kChunksPerRow;
    st_rowoff[x] = (uint32_t)(seg_a + r) * row_bytes;
    st_colb[x] = (uint32_t)(((p % Cfg::kChunksPerRow) ^ swz<D>(r)) * 16);
  }
  const bool is_lse = (wave & 1) == 0;
  const float* stat_src = uniform_ptr(is_lse ? lse2 : delta);
  const uint32_t stat_sentinel = (uint32_t)((const char*)(sentinel + (is_lse ? 0 : 1)) - (const char*)stat_src);
  int stat_row = seg_a + lane;                         // packed row this lane fetches next
  const uint32_t stat_head = (uint32_t)((size_t)head * total * 4u);
  const uint32_t smem_addr = lds_addr_of(smem);
  const uint32_t wave_lds = __builtin_amdgcn_readfirstlane(smem_addr + wave * 1024);
  const uint32_t stat_lds = __builtin_amdgcn_readfirstlane(smem_addr + Cfg::kStatBase + wave * (kBwdBQ * 4));
  auto issue_tile = [&](int stage) {
#pragma unroll
    for (int x = 0; x < LPW; ++x) {
      const uint32_t off = min(st_rowoff[x], last_row_off) + st_colb[x];
      const uint32_t dst = wave_lds + stage * SB + x * kBwdWaves * 1024;
      lds_dma16(qbase, off, dst);
      lds_dma16(dobase, off, dst + TB);
      st_rowoff[x] += kBwdBQ * row_bytes;
    }
    const uint32_t soff = stat_row < seg_b ? stat_head + (uint32_t)stat_row * 4u : stat_sentinel;
    lds_dma4(stat_src, soff, stat_lds + stage * Cfg::kStatBytes);
    stat_row += kBwdBQ;
  };

  // ---- per-lane LDS offsets within a tile.  The swizzle XORs low byte-offset bits with a
  // function of the low row bits only, so one base per lane serves every k-step / block:
  //   Q/dO rows as A operand (row ib*32 + c, columns ks*16 + 8g):
  //       off = (rbase ^ (ks << 5)) + ib*32*rowbytes
  //   Q^T/dO^T as A operand through transposing reads (same slot binding as the forward
  //   kernel's V^T operand):  off = (tbase[t] ^ (db << 6)) + (ib*32 + 16*s2)*rowbytes
  const int rbase = tile_off<D>(c, 8 * g);
  int tbase[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
    tbase[t] = tile_off<D>(8 * t + 4 * g + ((lane & 15) >> 2),
                           16 * ((lane >> 4) & 1) + 4 * (lane & 3));

  // Every swizzled LDS address the loop uses, held in a register of its own (made opaque so
  // that the compiler keeps them instead of recomputing them between the MFMAs): set 0 for
  // stages 0 and 1, set 1 for stage 2, whose tiles lie beyond the 64 KB an immediate reaches (head_dim 64: one set
  // reaches all three).
  constexpr int SETS = kBwdRing * SB > 65536 ? 2 : 1;
  uint32_t rb[SETS][KS], tb[SETS][2][DB];
#pragma unroll
  for (int hs = 0; hs < SETS; ++hs) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      rb[hs][ks] = smem_addr + hs * 2 * SB + (rbase ^ (ks << 5));
      asm volatile("" : "+v"(rb[hs][ks]));
    }
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        tb[hs][t][db] = smem_addr + hs * 2 * SB + (tbase[t] ^ (db << 6));
        asm volatile("" : "+v"(tb[hs][t][db]));
      }
  }

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 dkacc[DB], dvacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) { dkacc[db] = zero16; dvacc[db] = zero16; }

  const int n_tiles = (seg_b - seg_a + kBwdBQ - 1) / kBwdBQ;
  const int n_blocks = 2 * n_tiles;

  auto read_rows = [&](int stage, int ib, bf16x8 (&qa)[KS], bf16x8 (&da)[KS]) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint32_t a = rb[SETS == 2 ? stage >> 1 : 0][ks] + (SETS == 2 ? stage & 1 : stage) * SB + ib * 32 * RB;
      qa[ks] = lds_read_b128_at(a);
      da[ks] = lds_read_b128_at(a + TB);
    }
  };

  // ---- prologue: K, V rows, tiles 0 and 1 requested; S(0), dP(0); row operands of block 1.  K and V come through LDS
  // in whole rows like the tiles, not as operands (32 bytes of each of 32 rows per
  // instruction): whole backward call 1.5% less for 40 clips of 700 tokens x 16 heads, 1% for 100 of 512, level from
  // 4,096 tokens on
  const uint32_t own = smem_addr + wave * (32 * RB);   // this wavefront's rows, from kOwnK and kOwnV on
  {
    const __bf16* kbase = k + head_off;
    const __bf16* vbase = v + head_off;
    const uint32_t own_s = __builtin_amdgcn_readfirstlane(own);
#pragma unroll
    for (int x = 0; x < 32 * RB / 1024; ++x) {
      const int p = x * 64 + lane, r = p / Cfg::kChunksPerRow;
      const uint32_t off = (uint32_t)min(j0 + wave * 32 + r, kv_b - 1) * row_bytes +
                           (uint32_t)(((p % Cfg::kChunksPerRow) ^ swz<D>(r)) * 16);
      lds_dma16(kbase, off, own_s + Cfg::kOwnK + x * 1024);
      lds_dma16(vbase, off, own_s + Cfg::kOwnV + x * 1024);
    }
  }
  issue_tile(0); issue_tile(1);
  wait_vmcnt<0>();
  bf16x8 kreg[KS], vreg[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    kreg[ks] = lds_read_b128_at(own + Cfg::kOwnK + (rbase ^ (ks << 5)));
    vreg[ks] = lds_read_b128_at(own + Cfg::kOwnV + (rbase ^ (ks << 5)));
    if constexpr (kAsm) { to_agpr(kreg[ks]); to_agpr(vreg[ks]); }
    else { settle(kreg[ks]); settle(vreg[ks]); }
  }
  __syncthreads();

  // A wavefront whose 32 key rows all lie past the end of the sequence (ragged last tile) has
  // nothing to compute.  It still fetches its share of every Q/dO tile and meets every
  // barrier, in the order of the loop below: per tile the wait, the barrier, the request;
  // then the final wait (and the epilogue's barrier).
  if (j0 + wave * 32 >= kv_b) {
    for (int t = 0; t < n_tiles; ++t) {
      wait_vmcnt<0>();
      __syncthreads();
      issue_tile((t + 2) % kBwdRing);
    }
    wait_vmcnt<0>();
    __syncthreads();
    return;
  }

  bf16x8 qa_n[KS], da_n[KS];      // row operands of block b+1
  f32x16 s_cur, dp_cur;           // S(b), dP(b)
  {
    bf16x8 q0r[KS], d0r[KS];
    read_rows(0, 0, q0r, d0r);
    read_rows(0, 1, qa_n, da_n);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      if constexpr (kAsm) {
        mfma32_v(s_cur, q0r[ks], kreg[ks], ks == 0);
        mfma32_v(dp_cur, d0r[ks], vreg[ks], ks == 0);
      } else {
        s_cur = mfma32(q0r[ks], kreg[ks], ks == 0 ? zero16 : s_cur);
        dp_cur = mfma32(d0r[ks], vreg[ks], ks == 0 ? zero16 : dp_cur);
      }
    }
  }

  // One pipeline iteration; POS = b % 6 fixes every LDS stage at compile time.
  auto iteration = [&](auto pos_c) {
    constexpr int POS = decltype(pos_c)::value;
    constexpr int IB = POS & 1;                          // block b within its tile
    constexpr int ST_CUR = (POS / 2) % kBwdRing;         // stage of block b's tile
    constexpr int ST_ROW = ((POS + 2) / 2) % kBwdRing;   // stage of block b+2's tile
    if constexpr (IB == 0) {
      // Start of tile t = b/2: tile t+1 must have landed for every wave before anyone reads
      // block b+2's rows, and every wave is past tile t-1, whose stage takes tile t+2.
      wait_vmcnt<0>();
      __syncthreads();
      issue_tile((ST_CUR + 2) % kBwdRing);
    }
    const float* lse_s = reinterpret_cast<const float*>(smem + Cfg::kStatBase + ST_CUR * Cfg::kStatBytes);
    const float* delta_s = lse_s + kBwdBQ;               // wave 1's statistics follow wave 0's

    // ---- phase A: S(b+1), dP(b+1) | P(b) | statistics and transposed-operand reads of block b
    // One group per MFMA, in program order (see mfma32_v): group 0 fetches lse, every group
    // two transposed operands (dO^T first: phase B needs it first), the last two Delta; the
    // 16 values of P per lane are spread over groups 2.. so that lse has arrived.
    constexpr int NG = 2 * KS;
    f32x4 l4[4], d4[4];
    s16x4 dlo[2][DB], dhi[2][DB], qlo[2][DB], qhi[2][DB];
    f32x16 s_next, dp_next, p;
    u32x8 pw;
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
      const int ks = gi >> 1;
      if constexpr (kAsm) {
        if ((gi & 1) == 0) mfma32_v(s_next, qa_n[ks], kreg[ks], ks == 0, s_cur, p, pw);
        else mfma32_v(dp_next, da_n[ks], vreg[ks], ks == 0, s_cur, p, pw);
      } else {
        if ((gi & 1) == 0) s_next = mfma32(qa_n[ks], kreg[ks], ks == 0 ? zero16 : s_next);
        else dp_next = mfma32(da_n[ks], vreg[ks], ks == 0 ? zero16 : dp_next);
      }
      if (gi == 0) {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) l4[q4] = *reinterpret_cast<const f32x4*>(lse_s + IB * 32 + 8 * q4 + 4 * g);
      }
#pragma unroll
      for (int r = 2 * gi; r < 2 * gi + 2; ++r) {
        const int rr = r % (4 * DB), s2 = rr / (2 * DB), db = (rr >> 1) % DB, hi = rr & 1;
        const uint32_t o = tb[SETS == 2 ? ST_CUR >> 1 : 0][hi][db] + (SETS == 2 ? ST_CUR & 1 : ST_CUR) * SB + (IB * 32 + 16 * s2) * RB;
        if (r < 4 * DB) { if (hi) dhi[s2][db] = lds_read_tr_at(o + TB); else dlo[s2][db] = lds_read_tr_at(o + TB); }
        else { if (hi) qhi[s2][db] = lds_read_tr_at(o); else qlo[s2][db] = lds_read_tr_at(o); }
      }
      if (gi >= NG - 2) {
#pragma unroll
        for (int q4 = 2 * (gi - (NG - 2)); q4 < 2 * (gi - (NG - 2)) + 2; ++q4)
          d4[q4] = *reinterpret_cast<const f32x4*>(delta_s + IB * 32 + 8 * q4 + 4 * g);
      }
      // P for rows i = 8*(e/4) + 4g + e%4 of the block, column j = this lane's key; a pair
      // is converted one group after its exponentials (no transcendental-result stall)
#pragma unroll
      for (int e = 1; e < 16; e += 2)
        if (e * (NG - 2) / 16 + 3 == gi) {
          const f32x2 pr = {p[e - 1], p[e]};
          pw[e >> 1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2));
        }
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (e * (NG - 2) / 16 + 2 == gi) p[e] = fast_exp2(s_cur[e] * scale_log2 - l4[e >> 2][e & 3]);
      __builtin_amdgcn_sched_barrier(0);
    }
    {
      const f32x2 pr = {p[14], p[15]};   // the last pair's group would be NG
      pw[7] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2));
    }
    bf16x8 pb[2];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      const u32x4 w = {pw[4 * s2], pw[4 * s2 + 1], pw[4 * s2 + 2], pw[4 * s2 + 3]};
      pb[s2] = __builtin_bit_cast(bf16x8, w);
    }

    // ---- phase B: dV^T += dO(b)^T P(b) | dS(b) = P(b) o (dP(b) - Delta)
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int db = 0; db < DB; ++db)
        dvacc[db] = mfma32(join_tr(dlo[s2][db], dhi[s2][db]), pb[s2], dvacc[db]);
    bf16x8 dsb[2];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      f32x8 a;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int r = 8 * s2 + e;
        a[e] = p[r] * (dp_cur[r] - d4[r >> 2][r & 3]);
      }
      dsb[s2] = to_bf16x8(a);
    }
#pragma unroll
    for (int i = 0; i < 2 * DB; ++i) {
      __builtin_amdgcn_sched_group_barrier(kSgMfmaB, 1, 0);
      __builtin_amdgcn_sched_group_barrier(kSgValuB, 5, 0);
    }
    __builtin_amdgcn_sched_barrier(0);

    // ---- phase C: dK^T += Q(b)^T dS(b) | row operands of block b+2
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int db = 0; db < DB; ++db)
        dkacc[db] = mfma32(join_tr(qlo[s2][db], qhi[s2][db]), dsb[s2], dkacc[db]);
    bf16x8 qa_2[KS], da_2[KS];
    read_rows(ST_ROW, IB, qa_2, da_2);
#pragma unroll
    for (int i = 0; i < 2 * DB; ++i) {
      __builtin_amdgcn_sched_group_barrier(kSgMfmaB, 1, 0);
      __builtin_amdgcn_sched_group_barrier(kSgDsReadB, (2 * KS + 2 * DB - 1) / (2 * DB), 0);
    }
    __builtin_amdgcn_sched_barrier(0);

    s_cur = s_next;
    dp_cur = dp_next;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) { qa_n[ks] = qa_2[ks]; da_n[ks] = da_2[ks]; }
  };

  static_assert(kBwdRing == 3, "the block loop is unrolled over the ring");
  for (int b = 0; b < n_blocks; b += 6) {
    iteration(IntC<0>{});
    iteration(IntC<1>{});
    if (b + 2 < n_blocks) { iteration(IntC<2>{}); iteration(IntC<3>{}); }
    if (b + 4 < n_blocks) { iteration(IntC<4>{}); iteration(IntC<5>{}); }
  }
  wait_vmcnt<0>();   // no load may still be writing LDS when the workgroup ends

  // ---- epilogue: dK (scaled) and dV of this wavefront's key rows
  __syncthreads();   // the ring is free: each wavefront turns its tiles through a piece of it
  const int row0 = j0 + wave * 32;
  if constexpr (SPLIT) {
    char* turn = smem + wave * (32 * D * 4);
    float* dkp = dkv32 + ((size_t)row0 * n_heads + head) * D;
    add_tile_rows<D>(turn, dkacc, scale, dkp, row_stride, kv_b - row0);
    add_tile_rows<D>(turn, dvacc, 1.0f, dkp + kv_elems, row_stride, kv_b - row0);
  } else {
    char* turn = smem + wave * (32 * RB);
    store_tile_rows<D>(turn, dkacc, scale, dk + (size_t)row0 * row_stride + head_off, row_stride, kv_b - row0);
    store_tile_rows<D>(turn, dvacc, 1.0f, dv + (size_t)row0 * row_stride + head_off, row_stride, kv_b - row0);
  }
}

// head_dim 64: two workgroups per CU (252 registers, 67 KB of LDS each; one set of LDS addresses, every operand in a
// VGPR), so that the exponentials of one meet the products of the other.  Against one workgroup with its operands in
// AGPRs (272 registers), whole backward call: 32,768 tokens x 32 heads 27.7 -> 26.2 ms, 64 clips of 300 x 16
// 170 -> 145 us, 2 x 4,096 x 16 456 -> 447; calls of fewer tiles than CUs lose 2% (2 x 2,048 x 2 62 -> 64).
template <int D, class Segs, bool SPLIT>
__global__ __launch_bounds__(kBwdWaves * 64, D == 64 ? 2 : 1)
void attn_bwd_dkdv_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k,
                          const __bf16* __restrict__ v, const __bf16* __restrict__ dout,
                          const float* __restrict__ lse2, const float* __restrict__ delta,
                          const float* __restrict__ sentinel,
                          __bf16* __restrict__ dk, __bf16* __restrict__ dv,
                          const Segs segs, const UnitMap um, const TileIndex ti,
                          int total, int n_heads, float scale, float scale_log2,
                          float* __restrict__ dkv32, size_t kv_elems, int q_split) {
  int head, tile;
  if (!map_unit(um, blockIdx.x, head, tile)) return;
  int q_chunk = 0;
  if constexpr (SPLIT) { q_chunk = tile % q_split; tile /= q_split; }
  int seq, tk;
  locate_tile(ti, segs.n, tile, seq, tk);
  bwd_dkdv_unit<D, Segs, SPLIT>(q, k, v, dout, lse2, delta, sentinel, dk, dv, segs, total, n_heads, scale,
                                scale_log2, dkv32, kv_elems, q_split, head, seq, tk, q_chunk);
}

// The fp32 sums of a split dK/dV pass, dK's and dV's in one launch each (blockIdx.y): zeroed before, -> bf16 after
__global__ void fill_zero_f32x4_kernel(f32x4* p0, f32x4* p1, size_t n4) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const f32x4 z = {0.f, 0.f, 0.f, 0.f};
  if (i < n4) (blockIdx.y ? p1 : p0)[i] = z;
}
__global__ void f32_to_bf16_kernel(const f32x4* __restrict__ src0, const f32x4* __restrict__ src1,
                                   bf16x4* __restrict__ dst0, bf16x4* __restrict__ dst1, size_t n4) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n4) (blockIdx.y ? dst1 : dst0)[i] = to_bf16x4((blockIdx.y ? src1 : src0)[i]);
}

// ---------------------------------------------------------------- dQ
constexpr int kDqBC = 64;   // key/value rows per LDS tile

template <int D, int NI, int W>
struct DqCfg {
  static constexpr int kBR = W * NI * 32;        // query rows per workgroup
  static constexpr int kTileBytes = kDqBC * D * 2;      // one K or V tile
  static constexpr int kLdsBytes = 4 * kTileBytes;      // K, V x 2 stages
  static constexpr int kChunksPerRow = D / 8;
  static constexpr int kChunksPerThread = kDqBC * kChunksPerRow / (W * 64);
};

// Serves head_dim 64, where the exponentials weigh twice as much against the products as at 128: with 154 registers
// three workgroups of four wavefronts share a CU, and half as many rows per workgroup spread small calls
// over more CUs.  Against one workgroup of eight wavefronts per CU (whole backward call): 64 clips of 300 tokens x 16 heads
// 176 -> 145 us, 2 x 2,048 tokens x 2 heads 74 -> 64, 8,192 x 12 692 -> 655, 32,768 x 32 26.9 -> 26.2 ms, 2 x 4,096 x
// 16 440 -> 447; each K/V tile is staged twice as often.
// STATS: as in bwd_dq2_unit (the pass runs first and leaves Delta, lse in log2 units and the sentinels for the
// dK/dV pass; figures at bwd_order).
template <int D, int NI, int W, class Segs, bool STATS>
__global__ __launch_bounds__(W * 64, NI == 1 ? 3 : 1)
void attn_bwd_dq_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k,
                        const __bf16* __restrict__ v, const __bf16* __restrict__ dout,
                        const __bf16* __restrict__ out, const float* __restrict__ lse,
                        float* __restrict__ lse2g, float* __restrict__ delta, float* __restrict__ sentinel,
                        __bf16* __restrict__ dq, const Segs segs, const UnitMap um, const TileIndex ti,
                        int total, int n_heads, float scale, float scale_log2) {
  using Cfg = DqCfg<D, NI, W>;
  constexpr int KS = D / 16;
  constexpr int DB = D / 32;
  constexpr int JB = kDqBC / 32;
  constexpr int CPT = Cfg::kChunksPerThread;
  constexpr int RB = D * 2;

  extern __shared__ __attribute__((aligned(16))) char smem[];

  int head, tile;
  if (!map_unit(um, blockIdx.x, head, tile)) return;
  if (STATS && blockIdx.x == 0 && threadIdx.x == 0) {   // the dK/dV pass' statistics of rows past a clip's end
    sentinel[0] = INFINITY;
    sentinel[1] = 0.f;
  }
  // query rows of the range [.., q_b); keys and values are rows [seg_a, seg_b) of k, v
  int seq, tq;
  locate_tile(ti, segs.n, tile, seq, tq);
  const int q_b = segs.q_start(seq) + segs.q_len(seq);
  const int q0 = segs.q_start(seq) + tq * Cfg::kBR;
  const int seg_a = segs.kv_start(seq);
  const int seg_b = seg_a + segs.kv_len(seq);

  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  const int lane = tid & 63;
  const int c = lane & 31;
  const int g = lane >> 5;
  const size_t row_stride = (size_t)n_heads * D;
  const size_t head_off = (size_t)head * D;
  const __bf16* kbase = k + head_off;
  const __bf16* vbase = v + head_off;

  // ---- Q and dO rows as B operands; lse (log2 units) and Delta are per-lane scalars
  bf16x8 qreg[NI][KS], doreg[NI][KS];
  float lse2[NI], dlt[NI];
  int qrow[NI];
#pragma unroll
  for (int ib = 0; ib < NI; ++ib) {
    qrow[ib] = q0 + (wave * NI + ib) * 32 + c;
    const int r = min(qrow[ib], q_b - 1);
    const size_t off = (size_t)r * row_stride + head_off + 8 * g;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      qreg[ib][ks] = *reinterpret_cast<const bf16x8*>(q + off + ks * 16);
      doreg[ib][ks] = *reinterpret_cast<const bf16x8*>(dout + off + ks * 16);
    }
    const size_t stat = (size_t)head * total + r;
    if constexpr (STATS) {
      bf16x8 oreg[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) oreg[ks] = *reinterpret_cast<const bf16x8*>(out + off + ks * 16);
      lse2[ib] = lse[stat] * kLog2eB;
      // the order of bwd_prepare_kernel's sums (chunks of 8 columns, then pairs of chunks D/16, .., 2, 1 apart)
      float s[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        s[ks] = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) s[ks] = __builtin_fmaf((float)oreg[ks][e], (float)doreg[ib][ks][e], s[ks]);
      }
#pragma unroll
      for (int o = KS / 2; o > 0; o >>= 1)
#pragma unroll
        for (int ks = 0; ks < o; ++ks) s[ks] += s[ks + o];
      dlt[ib] = pair_sum(s[0]);
      const bool few = segs.kv_len(seq) <= kShortKeys;   // (already in place)
      if (few) dlt[ib] = delta[stat];
      if (g == 0 && qrow[ib] < q_b) {
        lse2g[stat] = lse2[ib];
        if (!few) delta[stat] = dlt[ib];
      }
    } else {
      lse2[ib] = lse2g[stat];
      dlt[ib] = delta[stat];
    }
  }

  // ---- K/V staging with direct global->LDS loads (same scheme as the forward kernel)
  const uint32_t row_bytes = (uint32_t)row_stride * 2u;
  const uint32_t last_row_off = (uint32_t)(seg_b - 1) * row_bytes;
  uint32_t st_rowoff[CPT], st_colb[CPT];
#pragma unroll
  for (int x = 0; x < CPT; ++x) {
    const int p = (x * W + wave) * 64 + lane;
    const int r = p / Cfg::kChunksPerRow;
    st_rowoff[x] = (uint32_t)(seg_a + r) * row_bytes;
    st_colb[x] = (uint32_t)(((p % Cfg::kChunksPerRow) ^ swz<D>(r)) * 16);
  }
  const uint32_t wave_lds = __builtin_amdgcn_readfirstlane(lds_addr_of(smem) + wave * 1024);
  auto issue_tile = [&](int stage) {   // tiles are requested in sequence
#pragma unroll
    for (int x = 0; x < CPT; ++x) {
      const uint32_t off = min(st_rowoff[x], last_row_off) + st_colb[x];
      const uint32_t dst = wave_lds + stage * 2 * Cfg::kTileBytes + x * W * 1024;
      lds_dma16(kbase, off, dst);
      lds_dma16(vbase, off, dst + Cfg::kTileBytes);
      st_rowoff[x] += kDqBC * row_bytes;
    }
  };

  // K/V rows as A operand: off = (rbase ^ (ks << 5)) + jb*32*RB
  // K^T as A operand (transposing reads): off = (tbase[t] ^ (db << 6)) + (jb*32 + 16*s2)*RB
  const int rbase = tile_off<D>(c, 8 * g);
  int tbase[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
    tbase[t] = tile_off<D>(8 * t + 4 * g + ((lane & 15) >> 2),
                           16 * ((lane >> 4) & 1) + 4 * (lane & 3));

  f32x16 dqacc[NI][DB];
#pragma unroll
  for (int ib = 0; ib < NI; ++ib)
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) dqacc[ib][db][r] = 0.f;
  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

  const int n_tiles = (seg_b - seg_a + kDqBC - 1) / kDqBC;
#pragma unroll
  for (int ib = 0; ib < NI; ++ib)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) { settle(qreg[ib][ks]); settle(doreg[ib][ks]); }
#pragma unroll
  for (int ib = 0; ib < NI; ++ib) asm volatile("" :: "v"(lse2[ib]), "v"(dlt[ib]));
  issue_tile(0);
  wait_vmcnt<0>();
  __syncthreads();

  auto tile_body = [&](auto stage_c, int t) {
    constexpr int STAGE = decltype(stage_c)::value;
    const int j0 = seg_a + t * kDqBC;
    if (t + 1 < n_tiles) issue_tile(STAGE ^ 1);   // lands while this tile is processed
    const char* kt = smem + STAGE * 2 * Cfg::kTileBytes;
    const char* vt = kt + Cfg::kTileBytes;
    const bool tail = (j0 + kDqBC > seg_b);

#pragma unroll
    for (int jb = 0; jb < JB; ++jb) {
      // all row operands of this key block are requested before the first MFMA
      bf16x8 ka[KS], va[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int off = (rbase ^ (ks << 5)) + jb * 32 * RB;
        ka[ks] = lds_read_b128(kt, off);
        va[ks] = lds_read_b128(vt, off);
      }
      __builtin_amdgcn_sched_barrier(0);
      f32x16 sacc[NI], dpacc[NI];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int ib = 0; ib < NI; ++ib) {
          sacc[ib] = mfma32(ka[ks], qreg[ib][ks], ks == 0 ? zero16 : sacc[ib]);
          dpacc[ib] = mfma32(va[ks], doreg[ib][ks], ks == 0 ? zero16 : dpacc[ib]);
        }
      // K^T operands for the dQ MFMAs, requested in the shadow of the MFMAs above
      s16x4 klo[2][DB], khi[2][DB];
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          klo[s2][db] = lds_read_tr(kt, (tbase[0] ^ (db << 6)) + (jb * 32 + 16 * s2) * RB);
          khi[s2][db] = lds_read_tr(kt, (tbase[1] ^ (db << 6)) + (jb * 32 + 16 * s2) * RB);
        }
      __builtin_amdgcn_sched_barrier(0);
      bf16x8 dsb[NI][2];
#pragma unroll
      for (int ib = 0; ib < NI; ++ib) {
        f32x16 ds;
        if (tail) {   // wave-uniform: only the clip's last tile pays for the key mask
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int j = j0 + jb * 32 + 8 * (r >> 2) + 4 * g + (r & 3);
            const float pv = (j < seg_b) ? fast_exp2(sacc[ib][r] * scale_log2 - lse2[ib]) : 0.f;
            ds[r] = pv * (dpacc[ib][r] - dlt[ib]);
          }
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float pv = fast_exp2(sacc[ib][r] * scale_log2 - lse2[ib]);
            ds[r] = pv * (dpacc[ib][r] - dlt[ib]);
          }
        }
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
          f32x8 a;
#pragma unroll
          for (int e = 0; e < 8; ++e) a[e] = ds[8 * s2 + e];
          dsb[ib][s2] = to_bf16x8(a);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          const bf16x8 kta = join_tr(klo[s2][db], khi[s2][db]);
#pragma unroll
          for (int ib = 0; ib < NI; ++ib) dqacc[ib][db] = mfma32(kta, dsb[ib][s2], dqacc[ib][db]);
        }
      __builtin_amdgcn_sched_barrier(0);
    }

    wait_vmcnt<0>();   // the next tile has landed ...
    __syncthreads();   // ... for every wave, and every wave is done reading this one
  };
  for (int t = 0; t < n_tiles; t += 2) {
    tile_body(IntC<0>{}, t);
    if (t + 1 < n_tiles) tile_body(IntC<1>{}, t + 1);
  }

  // ---- epilogue: dq = bf16(scale * dQ^T), whole rows per store; every wave is past the ring (the loop's last
  // barrier), each turns its tiles through a piece of it
#pragma unroll
  for (int ib = 0; ib < NI; ++ib) {
    const int row0 = q0 + (wave * NI + ib) * 32;
    store_tile_rows<D>(smem + wave * (32 * RB), dqacc[ib], scale, dq + (size_t)row0 * row_stride + head_off, row_stride,
                       q_b - row0);
  }
}

// ---------------------------------------------------------------- dQ, 64 query rows per wavefront
// Same mathematics as attn_bwd_dq_kernel, built to halve its LDS operand traffic (under this
// chip's power limit the energy per flop is what bounds the kernels, and one LDS operand read
// per MFMA is a third of it): a wavefront owns two 32-row query blocks, so every K, V row
// operand and every K^T operand read from LDS feeds two MFMAs.  That needs 512 registers,
// i.e. one wavefront per SIMD, with the register classes chosen by hand: Q, dO rows (128) and
// the dQ^T accumulators (128) live in AGPRs, which the MFMAs address directly; S^T, dP^T and
// everything the VALU touches live in VGPRs.  All MFMAs are therefore assembly statements.
// With a single wavefront per SIMD nothing else hides the VALU work, so the two query blocks
// alternate ("half-steps"): while the VALU turns block IB's S^T, dP^T of key block b into
// dS^T, the matrix pipe runs the other block's MFMAs,
//     groups  0..15 : S^T, dP^T of the other block's next key block   (assembly, VGPR results)
//     groups 16..23 : dQ^T += K^T dS^T of the other block's previous key block
// one group per MFMA; register tuples passed through the statements (the block's S^T, so that
// nothing reads it early, and the VALU's results) pin one element of the VALU work to each group.  The compiler inserts no wait states for readers of an assembly
// MFMA's result: S^T, dP^T are read a half-step later (>= 8 MFMAs), the accumulators after
// explicit wait states at the end.
// K/V tiles of 64 keys go through a ring of three LDS stages: tile t is read from the second
// half of key block 2t-1 to the end of key block 2t+1, the workgroup meets once per tile at
// the start of key block 2t-1 (tile t landed, everybody done with tile t-2) and requests
// tile t+1 there.
constexpr int kDq2Waves = 4;
constexpr int kDq2Ring = 3;

template <int D>
struct Dq2Cfg {
  static constexpr int kBR = kDq2Waves * 64;                 // query rows per workgroup
  static constexpr int kTileBytes = kDqBC * D * 2;           // one K or V tile
  static constexpr int kStageBytes = 2 * kTileBytes;         // K tile, V tile
  // a wavefront's 64 rows of Q and of dO on their way into registers: behind the ring's first stage
  static constexpr int kOwnBase = kStageBytes;
  static constexpr int kOwnBytes = 2 * 64 * D * 2;
  static constexpr int kLdsBytes = kOwnBase + kDq2Waves * kOwnBytes;
  static_assert(kLdsBytes >= kDq2Ring * kStageBytes && kLdsBytes <= 160 * 1024, "ring, LDS of one CU");
  static constexpr int kChunksPerRow = D / 8;
  static constexpr int kChunksPerThread = kDqBC * kChunksPerRow / (kDq2Waves * 64);
};

// Sum over a lane's row of 16 lanes, in every lane: v + the value 8, then 4, 2, 1 lanes away (rotations).
__device__ __forceinline__ float row16_sum(float v) {
  auto add = [&](auto ror) {
    constexpr int kRor = 0x120 + decltype(ror)::value;   // row_ror
    v += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), kRor, 0xf, 0xf, true));
  };
  add(IntC<8>{});
  add(IntC<4>{});
  add(IntC<2>{});
  add(IntC<1>{});
  return v;
}

// The work of one workgroup: query tile tq of sequence seq, one head.  STATS: form Delta and lse in log2
// units of the tile's rows here, from `out` and `lse`, and leave them for the dK/dV pass (Delta of a sequence
// with few keys is already in place).  The rows of dO are in LDS on their way into registers, so this costs the
// reads of `out`, where the separate pass reads dO as well and is one more launch.
template <int D, class Segs, bool STATS>
__device__ __forceinline__
void bwd_dq2_unit(const __bf16* __restrict__ q, const __bf16* __restrict__ k,
                  const __bf16* __restrict__ v, const __bf16* __restrict__ dout,
                  const __bf16* __restrict__ out, const float* __restrict__ lse,
                  float* __restrict__ lse2g, float* __restrict__ delta,
                  __bf16* __restrict__ dq, const Segs& segs, int total, int n_heads, float scale,
                  float scale_log2, int head, int seq, int tq) {
  using Cfg = Dq2Cfg<D>;
  constexpr int KS = D / 16;
  constexpr int DB = D / 32;
  constexpr int CPT = Cfg::kChunksPerThread;
  constexpr int RB = D * 2;
  constexpr int TB = Cfg::kTileBytes;
  constexpr int SB = Cfg::kStageBytes;
  constexpr int NG = 2 * KS + 2 * DB;   // MFMAs (groups) per half-step
  static_assert(D == 128, "tuned for head_dim 128");

  extern __shared__ __attribute__((aligned(16))) char smem[];

  const int q_b = segs.q_start(seq) + segs.q_len(seq);
  const int q0 = segs.q_start(seq) + tq * Cfg::kBR;
  const int seg_a = segs.kv_start(seq);
  const int seg_b = seg_a + segs.kv_len(seq);

  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  const int lane = tid & 63;
  const int c = lane & 31;
  const int g = lane >> 5;
  const size_t row_stride = (size_t)n_heads * D;
  const size_t head_off = (size_t)head * D;
  const __bf16* kbase = k + head_off;
  const __bf16* vbase = v + head_off;

  // ---- K/V staging with direct global->LDS loads; tiles are requested in sequence
  const uint32_t row_bytes = (uint32_t)row_stride * 2u;
  const uint32_t last_row_off = (uint32_t)(seg_b - 1) * row_bytes;
  uint32_t st_rowoff[CPT], st_colb[CPT];
#pragma unroll
  for (int x = 0; x < CPT; ++x) {
    const int p = (x * kDq2Waves + wave) * 64 + lane;
    const int r = p / Cfg::kChunksPerRow;
    st_rowoff[x] = (uint32_t)(seg_a + r) * row_bytes;
    st_colb[x] = (uint32_t)(((p % Cfg::kChunksPerRow) ^ swz<D>(r)) * 16);
  }
  const uint32_t smem_addr = lds_addr_of(smem);
  const uint32_t wave_lds = __builtin_amdgcn_readfirstlane(smem_addr + wave * 1024);
  auto issue_tile = [&](int stage) {
#pragma unroll
    for (int x = 0; x < CPT; ++x) {
      const uint32_t off = min(st_rowoff[x], last_row_off) + st_colb[x];
      const uint32_t dst = wave_lds + stage * SB + x * kDq2Waves * 1024;
      lds_dma16(kbase, off, dst);
      lds_dma16(vbase, off, dst + TB);
      st_rowoff[x] += kDqBC * row_bytes;
    }
  };

  // ---- swizzled LDS addresses, one register each (opaque, so they are kept, not recomputed)
  // (a second set for the third stage, which lies beyond the 64 KB an immediate offset
  // reaches: without it every read of that stage costs a v_add_u32, 16 per key block)
  uint32_t rb[KS], tb[2][DB], rb2[KS], tb2[2][DB];
  {
    const int rbase = tile_off<D>(c, 8 * g);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      rb[ks] = smem_addr + (rbase ^ (ks << 5));
      rb2[ks] = rb[ks] + 2 * SB;
      asm volatile("" : "+v"(rb[ks]), "+v"(rb2[ks]));
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int tbase = tile_off<D>(8 * t + 4 * g + ((lane & 15) >> 2), 16 * ((lane >> 4) & 1) + 4 * (lane & 3));
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        tb[t][db] = smem_addr + (tbase ^ (db << 6));
        tb2[t][db] = tb[t][db] + 2 * SB;
        asm volatile("" : "+v"(tb[t][db]), "+v"(tb2[t][db]));
      }
    }
  }

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 dqacc[2][DB];
#pragma unroll
  for (int ib = 0; ib < 2; ++ib)
#pragma unroll
    for (int db = 0; db < DB; ++db) dqacc[ib][db] = zero16;

  const int n_tiles = (seg_b - seg_a + kDqBC - 1) / kDqBC;
  const int n_blocks = 2 * n_tiles;
  const int tail_rows = seg_b - seg_a - (n_tiles - 1) * kDqBC;   // valid rows of the last tile

  // A wavefront whose 64 query rows all lie past the end of the sequence (ragged last tile)
  // has nothing to compute.  It still fetches its share of every K/V tile, takes part in
  // zeroing the last tile's tail rows and meets every barrier, in the order of the loop
  // below: the prologue's requests, wait and barrier; from the second tile on the wait, the
  // barrier, the request; the two barriers
  // around the zeroing; the epilogue's wait and barrier.
  if (q0 + wave * 64 >= q_b) {
    issue_tile(0);
    wait_vmcnt<0>();
    __syncthreads();
    issue_tile(1);
    for (int t = 1; t < n_tiles; ++t) {
      wait_vmcnt<0>();
      __syncthreads();
      if (t + 1 < n_tiles) issue_tile((t + 1) % kDq2Ring);
    }
    if (tail_rows < kDqBC) {
      __syncthreads();
      const u32x4 z = {0u, 0u, 0u, 0u};
      const int n16 = (kDqBC - tail_rows) * (RB / 16);
      for (int i = tid; i < n16; i += kDq2Waves * 64)
        *reinterpret_cast<__attribute__((address_space(3))) u32x4*>(
            smem_addr + ((n_tiles - 1) % kDq2Ring) * SB + tail_rows * RB + i * 16) = z;
      __syncthreads();
    }
    wait_vmcnt<0>();
    __syncthreads();
    return;
  }

  // ---- this wavefront's Q and dO rows as B operands (AGPRs); lse, Delta per lane.  The rows come through LDS
  // (direct loads of whole rows, four per instruction, chunk order as in a tile): loaded into registers
  // as operands, 32 bytes of each of 32 rows per instruction, a workgroup of 512 keys spent a third of its life on
  // them.  `out` comes in rows too.  (Backward call: 56,320 queries x 512 keys x 32 heads 1,781 -> 1,722 us, 8 x 1,000
  // tokens x 8 heads 126 -> 123, 300 x 4 19.8 -> 18.4; level from 4,096 tokens on.)
  const uint32_t own = smem_addr + Cfg::kOwnBase + wave * Cfg::kOwnBytes;   // Q rows, then dO rows
  const int row_w = q0 + wave * 64;
  {
    const __bf16* qbase = q + head_off;
    const __bf16* dobase = dout + head_off;
    const uint32_t own_s = __builtin_amdgcn_readfirstlane(own);
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      const int r = x * 4 + (lane >> 4);
      const uint32_t off = (uint32_t)min(row_w + r, q_b - 1) * row_bytes + (uint32_t)(((lane & 15) ^ swz<D>(r)) * 16);
      lds_dma16(qbase, off, own_s + x * 1024);
      lds_dma16(dobase, off, own_s + 64 * RB + x * 1024);
    }
  }
  issue_tile(0);
  bf16x8 qreg[2][KS], doreg[2][KS];
  float lse2[2], dlt[2];
  int qrow[2];
  size_t stat[2];
#pragma unroll
  for (int ib = 0; ib < 2; ++ib) {
    qrow[ib] = row_w + ib * 32 + c;
    stat[ib] = (size_t)head * total + min(qrow[ib], q_b - 1);
  }
  auto read_own = [&]() {
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const uint32_t a = own + (tile_off<D>(c, 8 * g) ^ (ks << 5)) + ib * 32 * RB;
        qreg[ib][ks] = lds_read_b128_at(a);
        doreg[ib][ks] = lds_read_b128_at(a + 64 * RB);
        to_agpr(qreg[ib][ks]);
        to_agpr(doreg[ib][ks]);
      }
  };
  if constexpr (STATS) {
    bf16x8 orow[16];
#pragma unroll
    for (int x = 0; x < 16; ++x)
      orow[x] = *reinterpret_cast<const bf16x8*>(out + (size_t)min(row_w + x * 4 + (lane >> 4), q_b - 1) * row_stride +
                                                 head_off + (lane & 15) * 8);
#pragma unroll
    for (int ib = 0; ib < 2; ++ib) lse2[ib] = lse[stat[ib]] * kLog2eB;
    wait_vmcnt<0>();
    // the order of bwd_prepare_kernel's sums (chunks of 8 columns, then pairs of chunks 8, 4, 2, 1 apart; the
    // one-pass kernel's too), so that a clip's gradients do not depend, to the bit, on what else is in
    // the pack.  (Rotations by 8, 4, 2, 1 within a row's 16 lanes: after each the sums repeat with that period.)
    float s[16];
#pragma unroll
    for (int x = 0; x < 16; ++x) {
      const bf16x8 d = lds_read_b128_at(own + 64 * RB + tile_off<D>(x * 4 + (lane >> 4), (lane & 15) * 8));
      s[x] = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) s[x] = __builtin_fmaf((float)orow[x][e], (float)d[e], s[x]);
      s[x] = row16_sum(s[x]);
    }
    read_own();
    asm volatile("" ::: "memory");   // (the sums take the place of rows read above)
    if ((lane & 15) == 0)
#pragma unroll
      for (int x = 0; x < 16; ++x)
        *reinterpret_cast<__attribute__((address_space(3))) float*>(own + (x * 4 + (lane >> 4)) * 4) = s[x];
    const bool few = segs.kv_len(seq) <= kShortKeys;
#pragma unroll
    for (int ib = 0; ib < 2; ++ib) {
      dlt[ib] = *reinterpret_cast<const __attribute__((address_space(3))) float*>(own + (ib * 32 + c) * 4);
      if (few) dlt[ib] = delta[stat[ib]];
      if (g == 0 && qrow[ib] < q_b) {
        lse2g[stat[ib]] = lse2[ib];
        if (!few) delta[stat[ib]] = dlt[ib];
      }
    }
  } else {
#pragma unroll
    for (int ib = 0; ib < 2; ++ib) { lse2[ib] = lse2g[stat[ib]]; dlt[ib] = delta[stat[ib]]; }
    wait_vmcnt<0>();
    read_own();
  }
#pragma unroll
  for (int ib = 0; ib < 2; ++ib) asm volatile("" :: "v"(lse2[ib]), "v"(dlt[ib]));
  __syncthreads();            // tile 0 has landed, everyone has its rows
  issue_tile(1);              // (re-requests the last rows when the clip has a single tile)

  // ---- state carried between half-steps
  f32x16 sacc[2], dpacc[2];   // S^T, dP^T of the current key block, per query block
  f32x16 dsf;                 // dS^T of the half-step at hand, fp32
  u32x8 pw[2];                // dS^T as bf16 pairs, per query block: B operands of the update
  bf16x8 ka[KS], va[KS];      // row operands of the key block whose scores come next
  s16x4 klo[2][DB], khi[2][DB];   // K^T operands of the key block whose update comes next
#pragma unroll
  for (int i = 0; i < 8; ++i) { pw[0][i] = 0u; pw[1][i] = 0u; }
#pragma unroll
  for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
    for (int db = 0; db < DB; ++db) { klo[s2][db] = s16x4{0, 0, 0, 0}; khi[s2][db] = s16x4{0, 0, 0, 0}; }
  dsf = zero16;

  // prologue: row operands of key block 0, S^T and dP^T of (key block 0, query block 0)
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    ka[ks] = lds_read_b128_at(rb[ks]);
    va[ks] = lds_read_b128_at(rb[ks] + TB);
  }
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    mfma32_v(sacc[0], ka[ks], qreg[0][ks], ks == 0);
    mfma32_v(dpacc[0], va[ks], doreg[0][ks], ks == 0);
  }
  sacc[1] = zero16;
  dpacc[1] = zero16;

  // One half-step.  POSB = b % 6 fixes every LDS stage at compile time; IB is the query block
  // whose dS^T the VALU forms.
  auto half_step = [&](auto posb_c, auto ib_c, int b) {
    constexpr int POSB = decltype(posb_c)::value;
    constexpr int IB = decltype(ib_c)::value;
    constexpr int OB = 1 - IB;                               // the block the matrix pipe works for
    constexpr int ST_CUR = (POSB / 2) % kDq2Ring;            // stage of key block b
    constexpr int ST_NEXT = ((POSB + 1) / 2) % kDq2Ring;     // stage of key block b+1
    constexpr int JB_CUR = POSB & 1, JB_NEXT = (POSB + 1) & 1;
    const float lse_i = lse2[IB];
    // Delta is made a new value here: the subtractions dP - Delta then cannot be moved up into the
    // previous half-step, where the MFMAs that produce dP are still running (dP itself is not
    // passed through the statements)
    float dlt_i = dlt[IB];
    asm volatile("" : "+v"(dlt_i));
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
      // ---- matrix pipe
      if (gi < 2 * KS) {
        const int ks = gi >> 1;
        if ((gi & 1) == 0) mfma32_v(sacc[OB], ka[ks], qreg[OB][ks], ks == 0, sacc[IB], dsf, pw[IB]);
        else mfma32_v(dpacc[OB], va[ks], doreg[OB][ks], ks == 0, sacc[IB], dsf, pw[IB]);
      } else {
        const int s2 = (gi - 2 * KS) / DB, db = (gi - 2 * KS) % DB;
        const u32x4 w = {pw[OB][4 * s2], pw[OB][4 * s2 + 1], pw[OB][4 * s2 + 2], pw[OB][4 * s2 + 3]};
        mfma32_acc(dqacc[OB][db], join_tr(klo[s2][db], khi[s2][db]), __builtin_bit_cast(bf16x8, w),
                   sacc[IB], dsf, pw[IB]);
      }
      // ---- LDS reads
      if (IB == 0) {
        // row operands of key block b+1, once the score MFMAs have consumed those of block b
        if (gi >= 2 * KS) {
          constexpr int per = (2 * KS) / (2 * DB);   // reads per group: 16 / 8
#pragma unroll
          for (int x = (gi - 2 * KS) * per; x < (gi - 2 * KS + 1) * per; ++x) {
            const int ks = x >> 1;
            const uint32_t a = (ST_NEXT == 2 ? rb2[ks] : rb[ks] + ST_NEXT * SB) + JB_NEXT * 32 * RB;
            if ((x & 1) == 0) ka[ks] = lds_read_b128_at(a); else va[ks] = lds_read_b128_at(a + TB);
          }
        }
      } else {
        // K^T operands of key block b (the updates of block b-1 were all issued a half-step ago)
        if (gi < 2 * DB) {
#pragma unroll
          for (int x = 2 * gi; x < 2 * gi + 2; ++x) {
            const int s2 = x / (2 * DB), db = (x >> 1) % DB, hi = x & 1;
            const uint32_t a = (ST_CUR == 2 ? tb2[hi][db] : tb[hi][db] + ST_CUR * SB) + (JB_CUR * 32 + 16 * s2) * RB;
            if (hi) khi[s2][db] = lds_read_tr_at(a); else klo[s2][db] = lds_read_tr_at(a);
          }
        }
      }
      // ---- VALU: one element of dS^T per group (keys i = 8*(e/4) + 4g + e%4 of the block, this
      // lane's query row): the exponential in group G(e), the product one group later (no
      // stall on the transcendental's result), the conversion of a pair one group after that
#pragma unroll
      for (int e = 1; e < 16; e += 2)
        if (1 + e * (NG - 2) / 16 + 2 == gi) {
          const f32x2 pr = {dsf[e - 1], dsf[e]};
          pw[IB][e >> 1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(pr, bf16x2));
        }
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (1 + e * (NG - 2) / 16 + 1 == gi) dsf[e] = dsf[e] * (dpacc[IB][e] - dlt_i);
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (1 + e * (NG - 2) / 16 == gi) dsf[e] = fast_exp2(sacc[IB][e] * scale_log2 - lse_i);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto block = [&](auto posb_c, int b) {
    constexpr int POSB = decltype(posb_c)::value;
    if constexpr ((POSB & 1) == 1) {
      // key block 2t-1: tile t has landed for every wave, every wave is done with tile t-2,
      // whose stage takes tile t+1
      const int t = (b + 1) >> 1;
      if (t < n_tiles) {
        wait_vmcnt<0>();
        __syncthreads();
        if (t + 1 < n_tiles) issue_tile(((POSB + 1) / 2 + 1) % kDq2Ring);
      }
    }
    half_step(posb_c, IntC<0>{}, b);
    if constexpr ((POSB & 1) == 0) {
      // Keys past the clip's end (last tile only).  Their K, V rows were fetched as copies of
      // the last valid row, so their S^T, dP^T are finite and so is dS^T; what keeps them out
      // of dQ is a zero K^T column.  All row reads of this tile have been issued by now and
      // its first K^T read follows: zero those K rows in LDS in between.
      if (b == n_blocks - 2 && tail_rows < kDqBC) {
        __syncthreads();
        const u32x4 z = {0u, 0u, 0u, 0u};
        const int n16 = (kDqBC - tail_rows) * (RB / 16);
        for (int i = tid; i < n16; i += kDq2Waves * 64)
          *reinterpret_cast<__attribute__((address_space(3))) u32x4*>(
              smem_addr + ((POSB / 2) % kDq2Ring) * SB + tail_rows * RB + i * 16) = z;
        __syncthreads();
      }
    }
    half_step(posb_c, IntC<1>{}, b);
  };
  for (int b = 0; b < n_blocks; b += 6) {
    block(IntC<0>{}, b);
    block(IntC<1>{}, b + 1);
    if (b + 2 < n_blocks) { block(IntC<2>{}, b + 2); block(IntC<3>{}, b + 3); }
    if (b + 4 < n_blocks) { block(IntC<4>{}, b + 4); block(IntC<5>{}, b + 5); }
  }
  // drain: the last key block's update for query block 1
#pragma unroll
  for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      const u32x4 w = {pw[1][4 * s2], pw[1][4 * s2 + 1], pw[1][4 * s2 + 2], pw[1][4 * s2 + 3]};
      mfma32_acc(dqacc[1][db], join_tr(klo[s2][db], khi[s2][db]), __builtin_bit_cast(bf16x8, w));
    }
  wait_vmcnt<0>();   // no load may still be writing LDS when the workgroup ends
  // the accumulators were written by assembly: wait out the last MFMA before they are read
#pragma unroll
  for (int ib = 0; ib < 2; ++ib) wait_mfma_a(dqacc[ib][0], dqacc[ib][1], dqacc[ib][2], dqacc[ib][3]);

  // ---- epilogue: dq = bf16(scale * dQ^T), whole rows per store
  __syncthreads();   // the ring is free: each wavefront turns its tiles through a piece of it
#pragma unroll
  for (int ib = 0; ib < 2; ++ib) {
    const int row0 = q0 + (wave * 2 + ib) * 32;
    store_tile_rows<D>(smem + wave * (32 * D * 2), dqacc[ib], scale,
                       dq + (size_t)row0 * row_stride + head_off, row_stride, q_b - row0);
  }
}

template <int D, class Segs, bool STATS>
__global__ __launch_bounds__(kDq2Waves * 64, 1)
void attn_bwd_dq2_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k,
                         const __bf16* __restrict__ v, const __bf16* __restrict__ dout,
                         const __bf16* __restrict__ out, const float* __restrict__ lse,
                         float* __restrict__ lse2g, float* __restrict__ delta, float* __restrict__ sentinel,
                         __bf16* __restrict__ dq, const Segs segs, const UnitMap um, const TileIndex ti,
                         int total, int n_heads, float scale, float scale_log2) {
  int head, tile;
  if (!map_unit(um, blockIdx.x, head, tile)) return;
  if (STATS && blockIdx.x == 0 && threadIdx.x == 0) {   // the dK/dV pass' statistics of rows past a clip's end
    sentinel[0] = INFINITY;
    sentinel[1] = 0.f;
  }
  int seq, tq;
  locate_tile(ti, segs.n, tile, seq, tq);
  bwd_dq2_unit<D, Segs, STATS>(q, k, v, dout, out, lse, lse2g, delta, dq, segs, total, n_heads, scale, scale_log2,
                               head, seq, tq);
}

// ---------------------------------------------------------------- short sequences: one launch
// For sequences of a few hundred tokens the two passes above are bound by the memory path, not
// by the matrix pipe: each reads q, k, v, dout of a (sequence, head) once, a millisecond apart,
// so the second pass finds nothing of it in L2.  This kernel runs the same two units from one
// grid: per (head, sequence) the key tiles' dK/dV units, then the query tiles' dQ units, as
// consecutive workgroups of one XCD, so that they run side by side and share the lines they
// fetch.  ti counts both kinds of tile per sequence (key tiles first).
template <int D, class Segs>
__global__ __launch_bounds__(kBwdWaves * 64, 1)
void attn_bwd_both_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k,
                          const __bf16* __restrict__ v, const __bf16* __restrict__ dout,
                          float* __restrict__ lse2, float* __restrict__ delta,
                          const float* __restrict__ sentinel, __bf16* __restrict__ dq,
                          __bf16* __restrict__ dk, __bf16* __restrict__ dv,
                          const Segs segs, const UnitMap um, const TileIndex ti,
                          int total, int n_heads, float scale, float scale_log2) {
  static_assert(kBwdWaves == kDq2Waves, "one workgroup shape for both units");
  int head, tile;
  if (!map_unit(um, blockIdx.x, head, tile)) return;
  int seq, t;
  locate_tile(ti, segs.n, tile, seq, t);
  const int key_tiles = (segs.kv_len(seq) + kBwdBC - 1) / kBwdBC;
  if (t < key_tiles)
    bwd_dkdv_unit<D, Segs, false>(q, k, v, dout, lse2, delta, sentinel, dk, dv, segs, total, n_heads, scale,
                                  scale_log2, nullptr, 0, 1, head, seq, t, 0);
  else
    bwd_dq2_unit<D, Segs, false>(q, k, v, dout, nullptr, nullptr, lse2, delta, dq, segs, total, n_heads, scale,
                                 scale_log2, head, seq, t - key_tiles);
}

// ---------------------------------------------------------------- sequences of up to 256 tokens: one pass
// Self-attention over clips of at most kOnePassMaxRows tokens: one workgroup owns a whole (clip, head), so
// that the five products of the backward are formed once (the two passes above form seven), every
// operand comes from memory once and Delta needs no pass of its own.  What bounds such packs is the
// memory path (eight tensors of the clip against 10 D flops per pair of few pairs).
//   prologue: K into LDS, V rows into registers, lse in log2 units of all rows into LDS; Delta likewise
//             (out and dO straight from memory; dO is read again below while it is in L2), but at head_dim 128
//             with eight wavefronts, where no other workgroup's products hide those loads: there out rides in
//             the ring and Delta(b+1) is formed in phase 2 of block b, behind a barrier that block b+1 has landed
//             before (288 clips of 256 tokens x 32 heads: backward call 1,418 -> 1,368 us, 300 of 130 x 16 442 -> 419).
//             Eight wavefronts have a CU to themselves at head_dim 64 too; there the barrier that would publish the
//             block is the one that the second dS removes (below), and Delta by blocks has not been tried
//   per block b of 32 query rows (Q, dO in a ring of three LDS stages, requested two blocks ahead; two stages where that lets two
//   workgroups share a CU):
//     phase 1  dQ(b-1) = dS(b-1) K, every wavefront 32 columns over all keys, to memory;
//              S(b) = Q K^T, dP(b) = dO V^T, P, dS of the wavefront's own 32 keys
//     barrier
//     phase 2  dS(b) to LDS, key-major; dV^T += dO^T P, dK^T += Q^T dS
//     barrier
// dS is written in phase 2 and read in phase 1 only, so it needs no second copy.  At head_dim 64 there is room for one,
// and with it the barrier between the phases goes (288 clips of 256 tokens x 32 heads 850 -> 810 us); at 128 it gave
// 1% with eight wavefronts and does not fit two workgroups with four.  Keys past the clip's end
// have dS = 0; query rows past it P = 0 (lse = +inf).  Four wavefronts serve 128 tokens in 73 KB of LDS (57 at
// head_dim 64), so that two workgroups share a CU and one's loads and stores meet the other's products;
// eight serve 256 tokens, one workgroup per CU (154 KB; 90 KB at head_dim 64, where 174 registers allow two wavefronts
// per SIMD, which is this one workgroup).  Everything the loop could recompute it does
// (opaque offsets): one spilled register tuple read back in the loop waits for the loads in flight.
// Whole backward call, statistics included, 256 clips x 32 heads, two-pass kernels -> this one:
// 256 tokens 1,558 -> 1,203 us (3.6 TB/s of the eight tensors), 128 tokens 810 -> 439, 64 tokens 528 -> 223,
// 16 tokens 448 -> 128; head_dim 64, 256 tokens 769 -> 721, 128 tokens 340 -> 228, 64 tokens 195 -> 138.
template <int D, int NW>
struct FusedCfg {
  static constexpr int kRows = NW * 32;                      // longest clip
  static constexpr int kBlockBytes = 32 * D * 2;             // 32 rows of one tensor
  static constexpr int kRing = D == 128 && NW == 4 ? 2 : 3;  // stages of (Q, dO) blocks
  // out rides in the ring beside Q and dO, and Delta is formed block by block
  static constexpr bool kStreamOut = D == 128 && NW == 8;
  static constexpr int kStageTensors = kStreamOut ? 3 : 2;
  static constexpr int kStageBytes = kStageTensors * kBlockBytes;
  static constexpr int kRingBase = kRows * D * 2;            // K first
  static constexpr int kDsBase = kRingBase + kRing * kStageBytes;
  static constexpr int kDsBufs = D == 128 ? 1 : 2;
  static_assert(!kStreamOut || (kDsBufs == 1 && kRing == 3), "the barrier between the phases publishes the next block");
  static constexpr int kStatBase = kDsBase + kDsBufs * kRows * 64;     // dS: [key][32 queries] bf16; then lse2, Delta
  static constexpr int kLdsBytes = kStatBase + 2 * kRows * 4;
  static constexpr int kLoads = kStageBytes / 1024 / NW;     // wave loads per block (all tensors of a stage)
  // Neighbouring (clip, head) units per XCD: one at head_dim 128 (256 bytes of a row each; groups of 8 take 3%
  // longer), 8 at head_dim 64 (1 KB of a row; single units take 2 to 4% longer).
  static constexpr int kGroup = D == 128 ? 1 : 8;
};

template <int D, int NW>
__global__ __launch_bounds__(NW * 64, 2)
void attn_bwd_fused_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ k,
                           const __bf16* __restrict__ v, const __bf16* __restrict__ out,
                           const float* __restrict__ lse, const __bf16* __restrict__ dout,
                           __bf16* __restrict__ dq, __bf16* __restrict__ dk, __bf16* __restrict__ dv,
                           const SegTable segs, int total, int n_heads, float scale, float scale_log2) {
  using Cfg = FusedCfg<D, NW>;
  constexpr int KS = D / 16, DB = D / 32, CPR = D / 8, RB = D * 2;
  constexpr int BB = Cfg::kBlockBytes;
  constexpr int NT = NW * 64;

  extern __shared__ __attribute__((aligned(16))) char smem[];

  // units run over the heads of a clip first, clips longest first
  const int unit = dealt_unit(blockIdx.x, Cfg::kGroup);
  if (unit >= segs.n * n_heads) return;
  const int seq = unit / n_heads, head = unit - seq * n_heads;
  const int a = segs.start[seq], n = segs.len[seq];
  const int n_blk = (n + 31) / 32;

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, c = lane & 31, g = lane >> 5;
  const size_t row_stride = (size_t)n_heads * D;
  const size_t clip_off = (size_t)a * row_stride + (size_t)head * D;
  const uint32_t row_bytes = (uint32_t)row_stride * 2u;
  const uint32_t smem_addr = lds_addr_of(smem);

  // ---- K rows to LDS (rows past the end: copies of the last one; blocks without a row are left out)
  const __bf16* kbase = k + clip_off;
#pragma unroll
  for (int x = 0; x < CPR / 2; ++x) {
    const int p = (x * NW + wave) * 64 + lane;
    const int r = p / CPR;
    if ((x * NW + wave) * 64 / CPR < n_blk * 32)
      lds_dma16(kbase, (uint32_t)min(r, n - 1) * row_bytes + (uint32_t)(((p % CPR) ^ swz<D>(r)) * 16),
                __builtin_amdgcn_readfirstlane(smem_addr + (x * NW + wave) * 1024));
  }

  // ---- blocks of Q and dO: wave instruction i of a block fills 1 KB, the first half of them Q
  const int jrow = wave * 32 + c;                 // this lane's key, relative to the clip
  const bool active = wave * 32 < n;              // (wave-uniform) some key of the wavefront exists
  const __bf16* src[Cfg::kLoads];
  uint32_t st_colb[Cfg::kLoads], st_lds[Cfg::kLoads];
  int st_row[Cfg::kLoads];
#pragma unroll
  for (int x = 0; x < Cfg::kLoads; ++x) {
    const int i = x * NW + wave;
    const int p = (i % (CPR / 2)) * 64 + lane;
    const int r = p / CPR;
    src[x] = uniform_ptr((i < CPR / 2 ? q : i < CPR ? dout : out) + clip_off);
    st_row[x] = r;
    st_colb[x] = (uint32_t)(((p % CPR) ^ swz<D>(r)) * 16);
    st_lds[x] = __builtin_amdgcn_readfirstlane(smem_addr + Cfg::kRingBase + i * 1024);
  }
  auto issue_block = [&](int stage) {   // strictly in order; blocks past the end re-read the last row
#pragma unroll
    for (int x = 0; x < Cfg::kLoads; ++x) {
      lds_dma16(src[x], (uint32_t)min(st_row[x], n - 1) * row_bytes + st_colb[x], st_lds[x] + stage * Cfg::kStageBytes);
      st_row[x] += 32;
    }
  };
  issue_block(0);
  issue_block(1);

  // ---- V rows as B operand
  bf16x8 vreg[KS];
  {
    const __bf16* vp = v + clip_off + (size_t)min(jrow, n - 1) * row_stride + 8 * g;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) vreg[ks] = *reinterpret_cast<const bf16x8*>(vp + ks * 16);
  }
  // ---- statistics: CPR lanes per row
  float* lse_s = reinterpret_cast<float*>(smem + Cfg::kStatBase);
  float* delta_s = lse_s + Cfg::kRows;
  static_assert(Cfg::kRows <= NT, "one thread per row for lse");
  const float lse_r = lse[(size_t)head * total + a + min(tid, n - 1)];
  auto row_delta = [&](const u32x4& o8, const u32x4& d8) {   // this lane's 8 columns, then the row's CPR lanes
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s = __builtin_fmaf(__builtin_bit_cast(float, o8[e] << 16), __builtin_bit_cast(float, d8[e] << 16), s);
      s = __builtin_fmaf(__builtin_bit_cast(float, o8[e] & 0xffff0000u), __builtin_bit_cast(float, d8[e] & 0xffff0000u), s);
    }
#pragma unroll
    for (int o = CPR / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, CPR);
    return s;
  };
  // Delta of the rows of one block, out and dO from its ring stage (both swizzled alike)
  auto block_delta = [&](int blk, int stg) {
    static_assert(!Cfg::kStreamOut || NT == 32 * CPR, "one chunk per thread");
    int t = tid;
    asm volatile("" : "+v"(t));
    const char* dt = smem + Cfg::kRingBase + stg * Cfg::kStageBytes + BB + tile_off<D>(t / CPR, (t % CPR) * 8);
    const float s = row_delta(*reinterpret_cast<const u32x4*>(dt + BB), *reinterpret_cast<const u32x4*>(dt));
    const int r = blk * 32 + t / CPR;
    if (t % CPR == 0) delta_s[r] = r < n ? s : 0.f;
  };
  if constexpr (!Cfg::kStreamOut) {   // of all rows at once, all loads in flight before the first sum
    constexpr int RP = NT / CPR, PASSES = Cfg::kRows / RP;
    u32x4 oa[PASSES], da[PASSES];
    const int chunk = tid % CPR;
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {   // (rows past the end: copies of the last one, no branch between the loads)
      const size_t off = clip_off + (size_t)min(i * RP + tid / CPR, n - 1) * row_stride + chunk * 8;
      oa[i] = *reinterpret_cast<const u32x4*>(out + off);
      da[i] = *reinterpret_cast<const u32x4*>(dout + off);
    }
#pragma unroll
    for (int i = 0; i < PASSES; ++i) {
      const int r = i * RP + tid / CPR;
      const float s = row_delta(oa[i], da[i]);
      if (chunk == 0) delta_s[r] = r < n ? s : 0.f;
    }
  }
  if (tid < Cfg::kRows) lse_s[tid] = tid < n ? lse_r * kLog2eB : INFINITY;
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) settle(vreg[ks]);

  // ---- per-lane LDS offsets (see the dK/dV unit for the first two)
  const int rbase = tile_off<D>(c, 8 * g);
  int tbase[2];
#pragma unroll
  for (int t = 0; t < 2; ++t)
    tbase[t] = tile_off<D>(8 * t + 4 * g + ((lane & 15) >> 2), 16 * ((lane >> 4) & 1) + 4 * (lane & 3));
  const char* kt = smem + wave * 32 * RB;
  // dS rows are 64 bytes, 16-byte chunk x of key j kept at x ^ (j/4 mod 4)
  // dQ: 16x16x32 products over 32 keys.  This wavefront's part of the 32 x D block: 32 columns, and one or
  // both of the 16-row halves
  constexpr int NROW = D / 32 >= NW ? 2 : 1;
  const int col0 = (wave % (D / 32)) * 32, half0 = NROW == 2 ? 0 : wave / (D / 32);
  const bool dq_part = half0 < 2;                          // (head_dim 64 has two parts per half only)
  auto block_dq = [&](int blk, int rows_valid) {           // dQ of block blk, whose dS is in LDS -> memory
    const int ds_buf = Cfg::kDsBufs == 2 ? (blk & 1) * (Cfg::kRows * 64) : 0;
    f32x4 acc[2][NROW];
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
      for (int h = 0; h < NROW; ++h) acc[x][h] = f32x4{0.f, 0.f, 0.f, 0.f};
    // The instruction sums its 32 products in four groups of 8, one per lane group l/16, in that order;
    // the order within a group does not matter (measured: the same bits).  Lane group h takes keys
    // 16 (h/2) + 4 (h%2) + {0..3, 8..11}, which are the groups of the two-pass kernels' two 32x32x16 products, so
    // that dq is theirs to the bit.  Odd lane groups read the upper four first: rows read together then
    // differ in row/4 mod 4, which keeps them on different banks.
    int ln = lane;
    asm volatile("" : "+v"(ln));
    int ktr[2], dtr[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int odd = (ln >> 4) & 1;
      const int row = 16 * (ln >> 5) + 4 * odd + 8 * (t ^ odd) + ((ln & 15) >> 2);
      ktr[t] = tile_off<D>(row, col0 + 4 * (ln & 3));
      dtr[t] = Cfg::kDsBase + row * 64 + (((half0 * 2 + ((ln & 3) >> 1)) ^ ((row >> 2) & 3)) << 4) + (ln & 1) * 8;
    }
    // the next block's operands are read ahead of this block's products
    bf16x8 kf[2][2], df[2][NROW];
    auto read = [&](int kk, bf16x8 (&kr)[2], bf16x8 (&dr)[NROW]) {
      const char* kb = smem + kk * 32 * RB;
      const char* db = smem + ds_buf + kk * 32 * 64;
#pragma unroll
      for (int x = 0; x < 2; ++x)
        kr[x] = join_tr(lds_read_tr(kb, ktr[0] ^ (x * 32)), lds_read_tr(kb, ktr[1] ^ (x * 32)));
#pragma unroll
      for (int h = 0; h < NROW; ++h)
        dr[h] = join_tr(lds_read_tr(db, dtr[0] ^ (h * 32)), lds_read_tr(db, dtr[1] ^ (h * 32)));
    };
    auto mul = [&](bf16x8 (&kr)[2], bf16x8 (&dr)[NROW]) {
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int h = 0; h < NROW; ++h)
          acc[x][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kr[x], dr[h], acc[x][h], 0, 0, 0);
    };
    if constexpr (NROW == 2) {   // (no registers left for a second set; the CU's other workgroup fills the gaps)
      for (int kk = 0; kk < n_blk; ++kk) {
        read(kk, kf[0], df[0]);
        mul(kf[0], df[0]);
      }
    } else {
      read(0, kf[0], df[0]);
      for (int kk = 0; kk < n_blk; kk += 2) {
        if (kk + 1 < n_blk) read(kk + 1, kf[1], df[1]);
        mul(kf[0], df[0]);
        if (kk + 1 >= n_blk) break;
        if (kk + 2 < n_blk) read(kk + 2, kf[0], df[0]);
        mul(kf[1], df[1]);
      }
    }
    // a lane holds 4 columns of row l%16 in either 16-column product; exchanging 16-lane rows between the
    // two leaves it 8 columns of one, so that a store writes 64 contiguous bytes of each row
#pragma unroll
    for (int h = 0; h < NROW; ++h) {
      u32x2 w[2];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        f32x4 f;
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = acc[x][h][e] * scale;
        w[x] = __builtin_bit_cast(u32x2, to_bf16x4(f));
      }
      u32x4 o;
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        auto r = __builtin_amdgcn_permlane16_swap(w[0][e], w[1][e], false, false);
        o[e] = r[0];
        o[2 + e] = r[1];
      }
      const int row = (half0 + h) * 16 + (ln & 15), col = col0 + 16 * ((ln >> 4) & 1) + 8 * (ln >> 5);
      if (row < rows_valid)
        *reinterpret_cast<u32x4*>(dq + clip_off + (size_t)(blk * 32 + row) * row_stride + col) = o;
    }
  };

  const f32x16 zero16 = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  f32x16 dkacc[DB], dvacc[DB];
#pragma unroll
  for (int db = 0; db < DB; ++db) { dkacc[db] = zero16; dvacc[db] = zero16; }

  const uint32_t key_mask = jrow < n ? 0xffffffffu : 0u;
  // the two wavefronts of a SIMD run phase 1 in different orders, so that one's matrix
  // instructions meet the other's exponentials
  const bool late_dq = NW == 8 && wave >= 4;
  wait_vmcnt<0>();          // K, the first two blocks
  int stage = 0;            // b mod the ring's stages
  if constexpr (Cfg::kStreamOut) {
    __syncthreads();
    block_delta(0, 0);
  }
  for (int b = 0; b < n_blk; ++b) {
    // block b has landed (only block b+1's loads may be outstanding; dq stores only make the wait
    // stricter), everyone is done with block b-1, dS(b-1) is complete
    if constexpr (!Cfg::kStreamOut) wait_vmcnt<(Cfg::kRing - 2) * Cfg::kLoads>();
    __syncthreads();
    const char* qt = smem + Cfg::kRingBase + stage * Cfg::kStageBytes;
    if (Cfg::kRing == 3 || b > 0) issue_block(stage == 0 ? Cfg::kRing - 1 : stage - 1);
    stage = stage == Cfg::kRing - 1 ? 0 : stage + 1;
    if (b > 0 && !late_dq && dq_part) block_dq(b - 1, 32);
    bf16x8 pb[2], dsb[2];
    if (active) {
      // (offsets recomputed per block on purpose: held in registers they would push V out of them)
      int ro = rbase;
      asm volatile("" : "+v"(ro));
      f32x16 s = zero16, dp = zero16;
      bf16x8 qa[2], ka[2], da[2];
      auto rows = [&](int ks) {
        qa[ks & 1] = lds_read_b128(qt, ro ^ (ks << 5));
        ka[ks & 1] = lds_read_b128(kt, ro ^ (ks << 5));
        da[ks & 1] = lds_read_b128(qt + BB, ro ^ (ks << 5));
      };
      rows(0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        if (ks + 1 < KS) rows(ks + 1);
        s = mfma32(qa[ks & 1], ka[ks & 1], s);
        dp = mfma32(da[ks & 1], vreg[ks], dp);
        __builtin_amdgcn_sched_barrier(0);
      }
      f32x16 p, dl;
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const f32x4 l4 = *reinterpret_cast<const f32x4*>(lse_s + b * 32 + 8 * q4 + 4 * g);
        const f32x4 d4 = *reinterpret_cast<const f32x4*>(delta_s + b * 32 + 8 * q4 + 4 * g);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          p[q4 * 4 + e] = fast_exp2(s[q4 * 4 + e] * scale_log2 - l4[e]);
          dl[q4 * 4 + e] = d4[e];
        }
      }
      if (n <= kShortKeys) {   // few keys: Delta in its cancellation-free form, sum_j P_ij dP_ij (order: see there)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float x = jrow < n ? mul_alone(p[r], dp[r]) : 0.f;
#pragma unroll
          for (int o = 1; o < 32; o <<= 1) x += __shfl_xor(x, o, 32);
          dl[r] = x;
        }
      }
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2) {
        f32x8 pf, df;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          pf[e] = p[8 * s2 + e];
          df[e] = pf[e] * (dp[8 * s2 + e] - dl[8 * s2 + e]);
        }
        pb[s2] = to_bf16x8(pf);
        u32x4 w = __builtin_bit_cast(u32x4, to_bf16x8(df));   // keys past the end: zero
#pragma unroll
        for (int e = 0; e < 4; ++e) w[e] &= key_mask;
        dsb[s2] = __builtin_bit_cast(bf16x8, w);
      }
    }
    if (b > 0 && late_dq && dq_part) block_dq(b - 1, 32);
    if constexpr (Cfg::kStreamOut) wait_vmcnt<Cfg::kLoads>();   // block b+1 has landed
    if constexpr (Cfg::kDsBufs == 1) __syncthreads();   // everyone has read dS(b-1)
    if constexpr (Cfg::kStreamOut) {
      if (b + 1 < n_blk) block_delta(b + 1, stage);
    }
    if (active) {
      int j = jrow;
      asm volatile("" : "+v"(j));
      char* ds_w = smem + Cfg::kDsBase + (Cfg::kDsBufs == 2 ? (b & 1) * (Cfg::kRows * 64) : 0) + j * 64 + 8 * g;
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const bf16x8 d = dsb[q4 >> 1];
        const bf16x4 w = (q4 & 1) ? __builtin_shufflevector(d, d, 4, 5, 6, 7) : __builtin_shufflevector(d, d, 0, 1, 2, 3);
        *reinterpret_cast<bf16x4*>(ds_w + ((q4 ^ ((j >> 2) & 3)) << 4)) = w;
      }
      int t0 = tbase[0], t1 = tbase[1];
      asm volatile("" : "+v"(t0), "+v"(t1));
      s16x4 tr[2][4];
      auto cols = [&](int i) {
        const int o0 = (t0 ^ ((i % DB) << 6)) + 16 * (i / DB) * RB, o1 = (t1 ^ ((i % DB) << 6)) + 16 * (i / DB) * RB;
        tr[i & 1][0] = lds_read_tr(qt + BB, o0);
        tr[i & 1][1] = lds_read_tr(qt + BB, o1);
        tr[i & 1][2] = lds_read_tr(qt, o0);
        tr[i & 1][3] = lds_read_tr(qt, o1);
      };
      cols(0);
#pragma unroll
      for (int i = 0; i < 2 * DB; ++i) {
        if (i + 1 < 2 * DB) cols(i + 1);
        dvacc[i % DB] = mfma32(join_tr(tr[i & 1][0], tr[i & 1][1]), pb[i / DB], dvacc[i % DB]);
        dkacc[i % DB] = mfma32(join_tr(tr[i & 1][2], tr[i & 1][3]), dsb[i / DB], dkacc[i % DB]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  wait_vmcnt<0>();   // no load may still be writing LDS when the workgroup ends
  __syncthreads();
  if (dq_part) block_dq(n_blk - 1, n - (n_blk - 1) * 32);
  __syncthreads();
  // K is no longer needed: each wavefront turns its dK, dV tiles through its own rows of it
  if (active) {
    const int row0 = wave * 32;
    store_tile_rows<D>(smem + row0 * RB, dkacc, scale, dk + clip_off + (size_t)row0 * row_stride, row_stride, n - row0);
    store_tile_rows<D>(smem + row0 * RB, dvacc, 1.0f, dv + clip_off + (size_t)row0 * row_stride, row_stride, n - row0);
  }
}

template <int D, int NW>
static hipError_t launch_bwd_fused(const __bf16* q, const __bf16* k, const __bf16* v, const __bf16* out,
                                   const float* lse, const __bf16* dout, const SegTable& segs, int total,
                                   int n_heads, float scale, __bf16* dq, __bf16* dk, __bf16* dv, hipStream_t stream) {
  constexpr int lds = FusedCfg<D, NW>::kLdsBytes;
  static_assert(lds <= 160 * 1024, "LDS of one CU");
  auto kern = attn_bwd_fused_kernel<D, NW>;
  hipError_t e = allow_lds(kern, lds);
  if (e != hipSuccess) return e;
  return launch(kern, dim3(dealt_grid(segs.n * n_heads, FusedCfg<D, NW>::kGroup)), dim3(NW * 64), lds, stream, q, k, v,
                out, lse, dout, dq, dk, dv, segs, total, n_heads, scale, scale * kLog2eB);
}

int compute_unit_count() {
  static std::atomic<int> cached{0};
  int n = cached.load(std::memory_order_relaxed);
  if (n > 0) return n;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
    n = 256;
  cached.store(n, std::memory_order_relaxed);
  return n;
}

// Delta, lse in log2 units and the sentinels for the query tokens [tok0, tok_end) of a run.
static hipError_t launch_bwd_prepare(const void* out, const void* dout, const float* lse, float* delta, float* lse2,
                                     float* sentinel, int total, int n_heads, int head_dim, int tok0, int tok_end,
                                     hipStream_t stream) {
  const int tok_per_block = 256 / (head_dim / 8);
  const dim3 grid((tok_end - tok0 + tok_per_block - 1) / tok_per_block, (n_heads + kPrepHeads - 1) / kPrepHeads);
  auto kern = head_dim == 128 ? bwd_prepare_kernel<128> : bwd_prepare_kernel<64>;
  return launch(kern, grid, dim3(256), 0, stream, (const u32x4*)out, (const u32x4*)dout, lse, delta, lse2, sentinel,
                total, n_heads, tok0, tok_end);
}

template <int D, class Segs>
static hipError_t launch_bwd_d(const void* q, const void* k, const void* v, const void* out,
                               const float* lse, const void* dout, const Segs& segs, int total,
                               int n_heads, float scale, void* dq, void* dk, void* dv,
                               float* delta, float* lse2, float* sentinel, float* dkv32, int total_kv,
                               int kv_lo, int kv_hi, hipStream_t stream) {
  const __bf16 *qb = (const __bf16*)q, *kb = (const __bf16*)k, *vb = (const __bf16*)v, *dob = (const __bf16*)dout;
  hipError_t e;
  if constexpr (std::is_same_v<Segs, SegTable>) {
    if (segs.n == 0) return hipSuccess;
    if (bwd_one_pass(segs, n_heads, D, compute_unit_count())) {
      if (segs.len[0] <= 128)
        return launch_bwd_fused<D, 4>(qb, kb, vb, (const __bf16*)out, lse, dob, segs, total, n_heads, scale,
                                      (__bf16*)dq, (__bf16*)dk, (__bf16*)dv, stream);
      return launch_bwd_fused<D, 8>(qb, kb, vb, (const __bf16*)out, lse, dob, segs, total, n_heads, scale,
                                    (__bf16*)dq, (__bf16*)dk, (__bf16*)dv, stream);
    }
  }
  const TileIndex ti = make_tile_index<true>(segs, kBwdBC);
  const int tiles = count_tiles(ti);
  // Few key tiles and long query ranges (cross-attention): split the queries over workgroups.
  int q_split = 1;
  const RunSpan span = run_span(segs);
  const int cus = compute_unit_count();
  if (dkv32 && tiles > 0 && tiles * n_heads < cus)
    q_split = std::min(std::min(16, (cus + tiles * n_heads - 1) / (tiles * n_heads)), std::max(1, span.max_q / 512));
  const auto [both, dq_first] = bwd_order(D, q_split, span.longest, dq == q || dq == dout);
  if (span.max_q > 0) {   // (with no queries at all only the keys' zero gradients remain to be written)
    if (!dq_first) {
      e = launch_bwd_prepare(out, dout, lse, delta, lse2, sentinel, total, n_heads, D, span.tok0, span.tok_end, stream);
      if (e != hipSuccess) return e;
    }
    if (span.few_keys) {   // sequences with a handful of keys: Delta in its cancellation-free form
      const TileIndex ti_few = make_few_key_index(segs);
      e = launch(bwd_short_delta_kernel<D, Segs>, dim3(count_tiles(ti_few), n_heads), dim3(64), 0,
                 stream, qb, kb, vb, dob, lse, delta, segs, ti_few, total, n_heads, scale * kLog2eB);
      if (e != hipSuccess) return e;
    }
  }
  if (tiles == 0) return hipSuccess;
  auto launch_dq = [&](auto stats_c) -> hipError_t {
    constexpr bool STATS = decltype(stats_c)::value != 0;
    if constexpr (D == 128) {
      using Cfg = Dq2Cfg<D>;
      const TileIndex tq = make_tile_index<false>(segs, Cfg::kBR);
      const int n = count_tiles(tq);
      if (n == 0) return hipSuccess;
      const UnitMap uq = make_unit_map(segs, tq, Cfg::kBR, n_heads);
      auto kern = attn_bwd_dq2_kernel<D, Segs, STATS>;
      hipError_t err = allow_lds(kern, Cfg::kLdsBytes);
      if (err != hipSuccess) return err;
      return launch(kern, dim3(uq.chunk * kNumXcd), dim3(kDq2Waves * 64), Cfg::kLdsBytes, stream, qb, kb, vb, dob,
                    (const __bf16*)out, lse, lse2, delta, sentinel, (__bf16*)dq, segs, uq, tq, total, n_heads, scale,
                    scale * kLog2eB);
    } else {
      constexpr int NI = 1;
      constexpr int W = 4;   // 128 query rows, three workgroups per CU (see the kernel)
      using Cfg = DqCfg<D, NI, W>;
      const TileIndex tq = make_tile_index<false>(segs, Cfg::kBR);
      const int n = count_tiles(tq);
      if (n == 0) return hipSuccess;
      const UnitMap uq = make_unit_map(segs, tq, Cfg::kBR, n_heads);
      auto kern = attn_bwd_dq_kernel<D, NI, W, Segs, STATS>;
      hipError_t err = allow_lds(kern, Cfg::kLdsBytes);
      if (err != hipSuccess) return err;
      return launch(kern, dim3(uq.chunk * kNumXcd), dim3(W * 64), Cfg::kLdsBytes, stream, qb, kb, vb, dob,
                    (const __bf16*)out, lse, lse2, delta, sentinel, (__bf16*)dq, segs, uq, tq, total, n_heads, scale, scale * kLog2eB);
    }
  };
  if (dq_first) {
    e = launch_dq(IntC<1>{});
    if (e != hipSuccess) return e;
  }
  {
    using Cfg = BwdCfg<D>;
    if constexpr (D == 128) {
      if (both) {   // short sequences: both passes from one grid
        TileIndex tb;
        int n_both = 0;
        for (int s2 = 0; s2 <= VFM_MAX_SEQS; ++s2) {
          tb.cu[s2] = n_both;
          if (s2 < segs.n)
            n_both += (segs.kv_len(s2) + kBwdBC - 1) / kBwdBC + (segs.q_len(s2) + Dq2Cfg<D>::kBR - 1) / Dq2Cfg<D>::kBR;
        }
        const UnitMap um = make_unit_map(n_both, n_heads);
        constexpr int lds = Cfg::kLdsBytes > Dq2Cfg<D>::kLdsBytes ? Cfg::kLdsBytes : Dq2Cfg<D>::kLdsBytes;
        auto kern = attn_bwd_both_kernel<D, Segs>;
        e = allow_lds(kern, lds);
        if (e != hipSuccess) return e;
        return launch(kern, dim3(um.chunk * kNumXcd), dim3(kBwdWaves * 64), lds, stream, qb, kb, vb, dob, lse2,
                      delta, sentinel, (__bf16*)dq, (__bf16*)dk, (__bf16*)dv, segs, um, tb, total, n_heads, scale,
                      scale * kLog2eB);
      }
    }
    if (q_split > 1) {
      // the accumulators and the conversion cover this run's key rows [kv_lo, kv_hi) only:
      // other runs of the same call own the rest of dk, dv
      const size_t kv_elems = (size_t)total_kv * n_heads * D;
      const size_t lo4 = (size_t)kv_lo * n_heads * D / 4, h4 = (size_t)(kv_hi - kv_lo) * n_heads * D / 4;
      const dim3 cgrid((unsigned)((h4 + 255) / 256), 2);
      f32x4* acc_k = (f32x4*)dkv32 + lo4;
      f32x4* acc_v = (f32x4*)(dkv32 + kv_elems) + lo4;
      e = launch(fill_zero_f32x4_kernel, cgrid, dim3(256), 0, stream, acc_k, acc_v, h4);
      if (e != hipSuccess) return e;
      const UnitMap um = make_unit_map(tiles * q_split, n_heads);
      auto kern = attn_bwd_dkdv_kernel<D, Segs, true>;
      e = allow_lds(kern, Cfg::kLdsBytes);
      if (e != hipSuccess) return e;
      e = launch(kern, dim3(um.chunk * kNumXcd), dim3(kBwdWaves * 64), Cfg::kLdsBytes, stream, qb, kb, vb, dob,
                 lse2, delta, sentinel, (__bf16*)dk, (__bf16*)dv, segs, um, ti, total, n_heads, scale,
                 scale * kLog2eB, dkv32, kv_elems, q_split);
      if (e != hipSuccess) return e;
      e = launch(f32_to_bf16_kernel, cgrid, dim3(256), 0, stream, (const f32x4*)acc_k, (const f32x4*)acc_v,
                 (bf16x4*)dk + lo4, (bf16x4*)dv + lo4, h4);
      if (e != hipSuccess) return e;
    } else {
      const UnitMap um = make_unit_map(segs, ti, kBwdBC, n_heads);
      auto kern = attn_bwd_dkdv_kernel<D, Segs, false>;
      e = allow_lds(kern, Cfg::kLdsBytes);
      if (e != hipSuccess) return e;
      e = launch(kern, dim3(um.chunk * kNumXcd), dim3(kBwdWaves * 64), Cfg::kLdsBytes, stream, qb, kb, vb, dob,
                 lse2, delta, sentinel, (__bf16*)dk, (__bf16*)dv, segs, um, ti, total, n_heads, scale,
                 scale * kLog2eB, (float*)nullptr, (size_t)0, 1);
      if (e != hipSuccess) return e;
    }
  }
  if (dq_first) return hipSuccess;
  return launch_dq(IntC<0>{});
}

template <class Segs>
hipError_t launch_attn_bwd(const void* q, const void* k, const void* v, const void* out,
                           const float* lse, const void* dout, const Segs& segs, int total,
                           int n_heads, int head_dim, float scale, void* dq, void* dk, void* dv,
                           float* delta, float* lse2, float* sentinel, float* dkv32, int total_kv,
                           int kv_lo, int kv_hi, hipStream_t stream) {
  if (head_dim == 128)
    return launch_bwd_d<128>(q, k, v, out, lse, dout, segs, total, n_heads, scale, dq, dk, dv, delta, lse2, sentinel, dkv32, total_kv, kv_lo, kv_hi, stream);
  return launch_bwd_d<64>(q, k, v, out, lse, dout, segs, total, n_heads, scale, dq, dk, dv, delta, lse2, sentinel, dkv32, total_kv, kv_lo, kv_hi, stream);
}
template hipError_t launch_attn_bwd<SegTable>(const void*, const void*, const void*, const void*, const float*,
                                              const void*, const SegTable&, int, int, int, float, void*, void*,
                                              void*, float*, float*, float*, float*, int, int, int, hipStream_t);
template hipError_t launch_attn_bwd<XSegTable>(const void*, const void*, const void*, const void*, const float*,
                                               const void*, const XSegTable&, int, int, int, float, void*, void*,
                                               void*, float*, float*, float*, float*, int, int, int, hipStream_t);

}  // namespace vfm
