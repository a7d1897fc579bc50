// Shared device helpers and launcher declarations for libvfm (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <tuple>
#include <utility>

#include "../../include/vfm.h"

namespace vfm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// MI355X: 8 XCDs, workgroups are dealt to them round-robin.  A compile-time constant on purpose: it
// is part of the device-side block -> unit mapping (the HIP runtime exposes no XCD count to ask for),
// and the library is built for this one chip.
constexpr int kNumXcd = 8;

// Non-empty clips, longest first.  Passed to kernels by value (kernel argument
// memory), so no device allocation or copy is needed for the schedule.  Self-attention:
// a clip's queries and keys are the same token range.
struct SegTable {
  int n;
  int start[VFM_MAX_SEQS];
  int len[VFM_MAX_SEQS];
  __device__ __host__ int q_start(int s) const { return start[s]; }
  __device__ __host__ int q_len(int s) const { return len[s]; }
  __device__ __host__ int kv_start(int s) const { return start[s]; }
  __device__ __host__ int kv_len(int s) const { return len[s]; }
};

// Cross-attention: sequence s owns a query range of one packed tensor and a key/value
// range of another.  Same size in kernel-argument memory as SegTable.
struct XSegTable {
  int n;
  int qs[VFM_MAX_XSEQS], ql[VFM_MAX_XSEQS], ks[VFM_MAX_XSEQS], kl[VFM_MAX_XSEQS];
  __device__ __host__ int q_start(int s) const { return qs[s]; }
  __device__ __host__ int q_len(int s) const { return ql[s]; }
  __device__ __host__ int kv_start(int s) const { return ks[s]; }
  __device__ __host__ int kv_len(int s) const { return kl[s]; }
};

// Clip table for RoPE: all clips in packed order.
struct RopeTable {
  int n;
  int cu[VFM_MAX_SEQS + 1];
  int hw[VFM_MAX_SEQS];  // H*W of the clip's latent grid
  int w[VFM_MAX_SEQS];   // W
};

// FP8 attention: keys and values are packed in units of 64 keys that never straddle a clip.
// Packed-order table for the packing pass ...
struct Fp8ClipTable {
  int n;
  int cu[VFM_MAX_SEQS + 1];     // first packed token of clip s
  int unit0[VFM_MAX_SEQS + 1];  // units of the clips before s
};
// ... and the forward kernel's schedule (non-empty clips, longest first).  The FP8 entry points
// cut a call into runs of kFp8MaxSeqs clips: with three arrays per clip and the tile index beside
// it, a 256-clip table would not fit the 4 KB of kernel arguments.
constexpr int kFp8MaxSeqs = 128;
struct Fp8SegTable {
  int n;
  int start[kFp8MaxSeqs];
  int len[kFp8MaxSeqs];
  int unit0[kFp8MaxSeqs];       // first unit of the clip in the packed buffers
  __device__ __host__ int q_start(int s) const { return start[s]; }
  __device__ __host__ int q_len(int s) const { return len[s]; }
  __device__ __host__ int kv_start(int s) const { return start[s]; }
  __device__ __host__ int kv_len(int s) const { return len[s]; }
};

// Clip table for temporal attention: packed token and pixel offsets of every clip.
struct TemporalTable {
  int n;
  int cu[VFM_MAX_SEQS + 1];      // first packed token of clip s
  int pix_cu[VFM_MAX_SEQS + 1];  // pixels (H*W) of the clips before s
  int hw[VFM_MAX_SEQS];          // H*W of clip s (1 for an empty clip)
};

// A clip's frame count picks its kernels.  Class 0: up to 16 frames (one wavefront per sequence); classes 1
// to 4: up to 32, 64, 96, 128 frames (one workgroup per sequence, as many 32-row blocks as the class
// says); class 5: more (a wavefront per 32-row block).  A run is one launch per class that it holds.
// With the longest clip picking the kernels of the whole run, every single-frame pixel beside a
// 100-frame clip took a 512-thread workgroup and 129 KB of LDS (200 images of 32 x 32 beside 100
// frames of 8 x 8, 8 heads, head_dim 128, forward and backward: 53.3 ms, now 5.9), and 262,144
// pixels x 32 heads were more threads than one launch can have.
constexpr int kTemporalClasses = 6;
inline int temporal_class(int frames) { return frames <= 16 ? 0 : frames <= 128 ? (frames + 31) / 32 : 5; }
inline int temporal_frames(const TemporalTable& tab, int s) { return (tab.cu[s + 1] - tab.cu[s]) / tab.hw[s]; }

// Another launch costs a call forward and backward 5 to 8 us, so a class of few sequences joins the next
// longer class of the run.  Up to class 4: no more of them than twice the workgroups of that class'
// backward that fit the chip's LDS at once, four times where the classes are neighbours and their kernels
// differ least.  The line lies where joined is still level (head_dim 128, forward and backward, joined
// against apart: 2,048 sequences of 16 frames beside 32-frame ones 35 us against 34, 1,024 beside 64
// frames 32 against 33, 512 beside 96 frames 36 against 35; 2,048 of 32 beside 64 frames 57 against 61,
// 1,024 of 96 beside 128 frames 113 against 112; head_dim 64: 2,048 of 16 beside 64 frames 27 against
// 33, 2,048 of 96 beside 128 frames 90 against 98).  Class 5: no more than 1,024 32-row blocks (head_dim
// 128, beside 200 frames: 1,024 x 16 frames 124 against 126, 64 x 128 frames 115 against 133).
inline bool temporal_joins(int cls, int into, long long sequences, int head_dim, int cus) {
  if (into == 5) return sequences * (cls == 0 ? 1 : cls) <= 4LL * cus;
  const int chipful = 160 * 1024 / (into * (head_dim + 1) * 256) * cus;   // LDS of a backward workgroup: into * 32 rows
  return sequences <= (long long)chipful * (into == cls + 1 ? 4 : 2);
}

// The launch (named by its class) that the clips of every class take; -1: the run has none of the class.
struct TemporalPlan { int launch_of[kTemporalClasses]; };
inline TemporalPlan make_temporal_plan(const TemporalTable& tab, int n_heads, int head_dim, int cus) {
  TemporalPlan p;
  long long seqs[kTemporalClasses] = {};
  for (int s = 0; s < tab.n; ++s)
    if (tab.pix_cu[s + 1] > tab.pix_cu[s]) seqs[temporal_class(temporal_frames(tab, s))] += (long long)tab.hw[s] * n_heads;
  for (int c = 0; c < kTemporalClasses; ++c) p.launch_of[c] = seqs[c] > 0 ? c : -1;
  for (int c = 0; c < kTemporalClasses; ++c) {
    int into = c + 1;
    while (into < kTemporalClasses && seqs[into] == 0) ++into;
    if (seqs[c] == 0 || into == kTemporalClasses || !temporal_joins(c, into, seqs[c], head_dim, cus)) continue;
    seqs[into] += seqs[c];
    seqs[c] = 0;
    for (int x = 0; x <= c; ++x)
      if (p.launch_of[x] == c) p.launch_of[x] = into;
  }
  return p;
}

// The clips of one launch as a table of their own: the other clips keep their place and have no pixels.
inline TemporalTable temporal_launch_table(const TemporalTable& tab, const TemporalPlan& plan, int launch) {
  TemporalTable t = tab;
  int pix = 0;
  for (int s = 0; s <= VFM_MAX_SEQS; ++s) {
    t.pix_cu[s] = pix;
    if (s < tab.n && tab.pix_cu[s + 1] > tab.pix_cu[s] && plan.launch_of[temporal_class(temporal_frames(tab, s))] == launch)
      pix += tab.hw[s];
  }
  return t;
}

// Workgroups and threads of launches 0 to 4.  A tensor holds at most 2^25 (token, head) rows; a class 0
// sequence is at least one of them and takes 64 threads, a class c sequence at least 32 c - 31 (c = 1:
// 17) and 128 c threads in the backward: 2^31 threads at most (few more with the sequences that joined),
// where one launch can have 2^32 - 1.
struct TemporalGrid { unsigned blocks, threads; };
inline TemporalGrid temporal_grid(const TemporalTable& t, int launch, int n_heads, bool backward) {
  const long long units = (long long)t.pix_cu[t.n] * n_heads;
  if (launch == 0) return {(unsigned)((units + 3) / 4), 256u};                 // four sequences per workgroup
  return {(unsigned)units, (unsigned)(launch * (backward ? 128 : 64))};        // one wave per block (and role)
}

// The clips of launch 5: a work unit is one 32-row block of one (pixel, head) sequence.
struct TemporalLTable {
  int n;
  int cu[VFM_MAX_SEQS + 1];      // first packed token of clip s
  int blk_cu[VFM_MAX_SEQS + 1];  // (pixel, block) pairs of the clips before s: sum of H*W * ceil(T / 32)
  int hw[VFM_MAX_SEQS];          // H*W of clip s (1 for an empty clip)
};

// Work unit u = head * tiles_per_head + tile, units split into kNumXcd
// contiguous chunks so that one XCD (one L2) walks the tiles of one head
// together.  Returns false if this workgroup has nothing to do.
struct UnitMap {
  int tiles_per_head;
  int n_units;
  int chunk;  // ceil(n_units / kNumXcd)
  int dealt_heads;  // 0, or the number of heads: units are dealt out (below)
};

// The launch geometry of a kernel that takes one (head, tile) unit per workgroup: units are
// numbered head-major and cut into kNumXcd contiguous chunks; workgroup b belongs to XCD
// b % kNumXcd and takes unit (b % kNumXcd) * chunk + b / kNumXcd, so that the workgroups
// sharing an L2 walk neighbouring tiles of the same head.  Grid = chunk * kNumXcd.
//
// Dealt units: tile-major, u = tile * n_heads + head, workgroup b takes unit b: every XCD gets its share of every
// clip (see deal_units for when).
__host__ inline UnitMap make_unit_map(int tiles_per_head, int n_heads, bool dealt = false) {
  UnitMap um;
  um.tiles_per_head = tiles_per_head;
  um.n_units = tiles_per_head * n_heads;
  um.chunk = (um.n_units + kNumXcd - 1) / kNumXcd;
  um.dealt_heads = dealt ? n_heads : 0;
  return um;
}

__host__ __device__ __forceinline__ bool map_unit(const UnitMap& um, int block, int& head, int& tile) {
  if (um.dealt_heads) {
    if (block >= um.n_units) return false;
    tile = block / um.dealt_heads;
    head = block - tile * um.dealt_heads;
    return true;
  }
  const int xcd = block % kNumXcd;
  const int local = block / kNumXcd;
  const int u = xcd * um.chunk + local;
  if (local >= um.chunk || u >= um.n_units) return false;
  head = u / um.tiles_per_head;
  tile = u - head * um.tiles_per_head;
  return true;
}

// The other way to deal units: in order, round-robin over the XCDs in groups of `group` neighbours.  For units
// that share no operand but differ in length, longest first: a contiguous chunk per XCD would give one
// XCD all the long ones.  Grid = dealt_grid(); workgroups whose unit is >= units have none.
__host__ __device__ __forceinline__ int dealt_unit(int block, int group) {
  const int local = block / kNumXcd;
  return (local / group * kNumXcd + block % kNumXcd) * group + local % group;
}
inline int dealt_grid(int units, int group) { return (units + kNumXcd * group - 1) / (kNumXcd * group) * kNumXcd * group; }

// Tiles of the sequences before s (table order) for one launch's tile height, built on the host
// and passed by value beside the sequence table.  A workgroup finds its sequence by binary
// search in it: walking the table instead costs a dependent scalar load per sequence, which with
// 256 clips in a call took as long as a short clip's whole key loop.  Tiles are cut from the
// query ranges (KV = false) or from the key/value ranges (KV = true).
struct TileIndex {
  int cu[VFM_MAX_SEQS + 1];   // cu[s] = tiles of sequences 0..s-1; entries past the table repeat the total
};

template <bool KV, class Segs>
inline TileIndex make_tile_index(const Segs& segs, int rows_per_tile) {
  TileIndex ti;
  int tiles = 0;
  for (int s = 0; s <= VFM_MAX_SEQS; ++s) {
    ti.cu[s] = tiles;
    if (s < segs.n) tiles += ((KV ? segs.kv_len(s) : segs.q_len(s)) + rows_per_tile - 1) / rows_per_tile;
  }
  return ti;
}
inline int count_tiles(const TileIndex& ti) { return ti.cu[VFM_MAX_SEQS]; }

// Tile index (over the n sequences of the table, in table order) -> sequence s and tile t within
// it: the last s with cu[s] <= tile, which skips sequences that have no tile.
__host__ __device__ __forceinline__ void locate_tile(const TileIndex& ti, int n, int tile, int& s, int& t) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (ti.cu[mid] <= tile) lo = mid; else hi = mid;
  }
  s = lo;
  t = tile - ti.cu[lo];
}

// When a self-attention launch deals its units out (make_unit_map).  Where the heads do not divide by the XCDs a contiguous
// chunk holds pieces of heads, and with clips of unequal length (longest first) some XCDs get the long clips of such a
// head and others the short ones.  Dealt out, every XCD gets its share, but walks n_heads / gcd(n_heads, kNumXcd) heads
// at a time instead of one or two, which costs where there is nothing to even out (head_dim 128, contiguous -> dealt:
// 4,096 + 4,095 tokens, forward, 12 heads 213 -> 215 us, 13 219 -> 225, 33 586 -> 594; 8,192 + 8,190 + 8,100, 33 heads,
// backward 9.6 -> 10.1 ms).  So both orders are weighed here: their units are handed in order to the 32 CUs of an
// XCD, a unit taking its clip's length, a little less for a tile with few rows (a quarter of the time goes with them),
// and units are dealt where the contiguous order ends over 3% later.  Measured over 312 forward and backward calls (2 to
// 33 heads, 2 to 48 clips of 260 to 20,000 tokens, both head_dims), against contiguous throughout: 0.934 of the time in
// the geometric mean, at worst 1.04 (24 us) and then 1.02; dealing every unequal call 0.936, at worst 1.09.
// Gains: 12 heads, 5,000 + 1,200 + 700 + 300 tokens, forward 245 -> 176 us, backward 666 -> 533;
// 9,000 + 7,000 + 1,100 tokens 886 -> 730 and 2,616 -> 2,302; 4 x 1,500 + 8 x 300, 4 heads, backward 120 -> 91.
// Left contiguous: 4 x 1,500 + 8 x 300, 12 heads, forward 81 (dealt 89), 5,697 + 1,143, 12 heads, 281 (294).
// Up to one unit per CU the orders end together.  Beyond kDealWeighed units per CU a launch ends when its
// heaviest XCD has done its work, whose sum takes no walk over the units (which costs the host 2 to 5 us, with an odd
// number of heads up to 12).
constexpr int kXcdCus = 32;
constexpr int kDealWeighed = 2;
struct XcdClock {   // when the CUs of one XCD are done: a heap, the first to be done on top
  float done[kXcdCus] = {}, last = 0.f;
  void take(float cost) {
    const float t = done[0] + cost;
    int i = 0;
    for (int c; (c = 2 * i + 1) < kXcdCus; i = c) {
      c += c + 1 < kXcdCus && done[c + 1] < done[c];
      if (done[c] >= t) break;
      done[i] = done[c];
    }
    done[i] = t;
    last = t > last ? t : last;
  }
};
inline bool deal_units(const SegTable& segs, const TileIndex& ti, int rows_per_tile, int n_heads) {
  if (n_heads % kNumXcd == 0 || segs.n == 0 || segs.len[segs.n - 1] == segs.len[0]) return false;
  const int tiles = count_tiles(ti);
  const long long units = (long long)tiles * n_heads, chunk = (units + kNumXcd - 1) / kNumXcd;
  if (chunk <= kXcdCus) return false;
  constexpr float kMargin = 1.03f;
  auto tile_cost = [&](int s, int t) {
    const int left = segs.len[s] - t * rows_per_tile;
    return segs.len[s] * (0.75f + 0.25f * (left < rows_per_tile ? left : rows_per_tile) / rows_per_tile);
  };
  if (chunk > kDealWeighed * kXcdCus) {
    auto tiles_cost = [&](int end) {   // of a head's tiles [0, end)
      double sum = 0.0;
      for (int s = 0; s < segs.n && ti.cu[s] < end; ++s) {
        const int last = (ti.cu[s + 1] < end ? ti.cu[s + 1] : end) - ti.cu[s] - 1;
        sum += (double)last * tile_cost(s, 0) + tile_cost(s, last);
      }
      return sum;
    };
    const double head = tiles_cost(tiles);
    auto units_cost = [&](long long end) { return (double)(end / tiles) * head + tiles_cost((int)(end % tiles)); };
    for (int x = 0; x < kNumXcd; ++x) {
      const long long a = x * chunk, b = a + chunk;
      if (a >= units) break;
      if ((units_cost(b < units ? b : units) - units_cost(a)) * kNumXcd > kMargin * head * n_heads) return true;
    }
    return false;
  }
  struct Cursor { int tile, s; };   // (tiles are asked for in order)
  auto cost_at = [&](Cursor& at, int tile) {
    if (tile < at.tile) at.s = 0;
    at.tile = tile;
    while (ti.cu[at.s + 1] <= tile) ++at.s;
    return tile_cost(at.s, tile - ti.cu[at.s]);
  };
  XcdClock dealt;   // XCD 0 has the first, longest unit of every eight
  Cursor at{0, 0};
  for (int u = 0; u < (int)units; u += kNumXcd) dealt.take(cost_at(at, u / n_heads));
  int first[kNumXcd];
  for (int x = 0; x < kNumXcd; ++x) {
    const int a = x * (int)chunk, b = (int)(a + chunk < units ? a + chunk : units);
    first[x] = a % tiles;
    bool seen = false;   // an XCD that starts at the same tile has done as much
    for (int y = 0; y < x; ++y) seen |= first[y] == first[x];
    if (seen) continue;
    XcdClock c;
    for (int u = a, tile = first[x]; u < b; ++u) {
      c.take(cost_at(at, tile));
      tile = tile + 1 < tiles ? tile + 1 : 0;
    }
    if (c.last > kMargin * dealt.last) return true;
  }
  return false;
}
// (Cross-attention tables are ordered by pairs, not by the range that a unit walks: dealt out in that order long units
// may come last.  The FP8 forward and the one-grid backward of short sequences do not ask and stay contiguous; dealing
// would serve them too: FP8, 24 x 1,000 + 24 x 300 tokens, 4 heads 79 us, dealt 56; that backward, 6 x 1,000 + 6 x 400 +
// 10 x 260 tokens, 2 heads 68, dealt 45, but 1,000 + 700 + 2 x 500 + 300 + 12 x 257, 20 heads 149, dealt 152.)
inline bool deal_units(const XSegTable&, const TileIndex&, int, int) { return false; }

// The unit map of an attention launch over the tiles of ti, rows_per_tile rows each.
template <class Segs>
inline UnitMap make_unit_map(const Segs& segs, const TileIndex& ti, int rows_per_tile, int n_heads) {
  return make_unit_map(count_tiles(ti), n_heads, deal_units(segs, ti, rows_per_tile, n_heads));
}

// Sequences with at most this many keys have their Delta formed in its cancellation-free form (backward); the
// tiles of 32 of their queries, none of the other sequences'.
constexpr int kShortKeys = 32;
template <class Segs>
inline TileIndex make_few_key_index(const Segs& segs) {
  TileIndex ti;
  int tiles = 0;
  for (int s = 0; s <= VFM_MAX_SEQS; ++s) {
    ti.cu[s] = tiles;
    if (s < segs.n && segs.kv_len(s) > 0 && segs.kv_len(s) <= kShortKeys) tiles += (segs.q_len(s) + 31) / 32;
  }
  return ti;
}

// What a run's backward is chosen by: its longest query range, its longest range of either kind, the query
// tokens [tok0, tok_end) of all its sequences, and whether one with queries has few keys.
struct RunSpan { int max_q, longest, tok0, tok_end; bool few_keys; };
template <class Segs>
inline RunSpan run_span(const Segs& segs) {
  RunSpan r{0, 0, 0x7fffffff, 0, false};
  for (int s = 0; s < segs.n; ++s) {
    const int nq = segs.q_len(s), nk = segs.kv_len(s), q0 = segs.q_start(s);
    if (nq > r.max_q) r.max_q = nq;
    if (nq > r.longest || nk > r.longest) r.longest = nq > nk ? nq : nk;
    if (nq == 0) continue;
    if (q0 < r.tok0) r.tok0 = q0;
    if (q0 + nq > r.tok_end) r.tok_end = q0 + nq;
    r.few_keys |= nk > 0 && nk <= kShortKeys;
  }
  return r;
}

// Query rows per workgroup of the forward kernel for the sequences of one launch.  Few keys
// per sequence (cross-attention on a text prompt, packs of images): a workgroup's loop is
// short against its prologue and epilogue, so 128-row workgroups are used, two of which share
// a CU and overlap one's loads and stores with the other's loop (0.59 -> 0.55 ms for 56,320
// queries x 512 keys x 32 heads; +3-5% on packs of 256- to 484-token clips).  Each
// wavefront's arithmetic is the same.  With longer sequences the 256-row workgroup's halved
// K/V staging traffic wins.  head_dim 64 always uses 128-row workgroups.
template <class Segs>
inline int fwd_tile_rows(const Segs& segs, int head_dim) {
  if (head_dim != 128) return 128;
  int longest_kv = 0;
  for (int s = 0; s < segs.n; ++s) longest_kv = longest_kv > segs.kv_len(s) ? longest_kv : segs.kv_len(s);
  return longest_kv <= 1024 ? 128 : 256;
}

// Whether a run of clips (longest first) takes the one-pass backward, which forms its own statistics: one
// workgroup per (clip, head), clips of at most 256 tokens.  At head_dim 64 it is faster to about 190 tokens at any
// number of units, and to 224 level with few of them (two passes, one pass: 2 and 256 units of 64 tokens 11.5, 8.4 and
// 13.2, 8.7 us; 160 tokens 13.5, 11.7 and 21.8, 15.1; 192 tokens 13.3, 13.6 and 22.5, 17.4; 224 tokens 15.2, 15.9 and
// 26.4, 21.4).  Beyond, its lone workgroup takes longer than the two passes as long as each CU has at most one of their
// dK/dV workgroups, two to a clip of more than 128 tokens (225 tokens x 128 units 18.3, 20.1, x 136 23.7, 20.6; 256 tokens
// x 2 15.2, 18.2, x 64 16.9, 19.4, x 128 18.5, 20.4, x 136 24.0, 21.1, x 256 28.2, 24.6, x 9,216 934, 827; units of 256 and
// of 64 tokens, 16 and 112 16.2, 19.5, 16 and 496 24.4, 21.1).  (Where a second round of lone
// workgroups has just begun the lead is gone: 320 units of 225 to 256 tokens 37 to 42, 41.)
// At head_dim 128 it is level or faster up to 96 tokens (2 units of 64 and 96
// tokens 10.1 and 12.0 against 10.4 and 12.2; 256 units 12.6 and 16 against 22 and 28).  Beyond, its lone
// workgroup takes longer than the two-pass kernel's, which spreads a (clip, head) over up to three, so a run
// whose two-pass workgroups fit the chip at once stays there (two passes, one pass: 128 tokens x 64 units
// 14.1, 15.6, x 112 16.4, 16.5, x 136 26.6, 16.9; 256 tokens x 80 units 24.6, 33.5, x 88 33.8, 33.2, x 256 60,
// 44).  A clip shorter than the longest counts for its share of it, down to 64 rows (one of 256 and 7 of 64
// tokens, 16 heads: 19, 30; with 31 of them 45, 35).
constexpr int kOnePassMaxRows = 256;
inline bool bwd_one_pass(const SegTable& segs, int n_heads, int head_dim, int cus) {
  const int longest = segs.len[0];
  if (longest > kOnePassMaxRows) return false;
  if (longest <= (head_dim == 64 ? 224 : 96)) return true;
  if (head_dim == 64) {
    long long tiles = 0;   // of 128 keys
    for (int s = 0; s < segs.n; ++s) tiles += segs.len[s] > 128 ? 2 : 1;
    return tiles * n_heads > cus;
  }
  long long rows = 0;   // two-pass workgroups (tiles of 128 keys, of 256 queries), each as the rows of its clip
  for (int s = 0; s < segs.n; ++s) rows += (segs.len[s] > 128 ? 3 : 2) * (segs.len[s] > 64 ? segs.len[s] : 64);
  return rows * n_heads > (long long)cus * longest;
}

// The passes of a run that does not take the one-pass backward.  both: dK/dV and dQ units from one grid,
// where no sequence has more than this many rows (queries or keys), head_dim 128.  dq_first: the dQ pass runs before
// the dK/dV pass and forms the statistics on the way (backward call, separate pass ->
// here: head_dim 128, 20,000 queries x 300 keys x 16 heads 413 -> 403 us, 2 x 4,096 tokens x 16 heads 785 -> 775, 12,000
// tokens x 4 heads level; head_dim 64, 300 tokens x 4 20.1 -> 18.2 us, 64 clips of 300 x 16 144 -> 138, 8,192 x
// 12 655 -> 630).  With neither the statistics come from a pass of their own and dQ
// comes last.  The dK/dV workgroups of a sequence read all of its q and dout rows: where dq takes the place
// of either it has to be written after all of them are done, so neither of the first two will do.
constexpr int kBothMaxRows = 1024;
struct BwdOrder { bool both, dq_first; };
inline BwdOrder bwd_order(int head_dim, int q_split, int longest, bool dq_over_input) {
  if (dq_over_input) return {false, false};
  const bool both = head_dim == 128 && q_split == 1 && longest <= kBothMaxRows;
  return {both, !both};
}

// LDS tiles hold rows of D bf16 without padding; the 16-byte chunk index within
// a row is XOR-ed with a function of the row so that both row-wise 16-byte reads
// (16 consecutive rows, one chunk) and transposing 8-byte reads (4 consecutive
// rows x 64 bytes) spread over all 64 banks.
template <int D>
__device__ __forceinline__ int swz(int row) {
  if constexpr (D == 128) {
    return ((row & 3) << 2) | ((row >> 2) & 3);
  } else {
    return (((row >> 1) & 1) << 2) | ((row >> 2) & 3);
  }
}

// Byte offset of element (row, col) in a swizzled [rows][D] bf16 tile; col is a
// multiple of 4 and the returned address is valid for an 8-byte access (or a
// 16-byte one when col is a multiple of 8).
template <int D>
__device__ __forceinline__ int tile_off(int row, int col) {
  const int chunk = (col >> 3) ^ swz<D>(row);
  return row * (D * 2) + chunk * 16 + (col & 7) * 2;
}

__device__ __forceinline__ bf16x8 lds_read_b128(const char* base, int off) {
  return *reinterpret_cast<const bf16x8*>(base + off);
}

// Transposing LDS read (ds_read_b64_tr_b16).  Within each group of 16 lanes the
// addresses name a 4 x 16 block of 16-bit elements (lane i: row i/4, columns
// 4*(i%4)..+3); lane i receives column i of that block (4 elements, rows 0..3).
__device__ __forceinline__ s16x4 lds_read_tr(const char* base, int off) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (__attribute__((address_space(3))) s16x4*)(base + off));
}

// The same two reads at an LDS byte address held as an integer (base + immediate offset).
__device__ __forceinline__ bf16x8 lds_read_b128_at(uint32_t addr) {
  return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(addr);
}
__device__ __forceinline__ s16x4 lds_read_tr_at(uint32_t addr) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<__attribute__((address_space(3))) s16x4*>(addr));
}

__device__ __forceinline__ bf16x8 join_tr(s16x4 lo, s16x4 hi) {
  s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}

// Value held by the lane 32 away (lane l <-> l^32).
__device__ __forceinline__ float other_half(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  // r[0] = {low half, low half}, r[1] = {high half, high half}
  const uint32_t lo = r[0], hi = r[1];
  const uint32_t o = (threadIdx.x & 32) ? lo : hi;
  return __builtin_bit_cast(float, o);
}

// max / sum over the lane pair (l, l^32); every lane gets the result.
__device__ __forceinline__ float pair_max(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const uint32_t lo = r[0], hi = r[1];
  return fmaxf(__builtin_bit_cast(float, lo), __builtin_bit_cast(float, hi));
}
__device__ __forceinline__ float pair_sum(float x) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const uint32_t lo = r[0], hi = r[1];
  return __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ bf16x8 to_bf16x8(f32x8 v) { return __builtin_convertvector(v, bf16x8); }
__device__ __forceinline__ bf16x4 to_bf16x4(f32x4 v) { return __builtin_convertvector(v, bf16x4); }

// Stores a wavefront's 32 x D fp32 tile, held in the 32x32 MFMA accumulator layout (lane: row
// lane & 31; register q4*4 + e of block db: column db*32 + q4*8 + 4*(lane >> 5) + e), as bf16
// rows.  The tile is turned through 32*D*2 bytes of LDS that belong to the wavefront (16-byte
// chunk x of row r kept at chunk x ^ (r mod chunks-per-row)), so that every store instruction
// writes complete rows instead of 16 bytes of each of 32 rows.  mul scales this lane's row;
// dst points at row 0 of the tile (first column of the head); rows >= rows_valid are not
// written.  A wavefront's LDS accesses complete in program order, so only the compiler has
// to be kept from moving the reads over the writes.
template <int D>
__device__ __forceinline__ void store_tile_rows(char* turn, const f32x16 (&acc)[D / 32], float mul,
                                                __bf16* dst, size_t row_stride, int rows_valid) {
  constexpr int CPR = D / 8, RB = D * 2;
  const int lane = threadIdx.x & 63, c = lane & 31, g = lane >> 5;
#pragma unroll
  for (int db = 0; db < D / 32; ++db)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      f32x4 a;
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = acc[db][q4 * 4 + e] * mul;
      *reinterpret_cast<bf16x4*>(turn + c * RB + (((db * 4 + q4) ^ (c & (CPR - 1))) << 4) + 8 * g) = to_bf16x4(a);
    }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const int rr = lane / CPR, cx = lane % CPR;
#pragma unroll
  for (int i = 0; i < 32 * CPR / 64; ++i) {
    const int r = i * (64 / CPR) + rr;
    const u32x4 w = *reinterpret_cast<const u32x4*>(turn + r * RB + ((cx ^ (r & (CPR - 1))) << 4));
    if (r < rows_valid) *reinterpret_cast<u32x4*>(dst + (size_t)r * row_stride + cx * 8) = w;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ---- direct global -> LDS loads, issued as inline assembly ------------------
// The compiler orders every LDS read that follows a compiler-visible LDS-writing load
// behind a full vmcnt(0) wait, which would expose the whole global latency each tile.
// Issued as assembly the loads stay in flight across the tile's LDS reads; the kernels
// wait for them explicitly (wait_vmcnt) before the barrier that publishes the tile.
// Lane L's bytes land at lds_addr + L*size; lds_addr and base are wave-uniform, the
// global address is base + byte_off (32-bit unsigned, per lane).  Extra outstanding
// loads the compiler does not know of can only make its own vmcnt waits stricter.
__device__ __forceinline__ uint32_t lds_addr_of(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)p;
}
__device__ __forceinline__ void lds_dma16(const void* base, uint32_t byte_off, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds_addr), "v"(byte_off), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void lds_dma4(const void* base, uint32_t byte_off, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
               :: "s"(lds_addr), "v"(byte_off), "s"(base) : "memory", "m0");
}
// A pointer the compiler cannot prove wave-uniform (it depends on the wave index), moved
// to scalar registers.
template <typename T>
__device__ __forceinline__ const T* uniform_ptr(const T* p) {
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  return reinterpret_cast<const T*>(((uint64_t)hi << 32) | lo);
}
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}
template <int V>
struct IntC { static constexpr int value = V; };
// Marks a loaded operand as used here, so that the compiler waits for its global load at
// this point (before the main loop) instead of keeping conservative vmcnt waits inside
// the loop, where they would also wait for the direct-to-LDS loads in flight.
__device__ __forceinline__ void settle(const bf16x8& x) { asm volatile("" :: "v"(x)); }

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// ---- MFMAs issued as assembly, for kernels that need more than 256 registers -------------
// In such a kernel the compiler gives every MFMA it selects an AGPR destination and then
// copies each score to a VGPR (VALU cannot read AGPRs).  Score MFMAs are therefore written as
// assembly with a VGPR destination and the loop-invariant B operand in an AGPR tuple (which
// an MFMA may read directly).  The compiler does not know that the statement is an MFMA, so
// it inserts no wait states for readers of d: every reader must be at least two MFMAs
// downstream in program order (tests/test_isa_hazards.py checks the emitted assembly for it).
__device__ __forceinline__ void mfma32_v(f32x16& d, const bf16x8& a, const bf16x8& b, bool first) {
  if (first) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(d) : "v"(a), "a"(b));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(d) : "v"(a), "a"(b));
}
// The same with three register tuples passed through unchanged.  Volatile statements keep
// their program order, so arithmetic that reads f0/f1/f2 after this call cannot be moved
// before the MFMA, and arithmetic that produced them cannot be moved after it: this is how
// the VALU work is spread evenly between the MFMAs.
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ void mfma32_v(f32x16& d, const bf16x8& a, const bf16x8& b, bool first,
                                         f32x16& f0, f32x16& f1, u32x8& f2) {
  if (first) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %4, %5, 0"
                          : "=&v"(d), "+v"(f0), "+v"(f1), "+v"(f2) : "v"(a), "a"(b));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %4, %5, %0"
                    : "+v"(d), "+v"(f0), "+v"(f1), "+v"(f2) : "v"(a), "a"(b));
}

// Rebinds a loaded operand to an AGPR tuple (and, like settle(), makes the compiler wait
// for its global load here).
__device__ __forceinline__ void to_agpr(bf16x8& x) { asm volatile("" : "=a"(x) : "0"(x)); }

// Accumulation as assembly: accumulator in an AGPR tuple, both operands in VGPRs; the tuples
// are passed through unchanged (see mfma32_v).  Readers of acc other than the next
// accumulation into it must wait out the MFMA themselves.
__device__ __forceinline__ void mfma32_acc(f32x16& acc, const bf16x8& a, const bf16x8& b,
                                           f32x16& f0, f32x16& f1, u32x8& f2) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %4, %5, %0"
               : "+a"(acc), "+v"(f0), "+v"(f1), "+v"(f2) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma32_acc(f32x16& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}

// Wait states after assembly MFMAs, before code the compiler generates reads their results (it
// does not know they were MFMA results).  The tuples are passed through, so that their readers
// cannot be scheduled above the wait.
__device__ __forceinline__ void wait_mfma_v(f32x16& a) {
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15" : "+v"(a));
}
__device__ __forceinline__ void wait_mfma_v(f32x16& a, f32x16& b) {
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15" : "+v"(a), "+v"(b));
}
__device__ __forceinline__ void wait_mfma_a(f32x16& a, f32x16& b, f32x16& c, f32x16& d) {
  asm volatile("s_nop 15\n\ts_nop 15\n\ts_nop 15\n\ts_nop 15" : "+a"(a), "+a"(b), "+a"(c), "+a"(d));
}

// ---- kernel launch ----------------------------------------------------------
// Every kernel of the library is launched through hipLaunchKernel, whose return value is that
// launch's own status.  The thread's sticky "last error" is neither read nor cleared, so an
// error other code left pending in the runtime stays where it is and is never mistaken for
// the library's.
template <class... P, size_t... I>
inline hipError_t launch_impl(void (*kern)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t stream,
                              std::tuple<P...>& vals, std::index_sequence<I...>) {
  void* ptrs[] = {static_cast<void*>(const_cast<std::remove_const_t<std::tuple_element_t<I, std::tuple<P...>>>*>(
      &std::get<I>(vals)))...};
  return hipLaunchKernel(reinterpret_cast<const void*>(kern), grid, block, ptrs, lds, stream);
}
template <class... P, class... A>
inline hipError_t launch(void (*kern)(P...), dim3 grid, dim3 block, size_t lds, hipStream_t stream,
                         const A&... args) {
  static_assert(sizeof...(P) == sizeof...(A), "one argument per kernel parameter");
  std::tuple<P...> vals{static_cast<P>(args)...};
  return launch_impl(kern, grid, block, lds, stream, vals, std::index_sequence_for<P...>{});
}

// Lets a kernel take `bytes` of dynamic LDS.  Up to 64 KB every kernel may; asking the runtime all the same was 1.4 us
// of each small call.  For more, as most kernels need at head_dim 128, it is still asked on every launch: the answer belongs
// to a device, and nothing is kept here.
template <class... P>
inline hipError_t allow_lds(void (*kern)(P...), int bytes) {
  if (bytes <= 64 * 1024) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

// ---- launchers (defined next to their kernels) -----------------------------
// Compute units of the current device (asked once; 256 on MI355X, also the fallback).
int compute_unit_count();

// The RoPE launchers work on the tokens [tab.cu[0], tab.cu[tab.n]) of the clips in tab.
hipError_t launch_rope3d(void* x, const RopeTable& tab, int n_heads, int head_dim,
                         int dim_t, int dim_h, int dim_w, float theta, int inverse,
                         hipStream_t stream);

hipError_t launch_qknorm_rope3d(const void* x, void* y, const float* gain, float eps,
                                const RopeTable& tab, int n_heads, int head_dim,
                                int dim_t, int dim_h, int dim_w, float theta, hipStream_t stream);

hipError_t launch_qknorm_rope3d_bwd(const void* x, const void* dy, void* dx, const float* gain,
                                    float eps, float* dgain, const RopeTable& tab,
                                    int n_heads, int head_dim, int dim_t, int dim_h, int dim_w,
                                    float theta, hipStream_t stream);   // accumulates into dgain
hipError_t launch_zero_f32(float* p, int n, hipStream_t stream);

hipError_t launch_tattn_fwd(const void* q, const void* k, const void* v, const TemporalTable& tab,
                            int n_heads, int head_dim, float scale, void* out, hipStream_t stream);

hipError_t launch_tattn_bwd(const void* q, const void* k, const void* v, const void* dout,
                            const TemporalTable& tab, int n_heads, int head_dim, float scale, void* dq,
                            void* dk, void* dv, hipStream_t stream);

// FP8 path.  scales: the q row exponents and the units' scale words (fp8_scales_bytes() bytes).
hipError_t launch_fp8_pack_q(const void* q, int total, int n_heads, int head_dim, float pre, void* q8,
                             void* scales, hipStream_t stream);
hipError_t launch_fp8_pack_kv(const void* k, const void* v, const Fp8ClipTable& clips, int n_units, int total,
                              int n_heads, int head_dim, void* k8, void* vT8, void* scales, hipStream_t stream);
hipError_t launch_attn_fwd_fp8(const void* q8, const void* k8, const void* vT8, const void* scales,
                               const Fp8SegTable& segs, int n_units, int total, int n_heads, int head_dim,
                               void* out, float* lse, hipStream_t stream);
size_t fp8_scales_bytes(int total, int n_heads, int n_units);

// Segs is SegTable (self-attention) or XSegTable (cross-attention); total_q is the number
// of query tokens (rows of lse, Delta).
template <class Segs>
hipError_t launch_attn_fwd(const void* q, const void* k, const void* v, const Segs& segs,
                           int total_q, int n_heads, int head_dim, float scale, void* out,
                           float* lse, hipStream_t stream);

// The sequences of segs (one run of a call's clips).  dkv32: optional fp32 dK, dV accumulators of
// total_kv rows each (query-split pass); [kv_lo, kv_hi) is the run's range of key rows.
template <class Segs>
hipError_t launch_attn_bwd(const void* q, const void* k, const void* v, const void* out,
                           const float* lse, const void* dout, const Segs& segs, int total_q,
                           int n_heads, int head_dim, float scale, void* dq, void* dk, void* dv,
                           float* delta, float* lse2, float* sentinel, float* dkv32, int total_kv,
                           int kv_lo, int kv_hi, hipStream_t stream);

}  // namespace vfm
