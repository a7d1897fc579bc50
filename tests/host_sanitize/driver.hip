// Host-only exercise of the library's argument validation, clip-table builders, run splitting and
// tile scheduler under AddressSanitizer and UndefinedBehaviorSanitizer (no GPU, nothing launched).
// Built by tests/test_host_sanitizers.py from csrc/vfm_api.hip plus the launcher stubs below, which
// stand in for the kernels' launchers and check what the tables they are handed contain.
#include <stdio.h>
#include <stdlib.h>

#include <algorithm>
#include <random>
#include <vector>

#include "rope_common.h"
#include "vfm_common.h"

static long g_launches = 0;
static int g_failures = 0;
#define EXPECT(cond)                                                              \
  do {                                                                            \
    if (!(cond)) { ++g_failures; fprintf(stderr, "FAILED %s:%d: %s\n", __FILE__, __LINE__, #cond); } \
  } while (0)

namespace vfm {

// Every table a launcher receives must be internally consistent: that is what the kernels rely on.
static void check_rope_table(const RopeTable& t) {
  EXPECT(t.n >= 0 && t.n <= VFM_MAX_SEQS);
  for (int s = 0; s < t.n; ++s) {
    EXPECT(t.cu[s] <= t.cu[s + 1]);
    EXPECT(t.hw[s] >= 1 && t.w[s] >= 1);
    if (t.cu[s + 1] > t.cu[s]) EXPECT((t.cu[s + 1] - t.cu[s]) % t.hw[s] == 0 && t.hw[s] % t.w[s] == 0);
  }
  for (int s = t.n; s < VFM_MAX_SEQS; ++s) EXPECT(t.cu[s + 1] == t.cu[t.n]);
}
template <class Segs>
static void check_segs(const Segs& segs, int total_q) {
  EXPECT(segs.n >= 0);
  for (int s = 0; s < segs.n; ++s) {
    EXPECT(segs.q_len(s) >= 0 && segs.kv_len(s) >= 0 && segs.q_len(s) + segs.kv_len(s) > 0);
    EXPECT(segs.q_start(s) >= 0 && segs.q_start(s) + segs.q_len(s) <= total_q);
    if (segs.q_len(s) > 0) EXPECT(segs.kv_len(s) > 0);
  }
}

// What the backward derives from a run's sequences: the span of its queries, and the tiles of those with few
// keys (every such tile found again by its index, no other).
template <class Segs>
static void check_run_span(const Segs& segs) {
  const RunSpan r = run_span(segs);
  const TileIndex ti = make_few_key_index(segs);
  int tiles = 0, max_q = 0, longest = 0, lo = 0x7fffffff, hi = 0;
  for (int s = 0; s < segs.n; ++s) {
    max_q = std::max(max_q, segs.q_len(s));
    longest = std::max({longest, segs.q_len(s), segs.kv_len(s)});
    if (segs.q_len(s) == 0) continue;
    lo = std::min(lo, segs.q_start(s));
    hi = std::max(hi, segs.q_start(s) + segs.q_len(s));
    if (segs.kv_len(s) > kShortKeys) continue;
    for (int t = 0; t * 32 < segs.q_len(s); ++t) {
      int seq = -1, tile = -1;
      locate_tile(ti, segs.n, tiles++, seq, tile);
      EXPECT(seq == s && tile == t);
    }
  }
  EXPECT(count_tiles(ti) == tiles && r.few_keys == (tiles > 0));
  EXPECT(r.max_q == max_q && r.longest == longest && r.tok0 == lo && r.tok_end == hi);
}

hipError_t launch_rope3d(void*, const RopeTable& tab, int, int, int, int, int, float, int, hipStream_t) {
  ++g_launches; check_rope_table(tab); return hipSuccess;
}
hipError_t launch_qknorm_rope3d(const void*, void*, const float*, float, const RopeTable& tab, int, int, int, int, int,
                                float, hipStream_t) { ++g_launches; check_rope_table(tab); return hipSuccess; }
hipError_t launch_qknorm_rope3d_bwd(const void*, const void*, void*, const float*, float, float*, const RopeTable& tab,
                                    int, int, int, int, int, float, hipStream_t) {
  ++g_launches; check_rope_table(tab); return hipSuccess;
}
hipError_t launch_zero_f32(float*, int, hipStream_t) { ++g_launches; return hipSuccess; }
// The launches by frame class: every pixel of every clip in exactly one launch table, at its place and with
// its own frame count, no clip in kernels too short for it, only few in kernels made for longer ones,
// and no launch of 2^32 threads or more.
static void check_temporal_launches(const TemporalTable& t, int heads, int hd) {
  const TemporalPlan plan = make_temporal_plan(t, heads, hd, 256);
  std::vector<int> seen(VFM_MAX_SEQS, 0);
  long pixels = 0;
  for (int l = 0; l < kTemporalClasses; ++l) {
    const TemporalTable c = temporal_launch_table(t, plan, l);
    EXPECT(c.n == t.n && c.pix_cu[0] == 0 && (c.pix_cu[t.n] > 0) == (plan.launch_of[l] == l));
    long long joined = 0;
    for (int s = 0; s < t.n; ++s) {
      const int pix = c.pix_cu[s + 1] - c.pix_cu[s];
      EXPECT(c.cu[s] == t.cu[s] && c.cu[s + 1] == t.cu[s + 1] && c.hw[s] == t.hw[s]);
      if (pix == 0) continue;
      const int frames = temporal_frames(c, s);
      EXPECT(pix == t.hw[s] && pix * frames == t.cu[s + 1] - t.cu[s]);
      EXPECT(l == 5 || frames <= (l == 0 ? 16 : 32 * l));
      if (temporal_class(frames) != l) joined += (long long)pix * heads;
      ++seen[s];
    }
    EXPECT(joined <= 256 * 9 * 4);
    pixels += c.pix_cu[t.n];
    if (l < 5)
      for (bool backward : {false, true}) {
        const TemporalGrid g = temporal_grid(c, l, heads, backward);
        const long long waves = (long long)c.pix_cu[t.n] * heads * (l == 0 ? 1 : l * (backward ? 2 : 1));
        EXPECT((long long)g.blocks * g.threads >= waves * 64 && (long long)g.blocks * g.threads < waves * 64 + 256);
        EXPECT((long long)g.blocks * g.threads < 1LL << 32);
      }
  }
  EXPECT(pixels == t.pix_cu[t.n]);
  for (int s = 0; s < t.n; ++s) EXPECT(seen[s] == (t.cu[s + 1] > t.cu[s]));
}
hipError_t launch_tattn_fwd(const void*, const void*, const void*, const TemporalTable& t, int heads, int hd, float, void*,
                            hipStream_t) {
  ++g_launches;
  EXPECT(t.n >= 0 && t.n <= VFM_MAX_SEQS);
  for (int s = 0; s < t.n; ++s) { EXPECT(t.hw[s] >= 1 && t.pix_cu[s] <= t.pix_cu[s + 1] && t.cu[s] <= t.cu[s + 1]); }
  check_temporal_launches(t, heads, hd);
  return hipSuccess;
}
hipError_t launch_tattn_bwd(const void* q, const void* k, const void* v, const void*, const TemporalTable& t, int h, int d,
                            float sc, void* o, void*, void*, hipStream_t st) { return launch_tattn_fwd(q, k, v, t, h, d, sc, o, st); }
hipError_t launch_fp8_pack_q(const void*, int, int, int, float, void*, void*, hipStream_t) { ++g_launches; return hipSuccess; }
hipError_t launch_fp8_pack_kv(const void*, const void*, const Fp8ClipTable& c, int n_units, int, int, int, void*, void*,
                              void*, hipStream_t) {
  ++g_launches;
  EXPECT(c.n >= 0 && c.n <= VFM_MAX_SEQS);
  for (int s = 0; s < c.n; ++s) {
    EXPECT(c.unit0[s + 1] - c.unit0[s] == (c.cu[s + 1] - c.cu[s] + 63) / 64);
    EXPECT(c.unit0[s + 1] <= n_units);
  }
  return hipSuccess;
}
hipError_t launch_attn_fwd_fp8(const void*, const void*, const void*, const void*, const Fp8SegTable& segs, int n_units,
                               int total, int, int, void*, float*, hipStream_t) {
  ++g_launches;
  for (int s = 0; s < segs.n; ++s) {
    EXPECT(segs.len[s] > 0 && segs.start[s] >= 0 && segs.start[s] + segs.len[s] <= total);
    EXPECT(segs.unit0[s] >= 0 && segs.unit0[s] + (segs.len[s] + 63) / 64 <= n_units);
    if (s) EXPECT(segs.len[s - 1] >= segs.len[s]);
  }
  return hipSuccess;
}
size_t fp8_scales_bytes(int total, int n_heads, int n_units) {
  return ((size_t)total * n_heads + 255) / 256 * 256 + (size_t)n_units * n_heads * 4;
}
template <class Segs>
hipError_t launch_attn_fwd(const void*, const void*, const void*, const Segs& segs, int total_q, int, int, float, void*,
                           float*, hipStream_t) { ++g_launches; check_segs(segs, total_q); return hipSuccess; }
template <class Segs>
hipError_t launch_attn_bwd(const void*, const void*, const void*, const void*, const float*, const void*, const Segs& segs,
                           int total_q, int, int, float, void*, void*, void*, float*, float*, float*, float*, int total_kv,
                           int kv_lo, int kv_hi, hipStream_t) {
  ++g_launches; check_segs(segs, total_q); check_run_span(segs); EXPECT(kv_lo >= 0 && kv_lo <= kv_hi && kv_hi <= total_kv + (total_kv == 0 ? kv_hi : 0));
  return hipSuccess;
}
template hipError_t launch_attn_fwd<SegTable>(const void*, const void*, const void*, const SegTable&, int, int, int, float,
                                              void*, float*, hipStream_t);
template hipError_t launch_attn_fwd<XSegTable>(const void*, const void*, const void*, const XSegTable&, int, int, int, float,
                                               void*, float*, hipStream_t);
template hipError_t launch_attn_bwd<SegTable>(const void*, const void*, const void*, const void*, const float*, const void*,
                                              const SegTable&, int, int, int, float, void*, void*, void*, float*, float*,
                                              float*, float*, int, int, int, hipStream_t);
template hipError_t launch_attn_bwd<XSegTable>(const void*, const void*, const void*, const void*, const float*, const void*,
                                               const XSegTable&, int, int, int, float, void*, void*, void*, float*, float*,
                                               float*, float*, int, int, int, hipStream_t);
}  // namespace vfm

// dq over q or dout must be written after every dK/dV workgroup has read them: never from the grid that
// holds both kinds of unit (head_dim 128), never first.  Any other call takes one of the two.
static void check_bwd_order() {
  for (int hd : {64, 128})
    for (int split : {1, 2, 16})
      for (int longest : {1, 32, 257, 1024, 1025, 56320})
        for (bool over : {false, true}) {
          const vfm::BwdOrder o = vfm::bwd_order(hd, split, longest, over);
          EXPECT(!(o.both && o.dq_first));
          if (over) EXPECT(!o.both && !o.dq_first);
          if (o.both) EXPECT(hd == 128 && split == 1 && longest <= 1024);
          if (!over) EXPECT(o.both || o.dq_first);
        }
}

// Units dealt over the XCDs: each exactly once, and with clips longest first no XCD has more rows than
// another beyond one group of the longest clip.
static void check_dealt_units() {
  for (int group : {1, 8})
    for (int heads : {1, 2, 5, 16, 33})
      for (int clips : {1, 3, 32, 255, 256})
        for (int n_long : {1, 32, 100}) {
          const int units = clips * heads, grid = vfm::dealt_grid(units, group);
          std::vector<int> seen(units, 0);
          long long rows[vfm::kNumXcd] = {};
          EXPECT(grid % vfm::kNumXcd == 0 && grid >= units && grid < units + vfm::kNumXcd * group);
          for (int b = 0; b < grid; ++b) {
            const int u = vfm::dealt_unit(b, group);
            EXPECT(u >= 0 && u < grid);
            if (u >= units) continue;
            ++seen[u];
            rows[b % vfm::kNumXcd] += u / heads < n_long ? 256 : 1;
          }
          for (int u = 0; u < units; ++u) EXPECT(seen[u] == 1);
          const auto [lo, hi] = std::minmax_element(rows, rows + vfm::kNumXcd);
          EXPECT(*hi - *lo <= 256 * group);
        }
}

// The unit maps of the attention kernels: every (head, tile) exactly once; dealt out, no XCD has more tiles of any
// range of tiles than another, but for one.
static void check_unit_maps() {
  for (int heads : {1, 2, 3, 4, 8, 12, 20, 33})
    for (int tiles : {1, 2, 7, 58, 441})
      for (bool dealt : {false, true}) {
        const vfm::UnitMap um = vfm::make_unit_map(tiles, heads, dealt);
        EXPECT((um.dealt_heads != 0) == dealt);
        std::vector<int> seen(heads * tiles, 0);
        std::vector<std::vector<int>> upto(vfm::kNumXcd, std::vector<int>(tiles + 1, 0));   // tiles [0, t) of an XCD
        for (int b = 0; b < um.chunk * vfm::kNumXcd; ++b) {
          int head = -1, tile = -1;
          if (!vfm::map_unit(um, b, head, tile)) continue;
          EXPECT(head >= 0 && head < heads && tile >= 0 && tile < tiles);
          ++seen[head * tiles + tile];
          ++upto[b % vfm::kNumXcd][tile + 1];
        }
        for (int n : seen) EXPECT(n == 1);
        if (!dealt) continue;
        for (auto& u : upto)
          for (int t = 0; t < tiles; ++t) u[t + 1] += u[t];
        for (int a = 0; a < tiles; ++a)
          for (int t = a + 1; t <= tiles; ++t) {
            int lo = seen.size(), hi = 0;
            for (const auto& u : upto) lo = std::min(lo, u[t] - u[a]), hi = std::max(hi, u[t] - u[a]);
            EXPECT(hi - lo <= 1);
          }
      }
}

// Which launches are dealt (the rule's choice by itself is checked against a model of its own in the scheduler's
// tests): never one whose heads divide by the XCDs, whose clips are all alike or which has a unit per CU at most; every
// table of random clips is walked without a read past its end.
static void check_deal_rule() {
  auto table = [](std::vector<int> lens) {
    std::sort(lens.rbegin(), lens.rend());
    vfm::SegTable t{};
    t.n = (int)lens.size();
    for (int s = 0, at = 0; s < t.n; at += lens[s++]) { t.len[s] = lens[s]; t.start[s] = at; }
    return t;
  };
  auto deal = [](const vfm::SegTable& t, int rows, int heads) {
    return vfm::deal_units(t, vfm::make_tile_index<false>(t, rows), rows, heads);
  };
  EXPECT(!deal(table({}), 256, 12));
  for (int rows : {128, 256}) {
    EXPECT(deal(table({5000, 1200, 700, 300}), rows, 12) && !deal(table({5000, 1200, 700, 300}), rows, 16));
    EXPECT(!deal(table(std::vector<int>(64, 3000)), rows, 12) && !deal(table({3000, 100}), rows, 4));
    EXPECT(!deal(table({33554432}), rows, 1) && !deal(table({33554431, 1}), rows, 1));
  }
  std::mt19937 rng(7);
  for (int trial = 0; trial < 2000; ++trial) {
    const int n = 1 + (int)(rng() % (trial % 5 ? 12 : VFM_MAX_SEQS)), most = 1 << (rng() % 15);
    std::vector<int> lens(n);
    for (int& l : lens) l = 1 + (int)(rng() % most);
    const vfm::SegTable t = table(lens);
    const int heads = 1 + (int)(rng() % 33), rows = rng() & 1 ? 128 : 256;
    const vfm::TileIndex ti = vfm::make_tile_index<false>(t, rows);
    const bool dealt = deal(t, rows, heads);
    if (dealt) EXPECT(heads % vfm::kNumXcd != 0 && t.len[0] != t.len[n - 1] && vfm::count_tiles(ti) * heads > 256);
    EXPECT((vfm::make_unit_map(t, ti, rows, heads).dealt_heads == heads) == dealt);
  }
}

// The one pass serves clips of up to 256 tokens; at head_dim 128 and more than 96 it needs more two-pass
// workgroups than the chip has places for, short clips counting for their share; at head_dim 64 and more than 224
// more dK/dV workgroups than CUs.
static void check_one_pass_rule() {
  auto run = [](int n, int len, int m, int other) {
    vfm::SegTable t{};
    t.n = n + m;
    for (int s = 0; s < t.n; ++s) t.len[s] = s < n ? len : other;
    return t;
  };
  EXPECT(!vfm::bwd_one_pass(run(1, 257, 255, 1), 32, 64, 256) && !vfm::bwd_one_pass(run(1, 257, 255, 1), 32, 128, 256));
  EXPECT(vfm::bwd_one_pass(run(1, 224, 0, 0), 1, 64, 256) && vfm::bwd_one_pass(run(1, 96, 0, 0), 1, 128, 256));
  for (int len : {225, 256}) {
    EXPECT(!vfm::bwd_one_pass(run(1, len, 0, 0), 1, 64, 256) && !vfm::bwd_one_pass(run(8, len, 0, 0), 16, 64, 256));
    EXPECT(vfm::bwd_one_pass(run(1, len, 0, 0), 129, 64, 256) && vfm::bwd_one_pass(run(256, len, 0, 0), 65535, 64, 256));
    EXPECT(!vfm::bwd_one_pass(run(1, len, 14, 128), 16, 64, 256) && vfm::bwd_one_pass(run(1, len, 15, 128), 16, 64, 256));
    EXPECT(vfm::bwd_one_pass(run(1, len, 14, 129), 16, 64, 256));
  }
  EXPECT(!vfm::bwd_one_pass(run(1, 256, 0, 0), 85, 128, 256) && vfm::bwd_one_pass(run(1, 256, 0, 0), 86, 128, 256));
  EXPECT(!vfm::bwd_one_pass(run(1, 128, 0, 0), 128, 128, 256) && vfm::bwd_one_pass(run(1, 128, 0, 0), 129, 128, 256));
  EXPECT(!vfm::bwd_one_pass(run(1, 256, 7, 64), 16, 128, 256) && vfm::bwd_one_pass(run(1, 256, 31, 64), 16, 128, 256));
  EXPECT(vfm::bwd_one_pass(run(256, 256, 0, 0), 65535, 128, 256));
}

// Heads per workgroup of the position encoding: batches of four, about 1,024 workgroups where there are too
// few tokens for that, and one slice from 725 blocks on.
static void check_rope_slices() {
  for (int heads : {1, 3, 4, 8, 24, 32, 48, 65535})
    for (int blocks : {1, 13, 63, 188, 256, 313, 375, 512, 625, 724, 725, 750, 897, 1024, 4000}) {
      const int per = vfm::rope_heads_per_block(blocks, heads), slices = (heads + per - 1) / per;
      EXPECT(per >= 4 && per % 4 == 0 && slices >= 1 && slices <= 65535);
      EXPECT((long long)slices * blocks <= 1449 || slices == 1);
      if (blocks >= 725) EXPECT(slices == 1);
      if (blocks < 600 && heads >= 8) EXPECT(slices >= 2);
    }
}

// The cut of heads over work items in the backward of the normalised position encoding: every head in one
// slice, the grid's limits, and no more than a quarter of the places' time idle once there is work for
// twenty passes of single heads.
static void check_qk_bwd_split() {
  for (int hd : {64, 128})
    for (int heads : {1, 2, 3, 4, 5, 8, 12, 16, 24, 33, 48, 64, 200, 65535})
      for (int count : {1, 2, 63, 200, 512, 1001, 2000, 2049, 6000, 8192, 10000, 12000, 16384, 16385, 20000, 28704, 40000, 56320, 262144}) {
        if ((long long)count * heads * hd * 2 > 0xffffffffLL) continue;
        const vfm::QkBwdSplit sp = vfm::qk_bwd_split(count, heads, hd);
        const int per = (heads + sp.slices - 1) / sp.slices;
        const long long items = (long long)count * sp.slices, places = 256LL * 1024 / (hd / 8);
        EXPECT(sp.slices >= 1 && (sp.slices - 1) * per < heads && items < 1LL << 31);
        EXPECT(sp.threads == 1024 || (sp.threads == 256 && per <= 4 && items <= places / 16));
        const long long passes = (items + places - 1) / places;
        if (heads >= 8 && (long long)count * heads >= 20 * places) EXPECT(passes * per * places * 3 <= 4LL * count * heads);
      }
}

int main() {
  check_rope_slices();
  check_qk_bwd_split();
  check_bwd_order();
  check_dealt_units();
  check_unit_maps();
  check_deal_rule();
  check_one_pass_rule();
  std::mt19937 rng(12345);
  void* const P = reinterpret_cast<void*>(0x10000);     // never dereferenced: the stubs launch nothing
  float* const F = reinterpret_cast<float*>(0x20000);
  const size_t big = (size_t)1 << 40;
  for (int trial = 0; trial < 400; ++trial) {
    // clip counts on both sides of every run boundary, lengths with many zeros
    const int n_opts[] = {0, 1, 2, 127, 128, 129, 255, 256, 257, 511, 512, 513, 700, 1025};
    const int n = n_opts[rng() % 14];
    const int heads = 1 + rng() % 5, hd = (rng() & 1) ? 128 : 64;
    std::vector<int32_t> cu(n + 1, 0), thw(3 * (n + 1), 0), cu_kv(n + 1, 0);
    for (int s = 0; s < n; ++s) {
      int T = rng() % 5, H = 1 + rng() % 6, W = 1 + rng() % 6;
      if (rng() % 7 == 0) { T = 1; H = 1; W = 1 + rng() % 300; }
      if (rng() % 23 == 0) T = 33 + rng() % 100;
      thw[3 * s] = T; thw[3 * s + 1] = H; thw[3 * s + 2] = W;
      cu[s + 1] = cu[s] + T * H * W;
      cu_kv[s + 1] = cu_kv[s] + (T * H * W > 0 ? 1 + (int)(rng() % 90) : (int)(rng() % 3));
    }
    const int total = cu[n], total_kv = cu_kv[n];
    const int d2 = hd / 4 * 2, d1 = hd - 2 * d2 >= 0 ? hd - 2 * d2 : 0;
    EXPECT(vfm_rope3d(P, thw.data(), cu.data(), n, total, heads, hd, d1, d2, d2, 1e4f, trial & 1, VFM_BF16, nullptr) == VFM_OK);
    EXPECT(vfm_qknorm_rope3d(P, F, 1e-6f, P, thw.data(), cu.data(), n, total, heads, hd, d1, d2, d2, 1e4f, VFM_BF16, nullptr) == VFM_OK);
    EXPECT(vfm_qknorm_rope3d_bwd(P, F, 1e-6f, F, F + 64, F, thw.data(), cu.data(), n, total, heads, hd, d1, d2, d2, 1e4f,
                                 VFM_BF16, nullptr) == VFM_OK);
    EXPECT(vfm_attn_fwd(P, P, P, cu.data(), n, total, heads, hd, 0.1f, P, F, VFM_BF16, nullptr) == VFM_OK);
    EXPECT(vfm_attn_bwd(P, P, P, P, F, P, cu.data(), n, total, heads, hd, 0.1f, P, P, P, P, big, VFM_BF16, nullptr) == VFM_OK);
    EXPECT(vfm_attn_bwd_noalloc(P, P, P, P, F, P, cu.data(), n, 0, heads, hd, 0.1f, P, P, P, VFM_BF16, nullptr) ==
           (total == 0 ? VFM_OK : VFM_ERR_CU_SEQLENS));
    EXPECT(vfm_xattn_fwd(P, P, P, cu.data(), cu_kv.data(), n, total, total_kv, heads, hd, 0.1f, P, F, VFM_BF16, nullptr) == VFM_OK);
    EXPECT(vfm_xattn_bwd(P, P, P, P, F, P, cu.data(), cu_kv.data(), n, total, total_kv, heads, hd, 0.1f, P, P, P, P, big,
                         VFM_BF16, nullptr) == VFM_OK);
    EXPECT(vfm_tattn_fwd(P, P, P, thw.data(), cu.data(), n, total, heads, hd, 0.1f, P, VFM_BF16, nullptr) == VFM_OK);
    EXPECT(vfm_tattn_bwd(P, P, P, P, thw.data(), cu.data(), n, total, heads, hd, 0.1f, P, P, P, VFM_BF16, nullptr) == VFM_OK);
    size_t a, b, c, d;
    EXPECT(vfm_fp8_pack_sizes(cu.data(), n, total, heads, hd, &a, &b, &c, &d) == VFM_OK);
    EXPECT(vfm_fp8_pack(P, P, P, cu.data(), n, total, heads, hd, 0.1f, P, P, P, P, VFM_BF16, nullptr) == VFM_OK);
    EXPECT(vfm_attn_fwd_fp8(P, P, P, P, cu.data(), n, total, heads, hd, P, F, nullptr) == VFM_OK);
    // the scheduler: ask for the size, then fill exactly that many entries (a too-small buffer is refused)
    const int rows = 32 << (rng() % 4);
    int n_blocks = -1;
    EXPECT(vfm_schedule_units(cu.data(), n, total, heads, rows, nullptr, 0, &n_blocks) == (n_blocks == 0 ? VFM_OK : VFM_ERR_SHAPE));
    std::vector<int32_t> units(3 * (size_t)(n_blocks > 0 ? n_blocks : 1));
    if (n_blocks > 1) EXPECT(vfm_schedule_units(cu.data(), n, total, heads, rows, units.data(), n_blocks - 1, &n_blocks) == VFM_ERR_SHAPE);
    int again = -1;
    EXPECT(vfm_schedule_units(cu.data(), n, total, heads, rows, units.data(), n_blocks, &again) == VFM_OK && again == n_blocks);
    long covered = 0;
    for (int bidx = 0; bidx < n_blocks; ++bidx)
      if (units[3 * bidx] >= 0) {
        EXPECT(units[3 * bidx] < heads && units[3 * bidx + 1] >= 0 && units[3 * bidx + 2] >= 1 && units[3 * bidx + 2] <= rows &&
               units[3 * bidx + 1] + units[3 * bidx + 2] <= total);
        covered += units[3 * bidx + 2];
      }
    EXPECT(covered == (long)total * heads);
    const int n_runs = n == 0 ? 1 : (n + VFM_MAX_SEQS - 1) / VFM_MAX_SEQS;
    int tr = 0;
    EXPECT(vfm_attn_fwd_tile_rows(cu.data(), n, total, hd, n_runs - 1, &tr) == VFM_OK && (tr == 128 || tr == 256));
    EXPECT(vfm_attn_fwd_tile_rows(cu.data(), n, total, hd, n_runs, &tr) == VFM_ERR_SHAPE);
    // malformed boundaries are refused before any table is built
    if (n >= 2) {
      std::vector<int32_t> bad(cu);
      bad[n / 2] = bad[n] + 1;
      const long before = g_launches;
      EXPECT(vfm_attn_fwd(P, P, P, bad.data(), n, total, heads, hd, 0.1f, P, F, VFM_BF16, nullptr) == VFM_ERR_CU_SEQLENS);
      EXPECT(vfm_rope3d(P, thw.data(), bad.data(), n, total, heads, hd, d1, d2, d2, 1e4f, 0, VFM_BF16, nullptr) == VFM_ERR_CU_SEQLENS);
      EXPECT(g_launches == before);
    }
  }
  // temporal attention at the size limit: the largest tensors (2^25 and 2^24 rows) as single frames, as the shortest
  // clips of every class, and as single frames beside one long clip
  for (int hd : {64, 128})
    for (int frames : {1, 16, 17, 32, 33, 64, 65, 96, 97, 128, 129, 300})
      for (int beside : {0, 100, 300}) {
        const int rows = (int)((1LL << 31) / hd) - 300, pix = (rows - beside) / frames;
        const int32_t thw[6] = {frames, 1, pix, beside, 1, beside ? 1 : 0}, cu[3] = {0, frames * pix, frames * pix + beside};
        EXPECT(vfm_tattn_bwd(P, P, P, P, thw, cu, 2, cu[2], 1, hd, 0.1f, P, P, P, VFM_BF16, nullptr) == VFM_OK);
      }
  printf("%s: %ld stub launches, %d failures\n", g_failures ? "FAILED" : "ok", g_launches, g_failures);
  return g_failures ? 1 : 0;
}
