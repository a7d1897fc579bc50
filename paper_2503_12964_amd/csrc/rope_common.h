// Token -> grid position -> rotation angles, shared by the RoPE kernels (gfx950 only).
#pragma once

#include <math.h>

#include <algorithm>

#include "vfm_common.h"

namespace vfm {

struct RopeFreq {
  double inv_freq[64];    // per pair index p = element/2: theta^(-2i/d_axis)
  unsigned char axis[64]; // 0 = t, 1 = h, 2 = w
};

// Host: per-pair inverse frequencies and axis of each pair for a (d_t, d_h, d_w) split.
inline RopeFreq make_rope_freq(int dim_t, int dim_h, int dim_w, float theta) {
  RopeFreq fr;
  const int dims[3] = {dim_t, dim_h, dim_w};
  int p = 0;
  for (int ax = 0; ax < 3; ++ax) {
    for (int i = 0; i < dims[ax] / 2; ++i, ++p) {
      fr.inv_freq[p] = pow((double)theta, -2.0 * (double)i / (double)dims[ax]);
      fr.axis[p] = (unsigned char)ax;
    }
  }
  for (; p < 64; ++p) { fr.inv_freq[p] = 0.0; fr.axis[p] = 0; }
  return fr;
}

// Heads per workgroup of the position-encoding kernels, whose blocks cover all tokens in x and
// slices of the heads in y.  A token's angles are worth computing once for all heads as long as
// the tokens alone fill the chip; with few blocks a workgroup's walk over its heads is a serial chain
// of memory round trips on an idle chip, so the heads are cut into slices of at least four (one batch of
// loads in flight), each forming the angles again.  The number of slices is the power of two nearest to
// what makes 1,024 workgroups (4 per CU); rounded up instead, 3 slices for 375 blocks or 2 for 897 lose more
// to the shorter walks than they fill.
// (512 tokens x 32 heads x 128, 32 blocks: 6.1 -> 3.7 us; 10,000 tokens x 16 heads, 625 blocks: normalised form
// 19.9 -> 17.7; 12,000 tokens x 32 heads x 64, 375 blocks: none 21.0, two 20.0, three 22.9; 28,704 tokens x
// 32 heads x 64, 897 blocks: none 53.1, two 59.4.)
constexpr int kRopeFillBlocks = 1024;
inline int rope_heads_per_block(int token_blocks, int n_heads) {
  int slices = 1;   // (sqrt 2: the middle between a power of two and the next)
  while (slices < n_heads && slices * token_blocks * 1.4142f < kRopeFillBlocks) slices *= 2;
  const int per = (n_heads + slices - 1) / slices;
  return (per + 3) / 4 * 4;
}

// Backward of the normalised form.  A work item is one slice of a token's heads, taken by D/8 lanes.  Every workgroup ends in one atomic per
// element of dgain, about 25 ns a workgroup on the same 64 or 128 addresses, so workgroups are few: up to 64
// of 256 threads where those have a place for every item (200 tokens x 1 head x 128: 5.2 us, in workgroups
// of 1024 threads 6.8), else up to one of 1024 threads per CU, looping (8,192 tokens x 16 heads x 128: 25 us,
// with up to 4,096 small workgroups 31).
constexpr int kQkBwdSmall = 256, kQkBwdLarge = 1024;
constexpr int kQkBwdSmallGrid = 64, kQkBwdLargeGrid = 256;

// Slices of a token's heads (at least two heads each) and the workgroup's size.  Items are walked in passes
// over all places of the grid; an item costs its heads and about two more for the angles, and the passes'
// start and end about a third of one.  The split with the least of it keeps the last pass full (20,000
// tokens x 48 heads x 128 in two passes of which the second is a fifth full 189 us, in five 141).
struct QkBwdSplit { int slices, threads; };
inline QkBwdSplit qk_bwd_split(int count, int n_heads, int head_dim) {
  const int lanes = head_dim / 8;
  const int small_places = kQkBwdSmallGrid * kQkBwdSmall / lanes, large_places = kQkBwdLargeGrid * kQkBwdLarge / lanes;
  const int max_slices = (n_heads + 1) / 2;
  if (count <= small_places) {
    const int s = std::min(small_places / count, max_slices), per = (n_heads + s - 1) / s;
    if (per <= 4) return {(n_heads + per - 1) / per, kQkBwdSmall};
  }
  int best = 0;
  long long least = 0;
  auto consider = [&](int s) {
    const int per = (n_heads + s - 1) / s;
    if (s > max_slices || (n_heads + per - 1) / per != s) return;   // (or the same slices as fewer)
    const long long passes = ((long long)count * s + large_places - 1) / large_places;
    const long long cost = (3 * passes + 1) * (per + 2);
    if (best == 0 || cost * 40 < least * 39) { least = cost; best = s; }   // (a finer split has to promise 2.5%)
  };
  for (int s = 1; s <= std::min(64, max_slices); ++s) consider(s);
  if (large_places / count > 64) {   // few tokens of very many heads: as many slices as one pass has places for
    const int s = std::min(large_places / count, max_slices), per = (n_heads + s - 1) / s;
    consider((n_heads + per - 1) / per);
  }
  return {best, kQkBwdLarge};
}

// (cos, sin) of the four adjacent pairs in 16-byte chunk `chunk` of token `tok`'s head
// vectors.  The angle is formed and reduced to [-pi, pi] in fp64 (a handful of operations
// per token, reused for every head), so the rotation stays accurate to fp32 rounding
// however large the grid position is.  negate != 0 gives the transpose rotation.
__device__ __forceinline__ void rope_cos_sin(const RopeTable& tab, const RopeFreq& fr, int tok,
                                             int chunk, int negate, float (&cs)[4], float (&sn)[4]) {
  // clip of this token: last s with cu[s] <= tok (skips empty clips)
  int lo = 0, hi = tab.n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (tab.cu[mid] <= tok) lo = mid; else hi = mid;
  }
  const int r = tok - tab.cu[lo];
  const int hw = tab.hw[lo], w = tab.w[lo];
  int pos[3];
  pos[0] = r / hw;
  const int rem = r - pos[0] * hw;
  pos[1] = rem / w;
  pos[2] = rem - pos[1] * w;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int p = chunk * 4 + e;
    const int ax = fr.axis[p];
    const double pa = (double)(ax == 0 ? pos[0] : (ax == 1 ? pos[1] : pos[2]));
    double ang = pa * fr.inv_freq[p];
    ang -= 6.283185307179586476925 * rint(ang * 0.15915494309189533577);
    float s, c;
    sincosf((float)ang, &s, &c);
    cs[e] = c;
    sn[e] = negate ? -s : s;
  }
}

// bf16 pair packed in a 32-bit word <-> two floats
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xffff0000u); }
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  f32x2 y = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(y, bf16x2));
}

}  // namespace vfm
