// What the two prefill-shaped tree attention kernels share (attn_tree.hip, attn_tree_short.hip): the
// layout (a wave holds 32 query rows, each a (query node, query head) pair of one KV head), the
// placement of the row blocks, the rows and their key range, the visibility of a key, the output.
#pragma once

#include "attn_common.h"
#include "mfma_tile.h"

namespace td {

constexpr int kTreeWaves = 4;  // (two groups of waves per CU: their barriers do not wait on each other)
constexpr int kTreeThreads = kTreeWaves * 64;
constexpr int kTreeRows = kTreeWaves * 32;  // query rows per row block
constexpr float kTreeNegBig = -1.0e30f;
constexpr float kTreeSlack = 8.0f;  // a row's shift moves for scores 2^8 above it

template <int D>
struct TreeGeom {
  static constexpr int KSTEPS = D / 16;    // 32x32x16 steps of S^T
  static constexpr int DT = D / 32;        // 32-wide d tiles of O^T
  static constexpr int CPR = D / 8;        // 16-byte chunks per node row
  static constexpr int NBLK = CPR / 4;     // 64-byte blocks per row
  static constexpr int HALF = 32 * D * 2;  // bytes of 32 K (or V) rows
};

// (trie, layer of the call, KV head) and row block of a WG; the row blocks of a unit go to one XCD
// where the units divide over them (AttnArgs::xcd_group), the deepest (longest) first.  (Going up
// again after half of them, so that a CU gets a long and a short block, measured slower past 66
// blocks per XCD: at d = 128, 91 blocks 65.1 us against 53.7, 127 blocks 175 and 165.)
struct TreeUnit {
  int t, li, g, rb;
};
__device__ inline TreeUnit tree_unit(const DevState& s, const AttnArgs& a) {
  const int x = blockIdx.x;
  int unit, rb;
  if (a.xcd_group) {
    const int xcd = x % 8, k = x / 8;
    unit = (k / a.row_blocks) * 8 + xcd;
    rb = a.row_blocks - 1 - k % a.row_blocks;
  } else {
    unit = x / a.row_blocks;
    rb = a.row_blocks - 1 - x % a.row_blocks;
  }
  return {unit / (s.Hkv * a.n_layers), (unit / s.Hkv) % a.n_layers, unit % s.Hkv, rb};
}

// A lane's query row (a row without a live query node is not ok), and its wave's deepest query slot
// + 1, shallowest and deepest query depth (live rows).
struct TreeRow {
  int r, owner, depth;
  bool ok;
  uint64_t mask;
  int hi, dmin, dmax;
};
__device__ inline TreeRow tree_row(const DevState& s, const AttnArgs& a, const TreeUnit& u, int N, int G,
                                   const uint64_t* maskp, const int32_t* depthp, int wave, int col) {
  TreeRow q;
  q.r = u.rb * kTreeRows + wave * 32 + col;
  q.owner = q.r / G;
  const int slot = q.r < a.qmax * G ? a.qslots[(size_t)u.t * a.qmax + q.owner] : -1;
  q.ok = slot >= 0 && slot < N;
  q.mask = 0;
  q.depth = -1;
  if (q.ok) {
    q.mask = maskp[slot];
    q.ok = q.mask != 0ull;
  }
  if (q.ok) q.depth = depthp[slot];
  int hi = q.ok ? slot + 1 : 0, dmin = q.ok ? q.depth : INT_MAX, dmax = q.ok ? q.depth : -1;
  for (int o = 16; o > 0; o >>= 1) {
    hi = max(hi, __shfl_xor(hi, o));
    dmin = min(dmin, __shfl_xor(dmin, o));
    dmax = max(dmax, __shfl_xor(dmax, o));
  }
  q.hi = __builtin_amdgcn_readfirstlane(hi);
  q.dmin = __builtin_amdgcn_readfirstlane(dmin);
  q.dmax = __builtin_amdgcn_readfirstlane(dmax);
  return q;
}

// The block's key range [lo, hi): from the window start of its shallowest query to its deepest query
// slot (ancestors precede their descendants in slot order).  Every thread calls it (red: scratch).
__device__ inline int2 tree_range(const DevState& s, const TreeUnit& u, const TreeRow& q, int base, int N, int lane,
                                  int wave, int (*red)[kTreeWaves]) {
  if (lane == 0) {
    red[0][wave] = q.hi;
    red[1][wave] = q.dmin;
  }
  __syncthreads();
  int hi = 0, dmin = INT_MAX;
  for (int w = 0; w < kTreeWaves; ++w) {
    hi = max(hi, red[0][w]);
    dmin = min(dmin, red[1][w]);
  }
  hi = __builtin_amdgcn_readfirstlane(hi);
  dmin = __builtin_amdgcn_readfirstlane(dmin);
  return make_int2(__builtin_amdgcn_readfirstlane(hi > 0 ? window_lo(s, u.t, base, N, dmin) : 0), hi);
}

// The lane's query row as B operands of S^T: half hh of its d range.
template <int D>
__device__ inline void tree_query(const DevState& s, const AttnArgs& a, const TreeUnit& u, const TreeRow& q, int G, int hh,
                                  bf16x8 (&qv)[D / 16]) {
  const uint4* qp = reinterpret_cast<const uint4*>(
      static_cast<const __bf16*>(a.q) +
      ((((size_t)u.li * s.T + u.t) * a.qmax + (q.ok ? q.owner : 0)) * s.Hq + u.g * G + q.r % G) * D + hh * (D / 2));
#pragma unroll
  for (int k = 0; k < D / 16; ++k) {
    const uint4 v = q.ok ? qp[k] : make_uint4(0, 0, 0, 0);
    qv[k] = __builtin_bit_cast(bf16x8, v);
  }
}

// Whether key i of a tile (whose depths and masks the lanes hold, key by key) is visible to a row:
// in the range, no deeper, on every beam's path that the query is on (MASKS; before the end of the
// shared prefix every key is), and inside the window.  Branch-free: the test only selects.
template <bool MASKS>
__device__ inline bool tree_visible(const DevState& s, const TreeRow& q, int i, bool in_range, int depths, int mlo, int mhi) {
  const int dn = __builtin_amdgcn_ds_bpermute(i << 2, depths);
  bool ok = in_range & (dn <= q.depth) & ((s.W <= 0) | (q.depth - dn < s.W));
  if constexpr (MASKS) {
    const uint32_t qlo = (uint32_t)q.mask, qhi = (uint32_t)(q.mask >> 32);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(i << 2, mlo);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(i << 2, mhi);
    ok &= ((lo & qlo) == qlo) & ((hi & qhi) == qhi);
  }
  return ok;
}

// A wave writes its own rows, O / l: zero for a row without keys or without a query; a NaN score makes
// l NaN, and the row with it.
template <int D>
__device__ inline void tree_output(const DevState& s, const AttnArgs& a, const TreeUnit& u, const TreeRow& q, int G, int hh,
                                   float lsum, const f32x16 (&o)[D / 32]) {
  lsum += __shfl_xor(lsum, 32);
  if (q.r >= a.qmax * G) return;
  const bool some = q.ok && lsum != 0.0f;
  const float inv = some ? 1.0f / lsum : 0.0f;
  __bf16* orow = static_cast<__bf16*>(a.out) +
                 ((((size_t)u.li * s.T + u.t) * a.qmax + q.owner) * s.Hq + u.g * G + q.r % G) * D;
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      bf16x4 y;
#pragma unroll
      for (int e = 0; e < 4; ++e) y[e] = (__bf16)(some ? o[dt][4 * q4 + e] * inv : 0.0f);
      *reinterpret_cast<bf16x4*>(orow + 32 * dt + 8 * q4 + 4 * hh) = y;
    }
}

}  // namespace td
