// Multi-query tree attention over short key ranges, prefill-shaped (gfx950 matrix cores).
//
// The contract, the row layout and the placement are those of k_attn_tree (attn_tree.hip): a WG
// of 4 waves holds 128 (query node, query head) rows of one KV head, 32 per wave, and streams
// 64-key tiles through two LDS buffers; the row blocks of a unit go to one XCD.  This kernel is
// the compact one: a tile's 32-key halves are one loop body, taken one after the other with one
// half's operands live at a time, where k_attn_tree unrolls both halves of two tiles.
//
// What bounds it: latency, of a chain of few tiles.  k_attn_tree's longer code and its repeated
// first weights (it takes no maximum) only pay over long chains.  Measured, 32 q / 8 KV heads at
// d = 128, every node a query: 60 nodes 8.0 us here, 9.9 there; 200 nodes, 448 blocks, 19.4
// and 20.7; 300 nodes, 80 blocks, 15.6 and 15.7; 1,000 nodes, 256 blocks, 35.4 and 28.1.
#include "attn_tree_common.h"

namespace td {

namespace {

template <int D>
struct TreeCfg : TreeGeom<D> {
  using TreeGeom<D>::HALF;
  static constexpr int TILE = 4 * HALF;                 // K half 0, K half 1, V half 0, V half 1
  static constexpr int LOADS = TILE / 16 / kTreeThreads;  // 16-byte loads per thread per tile
  static_assert(TILE % (16 * kTreeThreads) == 0, "a tile is a whole number of WG loads");
};

template <int D>
__global__ __launch_bounds__(kTreeThreads, 2) void k_attn_tree_short(DevState s, AttnArgs a) {
  using C = TreeCfg<D>;
  __shared__ __attribute__((aligned(16))) unsigned char lds[2 * C::TILE];
  __shared__ int wred[2][kTreeWaves];  // per wave: deepest query slot + 1, shallowest depth
  const TreeUnit u = tree_unit(s, a);
  const TrieHdr h = s.hdr[u.t];
  const int N = h.n_nodes, base = h.base;
  const int G = s.Hq / s.Hkv;
  const int lab = a.layer_begin + u.li;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = lane & 31, hh = lane >> 5;
  const uint64_t* maskp = s.mask + (size_t)u.t * s.cap + base;
  const int32_t* depthp = s.depth + (size_t)u.t * s.cap + base;

  const TreeRow q = tree_row(s, a, u, N, G, maskp, depthp, wave, col);
  const bool any_dead = __ballot(!q.ok) != 0ull;
  const int2 range = tree_range(s, u, q, base, N, lane, wave, wred);
  const int lo = range.x, hi = range.y;
  const int ntiles = hi > lo ? (hi - lo + 63) / 64 : 0;

  const __bf16* kpool = static_cast<const __bf16*>(s.k_pool) + pool_row(s, u.t, lab, u.g, base);
  const __bf16* vpool = static_cast<const __bf16*>(s.v_pool) + pool_row(s, u.t, lab, u.g, base);

  // Load j of this thread writes LDS chunk c = kTreeThreads j + threadIdx.x of the tile: part c /
  // (HALF / 16) (K half 0, K half 1, V half 0, V half 1), row and physical chunk inside it;
  // K rows rotated by one chunk per row, V rows by one 64-byte block per row (the decode
  // kernel's layout).  ld[j]: tile row (bits 0-7), element offset of the logical chunk in
  // its row (bits 8-15), V (bit 16).
  int ld[C::LOADS];
#pragma unroll
  for (int j = 0; j < C::LOADS; ++j) {
    const int c = j * kTreeThreads + (int)threadIdx.x;
    const int part = c / (C::HALF / 16), p = c % (C::HALF / 16);
    const int row = p / C::CPR, pc = p % C::CPR;
    const bool isv = part >= 2;
    const int off = isv ? (pc + C::CPR - 4 * (row % C::NBLK)) % C::CPR * 8 : (pc + C::CPR - row % C::CPR) % C::CPR * 8;
    ld[j] = ((part & 1) * 32 + row) | (off << 8) | (isv ? 1 << 16 : 0);
  }
  // key depth and mask of tile key lane (0..63), for the visibility test
  int kdep = 0;
  uint64_t kmk = 0;
  auto issue = [&](int tile, int buf) {
    const int tb = lo + tile * 64;
    unsigned char* dst = lds + buf * C::TILE;
#pragma unroll
    for (int j = 0; j < C::LOADS; ++j) {
      const int n = min(tb + (ld[j] & 255), hi - 1);
      const __bf16* src = ((ld[j] >> 16) ? vpool : kpool) + (size_t)n * D + ((ld[j] >> 8) & 255);
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                       (__attribute__((address_space(3))) void*)(dst + (j * kTreeThreads + wave * 64) * 16),
                                       16, 0, 0);
    }
    const int nn = min(tb + lane, hi - 1);
    kdep = depthp[nn];
    kmk = maskp[nn];
  };

  bf16x8 qv[C::KSTEPS];
  tree_query<D>(s, a, u, q, G, hh, qv);
  // operand geometry (as in the decode kernel): K rows read in MFMA layout; V read back
  // transposed by 16-lane groups
  const int grp = lane >> 4, tm = (lane & 15) >> 2, tq = lane & 3;
  const int krow = col * (2 * D), kc0 = hh * (C::CPR / 2) + col;  // K operand k: chunk (kc0 + k) % CPR

  const float scale = a.scale_log2;
  float m = kTreeNegBig, lsum = 0.0f;
  f32x16 o[C::DT];
#pragma unroll
  for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[dt][v] = 0.0f;

  if (ntiles > 0) issue(0, 0);
  for (int tile = 0; tile < ntiles; ++tile) {
    const int buf = tile & 1;
    __builtin_amdgcn_s_waitcnt(kWaitVmAll);  // this thread's loads of the tile have landed
    const int cdep = kdep;
    const uint64_t cmk = kmk;
    __syncthreads();  // every thread's loads have landed; the other buffer is free
    if (tile + 1 < ntiles) issue(tile + 1, buf ^ 1);
    const int tb = lo + tile * 64;
    const unsigned char* kb = lds + buf * C::TILE;
    const unsigned char* vb = kb + 2 * C::HALF;
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {  // (not unrolled: one half's operands live at a time)
      const int hb = tb + half * 32;  // first key of the half
      if (hb >= q.hi) continue;       // (wave-uniform) past the wave's deepest query
      const unsigned char* kh = kb + half * C::HALF;
      const __bf16* vh = reinterpret_cast<const __bf16*>(vb + half * C::HALF);
      bf16x8 kv[C::KSTEPS];
#pragma unroll
      for (int k = 0; k < C::KSTEPS; ++k) kv[k] = *reinterpret_cast<const bf16x8*>(kh + krow + (kc0 + k) % C::CPR * 16);
      bf16x8 va[2][C::DT];
#pragma unroll
      for (int uu = 0; uu < 2; ++uu) {
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt) {
          i16x4 part[2];
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            const int n = 16 * uu + 8 * hf + 4 * hh + tm;
            const int c = 4 * dt + 2 * (grp & 1) + (tq >> 1);
            const int pc = phys_chunk<C::CPR, C::NBLK>(n, c);
            part[hf] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(vh + n * D + pc * 8 + 4 * (tq & 1)));
          }
          va[uu][dt] = __builtin_bit_cast(bf16x8, __builtin_shufflevector(part[0], part[1], 0, 1, 2, 3, 4, 5, 6, 7));
        }
      }
      f32x16 acc;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
#pragma unroll
      for (int k = 0; k < C::KSTEPS; ++k) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kv[k], qv[k], acc, 0, 0, 0);

      // visibility of this lane's keys hb + 8(v/4) + 4hh + v%4 for its row.  Depth never
      // decreases along the slots, so the half's depth range is that of its first and last
      // key (lanes 32 half and 32 half + 31 hold them).
      const int dfirst = __builtin_amdgcn_readlane(cdep, 32 * half);
      const int dlast = __builtin_amdgcn_readlane(cdep, 32 * half + 31);
      const bool all_visible = hb + 32 <= hi && hb + 32 <= h.n_shared && dlast <= q.dmin &&
                               (s.W <= 0 || q.dmax - dfirst < s.W);
      if (all_visible) {
        if (any_dead) {
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[v] = q.ok ? acc[v] : -INFINITY;
        }
      } else {
        const int mlo = (int)(uint32_t)cmk, mhi = (int)(uint32_t)(cmk >> 32);
        uint32_t vis = 0;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int i = 32 * half + 8 * (v >> 2) + 4 * hh + (v & 3);
          vis |= (uint32_t)tree_visible<true>(s, q, i, tb + i < hi, cdep, mlo, mhi) << v;
        }
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = (vis >> v) & 1u ? acc[v] : -INFINITY;
      }
      float tmax = acc[0];
#pragma unroll
      for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, acc[v]);
      tmax = fmaxf(tmax, __shfl_xor(tmax, 32)) * scale;
      // The row's shift m moves up only when a score exceeds it by more than kTreeSlack
      // (log2 units): the probabilities stay <= 2^kTreeSlack, and O and l are rescaled on
      // few tiles instead of on nearly every one (softmax does not depend on the shift).
      const bool raise = tmax > m + kTreeSlack;
      float alpha = 1.0f;
      if (__any(raise)) {
        const float mn = raise ? tmax : m;
        alpha = __builtin_amdgcn_exp2f(m - mn);
        m = mn;
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
          for (int v = 0; v < 16; ++v) o[dt][v] *= alpha;
      }
      const float mn = m;
      bf16x8 pb[2];
#pragma unroll
      for (int v = 0; v < 16; ++v) pb[v >> 3][v & 7] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(acc[v], scale, -mn));
      float ps = 0.0f;
      const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        const bf16x2 pair = {pb[v >> 3][v & 7], pb[v >> 3][(v & 7) + 1]};
        ps = __builtin_amdgcn_fdot2_f32_bf16(pair, ones, ps, false);
      }
      lsum = lsum * alpha + ps;
#pragma unroll
      for (int uu = 0; uu < 2; ++uu)
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt)
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[uu][dt], pb[uu], o[dt], 0, 0, 0);
    }
  }

  tree_output<D>(s, a, u, q, G, hh, lsum, o);
}

}  // namespace

hipError_t launch_attn_tree_short(const DevState& s, const AttnArgs& a, hipStream_t st, hipEvent_t ev0,
                                  hipEvent_t ev1) {
  const dim3 grid(s.T * a.n_layers * s.Hkv * a.row_blocks), block(kTreeThreads);
  switch (s.D) {
    case 64: hipExtLaunchKernelGGL(k_attn_tree_short<64>, grid, block, 0, st, ev0, ev1, 0, s, a); break;
    case 96: hipExtLaunchKernelGGL(k_attn_tree_short<96>, grid, block, 0, st, ev0, ev1, 0, s, a); break;
    case 128: hipExtLaunchKernelGGL(k_attn_tree_short<128>, grid, block, 0, st, ev0, ev1, 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace td
