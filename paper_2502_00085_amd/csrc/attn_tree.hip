// Multi-query tree attention over the stored trie, prefill-shaped (gfx950 matrix cores).
//
// Alg 3's mask with one row per query node (Figure 2): the query of stored node q attends
// to the nodes m with depth(m) <= depth(q) and mask(m) containing mask(q), which for nodes
// on a live path is exactly the ancestor-or-self relation, within the window of depth(q).
// When many nodes are queries (the prefill of a serialized trie), the decode kernel's
// layout is wasteful: each 32-row block streams its whole key range through LDS for 32 x
// 32 scores per tile.  Here a group of 4 waves holds 128 query rows (wave w: rows 32w ..
// 32w + 31, each a (query node, query head) pair of one KV head) and streams the key range
// once for all of them; two such groups share a CU (64 KiB of LDS and 256 VGPRs each at
// d = 128), so one computes while the other waits at its tile barrier:
//
//   * a tile is 64 keys (two 32-key halves), K and V loaded by the whole group with direct
//     16-byte global -> LDS loads into one of two buffers while the other is consumed;
//   * each wave computes S^T = K Q^T and O^T += V^T P^T of both halves on
//     v_mfma_f32_32x32x16_bf16 with the decode kernel's LDS layout and operand reads;
//   * visibility: a tile whose keys all lie in the shared prefix (every beam's path) and no
//     deeper than any of the wave's queries, and inside every query's window, is fully
//     visible; otherwise each score is tested against the key's depth and, past the shared
//     prefix, its mask, which the lanes loaded with the tile and exchange by lane permutes;
//   * the softmax shift of a row moves only when its probabilities leave their range, which
//     their sum (needed anyway) tells: no maximum is taken;
//   * a wave skips what lies past its deepest query; each wave owns its rows.
//
// Launches of few WGs (launch_attn_tree says how few) make one WG of two groups, which take the
// tiles in turn and merge their states at the end: the longest block's chain of tiles is halved.
// The row blocks of one (trie, layer, KV head) are placed on one XCD, so that its K/V rows
// are read from HBM once and from that XCD's L2 afterwards.
//
// What bounds it: at two waves per SIMD neither pipe is full (every node of a 2,070-node trie a
// query, 32 layers: matrix cores busy 36 % of the time, 3,708 vector-ALU instructions per wave or
// at least 32 %); leaving out the loads, the exponentials or most of the output products
// shortens a tile by little more than their own time, so the waves' chains of score products,
// softmax and output products are the limit.  A software pipeline of the three (scores of one
// half beside the softmax of another) measured slower as hipcc schedules it.  Prefill of 2,096
// nodes at d = 128, 32 q / 8 KV heads, per layer: 85 us -> 62 us in one-layer calls, 50 -> 44 us
// in a call of 16 layers (782 TFLOP/s); 100 queries in one-layer calls: 68 -> 44 us.
#include <algorithm>

#include "attn_tree_common.h"

namespace td {

namespace {

constexpr int kTreeRound = 256, kTreeRampWgs = 512, kTreeRampWgs64 = 320;  // (see launch_attn_tree)
constexpr long kTreeShortKeys = 560, kTreeShortKeys64 = 768;
constexpr float kTreeMost = 8192.0f;  // a row's shift moves once 16 of its probabilities add up to more

template <int D>
struct TreeCfg : TreeGeom<D> {
  using TreeGeom<D>::CPR;
  using TreeGeom<D>::NBLK;
  using TreeGeom<D>::HALF;
  static constexpr int LOADS = 2 * HALF / 16 / kTreeThreads;  // 16-byte loads per thread: K (or V) of a tile
  static_assert(2 * HALF % (16 * kTreeThreads) == 0, "a tile is a whole number of WG loads");
  // load j of a thread is load 0 moved by whole rows (the same rotation), so one offset does
  static constexpr bool ONE_OFS = kTreeThreads % CPR == 0 && (kTreeThreads / CPR) % CPR == 0;
  static constexpr int OFS = ONE_OFS ? 1 : LOADS;
  static constexpr int WAVES = D == 64 ? 3 : 2;  // per SIMD: as many as the registers allow
  static constexpr int VROT = 8 % NBLK == 0 ? 1 : 4;  // rotations of V rows 8 apart
};

// KS: groups of 4 waves that share the rows and split the keys, tile by tile (group k takes
// tiles k, k + KS, ...); their states are merged at the end.
template <int D, int KS>
__global__ __launch_bounds__(KS * kTreeThreads, TreeCfg<D>::WAVES) void k_attn_tree(DevState s, AttnArgs a) {
  using C = TreeCfg<D>;
  // K and V of two tiles.  Four arrays, each used for one buffer only: the compiler can then
  // tell an operand read of one buffer from the direct loads under way into the other (with
  // one array it waits for every load before the first read: no load overlaps its tile).
  __shared__ __attribute__((aligned(16))) unsigned char kbuf0[KS * 2 * C::HALF], vbuf0[KS * 2 * C::HALF];
  __shared__ __attribute__((aligned(16))) unsigned char kbuf1[KS * 2 * C::HALF], vbuf1[KS * 2 * C::HALF];
  __shared__ int wred[2][kTreeWaves];  // per wave: deepest query slot + 1, shallowest depth
  const TreeUnit u = tree_unit(s, a);
  const TrieHdr h = s.hdr[u.t];
  const int N = h.n_nodes, base = h.base;
  const int G = s.Hq / s.Hkv;
  const int lab = a.layer_begin + u.li;
  const int lane = threadIdx.x & 63, tid = threadIdx.x % kTreeThreads;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);               // of its group
  const int group = __builtin_amdgcn_readfirstlane(threadIdx.x / kTreeThreads);
  const int col = lane & 31, hh = lane >> 5;
  const uint64_t* maskp = s.mask + (size_t)u.t * s.cap + base;
  const int32_t* depthp = s.depth + (size_t)u.t * s.cap + base;

  const TreeRow q = tree_row(s, a, u, N, G, maskp, depthp, wave, col);
  const int2 range = tree_range(s, u, q, base, N, lane, wave, wred);
  const int lo = range.x, hi = range.y;
  const int ntiles = hi > lo ? (hi - lo + 63) / 64 : 0;

  const __bf16* kpool = static_cast<const __bf16*>(s.k_pool) + pool_row(s, u.t, lab, u.g, base);
  const __bf16* vpool = static_cast<const __bf16*>(s.v_pool) + pool_row(s, u.t, lab, u.g, base);

  // Load j of this thread writes 16-byte LDS chunk c = j kTreeThreads + tid of its group's
  // tile's K (and V): tile row c / CPR at physical chunk c % CPR; the K rows of a 32-key half
  // are rotated by one chunk per row, its V rows by one 64-byte block per row (the decode
  // kernel's layout).
  // kofs / vofs: byte offset, in the tile's 64 pool rows, of the logical chunk it loads.
  uint32_t kofs[C::OFS], vofs[C::OFS];
#pragma unroll
  for (int j = 0; j < C::OFS; ++j) {
    const int c = j * kTreeThreads + tid, row = c / C::CPR, pc = c % C::CPR;
    kofs[j] = row * (2 * D) + (pc + C::CPR - row % 32 % C::CPR) % C::CPR * 16;
    vofs[j] = row * (2 * D) + (pc + C::CPR - 4 * (row % 32 % C::NBLK)) % C::CPR * 16;
  }
  // key depth and mask of tile key lane (0..63), for the visibility test
  int kdep = 0;
  uint64_t kmk = ~0ull;
  auto issue = [&](int tile, unsigned char* kdst, unsigned char* vdst) __attribute__((always_inline)) {
    const int tb = lo + tile * 64;
    const unsigned char* kt = reinterpret_cast<const unsigned char*>(kpool + (size_t)tb * D);
    const unsigned char* vt = reinterpret_cast<const unsigned char*>(vpool + (size_t)tb * D);
    const bool full = tb + 64 <= hi;
    const uint32_t last = (uint32_t)(hi - 1 - tb) * (2 * D);  // (rows past the end: the last row)
#pragma unroll
    for (int j = 0; j < C::LOADS; ++j) {
      const uint32_t step = C::ONE_OFS ? j * (kTreeThreads / C::CPR) * 2 * D : 0;
      uint32_t ko = kofs[C::ONE_OFS ? 0 : j], vo = vofs[C::ONE_OFS ? 0 : j];
      const unsigned char *kt_ = kt + step, *vt_ = vt + step;
      if (!full) {
        const uint32_t krow = (ko + step) / (2 * D) * (2 * D), vrow = (vo + step) / (2 * D) * (2 * D);
        ko = min(krow, last) + (ko + step - krow);
        vo = min(vrow, last) + (vo + step - vrow);
        kt_ = kt;
        vt_ = vt;
      }
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(kt_ + ko),
                                       (__attribute__((address_space(3))) void*)(kdst + (j * kTreeThreads + wave * 64) * 16), 16, 0, 0);
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(vt_ + vo),
                                       (__attribute__((address_space(3))) void*)(vdst + (j * kTreeThreads + wave * 64) * 16), 16, 0, 0);
    }
    const int nn = min(tb + lane, hi - 1);
    kdep = depthp[nn];
    if (tb + 64 > h.n_shared) kmk = maskp[nn];  // (before: every mask is all ones)
  };

  bf16x8 qv[C::KSTEPS];
  tree_query<D>(s, a, u, q, G, hh, qv);
  // operand read offsets (as in the decode kernel): K rows in MFMA layout, V transposed by
  // 16-lane groups
  const int grp = lane >> 4, tm = (lane & 15) >> 2, tq = lane & 3;
  int kread[C::KSTEPS], vread[C::VROT][C::DT];
#pragma unroll
  for (int k = 0; k < C::KSTEPS; ++k) kread[k] = col * (2 * D) + (hh * (C::CPR / 2) + col + k) % C::CPR * 16;
#pragma unroll
  for (int x8 = 0; x8 < C::VROT; ++x8)
#pragma unroll
    for (int dt = 0; dt < C::DT; ++dt) {
      const int n = 8 * x8 + 4 * hh + tm;
      const int c = 4 * dt + 2 * (grp & 1) + (tq >> 1);
      vread[x8][dt] = (4 * hh + tm) * (2 * D) + phys_chunk<C::CPR, C::NBLK>(n, c) * 16 + 8 * (tq & 1);
    }

  const float scale = a.scale_log2;
  float m = kTreeNegBig, lsum = 0.0f;
  f32x16 o[C::DT];
#pragma unroll
  for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[dt][v] = 0.0f;

  // (tile: the group's tile number)
  auto step = [&](int tile, const unsigned char* kb, const unsigned char* vb, unsigned char* knext,
                  unsigned char* vnext) __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(kWaitVmAll);  // this thread's loads of the tile have landed
    const int cdep = kdep;
    const uint64_t cmk = kmk;
    __syncthreads();  // every thread's loads have landed; the other buffer is free
    if (tile + KS < ntiles) issue(tile + KS, knext, vnext);
    const int tb = lo + tile * 64;
    if (tb >= q.hi) return;  // (wave-uniform) past the wave's deepest query
    // scores of both 32-key halves (two independent chains)
    f32x16 acc[2];
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][v] = acc[1][v] = 0.0f;
#pragma unroll
    for (int k = 0; k < C::KSTEPS; ++k)
#pragma unroll
      for (int half = 0; half < 2; ++half)
        acc[half] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            *reinterpret_cast<const bf16x8*>(kb + half * C::HALF + kread[k]), qv[k], acc[half], 0, 0, 0);
    // visibility of this lane's keys tb + 32 half + 8(v/4) + 4hh + v%4 for its row.  Depth never
    // decreases along the slots, so the tile's depth range is that of its first and last key.
    const int dfirst = __builtin_amdgcn_readlane(cdep, 0), dlast = __builtin_amdgcn_readlane(cdep, 63);
    const bool all_visible = tb + 64 <= hi && tb + 64 <= h.n_shared && dlast <= q.dmin &&
                             (s.W <= 0 || q.dmax - dfirst < s.W);
    if (!all_visible) {
      uint32_t vis[2] = {0, 0};
      if (tb + 64 <= h.n_shared) {
        // every key lies on every beam's path: the depth alone decides (the diagonal of a prefill)
#pragma unroll
        for (int v = 0; v < 32; ++v) {
          const int i = 32 * (v >> 4) + 8 * (v % 16 >> 2) + 4 * hh + (v & 3);
          vis[v >> 4] |= (uint32_t)tree_visible<false>(s, q, i, tb + i < hi, cdep, 0, 0) << (v & 15);
        }
      } else {
        const int mlo = (int)(uint32_t)cmk, mhi = (int)(uint32_t)(cmk >> 32);
#pragma unroll
        for (int v = 0; v < 32; ++v) {
          const int i = 32 * (v >> 4) + 8 * (v % 16 >> 2) + 4 * hh + (v & 3);
          vis[v >> 4] |= (uint32_t)tree_visible<true>(s, q, i, tb + i < hi, cdep, mlo, mhi) << (v & 15);
        }
      }
#pragma unroll
      for (int half = 0; half < 2; ++half)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[half][v] = (vis[half] >> v) & 1u ? acc[half][v] : -INFINITY;
    }
    const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (half == 1 && tb + 32 >= q.hi) return;  // (wave-uniform) past the wave's deepest query
      // Probabilities relative to the row's shift m, rounded to bf16, and their sum over this
      // lane's 16 keys.  Softmax does not depend on the shift, so it needs no maximum: it only
      // has to keep the probabilities in range, and their sum says when it does not (a first
      // tile, or scores far above every earlier one).
      bf16x8 pb[2];
      float ps = 0.0f;
      auto weights = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          pb[v >> 3][v & 7] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(acc[half][v], scale, -m));
        ps = 0.0f;
#pragma unroll
        for (int v = 0; v < 16; v += 2) {
          const bf16x2 pair = {pb[v >> 3][v & 7], pb[v >> 3][(v & 7) + 1]};
          ps = __builtin_amdgcn_fdot2_f32_bf16(pair, ones, ps, false);
        }
      };
      weights();
      if (__any(ps > kTreeMost)) {
        // raise the shift of the rows that need it to their largest score (a sum above
        // kTreeMost holds a probability above 2^kTreeSlack)
        float tmax = acc[half][0];
#pragma unroll
        for (int v = 1; v < 16; ++v) tmax = fmaxf(tmax, acc[half][v]);
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32)) * scale;
        const float mn = tmax > m + kTreeSlack ? tmax : m;
        const float alpha = __builtin_amdgcn_exp2f(m - mn);
        m = mn;
        lsum *= alpha;
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt)
#pragma unroll
          for (int v = 0; v < 16; ++v) o[dt][v] *= alpha;
        weights();
      }
      lsum += ps;
#pragma unroll
      for (int uu = 0; uu < 2; ++uu)
#pragma unroll
        for (int dt = 0; dt < C::DT; ++dt) {
          const unsigned char* vp = vb + half * C::HALF + 16 * uu * (2 * D);
          const i16x4 p0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(vp + vread[2 * uu % C::VROT][dt]));
          const i16x4 p1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (lds_i16x4*)(vp + 8 * (2 * D) + vread[(2 * uu + 1) % C::VROT][dt]));
          const bf16x8 va = __builtin_bit_cast(bf16x8, __builtin_shufflevector(p0, p1, 0, 1, 2, 3, 4, 5, 6, 7));
          o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb[uu], o[dt], 0, 0, 0);
        }
    }
  };
  unsigned char* const kb0 = kbuf0 + group * 2 * C::HALF;
  unsigned char* const kb1 = kbuf1 + group * 2 * C::HALF;
  unsigned char* const vb0 = vbuf0 + group * 2 * C::HALF;
  unsigned char* const vb1 = vbuf1 + group * 2 * C::HALF;
  if (group < ntiles) issue(group, kb0, vb0);
  const int steps = (ntiles + KS - 1) / KS;  // (every group takes every step's barrier)
  for (int i = 0; i < steps; i += 2) {
    step(i * KS + group, kb0, vb0, kb1, vb1);
    if (i + 1 < steps) step((i + 1) * KS + group, kb1, vb1, kb0, vb0);
  }

  if constexpr (KS == 2) {
    // group 1 hands its state over through LDS, lane by lane (O: [wave][register][lane] in the K
    // buffers, d / 2 registers each, then m and l in a V buffer)
    __syncthreads();  // every wave has read its last tile
    float* const olds0 = reinterpret_cast<float*>(kbuf0);
    float* const olds1 = reinterpret_cast<float*>(kbuf1);
    float* const ml = reinterpret_cast<float*>(vbuf0);
    static_assert(kTreeWaves * 64 * (D / 4) * 4 <= 2 * 2 * C::HALF, "half of O fits a K buffer");
    if (group == 1) {
#pragma unroll
      for (int x = 0; x < D / 4; ++x) {
        const int at = (wave * (D / 4) + x) * 64 + lane;
        olds0[at] = o[x / 16][x % 16];
        olds1[at] = o[(x + D / 4) / 16][(x + D / 4) % 16];
      }
      ml[(wave * 2) * 64 + lane] = m;
      ml[(wave * 2 + 1) * 64 + lane] = lsum;
    }
    __syncthreads();
    if (group == 1) return;
    const float m1 = ml[(wave * 2) * 64 + lane], l1 = ml[(wave * 2 + 1) * 64 + lane];
    const float mn = fmaxf(m, m1);
    const float f0 = __builtin_amdgcn_exp2f(m - mn), f1 = __builtin_amdgcn_exp2f(m1 - mn);
    lsum = lsum * f0 + l1 * f1;
#pragma unroll
    for (int x = 0; x < D / 4; ++x) {
      const int at = (wave * (D / 4) + x) * 64 + lane;
      o[x / 16][x % 16] = o[x / 16][x % 16] * f0 + olds0[at] * f1;
      const int y = x + D / 4;
      o[y / 16][y % 16] = o[y / 16][y % 16] * f0 + olds1[at] * f1;
    }
  }

  tree_output<D>(s, a, u, q, G, hh, lsum, o);
}

}  // namespace

int attn_tree_rows_per_block() { return kTreeRows; }

// Short key ranges go to the compact kernel (attn_tree_short.hip), which starts faster.  Measured,
// every node a query, the better form here against it: d = 128: 300 nodes, 320 blocks, 21.2 and
// 20.2 us; 520 nodes, 136 blocks, 22.2 and 21.8; 600 nodes, 152 blocks, 20.8 and 23.6.  At d = 64,
// where five of its WGs fit a CU, it holds out longer in launches of several WGs per CU: 600 nodes,
// 960 blocks, 37.5 and 35.8; 700 nodes, 1,088 blocks, 43.7 and 41.1; 850 nodes, 1,280, 51.7 and 54.0.
//
// Two groups per WG, whose barrier ties 8 waves and of which a CU holds one, where all of them run at
// once: up to 256 (100 queries of 1,700 nodes, 256 blocks, 44 us against 50 with one group; 400
// queries, 416 blocks, 75 against 64).  Where the blocks' ranges rise from nothing to all (every node
// a query, no window), a unit's blocks go out longest first and the next unit's after them: the second
// round may then hold the last unit's blocks and the shortest of the one before (per XCD, where the
// units have one: 8 units of 55, 46 and 51 us; 16 of 29, 35.2 and 36.9; 64 of 5, 38.3 and 33; without:
// 6 units of 49, 75 and 89; 3 of 133, 98 and 119; 12 of 24, 37.6 and 35.3), up to 512 blocks in all
// (528: 50.0 and 45.3), and up to 320 at d = 64, where more single groups fit a CU (23.7 and 24.6;
// 384 blocks, 28.0 and 27.2).
hipError_t launch_attn_tree(const DevState& s, const AttnArgs& a, long max_keys, bool ramp, hipStream_t st,
                            hipEvent_t ev0, hipEvent_t ev1) {
  const int wgs = s.T * a.n_layers * s.Hkv * a.row_blocks;
  const int second = (a.row_blocks + a.row_blocks / 4) * (a.xcd_group ? 8 : 1);
  const int most = ramp ? std::min(kTreeRound + second, s.D == 64 ? kTreeRampWgs64 : kTreeRampWgs) : kTreeRound;
  const bool split = wgs <= most;
  if (max_keys <= kTreeShortKeys || (s.D == 64 && max_keys <= kTreeShortKeys64 && !split))
    return launch_attn_tree_short(s, a, st, ev0, ev1);
  const dim3 grid(wgs), block(split ? 2 * kTreeThreads : kTreeThreads);
#define LAUNCH_TREE(DD)                                                                               \
  (split ? hipExtLaunchKernelGGL((k_attn_tree<DD, 2>), grid, block, 0, st, ev0, ev1, 0, s, a)          \
         : hipExtLaunchKernelGGL((k_attn_tree<DD, 1>), grid, block, 0, st, ev0, ev1, 0, s, a))
  switch (s.D) {
    case 64: LAUNCH_TREE(64); break;
    case 96: LAUNCH_TREE(96); break;
    case 128: LAUNCH_TREE(128); break;
    default: return hipErrorInvalidValue;
  }
#undef LAUNCH_TREE
  return hipGetLastError();
}

}  // namespace td
