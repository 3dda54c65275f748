// Trie attention on the fp32 matrix instructions (gfx950): fp32 storage, and bf16 storage at
// the head dims the bf16 matrix-core kernel does not implement; fp32 arithmetic throughout.
//
// The contract is that of the other decode kernels (Section 3.3, Alg 3's mask as one 64-bit
// ancestor mask per node).  A WG owns one (trie, layer, KV head, block of 16 or 32 query
// rows, node split); its waves take interleaved tiles of 16 nodes.  Both contractions run on
// v_mfma_f32_16x16x4_f32 (fp32 operands, products and sums), so a node's row meets every
// query row of the block in registers:
//
//   S^T[node][row] = K . Q^T    A = K rows (lane group l / 16 holds a quarter of the row, so
//                               one 16-byte LDS read feeds four or eight steps), B = Q from LDS
//   O^T[d][row]   += V^T . P^T  A = V straight from HBM: lane l % 16 holds D/16 consecutive
//                               elements of nodes 4 (l / 16) + v, one whole row per 16 lanes;
//                               B = P^T, the S^T accumulators as they are
//
// What bounds it: HBM, when the rows fill the block (32 rows at d = 128 need 16 bytes per
// clock and CU of K/V at the full fp32 matrix rate, more than HBM delivers), else latency.
// The vector-ALU kernel spends about 45 instructions per 4 nodes and query row and reads each
// node once per 8 rows; attn_kernel below says where it still is the better one.  Measured, 8 layers of
// 32 q / 8 KV heads at d = 128, 8 beams, 2,080 nodes in fp32 (139 MB), merge included: 293 us
// there, 48 us here (2.9 TB/s); bf16 at d = 32, 16 beams: 192 us and 27 us.  Error against
// 64 bits over d = 32 .. 256: 1.3e-7 .. 2.0e-7, there 1.3e-7 .. 2.7e-7.
//
// K goes HBM -> the wave's LDS tile by direct loads, V HBM -> registers.  The next tile's K is
// requested once this one's scores are done, its V once this one's products are: with two
// waves per SIMD one wave's loads overlap the other's matrix work.
#include <algorithm>
#include <type_traits>

#include "attn_common.h"
#include "mfma_tile.h"

namespace td {

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr float kNegBig32 = -1.0e30f;
constexpr int kTile32 = 16;  // nodes per wave tile

// Waves of a WG over rt 16-row tiles: past these d, 8 waves' merge buffers exceed the LDS, or their
// registers the file.
constexpr int waves32(int d, int rt) { return d > (rt == 2 ? 128 : 192) ? 4 : 8; }

template <typename T, int D, int RT>
struct Cfg32 {
  static constexpr int NW = waves32(D, RT);
  static constexpr int ROWS = 16 * RT;
  static constexpr int EPC = 16 / (int)sizeof(T);       // elements per 16-byte chunk
  static constexpr int CPR = D / EPC;                   // chunks per node row
  static constexpr int KL = kTile32 * CPR / 64;         // 16-byte loads per lane of a K tile
  static constexpr int EPL = D / 16;                    // V elements per lane and node
  static constexpr int VWORDS = EPL * (int)sizeof(T) / 4;
  static constexpr int K_TILE = kTile32 * D * (int)sizeof(T);  // bytes of a wave's K tile
  static constexpr int QSTRIDE = D * 4 + 16;               // bytes of an LDS Q row (fp32)
  static constexpr int OS = D + 4;                         // floats of an LDS O row
  static constexpr int Q_LDS = ROWS * QSTRIDE;
  static constexpr int K_LDS = NW * K_TILE;
  static constexpr int O_LDS = NW * ROWS * OS * 4 + (3 * NW + 2) * ROWS * 4;
  static constexpr int LDS = Q_LDS + K_LDS > O_LDS ? Q_LDS + K_LDS : O_LDS;
  static_assert(LDS <= 160 * 1024 - 256, "LDS of one WG per CU");
};

template <typename T>
__device__ inline float word_elem(uint32_t w, int e) {
  if constexpr (sizeof(T) == 4) return __uint_as_float(w);
  return __uint_as_float(e == 0 ? w << 16 : w & 0xffff0000u);
}

// W consecutive words by the widest loads their count allows (the address is aligned to them).
template <int W>
__device__ inline void load_words(const uint32_t* p, uint32_t* w) {
  if constexpr (W % 4 == 0) {
#pragma unroll
    for (int i = 0; i < W / 4; ++i) {
      const u32x4 x = reinterpret_cast<const u32x4*>(p)[i];
#pragma unroll
      for (int e = 0; e < 4; ++e) w[4 * i + e] = x[e];
    }
  } else if constexpr (W % 2 == 0) {
#pragma unroll
    for (int i = 0; i < W / 2; ++i) {
      const uint2 x = reinterpret_cast<const uint2*>(p)[i];
      w[2 * i] = x.x;
      w[2 * i + 1] = x.y;
    }
  } else {
#pragma unroll
    for (int i = 0; i < W; ++i) w[i] = p[i];
  }
}

template <typename T, int D, int RT>
__global__ __launch_bounds__((Cfg32<T, D, RT>::NW * 64), (Cfg32<T, D, RT>::NW / 4)) void k_attn_mfma32(DevState s, AttnArgs a) {
  using C = Cfg32<T, D, RT>;
  constexpr int NW = C::NW;
  constexpr int EW = 4 / (int)sizeof(T);  // elements per 32-bit word
  __shared__ __attribute__((aligned(16))) unsigned char lds[C::LDS];
  const AttnUnit u = attn_unit(s, a);
  const TrieHdr h = s.hdr[u.t];
  const int N = h.n_nodes, base = h.base, n_live = h.n_live;
  const int G = s.Hq / s.Hkv;
  const int lab = a.layer_begin + u.li;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, grp = lane >> 4;

  // rows moved by the last compaction (this WG is the only one of its layer and head), before
  // the leaf store, whose slots may be sources of moves
  if (a.moves) move_rows_block<T>(s, u.t, lab, u.g, reinterpret_cast<uint4*>(lds), C::LDS / 16);
  if (a.kv_pending && u.split == 0 && u.rb == 0) store_leaf_kv<T>(s, a, u, base, N, n_live);

  // this WG's nodes: whole tiles, over only as many splits as give each wave one (unless the
  // split count is forced); the other splits mark their partials empty and leave
  const int lo = window_lo(s, u.t, base, N, h.leaf_depth, reinterpret_cast<int*>(lds));
  const int span = N - lo, tiles = (span + kTile32 - 1) / kTile32;
  const int act = a.all_splits ? a.splits : min(a.splits, max(1, (tiles + NW - 1) / NW));
  float* part = s.attn_part + ((size_t)u.unit * a.splits + u.split) * C::ROWS * (D + 2);
  if (u.split >= act) {
    if ((int)threadIdx.x < C::ROWS) {
      part[threadIdx.x * (D + 2) + D] = kNegBig32;
      part[threadIdx.x * (D + 2) + D + 1] = 0.0f;
    }
    return;
  }
  const int per = (tiles + act - 1) / act * kTile32;
  const int n0 = lo + u.split * per, n1 = min(N, n0 + per);
  const int ntiles = n1 > n0 ? (n1 - n0 + kTile32 - 1) / kTile32 : 0;
  const int my_tiles = ntiles > wave ? (ntiles - wave + NW - 1) / NW : 0;

  const T* kpool = static_cast<const T*>(s.k_pool) + pool_row(s, u.t, lab, u.g, base);
  const T* vpool = static_cast<const T*>(s.v_pool) + pool_row(s, u.t, lab, u.g, base);
  const size_t leaf_off = (((size_t)u.li * s.T + u.t) * s.b * s.Hkv + u.g) * D;  // leaf 0 of k_new
  const T* knew = static_cast<const T*>(a.k_new) + leaf_off;
  const T* vnew = static_cast<const T*>(a.v_new) + leaf_off;
  const int leaf_stride = s.Hkv * D;
  const int leaf0 = a.kv_pending ? N - n_live : N;
  const uint64_t* maskp = s.mask + (size_t)u.t * s.cap + base;

  // K of a tile: direct global -> LDS loads, 1 KiB per instruction; LDS chunk p = 64 i + lane
  // is tile row p / CPR at physical chunk p % CPR, each row rotated by its number, so that
  // the operand reads of 16 rows use different banks
  unsigned char* kbuf = lds + C::Q_LDS + wave * C::K_TILE;
  auto load_k = [&](int tile) __attribute__((always_inline)) {
    const int tb = n0 + tile * kTile32;
    const bool inside = tb + kTile32 <= n1 && tb + kTile32 <= leaf0;  // 16 pool rows in place
#pragma unroll
    for (int i = 0; i < C::KL; ++i) {
      int ln = lane;
      asm volatile("" : "+v"(ln));  // (the geometry is recomputed per load, not held)
      const int p = 64 * i + ln, row = p / C::CPR;
      const int c = (p % C::CPR + C::CPR - row % C::CPR) % C::CPR;
      const T* src;
      if (inside) {
        src = kpool + (size_t)tb * D + (row * D + c * C::EPC);
      } else {  // (rows past the end repeat the last node, and are masked out)
        const int n = min(tb + row, n1 - 1);
        src = (n >= leaf0 ? knew + (size_t)(n - leaf0) * leaf_stride : kpool + (size_t)n * D) + c * C::EPC;
      }
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                       (__attribute__((address_space(3))) void*)(kbuf + i * 1024), 16, 0, 0);
    }
  };
  // V of a tile (nodes 4 grp + v of it) into registers, and past the shared prefix the masks
  uint32_t vr[4][C::VWORDS];
  uint64_t mk[4] = {~0ull, ~0ull, ~0ull, ~0ull};
  auto load_v = [&](int tile) __attribute__((always_inline)) {
    const int tb = n0 + tile * kTile32;
    if (tb + kTile32 <= n1 && tb + kTile32 <= leaf0) {
      const T* vp = vpool + (size_t)tb * D + (4 * grp * D + col * C::EPL);
#pragma unroll
      for (int v = 0; v < 4; ++v) load_words<C::VWORDS>(reinterpret_cast<const uint32_t*>(vp + v * D), vr[v]);
    } else {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int n = min(tb + 4 * grp + v, n1 - 1);
        const T* row = n >= leaf0 ? vnew + (size_t)(n - leaf0) * leaf_stride : vpool + (size_t)n * D;
        load_words<C::VWORDS>(reinterpret_cast<const uint32_t*>(row + col * C::EPL), vr[v]);
      }
    }
    if (tb + kTile32 > n1 || tb + kTile32 > h.n_shared) {
#pragma unroll
      for (int v = 0; v < 4; ++v) mk[v] = maskp[min(tb + 4 * grp + v, n1 - 1)];
    }
  };
  __syncthreads();  // the search's scratch is free
  if (my_tiles > 0) {
    load_k(wave);
    load_v(wave);
  }

  // the block's query rows in fp32: row r is beam r / G, query head g * G + r % G
  unsigned char* qlds = lds;
  {
    const T* qb = static_cast<const T*>(a.q);
    for (int idx = threadIdx.x; idx < C::ROWS * (D / C::EPC); idx += NW * 64) {
      const int i = idx / (D / C::EPC), c = idx % (D / C::EPC);
      const int r = u.rb * C::ROWS + i, bm = r / G;
      u32x4 x = {0, 0, 0, 0};
      if (r < s.b * G && bm < n_live)
        x = *reinterpret_cast<const u32x4*>(
            qb + ((((size_t)u.li * s.T + u.t) * s.b + bm) * s.Hq + u.g * G + r % G) * D + c * C::EPC);
      float* dst = reinterpret_cast<float*>(qlds + i * C::QSTRIDE) + c * C::EPC;
#pragma unroll
      for (int w = 0; w < 4; w += 4 / EW) {
        f32x4 f;
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e] = word_elem<T>(x[w + e / EW], e % EW);
        *reinterpret_cast<f32x4*>(dst + w * EW) = f;
      }
    }
  }
  __syncthreads();

  // this lane's query rows (one per 16-row tile) and their beams' bits
  int bit[RT];
  bool rok[RT];
#pragma unroll
  for (int k = 0; k < RT; ++k) {
    const int r = u.rb * C::ROWS + 16 * k + col;
    bit[k] = r / G < 64 ? r / G : 63;
    rok[k] = r < s.b * G && r / G < n_live;
  }
  const unsigned char* qread = qlds + col * C::QSTRIDE + grp * D;
  const float scale = a.scale_log2;
  float m[RT], lsum[RT];
  f32x4 o[RT][C::EPL];
#pragma unroll
  for (int k = 0; k < RT; ++k) {
    m[k] = kNegBig32;
    lsum[k] = 0.0f;
#pragma unroll
    for (int e = 0; e < C::EPL; ++e) o[k][e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }

  for (int it = 0; it < my_tiles; ++it) {
    const int tile = wave + NW * it, tb = n0 + tile * kTile32;
    __builtin_amdgcn_s_waitcnt(kWaitVmAll);  // this tile has landed
    // A score's sum over d: pieces of 8 elements (two steps from a fresh accumulator), four of
    // them added pairwise, then added up.  One long chain would round half as much again as the
    // vector-ALU kernel's 8 elements per lane and tree over the lanes; this rounds no more.
    f32x4 acc[RT];
#pragma unroll
    for (int k = 0; k < RT; ++k) acc[k] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
    for (int c = 0; c < D / 32; ++c) {  // (a loop: unrolled, its operands spill)
      f32x4 piece[RT][4];
      u32x4 kc[8 / C::EPC];
#pragma unroll
      for (int i = 0; i < 8 / C::EPC; ++i) {
        // (logical chunk of row col, rotated by col; an unsigned minimum wraps it)
        const uint32_t u0 = grp * (C::CPR / 4) + c * (8 / C::EPC) + i + col % C::CPR;
        kc[i] = *reinterpret_cast<const u32x4*>(kbuf + col * (D * (int)sizeof(T)) + min(u0, u0 - C::CPR) * 16);
      }
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int k = 0; k < RT; ++k) {
          const f32x4 qc = *reinterpret_cast<const f32x4*>(qread + 16 * k * C::QSTRIDE + (2 * c + x) * 16);
          piece[k][2 * x] = piece[k][2 * x + 1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int w = 4 * x + e;  // element of the group's 8
            const float ke = word_elem<T>(kc[w / C::EPC][w % C::EPC / EW], w % EW);
            f32x4& f = piece[k][2 * x + (e & 1)];
            f = __builtin_amdgcn_mfma_f32_16x16x4f32(ke, qc[e], f, 0, 0, 0);
          }
        }
#pragma unroll
      for (int k = 0; k < RT; ++k) acc[k] += (piece[k][0] + piece[k][1]) + (piece[k][2] + piece[k][3]);
    }
    __builtin_amdgcn_s_waitcnt(kWaitLgkmAll);  // the tile's K has been read: the next one's K
    if (it + 1 < my_tiles) load_k(tile + NW);
    const bool masked = tb + kTile32 > n1 || tb + kTile32 > h.n_shared;
    float p[RT][4];
    uint32_t vis[RT];  // bit v: node 4 grp + v is visible to this lane's row
#pragma unroll
    for (int k = 0; k < RT; ++k) {
      float sc[4];
      vis[k] = 15u;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        sc[v] = acc[k][v];
        if (masked) {
          const int n = tb + 4 * grp + v;
          const bool ok = (n < n1) & ((n < h.n_shared) | (((mk[v] >> bit[k]) & 1ull) != 0));
          vis[k] &= ok ? 15u : ~(1u << v);
          sc[v] = ok ? sc[v] : -INFINITY;
        }
      }
      float t = fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3]));
      t = fmaxf(t, __shfl_xor(t, 16));
      t = fmaxf(t, __shfl_xor(t, 32));
      const float mn = fmaxf(m[k], t * scale);
      const float alpha = __builtin_amdgcn_exp2f(m[k] - mn);
      m[k] = mn;
      float ps = 0.0f;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        p[k][v] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[v], scale, -mn));
        ps += p[k][v];
      }
      lsum[k] = lsum[k] * alpha + ps;
      if (__any(alpha != 1.0f)) {
#pragma unroll
        for (int e = 0; e < C::EPL; ++e) o[k][e] *= alpha;
      }
    }
    // A hidden node weighs 0, but 0 times an infinite or NaN V is NaN: a tile with hidden nodes
    // and such a V adds its products node by node, where the node is visible.
    bool slow = false;
    if (masked) {
      bool odd = false;
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int e = 0; e < C::EPL; ++e) odd |= !(fabsf(word_elem<T>(vr[v][e / EW], e % EW)) < INFINITY);
      slow = __any(odd);
      if (slow) {
#pragma unroll 1
        for (int g = 0; g < 4; ++g) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
#pragma unroll
            for (int k = 0; k < RT; ++k) {
              const bool own = __shfl((int)((vis[k] >> v) & 1u), g * 16 + col) != 0;
#pragma unroll
              for (int e = 0; e < C::EPL; ++e) {
                uint32_t w = vr[v][e / EW];
                asm volatile("" : "+v"(w));  // (nothing of this rare path is prepared ahead)
                const float ve = grp == g ? word_elem<T>(w, e % EW) : 0.0f;
                const f32x4 f = __builtin_amdgcn_mfma_f32_16x16x4f32(ve, grp == g ? p[k][v] : 0.0f,
                                                                     f32x4{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
#pragma unroll
                for (int x = 0; x < 4; ++x) o[k][e][x] += own ? f[x] : 0.0f;
                __builtin_amdgcn_sched_barrier(0);
              }
            }
          }
        }
      }
    }
    if (!slow) {
    // (a tile's products in two accumulators of their own, then two additions: the output's
    // rounding error grows with the tiles, not with the nodes)
#pragma unroll
    for (int e = 0; e < C::EPL; ++e) {
#pragma unroll
      for (int k = 0; k < RT; ++k) {
        f32x4 f[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};
#pragma unroll
        for (int v = 0; v < 4; ++v)
          f[v & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(word_elem<T>(vr[v][e / EW], e % EW), p[k][v], f[v & 1], 0, 0, 0);
        o[k][e] += f[0] + f[1];
      }
      // (only vector-ALU work moves across: the products of two elements at a time are in flight)
      if (e % 2 == 1) __builtin_amdgcn_sched_barrier(6);
    }
    }
    if (it + 1 < my_tiles) load_v(tile + NW);
  }

  // ---- merge the waves: every wave stores its state, one combine ----
  // (lane: row col, elements (4 grp + v) EPL + e of d, i.e. the quarter grp of the row)
#pragma unroll
  for (int k = 0; k < RT; ++k) {
    lsum[k] += __shfl_xor(lsum[k], 16);
    lsum[k] += __shfl_xor(lsum[k], 32);
  }
  __syncthreads();
  float* obuf = reinterpret_cast<float*>(lds);  // [NW][ROWS][OS]
  float* smx = obuf + NW * C::ROWS * C::OS;      // [NW][ROWS] running max
  float* ssum = smx + NW * C::ROWS;              // [NW][ROWS] weight sum
  float* fw = ssum + NW * C::ROWS;               // [NW][ROWS] wave weight 2^(m_w - M)
  float* rowm = fw + NW * C::ROWS;               // [ROWS]
  float* rowl = rowm + C::ROWS;                  // [ROWS]
#pragma unroll
  for (int k = 0; k < RT; ++k) {
    const int i = wave * C::ROWS + 16 * k + col;
    if (grp == 0) {
      smx[i] = m[k];
      ssum[i] = rok[k] ? lsum[k] : 0.0f;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
      for (int e = 0; e < C::EPL; ++e) obuf[i * C::OS + (4 * grp + v) * C::EPL + e] = o[k][e][v];
  }
  __syncthreads();
  if ((int)threadIdx.x < C::ROWS) {
    const int i = threadIdx.x;
    float M = smx[i];
    for (int w = 1; w < NW; ++w) M = fmaxf(M, smx[w * C::ROWS + i]);
    float L = 0.0f;
    for (int w = 0; w < NW; ++w) {
      const float f = __builtin_amdgcn_exp2f(smx[w * C::ROWS + i] - M);
      fw[w * C::ROWS + i] = f;
      L += ssum[w * C::ROWS + i] * f;  // fixed wave order
    }
    rowm[i] = M;
    rowl[i] = L;
  }
  __syncthreads();
  T* outp = static_cast<T*>(a.out);
  for (int idx = threadIdx.x; idx < C::ROWS * (D / 4); idx += NW * 64) {
    const int i = idx / (D / 4), c = idx % (D / 4) * 4;
    f32x4 O = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = fw[w * C::ROWS + i];
      O += *reinterpret_cast<const f32x4*>(obuf + (w * C::ROWS + i) * C::OS + c) * f;
    }
    const float L = rowl[i];
    if (a.splits == 1) {
      const int r = u.rb * C::ROWS + i;
      if (r < s.b * G) {
        const int bm = r / G;
        const bool live = bm < n_live && L > 0.0f;
        T* dst = outp + ((((size_t)u.li * s.T + u.t) * s.b + bm) * s.Hq + u.g * G + r % G) * D + c;
        typedef T t4 __attribute__((ext_vector_type(4)));
        t4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = (T)(live ? O[e] / L : 0.0f);
        *reinterpret_cast<t4*>(dst) = y;
      }
    } else {
      float* pp = part + i * (D + 2);
#pragma unroll
      for (int e = 0; e < 4; ++e) pp[c + e] = O[e];
      if (c == 0) {
        pp[D] = rowm[i];
        pp[D + 1] = L;
      }
    }
  }
}

template <typename T, int RT>
hipError_t launch_rt(const DevState& s, const AttnArgs& a, dim3 grid, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1) {
  switch (s.D) {
#define MFMA32_CASE(DD)                                                                                        \
    case DD:                                                                                                   \
      hipExtLaunchKernelGGL((k_attn_mfma32<T, DD, RT>), grid, dim3(Cfg32<T, DD, RT>::NW * 64), 0, st, ev0, ev1, 0, \
                            s, a);                                                                              \
      break;
    MFMA32_CASE(32) MFMA32_CASE(160) MFMA32_CASE(192) MFMA32_CASE(224) MFMA32_CASE(256)
    case 64: case 96: case 128:
      if constexpr (sizeof(T) == 4) {  // (bf16: the bf16 matrix-core kernel's head dims)
        switch (s.D) { MFMA32_CASE(64) MFMA32_CASE(96) MFMA32_CASE(128) }
        break;
      }
      return hipErrorInvalidValue;
#undef MFMA32_CASE
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

// 32 query rows per WG, or 16 when there are no more.
int attn_mfma32_rows_per_block(const DevState& s) { return s.b * (s.Hq / s.Hkv) <= 16 ? 16 : 32; }

// Nodes of one round of a WG: a tile per wave.
static int round_nodes32(const DevState& s) {
  return waves32(s.D, attn_mfma32_rows_per_block(s) / 16) * kTile32;
}

// (a trie of at most one tile per wave of a WG needs no split, no partials and no merge launch)
int attn_mfma32_splits(const DevState& s, int n_layers, int row_blocks, long max_nodes) {
  const long round = round_nodes32(s), need = (max_nodes + round - 1) / round;
  return (int)std::max(1l, std::min<long>(attn_choose_splits(s, n_layers, row_blocks), need));
}

// bf16 at the bf16 kernel's head dims: that one.  Else this kernel or the vector-ALU one, by an
// estimate of either's chain of dependent work, in units of about 0.3 us.
//
//   vector ALU      its iterations (16 nodes of a WG's split) times 1 + 0.75 per query row of its
//                   block, twice as long for each further 512 WGs
//   this kernel     16 per round of tiles at d = 256 and 16 query rows (in proportion for other d;
//                   twice that for 32 rows), once per 256 WGs (its LDS leaves room for one per CU);
//                   a split launch: 8 more, for the merge of its partials
//
// This one wins wherever the rows fill its tiles and the nodes its waves.  It loses where a tile
// round is long beside the little there is to do: d past 128, where a WG has 4 waves and multiplies
// 16 or 32 rows whether they exist or not, and 32 rows at d = 96 and 128 in small calls.  One of its
// WGs with one round of 16 rows answers first at any d, and at d <= 128 no call of up to 16 rows was
// slower on it.
//
// Measured over 16,349 one-layer calls (both types, d = 64 .. 256, 1 .. 96 rows, 1 .. 512 units of 17
// .. 12,000 nodes), us, vector ALU and this kernel:
//   d = 256  32 rows, 1 unit, 190 nodes  12.3, 20.3 (bf16)     1 row, 352 units, 330 nodes  34.3, 79.6 (bf16)
//            16 rows, 24 units, 600 nodes  30.8, 17.2 (bf16)   4 rows, 128 units, 3,000 nodes  168, 152 (bf16)
//   d = 160  6 rows, 1 unit, 190 nodes  10.9, 13.2; 3,000 nodes  22.9, 17.1 (bf16)
//   d = 128  32 rows, 1 unit, 190 nodes  13.1, 16.4; 800 nodes  18.6, 15.9 (fp32)
// Over 6,529 other ones its choice takes 0.7 % longer than the faster kernel in the mean; always this
// one 5 %, always the vector ALU 55 %.
AttnKernel attn_kernel(const DevState& s, int attn_impl, int n_layers, long max_nodes) {
  if (attn_impl == TD_ATTN_VALU) return AttnKernel::kValu;
  if (s.dtype == TD_BF16 && mfma_head_dim(s.D)) return AttnKernel::kMfma;
  const int rows = s.b * (s.Hq / s.Hkv), tiles = attn_mfma32_rows_per_block(s) / 16;
  if (s.D <= 128 && tiles == 1) return AttnKernel::kMfma32;
  const long units = (long)s.T * n_layers * s.Hkv;
  auto up = [](long x, long y) { return (x + y - 1) / y; };

  const int vrows = attn_valu_rows_per_block(s.D), vblocks = (int)up(rows, vrows);
  const int vsplits = attn_choose_splits(s, n_layers, vblocks);
  const double valu = up(max_nodes, 16 * vsplits) * std::max(1.0, units * vblocks * vsplits / 512.0) *
                      (1.0 + 0.75 * std::min(rows, vrows));

  const int blocks = (int)up(rows, 16 * tiles);
  const int splits = attn_mfma32_splits(s, n_layers, blocks, max_nodes);
  const long rounds = up(max_nodes, (long)splits * round_nodes32(s)), wgs = units * blocks * splits;
  if (splits == 1 && rounds == 1 && tiles == 1 && wgs <= 256) return AttnKernel::kMfma32;
  const double mfma = 16.0 * rounds * up(wgs, 256) * tiles * s.D / 256 - (splits == 1 ? 8.0 : 0.0);
  return valu <= mfma ? AttnKernel::kValu : AttnKernel::kMfma32;
}

hipError_t launch_attn_mfma32(const DevState& s, const AttnArgs& a, hipStream_t st, hipEvent_t ev0,
                              hipEvent_t ev1) {
  const dim3 grid(s.T * a.n_layers * s.Hkv * a.row_blocks * a.splits);
  const bool one = attn_mfma32_rows_per_block(s) == 16;
  if (s.dtype == TD_F32)
    return one ? launch_rt<float, 1>(s, a, grid, st, ev0, ev1)
               : launch_rt<float, 2>(s, a, grid, st, ev0, ev1);
  return one ? launch_rt<__bf16, 1>(s, a, grid, st, ev0, ev1)
             : launch_rt<__bf16, 2>(s, a, grid, st, ev0, ev1);
}

}  // namespace td
