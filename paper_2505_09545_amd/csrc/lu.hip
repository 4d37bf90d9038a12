// Step (b) of the hot path: dense complex LU with partial pivoting and the
// multi-right-hand-side solve (arXiv:2505.09545, Sec. "Numerical solution": the
// system M F = F0 is solved by LU decomposition; many illuminations are solved
// at once, Sec. "Implementation technical details", batch evaluation).
//
// Algorithm: blocked right-looking getrf.  For each block of w columns at k0
//   1. panel: factor A[k0:n, k0:k0+w] with partial pivoting (pivot = largest
//      |re|+|im| in the column, lowest row on ties).  One cooperative launch of
//      G workgroups; each holds R rows of the panel in LDS and the workgroups
//      agree on every pivot through one device-wide exchange per column.
//   2. the panel also lists the block's net row permutation (<= 2w rows move,
//      read off the row labels), which is applied to the trailing columns and,
//      in the solve, to the right-hand sides.  Interchanges are never applied
//      to the columns left of the block: the factors are kept in the factored
//      form
//          M = P1^T L1 P2^T L2 ... Pk^T Lk U
//      and the solve applies P_b before using L_b, which is equivalent.
//   3. U12 = L11^-1 A12 (tiles.hip), 4. A22 -= L21 U12 (complex GEMM on MFMA,
//      gemm.hip; FP32 factors that are refined: update_split.hip; small updates:
//      solve_step.hip).  With look-ahead, step 3 and step 4 for the next panel's
//      columns run on the main stream and the rest of step 4 on a side stream,
//      overlapping the next panel.
//   5. after the last block, the solve-ready form of all blocks (tiles.hip).
//
// Layout: column-major interleaved complex, leading dimension ld.  ipiv holds
// 0-based global row indices (LAPACK semantics otherwise).
#include <algorithm>
#include <climits>
#include <map>
#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "gdm_common.hpp"
#include "gdm_kernels.hpp"
#include "lu_common.hpp"

namespace gdm {

constexpr uint32_t SPIN_LIMIT = 1u << 22;

__global__ void zero_u64_kernel(unsigned long long* a, size_t na, unsigned long long* b, size_t nb,
                                int32_t* c, size_t nc) {
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < na) a[i] = 0;
  if (i < nb) b[i] = 0;
  if (i < nc) c[i] = 0;
}

__global__ void init_err_kernel(int32_t* err) {
  if (threadIdx.x == 0) {
    err[0] = 0;
    err[1] = INT32_MAX;
  }
}

// ---------------------------------------------------------------------------
// 1. panel factorisation (cooperative, one device-wide exchange per column)
// ---------------------------------------------------------------------------
// Cross-workgroup exchange uses self-validating 64-bit words: the high 32 bits
// hold an epoch (unique per column of the whole factorisation), the low 32 bits
// the payload.  Words are written and read with agent-scope relaxed atomics; a
// reader spins on each word until it carries the epoch it expects, so no
// release/acquire fences (L2 write-back / invalidate) are needed.  Every buffer
// is double-buffered by column parity: a workgroup can only overwrite a slot of
// parity j%2 at column j+2, after every other workgroup has published its
// column j+1 key, i.e. after they all finished reading column j.
typedef unsigned long long u64;
// each workgroup's key words get their own 128-byte line (no false sharing
// between the atomic stores of different workgroups)
constexpr int KEY_STRIDE = 16;

__device__ inline void ll_put(u64* p, uint32_t epoch, uint32_t payload) {
  __hip_atomic_store(p, ((u64)epoch << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Spin until the word carries `epoch`; returns the payload (0 and sets *bad on timeout).
__device__ inline uint32_t ll_get(const u64* p, uint32_t epoch, int* bad) {
  uint32_t it = 0;
  while (true) {
    const u64 v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((uint32_t)(v >> 32) == epoch) return (uint32_t)v;
    if (++it > SPIN_LIMIT) {
      *bad = 1;
      return 0;
    }
  }
}
// Several words at once: all loads are in flight together (one round trip when
// the data is already there); only words not yet carrying `epoch` are re-read.
template <int K>
__device__ inline void ll_get_n(const u64* const (&p)[K], uint32_t epoch, uint32_t (&out)[K], int* bad) {
  u64 v[K];
#pragma unroll
  for (int i = 0; i < K; ++i) v[i] = __hip_atomic_load(p[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  uint32_t it = 0;
  while (true) {
    bool all = true;
#pragma unroll
    for (int i = 0; i < K; ++i) all = all && (uint32_t)(v[i] >> 32) == epoch;
    if (all) break;
    if (++it > SPIN_LIMIT) {
      *bad = 1;
      break;
    }
#pragma unroll
    for (int i = 0; i < K; ++i)
      if ((uint32_t)(v[i] >> 32) != epoch) v[i] = __hip_atomic_load(p[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
#pragma unroll
  for (int i = 0; i < K; ++i) out[i] = (uint32_t)v[i];
}

// CPT records of KW consecutive words each (record u at base[u]), returned once
// every word carries `epoch`; all loads in flight together.  While some word is
// stale every word is loaded again (a word that already carries the epoch keeps
// it until this reader is done, so reloading it is harmless).
template <int KW, int CPT>
__device__ inline void ll_get_rec(const u64* const (&base)[CPT], uint32_t epoch, uint32_t (&out)[CPT * KW], int* bad) {
  u64 v[CPT * KW];
  auto load_all = [&]() {
    static_for<CPT * KW>([&](auto i) {
      v[i] = __hip_atomic_load(base[i / KW] + i % KW, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    });
  };
  load_all();
  uint32_t it = 0;
  while (true) {
    bool all = true;
    static_for<CPT * KW>([&](auto i) { all = all && (uint32_t)(v[i] >> 32) == epoch; });
    if (all) break;
    if (++it > SPIN_LIMIT) {
      *bad = 1;
      break;
    }
    load_all();
  }
  static_for<CPT * KW>([&](auto i) { out[i] = (uint32_t)v[i]; });
}

// K words at p[i] (any addresses), as ll_get_rec.
template <int K>
__device__ inline void ll_get_sel(const u64* const (&p)[K], uint32_t epoch, uint32_t (&out)[K], int* bad) {
  u64 v[K];
  auto load_all = [&]() {
    static_for<K>([&](auto i) { v[i] = __hip_atomic_load(p[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); });
  };
  load_all();
  uint32_t it = 0;
  while (true) {
    bool all = true;
    static_for<K>([&](auto i) { all = all && (uint32_t)(v[i] >> 32) == epoch; });
    if (all) break;
    if (++it > SPIN_LIMIT) {
      *bad = 1;
      break;
    }
    load_all();
  }
  static_for<K>([&](auto i) { out[i] = (uint32_t)v[i]; });
}

// complex values travel as their 32-bit words (2 for complex float, 4 for
// complex double), little-endian order of the (re, im) storage.
template <typename CT> __device__ inline uint32_t cword(const CT& v, int k) {
  return reinterpret_cast<const uint32_t*>(&v)[k];
}

// Rows never move between workgroups inside the panel: each local row carries a
// label, the position it will be written back to.  The interchange of column j
// (positions gj <-> p) swaps the labels of the two rows involved, which their
// owners do locally; the pivot row's values are the only data exchanged.
template <typename CT>
__device__ inline u64 pivot_key(const CT& v, uint32_t label) {
  const float a = (float)(fabs(v.x) + fabs(v.y));
  return ((u64)__float_as_uint(a) << 32) | (0xffffffffu - label);
}

// Wave-wide max of a 64-bit key with DPP moves: xor-1 and xor-2 within quads,
// then mirrors within 8 and 16 lanes leave every lane with the max of its row
// of 16; the four row maxima are combined with readlane.
template <int CTRL>
__device__ inline u64 dpp_u64(u64 v) {
  const int lo = __builtin_amdgcn_mov_dpp((int)(uint32_t)v, CTRL, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_mov_dpp((int)(uint32_t)(v >> 32), CTRL, 0xf, 0xf, false);
  return ((u64)(uint32_t)hi << 32) | (uint32_t)lo;
}
__device__ inline u64 wave_max_u64(u64 v) {
  u64 o;
  o = dpp_u64<0xb1>(v);  // quad_perm [1,0,3,2]
  v = o > v ? o : v;
  o = dpp_u64<0x4e>(v);  // quad_perm [2,3,0,1]
  v = o > v ? o : v;
  o = dpp_u64<0x141>(v);  // row_half_mirror
  v = o > v ? o : v;
  o = dpp_u64<0x140>(v);  // row_mirror
  v = o > v ? o : v;
  u64 r = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, 16 * q);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), 16 * q);
    const u64 x = ((u64)hi << 32) | lo;
    r = x > r ? x : r;
  }
  return r;
}

// Workgroup-wide argmax of (key, idx); one barrier.  Keys are unique (they end
// with the row label), so only the key is reduced and the lane holding the
// winning key publishes its idx.  skey/sidx: LDS arrays (4 entries) that the
// caller does not touch again before the next barrier.
__device__ inline void block_argmax(u64& key, int& idx, u64* skey, int* sidx) {
  const u64 k = wave_max_u64(key);
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) skey[wv] = k;
  if (key == k && k != 0) sidx[wv] = idx;
  __syncthreads();
  key = skey[0];
  int wbest = 0;
#pragma unroll
  for (int i = 1; i < 4; ++i)
    if (skey[i] > key) {
      key = skey[i];
      wbest = i;
    }
  idx = key ? sidx[wbest] : -1;
}

// The panel also lists the rows it moved, as (final position, original
// position) pairs: a row's label is its final position, so a workgroup knows
// its moved rows without replaying the interchanges.  Slots are claimed with an
// atomic counter (zeroed before the factorisation); the order of the list is
// irrelevant, since the permutation gathers every source before it scatters.
template <typename T>
__global__ void __launch_bounds__(256) panel_kernel(cplx<T>* __restrict__ A, int64_t ld, int64_t n, int64_t k0, int w,
                                                     int R, int G, int32_t* __restrict__ ipiv, LUWork ws,
                                                     uint32_t epoch0, int64_t sA, int64_t sipiv,
                                                     int32_t* __restrict__ mdst, int32_t* __restrict__ msrc,
                                                     int32_t* __restrict__ mcount, int mcap) {
  using CT = cplx<T>;
  // batch item blockIdx.y: its own matrix, pivots and exchange buffers
  A += (int64_t)blockIdx.y * sA;
  ipiv += (int64_t)blockIdx.y * sipiv;
  ws.cand += (int64_t)blockIdx.y * ws.s_cand;
  ws.rows += (int64_t)blockIdx.y * ws.s_rows;
  mdst += (int64_t)blockIdx.y * ws.s_pairs;
  msrc += (int64_t)blockIdx.y * ws.s_pairs;
  mcount += (int64_t)blockIdx.y * ws.s_npairs;
  constexpr int NW = sizeof(CT) / 4;  // payload words per complex
  extern __shared__ unsigned char smem_raw[];
  CT* tile = reinterpret_cast<CT*>(smem_raw);           // [w][R], column c at tile + c*R
  CT* prow = tile + (size_t)w * R;                      // [w] pivot row
  int32_t* lab = reinterpret_cast<int32_t*>(prow + w);  // [R] row labels (final positions)
  int32_t* pl = lab + R;                                // [w] pivot positions of this panel
  __shared__ u64 skey1[4], skey2[4];
  __shared__ int sidx1[4], sidx2[4];
  __shared__ int bad;
  const int g = blockIdx.x, tid = threadIdx.x;
  const int64_t rbase = k0 + (int64_t)g * R;
  const int myR = (int)(n - rbase < (int64_t)R ? (n - rbase > 0 ? n - rbase : 0) : R);
  if (tid == 0) bad = 0;
  // columns in batches of LB loads in flight per thread (a load followed by its
  // LDS store in one loop body would put one memory latency per column on the
  // panel's critical path)
  constexpr int LB = 128 / (int)sizeof(CT);
  const int wfull = w - w % LB;
  for (int lr = tid; lr < myR; lr += 256) {
    const CT* src = A + (rbase + lr) + k0 * ld;
    for (int c0 = 0; c0 < wfull; c0 += LB) {
      CT v[LB];
#pragma unroll
      for (int u = 0; u < LB; ++u) v[u] = src[(c0 + u) * ld];
#pragma unroll
      for (int u = 0; u < LB; ++u) tile[(c0 + u) * R + lr] = v[u];
    }
    for (int c = wfull; c < w; ++c) tile[c * R + lr] = src[c * ld];
  }
  for (int lr = tid; lr < myR; lr += 256) lab[lr] = (int32_t)(rbase + lr);
  // 2D mapping for the rank-1 update: RP rows x CG column groups
  int RP = 1;
  while (RP < myR && RP < 256) RP <<= 1;
  const int CG = 256 / RP;
  const int ulr0 = tid & (RP - 1), ucg = tid / RP;
  __syncthreads();
  // candidate of column 0
  u64 best = 0;
  int brow = -1;
  for (int lr = tid; lr < myR; lr += 256) {
    const u64 kk = pivot_key(tile[lr], (uint32_t)lab[lr]);
    if (kk > best) {
      best = kk;
      brow = lr;
    }
  }
  int zero_col = -1;
  // Column j's rank-1 update is split: column j + 1 right after the pivot is
  // known (it holds the next pivot candidates), the rest of the trailing
  // columns after the next candidate has been published, so that it runs while
  // the other workgroups' keys for column j + 1 are on their way.  Every row
  // receives every update exactly once: the candidate row gets its deferred part
  // when it is published, the other rows in the bulk step.
  for (int j = 0; j < w; ++j) {
    const int64_t gj = k0 + j;
    const uint32_t E = epoch0 + (uint32_t)j;
    const int par = j & 1;
    u64* cand = ws.cand + (size_t)par * ws.gitem * KEY_STRIDE;
    u64* rows = ws.rows + (size_t)par * ws.gitem * ws.wwmax;
    // workgroup candidate over its active rows (labels >= gj); column j is final
    block_argmax(best, brow, skey1, sidx1);
    const u64 mybest = best;
    const int lrow = best ? brow : -1;
    // publish key (value, label) and columns j.. of the candidate row; its
    // columns j + 1.. first receive the deferred update by pivot j - 1 (the
    // multipliers of pivot j - 1 sit in tile column j - 1)
    if (tid == 0) {
      ll_put(&cand[KEY_STRIDE * g + 0], E, mybest ? (uint32_t)(mybest >> 32) : 0u);
      ll_put(&cand[KEY_STRIDE * g + 1], E, mybest ? (0xffffffffu - (uint32_t)(mybest & 0xffffffffu)) : 0xffffffffu);
    }
    const int WC = w - j;  // columns still needed by the others
    if (lrow >= 0)
      for (int tc = tid; tc < WC; tc += 256) {
        const int c = j + tc;
        CT v = tile[c * R + lrow];
        if (j > 0 && tc > 0) {
          v = r1_upd(v, tile[(j - 1) * R + lrow], prow[c]);
          tile[c * R + lrow] = v;
        }
#pragma unroll
        for (int q = 0; q < NW; ++q) ll_put(&rows[(size_t)g * ws.wwmax + (size_t)tc * NW + q], E, cword(v, q));
      }
    // deferred part of pivot j - 1's update: columns j + 1.. of the other active rows
    if (j > 0) {
      for (int lr = ulr0; lr < myR; lr += RP) {
        if (lab[lr] <= (int32_t)(gj - 1) || lr == lrow) continue;
        const CT l = tile[(j - 1) * R + lr];
        int c = j + 1 + ucg;
        // FP32: batches of UB columns, all reads first, then the updates, then
        // all writes (written one column at a time, each read would wait for
        // the previous column's write, since the compiler cannot tell them
        // apart).  The same batching makes the FP64 panel slower, so FP64 keeps
        // the column-at-a-time loop.
        constexpr int UB = 8;
        if constexpr (sizeof(T) == 4) {
          for (; c + (UB - 1) * CG < w; c += UB * CG) {
            CT t[UB], u[UB];
#pragma unroll
            for (int e = 0; e < UB; ++e) {
              u[e] = prow[c + e * CG];
              t[e] = tile[(c + e * CG) * R + lr];
            }
#pragma unroll
            for (int e = 0; e < UB; ++e) t[e] = r1_upd(t[e], l, u[e]);
#pragma unroll
            for (int e = 0; e < UB; ++e) tile[(c + e * CG) * R + lr] = t[e];
          }
          for (; c < w; c += CG) tile[c * R + lr] = r1_upd(tile[c * R + lr], l, prow[c]);
        } else {
#pragma unroll 8
          for (; c < w; c += CG) tile[c * R + lr] = r1_upd(tile[c * R + lr], l, prow[c]);
        }
      }
    }
    // gather all keys; winner = largest |re|+|im|, lowest label on ties (the
    // barrier inside block_argmax also ends every read of prow above)
    u64 k = 0;
    int owner = -1;
    if (tid < G) {
      const u64* const pk[2] = {&cand[KEY_STRIDE * tid + 0], &cand[KEY_STRIDE * tid + 1]};
      uint32_t vk[2];
      ll_get_n<2>(pk, E, vk, &bad);
      k = ((u64)vk[0] << 32) | (0xffffffffu - vk[1]);
      owner = tid;
    }
    block_argmax(k, owner, skey2, sidx2);
    const int gp = owner;
    const uint32_t plabel = 0xffffffffu - (uint32_t)(k & 0xffffffffu);
    // pivot row, columns j..
    if (gp >= 0) {
      const int WW = WC * NW;
      const u64* src = rows + (size_t)gp * ws.wwmax;
      uint32_t* dstw = reinterpret_cast<uint32_t*>(prow + j);
      int t = tid;
      for (; t + 256 < WW; t += 512) {
        const u64* const pw[2] = {src + t, src + t + 256};
        uint32_t vw[2];
        ll_get_n<2>(pw, E, vw, &bad);
        dstw[t] = vw[0];
        dstw[t + 256] = vw[1];
      }
      if (t < WW) dstw[t] = ll_get(src + t, E, &bad);
    }
    // interchange of positions gj <-> plabel: swap labels (each row by one thread)
    if (plabel != (uint32_t)gj) {
      for (int lr = tid; lr < myR; lr += 256) {
        const int32_t lb = lab[lr];
        if (lb == (int32_t)gj) lab[lr] = (int32_t)plabel;
        else if (g == gp && lr == lrow) lab[lr] = (int32_t)gj;
      }
    }
    if (tid == 0) pl[j] = (int32_t)plabel;
    __syncthreads();
    if (bad || gp < 0) {
      if (tid == 0) __hip_atomic_store(&ws.err[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    const CT piv = prow[j];
    const bool zero = piv.x == 0 && piv.y == 0;
    if (zero && zero_col < 0) zero_col = j;
    CT inv;
    if (zero) { inv.x = 0; inv.y = 0; } else inv = cinv_t(piv);
    // multipliers of the rows below (labels > gj) into tile column j, and the
    // update of column j + 1 with the next pivot candidates
    best = 0;
    brow = -1;
    const bool nxt = j + 1 < w;
    const CT u1 = nxt ? prow[j + 1] : piv;
    for (int lr = tid; lr < myR; lr += 256) {
      const int32_t lb = lab[lr];
      if (lb <= (int32_t)gj) continue;
      const CT l = cmul_t(tile[j * R + lr], inv);
      tile[j * R + lr] = l;
      if (nxt) {
        const CT t = r1_upd(tile[(j + 1) * R + lr], l, u1);
        tile[(j + 1) * R + lr] = t;
        const u64 kk = pivot_key(t, (uint32_t)lb);
        if (kk > best) {
          best = kk;
          brow = lr;
        }
      }
    }
    // (the barrier inside the next block_argmax orders these writes before any read)
  }
  __syncthreads();
  if (g == 0) {
    for (int j = tid; j < w; j += 256) ipiv[k0 + j] = pl[j];
    if (tid == 0 && zero_col >= 0) atomicMin(&ws.err[1], (int)(k0 + zero_col));
  }
  for (int lr = tid; lr < myR; lr += 256) {
    const int32_t orig = (int32_t)(rbase + lr);
    if (lab[lr] != orig) {
      const int slot = __hip_atomic_fetch_add(mcount, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (slot < mcap) {
        mdst[slot] = lab[lr];
        msrc[slot] = orig;
      }
    }
  }
  for (int lr = tid; lr < myR; lr += 256) {
    CT* dst = A + lab[lr] + k0 * ld;
    for (int c0 = 0; c0 < wfull; c0 += LB) {
      CT v[LB];
#pragma unroll
      for (int u = 0; u < LB; ++u) v[u] = tile[(c0 + u) * R + lr];
#pragma unroll
      for (int u = 0; u < LB; ++u) dst[(c0 + u) * ld] = v[u];
    }
    for (int c = wfull; c < w; ++c) dst[c * ld] = tile[c * R + lr];
  }
}

// ---------------------------------------------------------------------------
// 1a. the same panel with the column loop in one wave (at most 64 rows per workgroup)
// ---------------------------------------------------------------------------
// The panel is taken in sub-panels of SUBW columns.  Wave 0 runs a sub-panel's
// columns by itself, one row per lane with its SUBW entries in registers, so a
// column has no barrier: choice of the candidate (DPP), its key, then its row
// and the reciprocal of its pivot published; the other workgroups' keys; the
// winner's row, which goes through LDS to every lane; multipliers and the rank-1
// update of at most SUBW - 1 columns.  The remaining columns of the panel are
// updated once per sub-panel, by all four waves: the owners publish the pivot
// rows' entries there, every workgroup subtracts L11 times the earlier U rows (one
// column per thread), then the rank-SUBW update goes to the matrix cores.
// What bounds it is the chain of a column: the key's trip through memory to
// workgroups on other dies (0.75 us of waiting behind the rank-1 update that it
// overlaps), the load of the winner's row (0.4) and the choice of the next
// candidate (0.35).  n = 3001: 2.5 us per column in FP32, 2.8 in FP64; panel_kernel,
// with three barriers per column and all remaining columns updated from LDS, 2.9
// and 5.1.  (Any 24 to 56 rows per workgroup measure the same.)
//
// Exchange buffers: keys as in panel_kernel; rows [2][gitem][SUBW NW] words, the
// record of a workgroup's candidate: multipliers of the sub-panel's columns before
// j, the reciprocal of the pivot in place of column j, the columns after it; then the pivot
// rows' remaining columns [2][SUBW][wwmax], double-buffered by the parity of the
// sub-panel (an owner writes a slot again after the keys of a whole sub-panel,
// which every workgroup publishes after it has read the slot).
constexpr int SUBW = 16;
// words between two workgroups' keys: 4 workgroups to a 128-byte line (a line each: 12.0
// instead of 11.7 ms for n = 3001 in FP64, since every workgroup reads them all)
constexpr int PW_KEYS = 4;

template <typename CT>
static __host__ __device__ inline size_t panel_wave_lds(int w, int R) {
  const int rest = w > SUBW ? w - SUBW : 0;
  return ((size_t)w * R + (size_t)SUBW * rest + SUBW * (SUBW + 1) + 64) * sizeof(CT) + (size_t)(R + w + SUBW) * 4;
}

__device__ inline uint32_t wave_max_u32(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xb1, 0xf, 0xf, false));   // quad_perm [1,0,3,2]
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4e, 0xf, 0xf, false));   // quad_perm [2,3,0,1]
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xf, 0xf, false));  // row_half_mirror
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xf, 0xf, false));  // row_mirror
  const uint32_t a = __builtin_amdgcn_readlane((int)v, 0), b = __builtin_amdgcn_readlane((int)v, 16);
  const uint32_t c = __builtin_amdgcn_readlane((int)v, 32), d = __builtin_amdgcn_readlane((int)v, 48);
  return max(max(a, b), max(c, d));
}
// The largest key of the wave and a lane that holds it (-1 if it is 0): the upper
// words first, the lower ones only if they tie.
__device__ inline u64 wave_argmax(u64 key, int& src) {
  const uint32_t hi = wave_max_u32((uint32_t)(key >> 32));
  unsigned long long who = __ballot((uint32_t)(key >> 32) == hi);
  if (__builtin_popcountll(who) != 1) {
    const uint32_t lo = wave_max_u32((uint32_t)(key >> 32) == hi ? (uint32_t)key : 0u);
    who = __ballot((uint32_t)(key >> 32) == hi && (uint32_t)key == lo);
  }
  const int l = (int)__builtin_ctzll(who);
  const u64 k = ((u64)hi << 32) | (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)key, l);
  src = k ? l : -1;
  return k;
}

// the keys of all workgroups, KPL per lane: the winner's key and workgroup
template <int KPL>
__device__ inline u64 gather_keys(const u64* cand, int G, uint32_t E, int lane, int& gp, int* bad) {
  const u64* pk[2 * KPL];
  uint32_t v[2 * KPL];
#pragma unroll
  for (int i = 0; i < KPL; ++i) {
    const int g = lane + 64 * i < G ? lane + 64 * i : lane % G;
    pk[2 * i] = cand + PW_KEYS * g;
    pk[2 * i + 1] = pk[2 * i] + 1;
  }
  ll_get_n<2 * KPL>(pk, E, v, bad);
  u64 best = 0;
  int bg = 0;
#pragma unroll
  for (int i = 0; i < KPL; ++i) {
    const u64 k = ((u64)v[2 * i] << 32) | (0xffffffffu - v[2 * i + 1]);
    if (k > best) {
      best = k;
      bg = lane + 64 * i < G ? lane + 64 * i : lane % G;
    }
  }
  int src;
  const u64 k = wave_argmax(best, src);
  gp = src >= 0 ? __builtin_amdgcn_readlane(bg, src) : -1;
  return k;
}

template <typename T>
__global__ void __launch_bounds__(256) panel_wave_kernel(cplx<T>* __restrict__ A, int64_t ld, int64_t n, int64_t k0, int w,
                                                          int R, int G, int32_t* __restrict__ ipiv, LUWork ws,
                                                          uint32_t epoch0, int32_t* __restrict__ mdst,
                                                          int32_t* __restrict__ msrc, int32_t* __restrict__ mcount, int mcap) {
  using CT = cplx<T>;
  constexpr int NW = sizeof(CT) / 4, RW = SUBW * NW;  // words per complex, per record
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int restmax = w > SUBW ? w - SUBW : 0;
  CT* tile = reinterpret_cast<CT*>(smem_raw);              // [w][R]
  CT* ub = tile + (size_t)w * R;                           // [SUBW][restmax] pivot rows, then U, right of the sub-panel
  CT* lp = ub + (size_t)SUBW * restmax;                    // [SUBW][SUBW] the pivot rows' records, SUBW unused
  CT* spare = lp + SUBW * (SUBW + 1);                      // [64] takes the stores past a sub-panel's last column
  int32_t* lab = reinterpret_cast<int32_t*>(spare + 64);   // [R] row labels (final positions)
  int32_t* pl = lab + R;                                   // [w] pivot positions
  int32_t* mine = pl + w;                                  // [SUBW] local row of the sub-panel's pivot, or -1
  __shared__ int bad;
  const int g = blockIdx.x, tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t rbase = k0 + (int64_t)g * R;
  const int myR = (int)(n - rbase < (int64_t)R ? (n - rbase > 0 ? n - rbase : 0) : R);
  if (tid == 0) bad = 0;
  // a wave's lanes are rows; columns dealt to the waves, LB loads in flight
  constexpr int LB = 128 / (int)sizeof(CT);
  if (lane < myR) {
    const CT* src = A + rbase + lane + k0 * ld;
    for (int c0 = wave; c0 < w; c0 += 4 * LB) {
      CT v[LB];
#pragma unroll
      for (int u = 0; u < LB; ++u) v[u] = src[(int64_t)(c0 + 4 * u < w ? c0 + 4 * u : w - 1) * ld];
#pragma unroll
      for (int u = 0; u < LB; ++u)
        if (c0 + 4 * u < w) tile[(c0 + 4 * u) * R + lane] = v[u];
    }
  }
  if (tid < myR) lab[tid] = (int32_t)(rbase + tid);
  __syncthreads();
  int zero_col = -1;  // wave 0
  u64* const ubase = ws.rows + 2 * (size_t)ws.gitem * RW;
  for (int s0 = 0, sp = 0; s0 < w; s0 += SUBW, sp ^= 1) {
    const int sw = w - s0 < SUBW ? w - s0 : SUBW;
    if (wave == 0) {
      int32_t mylab = lane < myR ? lab[lane] : -1;
      if (lane < SUBW) mine[lane] = -1;
      CT x[SUBW];  // this row's columns j, j + 1, ... (shifted along with j)
#pragma unroll
      for (int c = 0; c < SUBW; ++c) {
        x[c].x = x[c].y = 0;
        if (lane < myR && c < sw) x[c] = tile[(s0 + c) * R + lane];
      }
      // this workgroup's candidate of column j (its entries in v), its key published
      auto candidate = [&](int j, const CT& v) -> int {
        const uint32_t E = epoch0 + (uint32_t)(s0 + j);
        u64* cand = ws.cand + (size_t)((s0 + j) & 1) * ws.gitem * PW_KEYS + PW_KEYS * g;
        int src;
        const u64 k = wave_argmax(mylab >= (int32_t)(k0 + s0 + j) ? pivot_key(v, (uint32_t)mylab) : 0, src);
        if (lane < 2)
          ll_put(cand + lane, E, lane ? (k ? 0xffffffffu - (uint32_t)k : 0xffffffffu) : (uint32_t)(k >> 32));
        return src;
      };
      int lrow = candidate(0, x[0]);
      int late = 0;  // a word did not come
      for (int j = 0; j < sw; ++j) {
        const int32_t gj = (int32_t)(k0 + s0 + j);
        const uint32_t E = epoch0 + (uint32_t)(s0 + j);
        const int par = (s0 + j) & 1;
        const u64* cand = ws.cand + (size_t)par * ws.gitem * PW_KEYS;
        u64* rows = ws.rows + (size_t)par * ws.gitem * RW;
        if (lrow >= 0 && lane < RW) {
          // (the row's earlier columns are its multipliers, the later ones are current)
          const int c = s0 + lane / NW;
          const CT* e = tile + (size_t)(c < w ? c : w - 1) * R + lrow;
          uint32_t word = reinterpret_cast<const uint32_t*>(e)[lane % NW];
          const CT piv = tile[(size_t)(s0 + j) * R + lrow];
          CT inv;
          inv.x = inv.y = 0;
          if (piv.x != 0 || piv.y != 0) inv = cinv_t(piv);
#pragma unroll
          for (int q = 0; q < NW; ++q) word = lane == j * NW + q ? cword(inv, q) : word;
          ll_put(&rows[(size_t)g * RW + lane], E, word);
        }
        int gp;
        u64 k;
        if (G <= 64) k = gather_keys<1>(cand, G, E, lane, gp, &late);
        else if (G <= 128) k = gather_keys<2>(cand, G, E, lane, gp, &late);
        else k = gather_keys<4>(cand, G, E, lane, gp, &late);
        if (gp < 0 || __any(late)) {
          late = 1;
          break;
        }
        if (lane < RW) reinterpret_cast<uint32_t*>(lp + j * SUBW)[lane] = ll_get(rows + (size_t)gp * RW + lane, E, &late);
        const int32_t plabel = (int32_t)(0xffffffffu - (uint32_t)(k & 0xffffffffu));
        // interchange of positions gj <-> plabel
        if (g == gp && lane == lrow) {
          mylab = gj;
          mine[j] = lrow;
        } else if (mylab == gj) {
          mylab = plabel;
        }
        if (lane == 0) pl[s0 + j] = plabel;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const CT* urow = lp + j * SUBW + j;
        CT u[SUBW];  // the reciprocal, then the pivot row (the last ones past its end: not used)
#pragma unroll
        for (int c = 0; c < SUBW; ++c) u[c] = urow[c];
        if (u[0].x == 0 && u[0].y == 0 && zero_col < 0) zero_col = s0 + j;
        const bool active = mylab > gj;
        const CT l = cmul_t(x[0], u[0]);
        // the next column first: its candidate's key travels while the rest is updated
        x[0] = r1_upd(x[1], l, u[1]);
        const CT x1 = x[0];
        if (j + 1 < sw) lrow = candidate(j + 1, x1);
        static_for<SUBW - 2>([&](auto c) { x[c + 1] = r1_upd(x[c + 2], l, u[c + 2]); });
        if (active) {
          CT* trow = tile + (size_t)(s0 + j) * R + lane;
          trow[0] = l;
          static_for<SUBW - 1>([&](auto c) {
            CT* p = j + c + 1 < sw ? trow + (c + 1) * R : spare + lane;
            *p = x[c];
          });
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
      if (lane < myR) lab[lane] = mylab;
      if (late) bad = 1;
    }
    __syncthreads();
    if (bad) {
      if (tid == 0) __hip_atomic_store(&ws.err[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    const int c1 = s0 + sw, rest = w - c1;
    if (rest <= 0) break;
    // the pivot rows' remaining columns: owners publish theirs, everyone reads all
    const uint32_t E = epoch0 + (uint32_t)(c1 - 1);
    u64* const uw = ubase + (size_t)sp * SUBW * ws.wwmax;
    const int words = rest * NW;
    const int own = mine[lane % SUBW];
    const uint32_t ours = (uint32_t)__ballot(own >= 0) & ((1u << SUBW) - 1);  // pivots that are rows of this workgroup
    for (uint32_t left = ours; left; left &= left - 1) {
      const int i = __builtin_ctz(left), lr = __builtin_amdgcn_readlane(own, i);
      for (int t = tid; t < words; t += 256)
        ll_put(uw + (size_t)i * ws.wwmax + t, E, reinterpret_cast<const uint32_t*>(tile + (size_t)(c1 + t / NW) * R + lr)[t % NW]);
    }
    {
      // wave v reads rows 4 v .. 4 v + 3, 64 B words of each in flight together
      uint32_t* const dst = reinterpret_cast<uint32_t*>(ub);
      constexpr int B = 4;  // one round trip for 112 columns in FP32, two in FP64
      for (int t0 = 0; t0 < words; t0 += 64 * B) {
        const u64* p[4 * B];
        uint32_t v[4 * B];
#pragma unroll
        for (int b = 0; b < 4 * B; ++b) {
          const int t = t0 + 64 * (b % B) + lane;
          p[b] = uw + (size_t)(4 * wave + b / B) * ws.wwmax + (t < words ? t : lane % words);
        }
        ll_get_n<4 * B>(p, E, v, &bad);
#pragma unroll
        for (int b = 0; b < 4 * B; ++b) {
          const int t = t0 + 64 * (b % B) + lane;
          if (t < words) dst[(size_t)(4 * wave + b / B) * restmax * NW + t] = v[b];
        }
      }
    }
    __syncthreads();
    if (bad) {
      if (tid == 0) __hip_atomic_store(&ws.err[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    // U rows: one column per thread
    if (tid < rest) {
      CT u[SUBW];
#pragma unroll
      for (int i = 0; i < SUBW; ++i) u[i] = ub[i * restmax + tid];
      static_for<SUBW>([&](auto i) {
        static_for<decltype(i)::value>([&](auto p) { u[i] = r1_upd(u[i], lp[i * SUBW + p], u[p]); });
        ub[i * restmax + tid] = u[i];
      });
    }
    __syncthreads();
    const int32_t last = (int32_t)(k0 + c1 - 1);
    for (uint32_t left = ours; left; left &= left - 1) {
      const int i = __builtin_ctz(left), lr = __builtin_amdgcn_readlane(own, i);
      for (int c = tid; c < rest; c += 256) tile[(size_t)(c1 + c) * R + lr] = ub[i * restmax + c];
    }
    // rank-SUBW update of the rows still active: 16 x 16 tiles dealt to the waves
    {
      const int lr16 = lane & 15, lk = lane >> 4;
      const int rt = (myR + 15) >> 4, nt = rt * ((rest + 15) >> 4);
      for (int t = wave; t < nt; t += 4) {
        const int row = 16 * (t % rt) + lr16, crow = row < myR ? row : myR - 1;
        const int cc = 16 * (t / rt);
        const int uc = cc + lr16 < rest ? cc + lr16 : rest - 1;
        typename acc_of<T>::type re = {0, 0, 0, 0}, im = {0, 0, 0, 0};
        CT l[4], u[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          l[q] = tile[(size_t)(s0 + 4 * q + lk) * R + crow];
          u[q] = ub[(4 * q + lk) * restmax + uc];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          re = mfma16(u[q].x, l[q].x, re);
          im = mfma16(u[q].x, l[q].y, im);
          re = mfma16(-u[q].y, l[q].y, re);
          im = mfma16(u[q].y, l[q].x, im);
        }
        if (row < myR && lab[row] > last) {
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int c = cc + (sizeof(T) == 8 ? lk + 4 * q : 4 * lk + q);
            if (c < rest) {
              CT* p = tile + (size_t)(c1 + c) * R + row;
              CT v = *p;
              v.x -= re[q];
              v.y -= im[q];
              *p = v;
            }
          }
        }
      }
    }
    __syncthreads();
  }
  if (g == 0) {
    for (int j = tid; j < w; j += 256) ipiv[k0 + j] = pl[j];
    if (tid == 0 && zero_col >= 0) atomicMin(&ws.err[1], (int)(k0 + zero_col));
  }
  if (tid < myR) {
    const int32_t orig = (int32_t)(rbase + tid);
    if (lab[tid] != orig) {
      const int slot = __hip_atomic_fetch_add(mcount, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (slot < mcap) {
        mdst[slot] = lab[tid];
        msrc[slot] = orig;
      }
    }
  }
  if (lane < myR) {
    CT* dst = A + lab[lane] + k0 * ld;
    for (int c = wave; c < w; c += 4) dst[c * ld] = tile[c * R + lane];
  }
}

// ---------------------------------------------------------------------------
// 1b. panel factorisation with tournament pivoting: one exchange per PB columns
// ---------------------------------------------------------------------------
// The columns of the panel are taken in inner steps of PB.  For the step's
// columns [j0, j0 + pw) the pivots are chosen by a tournament of partial
// pivotings, each on the original values of its candidates:
//   * every row workgroup picks up to PB candidate rows among its active rows
//     (one wave, partial pivoting on the step's columns) and publishes them:
//     their labels and step values, and their remaining columns;
//   * root workgroups (one per TP_ROOT_SPAN row workgroups, launched after
//     them) hold one candidate per thread; each wave picks PB among its 64,
//     then one wave PB among the 4 PB winners, and the root publishes them;
//   * every row workgroup reads the roots' winners (one per lane of one wave)
//     and picks the step's PB pivots among them.  The arithmetic is identical
//     everywhere, so all row workgroups agree on the pivots and on the factored
//     PB x PB pivot block (L11 strictly below the diagonal, U11 on and above).
// Then the U rows of the step (a pivot row's remaining columns, fetched from
// its owner, minus L11 times the earlier U rows) and, for every other active
// row, the multipliers l = a U11^-1 and the rank-pw update of its remaining
// columns: the next step's columns first (they decide its candidates), the
// candidates' remaining columns next (they are published), the rest after the
// publication, while the roots work.
// This is the tree form of communication-avoiding LU (tournament pivoting);
// with PB = 1 it would be plain partial pivoting, which panel_kernel
// implements.  Pivot keys and ties follow panel_kernel (largest |re| + |im| in
// FP32, lowest label); rows never move between workgroups, and interchanges
// swap labels.
//
// Exchange buffers (per batch item, double-buffered by the parity of the inner
// step; every 32-bit payload travels in an epoch-tagged 64-bit word):
//   records ws.cand [2][gitem][PB][K], K = 1 + PB NW: label, PB step values
//     (label 0xffffffff: no candidate);
//   root results after them, [2][ceil(gitem / TP_ROOT_SPAN)][PB][KR],
//     KR = 2 + PB NW: candidate index (workgroup PB + slot, 0xffffffff: none),
//     label, PB step values;
//   rows ws.rows [2][gitem][PB][wwmax]: a candidate's columns after the step.
constexpr int TP_ROOT_SPAN = 32;

template <typename CT>
__device__ inline CT rdlane(CT v, int l) {
  if constexpr (sizeof(CT) == 8) {
    CT r;
    r.x = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v.x), l));
    r.y = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v.y), l));
    return r;
  } else {
    auto rd = [&](double d) {
      const long long b = __double_as_longlong(d);
      const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), l);
      const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
      return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
    };
    CT r;
    r.x = rd(v.x);
    r.y = rd(v.y);
    return r;
  }
}

// One step of partial pivoting inside a wave over the candidates its lanes hold
// (RL per lane: values v[r][0..PB), labels lab[r], live flags alive[r]): the
// live candidate with the largest |re| + |im| in column c (lowest label on ties)
// is chosen; its values pv (multipliers of the earlier steps before column c,
// its U row from c on) reach every lane; every other live candidate is
// eliminated.  wl / wsl: lane and slot of the chosen one (wave-uniform); inv:
// 1 / pv[c] (0 for a zero pivot).  Returns false if no live candidate is left.
template <typename CT, int PB, int RL>
__device__ __forceinline__ bool wave_pivot_step(int c, int pw, CT (&v)[RL][PB], const uint32_t (&lab)[RL], bool (&alive)[RL],
                                       CT (&pv)[PB], CT& inv, int& wl, int& wsl) {
  const int lane = threadIdx.x & 63;
  u64 best = 0;
  int bs = 0;
#pragma unroll
  for (int r = 0; r < RL; ++r)
    if (alive[r]) {
      const u64 k = pivot_key(v[r][c], lab[r]);
      if (k > best) {
        best = k;
        bs = r;
      }
    }
  const u64 wb = wave_max_u64(best);
  if (wb == 0) return false;
  const unsigned long long m = __ballot(best == wb);  // one lane: keys are unique
  wl = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)m) - 1);
  wsl = __builtin_amdgcn_readlane(bs, wl);
  // the lane's chosen slot by register selects (the empty asm keeps the
  // compiler from turning the select chain into an indexed load from a stack
  // copy of v)
  CT mine[PB];
#pragma unroll
  for (int cc = 0; cc < PB; ++cc) {
    mine[cc] = v[0][cc];
#pragma unroll
    for (int r = 1; r < RL; ++r) {
      CT t = v[r][cc];
      asm volatile("" : "+v"(t.x), "+v"(t.y));
      mine[cc].x = bs == r ? t.x : mine[cc].x;
      mine[cc].y = bs == r ? t.y : mine[cc].y;
    }
  }
#pragma unroll
  for (int cc = 0; cc < PB; ++cc) pv[cc] = rdlane(mine[cc], wl);
  if (lane == wl)
#pragma unroll
    for (int r = 0; r < RL; ++r)
      if (r == bs) alive[r] = false;
  if (pv[c].x == 0 && pv[c].y == 0) {
    inv.x = 0;
    inv.y = 0;
  } else {
    inv = cinv_t(pv[c]);
  }
#pragma unroll
  for (int r = 0; r < RL; ++r)
    if (alive[r]) {
      const CT l = cmul_t(v[r][c], inv);
      v[r][c] = l;
#pragma unroll
      for (int cc = 0; cc < PB; ++cc)
        if (cc > c && cc < pw) v[r][cc] = r1_upd(v[r][cc], l, pv[cc]);
    }
  return true;
}

template <typename T, int PB>
__global__ void __launch_bounds__(256) panel_tp_kernel(cplx<T>* __restrict__ A, int64_t ld, int64_t n, int64_t k0,
                                                        int w, int R, int G, int32_t* __restrict__ ipiv, LUWork ws,
                                                        uint32_t epoch0, int64_t sA, int64_t sipiv,
                                                        int32_t* __restrict__ mdst, int32_t* __restrict__ msrc,
                                                        int32_t* __restrict__ mcount, int mcap) {
  using CT = cplx<T>;
  constexpr int NW = sizeof(CT) / 4;
  constexpr int K = 1 + PB * NW;   // words of a candidate record
  constexpr int KR = 2 + PB * NW;  // words of a root's winner
  A += (int64_t)blockIdx.y * sA;
  ipiv += (int64_t)blockIdx.y * sipiv;
  ws.cand += (int64_t)blockIdx.y * ws.s_cand;
  ws.rows += (int64_t)blockIdx.y * ws.s_rows;
  mdst += (int64_t)blockIdx.y * ws.s_pairs;
  msrc += (int64_t)blockIdx.y * ws.s_pairs;
  mcount += (int64_t)blockIdx.y * ws.s_npairs;
  const int g = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  // an earlier panel's exchange failed (flag set before this launch): the
  // factorisation is lost, so do not wait out another exchange
  if (__hip_atomic_load(&ws.err[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return;
  const int NR = (G + TP_ROOT_SPAN - 1) / TP_ROOT_SPAN;
  const int nrmax = (ws.gitem + TP_ROOT_SPAN - 1) / TP_ROOT_SPAN;
  const size_t rec_par = (size_t)ws.gitem * PB * K;
  u64* const res_all = ws.cand + 2 * rec_par;
  const size_t res_par = (size_t)nrmax * PB * KR;
  const int nsteps = (w + PB - 1) / PB;
  __shared__ int bad;
  if (tid == 0) bad = 0;

  // ------------------------------------------------------------------ roots
  if (g >= G) {
    __shared__ uint32_t l1ci[4][PB], l1lab[4][PB];
    __shared__ CT l1v[4][PB][PB];
    const int r = g - G;
    const int cg = r * TP_ROOT_SPAN + tid / PB, cs = tid % PB;
    const bool have = tid < TP_ROOT_SPAN * PB && cg < G;
    __syncthreads();
    for (int s = 0; s < nsteps; ++s) {
      const int j0 = s * PB, pw = w - j0 < PB ? w - j0 : PB;
      const uint32_t E = epoch0 + (uint32_t)s;
      const int par = s & 1;
      const u64* rec = ws.cand + par * rec_par;
      const u64* base[1] = {rec + (size_t)(have ? cg * PB + cs : 0) * K};  // record 0 is always published
      uint32_t wd[K];
      ll_get_rec<K, 1>(base, E, wd, &bad);
      CT v[1][PB], v0[PB];
      uint32_t lb[1] = {wd[0]};
      bool al[1] = {have && wd[0] != 0xffffffffu};
#pragma unroll
      for (int c = 0; c < PB; ++c) {
        uint32_t* d = reinterpret_cast<uint32_t*>(&v0[c]);
#pragma unroll
        for (int q = 0; q < NW; ++q) d[q] = wd[1 + c * NW + q];
        v[0][c] = v0[c];
      }
      // level 1: PB winners of each wave, with their original values
      bool more = true;
#pragma unroll
      for (int c = 0; c < PB; ++c) {
        CT pv[PB], inv;
        int wl = 0, wsl = 0;
        if (c < pw && more) more = wave_pivot_step<CT, PB, 1>(c, pw, v, lb, al, pv, inv, wl, wsl);
        if (c < pw && more) {
          if (lane == wl) {
            l1ci[wv][c] = (uint32_t)(cg * PB + cs);
            l1lab[wv][c] = lb[0];
#pragma unroll
            for (int cc = 0; cc < PB; ++cc) l1v[wv][c][cc] = v0[cc];
          }
        } else if (lane == 0) {
          l1ci[wv][c] = 0xffffffffu;
        }
      }
      __syncthreads();
      // level 2 (wave 0): PB winners among the 4 PB, published with their original values
      if (wv == 0) {
        const int sw = lane / PB, sc = lane % PB;
        const bool in = lane < 4 * PB;
        uint32_t ci2 = in ? l1ci[sw][sc] : 0xffffffffu;
        uint32_t lb2[1] = {in ? l1lab[sw][sc] : 0u};
        bool al2[1] = {ci2 != 0xffffffffu};
        CT u0[PB], u[1][PB];
#pragma unroll
        for (int cc = 0; cc < PB; ++cc) {
          if (in) {
            u0[cc] = l1v[sw][sc][cc];
          } else {
            u0[cc].x = 0;
            u0[cc].y = 0;
          }
          u[0][cc] = u0[cc];
        }
        u64* res = res_all + par * res_par + (size_t)r * PB * KR;
        bool more2 = true;
#pragma unroll
        for (int c = 0; c < PB; ++c) {
          CT pv[PB], inv;
          int wl = 0, wsl = 0;
          if (c < pw && more2) more2 = wave_pivot_step<CT, PB, 1>(c, pw, u, lb2, al2, pv, inv, wl, wsl);
          const bool got = c < pw && more2;
          // the winner's lane (lane 0 for an empty slot) writes the slot's KR words
          if ((got && lane == wl) || (!got && lane == 0)) {
            u64* o = res + (size_t)c * KR;
            ll_put(&o[0], E, got ? ci2 : 0xffffffffu);
            ll_put(&o[1], E, got ? lb2[0] : 0u);
#pragma unroll
            for (int cc = 0; cc < PB; ++cc)
#pragma unroll
              for (int q = 0; q < NW; ++q) ll_put(&o[2 + cc * NW + q], E, got ? cword(u0[cc], q) : 0u);
          }
        }
      }
      __syncthreads();  // the level-1 slots are rewritten next step
      if (bad) break;
    }
    if (bad && tid == 0) __hip_atomic_store(&ws.err[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }

  // ------------------------------------------------------------ row workgroups
  extern __shared__ unsigned char smem_raw[];
  CT* tile = reinterpret_cast<CT*>(smem_raw);                        // [w][R], column c at tile + c R
  CT* prow = tile + (size_t)w * R;                                   // [PB][w] U rows of the step
  CT* sel = prow + (size_t)PB * w;                                   // [PB][R] scratch of the local choice (R > 256)
  int32_t* lab = reinterpret_cast<int32_t*>(sel + (size_t)PB * R);  // [R] row labels (final positions)
  int32_t* pl = lab + R;                                             // [w] pivot positions of this panel
  __shared__ CT blk[PB][PB];  // factored pivot block of the step
  __shared__ CT binv[PB];     // 1 / U11[c][c] (0 for a zero pivot)
  __shared__ int pci[PB];     // candidate index (workgroup PB + slot) of pivot c
  __shared__ int32_t plab[PB];  // label of pivot c's row when the step starts
  __shared__ int chosen[PB];  // local rows offered as candidates
  __shared__ int nch;
  __shared__ int zcol;        // first zero pivot column of this panel (-1: none)
  const int64_t rbase = k0 + (int64_t)g * R;
  const int myR = (int)(n - rbase < (int64_t)R ? (n - rbase > 0 ? n - rbase : 0) : R);
  if (tid == 0) zcol = -1;
  constexpr int LB = 128 / (int)sizeof(CT);
  const int wfull = w - w % LB;
  for (int lr = tid; lr < myR; lr += 256) {
    const CT* src = A + (rbase + lr) + k0 * ld;
    for (int c0 = 0; c0 < wfull; c0 += LB) {
      CT v[LB];
#pragma unroll
      for (int u = 0; u < LB; ++u) v[u] = src[(c0 + u) * ld];
#pragma unroll
      for (int u = 0; u < LB; ++u) tile[(c0 + u) * R + lr] = v[u];
    }
    for (int c = wfull; c < w; ++c) tile[c * R + lr] = src[c * ld];
  }
  for (int lr = tid; lr < myR; lr += 256) lab[lr] = (int32_t)(rbase + lr);
  // 2D mapping of the bulk update: RP rows x CG column groups
  int RP = 1;
  while (RP < myR && RP < 256) RP <<= 1;
  const int CG = 256 / RP;
  const int ulr0 = tid & (RP - 1), ucg = tid / RP;
  __syncthreads();

  // Local choice (wave 0): partial pivoting on columns [j1, j1 + pw1) of the
  // active rows (labels >= k0 + j1).  Up to 128 rows the lanes keep their rows
  // (lane, lane + 64) in registers; beyond that, in the LDS scratch.
  // Writes chosen[] and nch.
  auto local_choice = [&](int j1, int pw1) {
    if (wv != 0) return;
    const int32_t gj1 = (int32_t)(k0 + j1);
    int cnt = 0;
    if (myR <= 128) {
      constexpr int RL = 2;
      CT v[RL][PB];
      uint32_t lb[RL];
      bool al[RL];
#pragma unroll
      for (int i = 0; i < RL; ++i) {
        const int lr = lane + 64 * i;
        al[i] = lr < myR && lab[lr] >= gj1;
        lb[i] = al[i] ? (uint32_t)lab[lr] : 0u;
#pragma unroll
        for (int c = 0; c < PB; ++c) {
          v[i][c].x = 0;
          v[i][c].y = 0;
          if (al[i] && c < pw1) v[i][c] = tile[(j1 + c) * R + lr];
        }
      }
      bool more = true;
#pragma unroll
      for (int c = 0; c < PB; ++c) {
        CT pv[PB], inv;
        int wl = 0, wsl = 0;
        if (c < pw1 && more) more = wave_pivot_step<CT, PB, RL>(c, pw1, v, lb, al, pv, inv, wl, wsl);
        if (c < pw1 && more) {
          if (lane == 0) chosen[c] = wl + 64 * wsl;
          cnt = c + 1;
        }
      }
    } else {
      for (int lr = lane; lr < myR; lr += 64)
#pragma unroll
        for (int c = 0; c < PB; ++c)
          if (c < pw1) sel[c * R + lr] = tile[(j1 + c) * R + lr];
      uint32_t taken = 0;  // bit i: row lane + 64 i already chosen
      bool more = true;
#pragma unroll
      for (int c = 0; c < PB; ++c) {
        if (c < pw1 && more) {
          u64 best = 0;
          int blr = -1;
          for (int lr = lane, i = 0; lr < myR; lr += 64, ++i) {
            if (lab[lr] < gj1 || ((taken >> i) & 1u)) continue;
            const u64 kk = pivot_key(sel[c * R + lr], (uint32_t)lab[lr]);
            if (kk > best) {
              best = kk;
              blr = lr;
            }
          }
          const u64 wbest = wave_max_u64(best);
          if (wbest == 0) {
            more = false;  // no active row left
          } else {
            const int wl = __ffsll((unsigned long long)__ballot(best == wbest)) - 1;
            const int wlr = __shfl(blr, wl);
            if (lane == wl) taken |= 1u << ((wlr - lane) >> 6);
            if (lane == 0) chosen[c] = wlr;
            cnt = c + 1;
            CT pv[PB];
#pragma unroll
            for (int cc = 0; cc < PB; ++cc) {
              CT v = {0, 0};
              if (lane == wl && cc >= c && cc < pw1) v = sel[cc * R + wlr];
              pv[cc].x = __shfl(v.x, wl);
              pv[cc].y = __shfl(v.y, wl);
            }
            CT inv;
            if (pv[c].x == 0 && pv[c].y == 0) {
              inv.x = 0;
              inv.y = 0;
            } else {
              inv = cinv_t(pv[c]);
            }
            for (int lr = lane, i = 0; lr < myR; lr += 64, ++i) {
              if (lab[lr] < gj1 || ((taken >> i) & 1u)) continue;
              const CT l = cmul_t(sel[c * R + lr], inv);
#pragma unroll
              for (int cc = 0; cc < PB; ++cc)
                if (cc > c && cc < pw1) sel[cc * R + lr] = r1_upd(sel[cc * R + lr], l, pv[cc]);
            }
          }
        }
      }
    }
    if (lane == 0) nch = cnt;
  };
  auto is_chosen = [&](int lr) {
    bool r = false;
#pragma unroll
    for (int c = 0; c < PB; ++c) r = r || (c < nch && chosen[c] == lr);
    return r;
  };
  // Publish the candidates of step s (columns [j1, j1 + pw1)): records, then
  // the columns after the step.
  auto publish = [&](int s, int j1, int pw1) {
    const uint32_t E = epoch0 + (uint32_t)s;
    const int par = s & 1;
    u64* rec = ws.cand + par * rec_par + (size_t)g * PB * K;
    u64* rws = ws.rows + (size_t)par * ws.gitem * PB * ws.wwmax + (size_t)g * PB * ws.wwmax;
    for (int t = tid; t < PB * K; t += 256) {
      const int c = t / K, k = t % K;
      uint32_t v;
      if (c >= nch) {
        v = k == 0 ? 0xffffffffu : 0u;
      } else {
        const int lr = chosen[c];
        if (k == 0) {
          v = (uint32_t)lab[lr];
        } else {
          const int cc = (k - 1) / NW;
          v = cc < pw1 ? cword(tile[(j1 + cc) * R + lr], (k - 1) % NW) : 0u;
        }
      }
      ll_put(&rec[t], E, v);
    }
    const int WR = (w - j1 - pw1) * NW;
    for (int t = tid; t < nch * WR; t += 256) {
      const int c = t / WR, k = t % WR;
      ll_put(&rws[(size_t)c * ws.wwmax + k], E, cword(tile[(j1 + pw1 + k / NW) * R + chosen[c]], k % NW));
    }
  };

  local_choice(0, PB < w ? PB : w);
  __syncthreads();
  publish(0, 0, PB < w ? PB : w);
  for (int s = 0; s < nsteps; ++s) {
    const int j0 = s * PB, pw = w - j0 < PB ? w - j0 : PB;
    const int j1 = j0 + pw, pw1 = w - j1 < PB ? w - j1 : PB;
    const int32_t gj0 = (int32_t)(k0 + j0), gj1 = (int32_t)(k0 + j1);
    const uint32_t E = epoch0 + (uint32_t)s;
    const int par = s & 1;
    // --- the step's pivots: wave 0 chooses among the roots' winners ---
    if (wv == 0) {
      const bool in = lane < NR * PB;
      const u64* res = res_all + par * res_par;
      const u64* base[1] = {res + (size_t)(in ? lane : 0) * KR};  // root 0's slot 0 is always published
      uint32_t wd[KR];
      ll_get_rec<KR, 1>(base, E, wd, &bad);
      const uint32_t ci = in ? wd[0] : 0xffffffffu;
      uint32_t lb[1] = {wd[1]};
      bool al[1] = {ci != 0xffffffffu};
      CT v[1][PB];
#pragma unroll
      for (int c = 0; c < PB; ++c) {
        uint32_t* d = reinterpret_cast<uint32_t*>(&v[0][c]);
#pragma unroll
        for (int q = 0; q < NW; ++q) d[q] = wd[2 + c * NW + q];
      }
      bool more = true;
#pragma unroll
      for (int c = 0; c < PB; ++c) {
        CT pv[PB], inv;
        int wl = 0, wsl = 0;
        const uint32_t cic = ci, lbc = lb[0];  // before the step retires the winner
        if (c < pw && more) more = wave_pivot_step<CT, PB, 1>(c, pw, v, lb, al, pv, inv, wl, wsl);
        if (c < pw) {
          if (!more) {
            if (lane == 0) bad = 1;  // fewer candidates than columns: cannot happen
          } else {
            const uint32_t wci = (uint32_t)__builtin_amdgcn_readlane((int)cic, wl);
            const uint32_t wlb = (uint32_t)__builtin_amdgcn_readlane((int)lbc, wl);
            if (lane == 0) {
              pci[c] = (int)wci;
              plab[c] = (int32_t)wlb;
              binv[c] = inv;
#pragma unroll
              for (int cc = 0; cc < PB; ++cc) blk[c][cc] = pv[cc];
              if (pv[c].x == 0 && pv[c].y == 0 && zcol < 0) zcol = j0 + c;
            }
          }
        }
      }
    }
    __syncthreads();
    if (bad) {
      if (tid == 0) __hip_atomic_store(&ws.err[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    // --- positions of the pivots before their interchanges (LAPACK ipiv) ---
    int32_t ppos[PB];
#pragma unroll
    for (int c = 0; c < PB; ++c) {
      int32_t p = plab[c < pw ? c : 0];
#pragma unroll
      for (int cc = 0; cc < PB; ++cc)
        if (cc < c && p == gj0 + cc) p = ppos[cc];
      ppos[c] = p;
    }
    if (tid == 0)
#pragma unroll
      for (int c = 0; c < PB; ++c)
        if (c < pw) pl[j0 + c] = ppos[c];
    // which local row is pivot c (-1 if another workgroup owns it)
    int own[PB];
#pragma unroll
    for (int c = 0; c < PB; ++c) own[c] = (c < pw && pci[c] / PB == g) ? chosen[pci[c] % PB] : -1;
    // --- fetch the pivot rows' columns [j1, w) from their owners (at most 8
    // words per thread, all in flight together) ---
    {
      const int WR = (w - j1) * NW;
      const int tot = pw * WR;
      if (tot > 0) {
        const u64* rws = ws.rows + (size_t)par * ws.gitem * PB * ws.wwmax;
        uint32_t* p32 = reinterpret_cast<uint32_t*>(prow);
        constexpr int FB = 8;  // PB w NW <= 8 x 128 x 2 = 4 x 128 x 4 = 2048 = 8 x 256
        const u64* pp[FB];
#pragma unroll
        for (int i = 0; i < FB; ++i) {
          const int t = tid + 256 * i < tot ? tid + 256 * i : 0;
          const int c = t / WR, k = t % WR;
          const int ci = pci[c];
          pp[i] = rws + (size_t)(ci / PB) * PB * ws.wwmax + (size_t)(ci % PB) * ws.wwmax + k;
        }
        uint32_t wd[FB];
        ll_get_sel<FB>(pp, E, wd, &bad);
#pragma unroll
        for (int i = 0; i < FB; ++i) {
          const int t = tid + 256 * i;
          if (t < tot) p32[((size_t)(t / WR) * w + j1) * NW + t % WR] = wd[i];
        }
      }
    }
    // --- interchanges: labels of the pivot rows and of the rows they displace ---
    for (int lr = tid; lr < myR; lr += 256) {
      int32_t L = lab[lr];
      if (L < gj0) continue;
#pragma unroll
      for (int c = 0; c < PB; ++c) {
        if (c < pw) {
          if (own[c] == lr) L = gj0 + c;
          else if (L == gj0 + c) L = ppos[c];
        }
      }
      lab[lr] = L;
    }
    __syncthreads();
    // --- U rows: columns [j1, w) of pivot c minus L11[c][:c] times the earlier ones ---
    for (int col = j1 + tid; col < w; col += 256)
#pragma unroll
      for (int c = 1; c < PB; ++c) {
        if (c < pw) {
          CT u = prow[c * w + col];
#pragma unroll
          for (int cc = 0; cc < PB; ++cc)
            if (cc < c) u = r1_upd(u, blk[c][cc], prow[cc * w + col]);
          prow[c * w + col] = u;
        }
      }
    __syncthreads();
    // --- the step's rows: pivot rows get their factored values, every other
    // active row its multipliers and the update of the next step's columns ---
    for (int t = tid; t < pw * (w - j0); t += 256) {
      const int c = t / (w - j0), col = j0 + t % (w - j0);
      int lr = -1;
#pragma unroll
      for (int cc = 0; cc < PB; ++cc)
        if (cc == c) lr = own[cc];
      if (lr >= 0) tile[col * R + lr] = col < j1 ? blk[c][col - j0] : prow[c * w + col];
    }
    for (int lr = tid; lr < myR; lr += 256) {
      if (lab[lr] < gj1) continue;
      CT l[PB];
#pragma unroll
      for (int c = 0; c < PB; ++c) {
        l[c].x = 0;
        l[c].y = 0;
        if (c < pw) {
          CT a = tile[(j0 + c) * R + lr];
#pragma unroll
          for (int cc = 0; cc < PB; ++cc)
            if (cc < c) a = r1_upd(a, l[cc], blk[cc][c]);
          l[c] = cmul_t(a, binv[c]);
          tile[(j0 + c) * R + lr] = l[c];
        }
      }
#pragma unroll
      for (int cc = 0; cc < PB; ++cc) {
        if (cc < pw1) {
          CT a = tile[(j1 + cc) * R + lr];
#pragma unroll
          for (int c = 0; c < PB; ++c)
            if (c < pw) a = r1_upd(a, l[c], prow[c * w + j1 + cc]);
          tile[(j1 + cc) * R + lr] = a;
        }
      }
    }
    __syncthreads();
    if (j1 >= w) break;
    // --- candidates of the next step, their remaining columns, publication ---
    local_choice(j1, pw1);
    __syncthreads();
    {
      const int WC = w - j1 - pw1;
      for (int t = tid; t < nch * WC; t += 256) {
        const int c = t / WC, col = j1 + pw1 + t % WC;
        const int lr = chosen[c];
        CT a = tile[col * R + lr];
#pragma unroll
        for (int cc = 0; cc < PB; ++cc)
          if (cc < pw) a = r1_upd(a, tile[(j0 + cc) * R + lr], prow[cc * w + col]);
        tile[col * R + lr] = a;
      }
    }
    __syncthreads();
    publish(s + 1, j1, pw1);
    // --- the rest of the update, while the roots choose ---
    for (int lr = ulr0; lr < myR; lr += RP) {
      if (lab[lr] < gj1 || is_chosen(lr)) continue;
      CT l[PB];
#pragma unroll
      for (int c = 0; c < PB; ++c) {
        if (c < pw) {
          l[c] = tile[(j0 + c) * R + lr];
        } else {
          l[c].x = 0;
          l[c].y = 0;
        }
      }
      for (int col = j1 + pw1 + ucg; col < w; col += CG) {
        CT a = tile[col * R + lr];
#pragma unroll
        for (int c = 0; c < PB; ++c)
          if (c < pw) a = r1_upd(a, l[c], prow[c * w + col]);
        tile[col * R + lr] = a;
      }
    }
  }
  __syncthreads();
  if (bad && tid == 0) __hip_atomic_store(&ws.err[0], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (g == 0) {
    for (int j = tid; j < w; j += 256) ipiv[k0 + j] = pl[j];
    if (tid == 0 && zcol >= 0) atomicMin(&ws.err[1], (int)(k0 + zcol));
  }
  for (int lr = tid; lr < myR; lr += 256) {
    const int32_t orig = (int32_t)(rbase + lr);
    if (lab[lr] != orig) {
      const int slot = __hip_atomic_fetch_add(mcount, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (slot < mcap) {
        mdst[slot] = lab[lr];
        msrc[slot] = orig;
      }
    }
  }
  for (int lr = tid; lr < myR; lr += 256) {
    CT* dst = A + lab[lr] + k0 * ld;
    for (int c0 = 0; c0 < wfull; c0 += LB) {
      CT v[LB];
#pragma unroll
      for (int u = 0; u < LB; ++u) v[u] = tile[(c0 + u) * R + lr];
#pragma unroll
      for (int u = 0; u < LB; ++u) dst[(c0 + u) * ld] = v[u];
    }
    for (int c = wfull; c < w; ++c) dst[c * ld] = tile[c * R + lr];
  }
}

// ---------------------------------------------------------------------------
// 2. row permutations (a block's moved rows, listed by its panel)
// ---------------------------------------------------------------------------
// X[dst[t], col] = Xold[src[t], col] for the columns [c0, c0 + ncols).
template <typename T>
__global__ void __launch_bounds__(256) row_permute_kernel(cplx<T>* __restrict__ X, int64_t ld, int64_t c0,
                                                          const int32_t* __restrict__ dst, const int32_t* __restrict__ src,
                                                          const int32_t* __restrict__ npairs, int64_t sX, int64_t spairs,
                                                          int64_t snpairs) {
  using CT = cplx<T>;
  X += (int64_t)blockIdx.y * sX;  // batch item blockIdx.y
  dst += (int64_t)blockIdx.y * spairs;
  src += (int64_t)blockIdx.y * spairs;
  npairs += (int64_t)blockIdx.y * snpairs;
  const int np = *npairs;
  const int64_t col = c0 + blockIdx.x;
  CT* x = X + col * ld;
  CT v[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int t = threadIdx.x + 256 * i;
    if (t < np) v[i] = x[src[t]];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int t = threadIdx.x + 256 * i;
    if (t < np) x[dst[t]] = v[i];
  }
}

// inverse: Xnew[src[t]] = Xold[dst[t]] (for the transposed solve)
template <typename T>
__global__ void __launch_bounds__(256) row_permute_inv_kernel(cplx<T>* __restrict__ X, int64_t ld, int64_t c0,
                                                              const int32_t* __restrict__ dst, const int32_t* __restrict__ src,
                                                              const int32_t* __restrict__ npairs, int64_t sX,
                                                              int64_t spairs, int64_t snpairs) {
  using CT = cplx<T>;
  X += (int64_t)blockIdx.y * sX;  // batch item blockIdx.y
  dst += (int64_t)blockIdx.y * spairs;
  src += (int64_t)blockIdx.y * spairs;
  npairs += (int64_t)blockIdx.y * snpairs;
  const int np = *npairs;
  const int64_t col = c0 + blockIdx.x;
  CT* x = X + col * ld;
  CT v[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int t = threadIdx.x + 256 * i;
    if (t < np) v[i] = x[dst[t]];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int t = threadIdx.x + 256 * i;
    if (t < np) x[src[t]] = v[i];
  }
}

// ---------------------------------------------------------------------------
// planning and workspace
// ---------------------------------------------------------------------------
static const int LDS_RESERVE = 2048;
// the tournament panel's static LDS (pivot block, wave slots) is larger
static const int LDS_RESERVE_TP = 4096;
// rows per workgroup of the local choice (a 32-bit mask of each lane's rows)
static const int TP_MAX_ROWS = 2048;

// dynamic LDS of a panel workgroup: tile, pivot row(s), scratch, labels, pivots
static size_t panel_lds_bytes(int w, int R, size_t cbytes, int pb) {
  if (pb <= 1) return ((size_t)w * R + w) * cbytes + (size_t)(R + w) * 4;
  return ((size_t)w * R + (size_t)pb * w + (size_t)pb * R) * cbytes + (size_t)(R + w) * 4;
}
static int lds_reserve(int pb) { return pb <= 1 ? LDS_RESERVE : LDS_RESERVE_TP; }
// most rows of one panel workgroup that fit its LDS
static int64_t panel_rows_max(int w, int64_t lds_bytes, int cbytes, int pb) {
  if (pb <= 1) return (lds_bytes - LDS_RESERVE - (int64_t)w * (cbytes + 4)) / ((int64_t)(w + 1) * cbytes + 4);
  const int64_t r = (lds_bytes - LDS_RESERVE_TP - (int64_t)w * (pb * cbytes + 4)) / ((int64_t)(w + pb) * cbytes + 4);
  return r < TP_MAX_ROWS ? r : TP_MAX_ROWS;
}

// root workgroups of a tournament panel over G row workgroups
static int tp_roots(int G) { return (G + 31) / 32; }

LUPlan lu_plan(int64_t n, int elem_bytes, int num_cu, int lds_bytes, int nbatch, int nb_max, int pb, bool refined) {
  LUPlan p;
  p.n = n;
  if (nbatch < 1) nbatch = 1;
  p.spec = pb == 0;
  if (pb != 1 && pb != 2 && pb != 4 && pb != 8) pb = 1;
  if (elem_bytes == 8 && pb > 4) pb = 4;  // FP64 candidates of 8 columns would need too many registers
  p.pb = pb;
  // the panels of all items run in one launch and must all be resident
  p.max_wg = num_cu / nbatch > 0 ? num_cu / nbatch : 1;
  p.nbatch = nbatch;
  p.lds_bytes = lds_bytes;
  // row workgroups of one panel: with tournament pivoting, one root workgroup
  // per 32 of them must be resident too (G + ceil(G / 32) <= max_wg)
  const int avail = pb > 1 ? std::max(1, 32 * p.max_wg / 33) : p.max_wg;
  const int cbytes = 2 * elem_bytes;
  const int nb_want = nb_max >= 16 && nb_max <= 128 ? nb_max : 128;
  // a searching panel must fit: ceil(n / avail) rows x nb columns in LDS
  int nb_fit = nb_want;
  while (nb_fit > 16 && (n + avail - 1) / avail > panel_rows_max(nb_fit, lds_bytes, cbytes, pb)) nb_fit /= 2;
  // (not a speculative one, which keeps no rows there; a failed factorisation is
  // repeated with a plan of its own.  128 instead of 64 columns halve the traffic of
  // the updates: spectra of four structures up to n = 4500, 16 systems at a time,
  // 64.9 -> 53.0 ms; one FP32 factorisation of n = 69 000 7.5 -> 4.1 s)
  const int nb = p.spec ? nb_want : nb_fit;
  p.nb = nb;
  // wide blocks need no more workspace than blocks of nb_fit columns with an
  // inverse, a copied panel and a solve's scratch of that width did
  p.tmp_cols = p.spec ? std::min(nb, 3 * nb_fit) : nb;
  // (whole blocks of 128 or 64 columns; the planes hold no others)
  p.split = refined && elem_bytes == 4 && (nb == 128 || nb == 64) && nb < n;
  // Workgroups of one panel.  Measured on n = 12 000: an FP32 panel over at most
  // 128 CUs is as fast per column as one over all 256 and leaves the other CUs
  // to the look-ahead update (140 vs 150 ms per factorisation + solve step); an
  // FP64 panel (twice the bytes per row) is fastest spread over every CU.  The
  // cap is raised when the panel's rows would not fit the LDS of fewer
  // workgroups.
  int cap = avail;
  if (elem_bytes == 4 && nbatch == 1) {
    const int64_t rmax = panel_rows_max(nb, lds_bytes, cbytes, pb);
    const int64_t need = rmax > 0 ? (n + rmax - 1) / rmax : avail;
    cap = (int)std::min<int64_t>(avail, std::max<int64_t>(128, need));
  }
  for (int64_t k0 = 0; k0 < n; k0 += nb) {
    LUBlock b;
    b.k0 = k0;
    b.w = (int)(n - k0 < nb ? n - k0 : nb);
    const int64_t m = n - k0;
    int64_t R = (m + cap - 1) / cap;
    if (R < 32) R = 32;
    const int64_t Rmax = panel_rows_max(b.w, lds_bytes, cbytes, pb);
    if (R > Rmax) R = Rmax;
    b.R = (int)R;
    b.G = (int)((m + R - 1) / R);
    p.blocks.push_back(b);
  }
  return p;
}

bool lu_plan_fits(const LUPlan& p) {
  if (p.spec) return true;
  for (const LUBlock& b : p.blocks)
    if (b.G + (p.pb > 1 ? tp_roots(b.G) : 0) > p.max_wg || (int64_t)b.G * b.R < p.n - b.k0) return false;
  return true;
}

// rows of the complex scratch `tmp` (x plan.tmp_cols): the sweeps of a solve need
// n; the split-k partial sums of the transposed solve more than n for small n
static int64_t tmp_rows(const LUPlan& p) { return p.n > 512 ? p.n : 512; }

static size_t al256(size_t b) { return (b + 255) / 256 * 256; }

// bytes of one split operand (the updates read whole 128-wide tiles from any
// multiple of 64 columns on)
static int64_t lu_plane_stride(const LUPlan& p) { return p.split ? split_bytes(p.n - p.nb + 128, p.nb) : 0; }
size_t lu_planes_bytes(const LUPlan& p, int nbatch) { return (size_t)nbatch * 3 * lu_plane_stride(p); }

size_t lu_workspace_bytes(const LUPlan& p, int elem_bytes, int num_cu, int nbatch) {
  LUWork w;
  lu_workspace_carve(nullptr, p, elem_bytes, num_cu, w, nbatch);
  return w.bytes;
}

// Every per-item field is nbatch consecutive copies `s_*` elements apart.
void lu_workspace_carve(void* base, const LUPlan& p, int elem_bytes, int num_cu, LUWork& w, int nbatch) {
  if (nbatch < 1) nbatch = 1;
  const size_t nb = (size_t)p.nb, nblk = p.blocks.size();
  const size_t ww = nb * (2 * (size_t)elem_bytes / 4);
  const size_t cb = 2 * (size_t)elem_bytes;
  char* b = static_cast<char*>(base);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* r = b ? b + off : nullptr;
    off += al256(bytes) + 256;
    return r;
  };
  w.nbatch = nbatch;
  w.gmax = num_cu;
  w.gitem = p.max_wg > 0 ? p.max_wg : num_cu;
  w.pb = p.pb;
  w.wwmax = (int)ww;
  const size_t pbz = (size_t)(p.pb > 1 ? p.pb : 1);
  const size_t nwc = 2 * (size_t)elem_bytes / 4;  // 32-bit words per complex
  // tournament: records [2][gitem][pb][1 + pb nwc], then the roots' winners
  // [2][ceil(gitem / 32)][pb][2 + pb nwc]; partial pivoting: keys [2][gitem][KEY_STRIDE]
  // (speculative panels exchange nothing)
  const size_t cand_words = p.spec ? 0 : p.pb > 1 ? 2 * (size_t)w.gitem * pbz * (1 + pbz * nwc) +
                                           2 * (size_t)tp_roots(w.gitem) * pbz * (2 + pbz * nwc)
                                     : 2 * (size_t)w.gitem * KEY_STRIDE;
  w.s_cand = (int64_t)(al256(cand_words * 8) / 8);
  w.s_rows = p.spec ? 0 : (int64_t)(al256(2 * (size_t)w.gitem * pbz * ww * 8) / 8);
  w.cand = reinterpret_cast<unsigned long long*>(take((size_t)nbatch * w.s_cand * 8));
  w.rows = reinterpret_cast<unsigned long long*>(take((size_t)nbatch * w.s_rows * 8));
  w.err = reinterpret_cast<int32_t*>(take(64));
  w.s_pairs = (int64_t)(al256(nblk * 2 * 2 * nb * 4) / 4);
  w.s_npairs = (int64_t)(al256(2 * nblk * 4) / 4);  // moved-row counts, then the speculative panels' flags
  w.pairs = reinterpret_cast<int32_t*>(take((size_t)nbatch * w.s_pairs * 4));
  w.npairs = reinterpret_cast<int32_t*>(take((size_t)nbatch * w.s_npairs * 4));
  w.spec = w.npairs ? w.npairs + nblk : nullptr;
  w.tmp_elems = tmp_rows(p) * (int64_t)p.tmp_cols;
  w.s_tmp = (int64_t)(al256((size_t)w.tmp_elems * cb) / cb);
  w.s_tinv = (int64_t)(al256(nblk * (size_t)tinv_block_elems(p.nb) * cb) / cb);
  w.tmp = w.tinv = take((size_t)nbatch * std::max(w.s_tmp, w.s_tinv) * cb);
  w.s_split = lu_plane_stride(p);
  w.events = nullptr;
  w.bytes = off + 256;
}

// The panel kernel of a plan (pb columns per exchange).
template <typename T>
static const void* panel_fn(int pb) {
  switch (pb) {
    case 2: return reinterpret_cast<const void*>(&panel_tp_kernel<T, 2>);
    case 4: return reinterpret_cast<const void*>(&panel_tp_kernel<T, 4>);
    case 8:
      if constexpr (sizeof(T) == 4) return reinterpret_cast<const void*>(&panel_tp_kernel<T, 8>);
      return nullptr;
    default: return reinterpret_cast<const void*>(&panel_kernel<T>);
  }
}

// Whether block b's panel takes the kernel whose columns are one wave's work: one
// system, pivots one column at a time, a workgroup's rows one per lane, its LDS
// and exchange buffers as they are.  (FP32 from n = 8192 on and FP64 from about 14 000
// have more rows per workgroup in the first blocks.)
template <typename T>
static bool panel_in_wave(const LUPlan& p, const LUBlock& b, int gitem) {
  return p.pb <= 1 && p.nbatch == 1 && b.R <= 64 && b.G <= 256 &&
         (p.nb <= SUBW || (int64_t)gitem * (p.nb - SUBW) >= (int64_t)SUBW * p.nb) &&
         panel_wave_lds<cplx<T>>(b.w, b.R) + 256 <= (size_t)p.lds_bytes;
}

// One panel launch: G row workgroups (plus the roots of a tournament panel) per item.
template <typename T>
static void launch_panel(int pb, bool in_wave, const LUBlock& b, int NB, size_t lds, hipStream_t st, cplx<T>* A, int64_t ld,
                         int64_t n, int32_t* ipiv, const LUWork& ws, uint32_t epoch, int64_t sA, int64_t sipiv,
                         int32_t* dst, int32_t* src, int32_t* npr, int mcap) {
  if (in_wave) {
    hipLaunchKernelGGL(panel_wave_kernel<T>, dim3(b.G), dim3(256), panel_wave_lds<cplx<T>>(b.w, b.R), st, A, ld, n, b.k0,
                       b.w, b.R, b.G, ipiv, ws, epoch, dst, src, npr, mcap);
    return;
  }
  const dim3 grid(b.G + (pb > 1 ? tp_roots(b.G) : 0), NB);
#define GDM_PANEL_ARGS A, ld, n, b.k0, b.w, b.R, b.G, ipiv, ws, epoch, sA, sipiv, dst, src, npr, mcap
  switch (pb) {
    case 2: hipLaunchKernelGGL((panel_tp_kernel<T, 2>), grid, dim3(256), lds, st, GDM_PANEL_ARGS); break;
    case 4: hipLaunchKernelGGL((panel_tp_kernel<T, 4>), grid, dim3(256), lds, st, GDM_PANEL_ARGS); break;
    case 8:
      if constexpr (sizeof(T) == 4) {
        hipLaunchKernelGGL((panel_tp_kernel<T, 8>), grid, dim3(256), lds, st, GDM_PANEL_ARGS);
        break;
      }
      [[fallthrough]];
    default: hipLaunchKernelGGL(panel_kernel<T>, grid, dim3(256), lds, st, GDM_PANEL_ARGS); break;
  }
#undef GDM_PANEL_ARGS
}

// Panels may need more than the default 64 KB of dynamic LDS: raise each panel
// kernel's limit once (a host-side setting; done before any graph capture).
template <typename T>
hipError_t lu_prepare(const LUPlan& plan) {
  static std::map<const void*, size_t> lds_set;
  static std::mutex mu;
  std::lock_guard<std::mutex> lk(mu);
  if (plan.spec) {
    static bool diag_set = false;
    if (!diag_set) {
      hipError_t e = prepare_diag_lu<T>();
      if (e != hipSuccess) return e;
      diag_set = true;
    }
  }
  if (plan.spec) return hipSuccess;
  for (const LUBlock& b : plan.blocks) {
    const bool in_wave = panel_in_wave<T>(plan, b, plan.max_wg);
    const size_t need = in_wave ? panel_wave_lds<cplx<T>>(b.w, b.R) : panel_lds_bytes(b.w, b.R, sizeof(cplx<T>), plan.pb);
    const void* fn = in_wave ? reinterpret_cast<const void*>(&panel_wave_kernel<T>) : panel_fn<T>(plan.pb);
    if (!fn) return hipErrorInvalidValue;
    size_t& cur = lds_set[fn];
    if (need > 64 * 1024 && need > cur) {
      hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)need);
      if (e != hipSuccess) return e;
      cur = need;
    }
  }
  return hipSuccess;
}
template hipError_t lu_prepare<double>(const LUPlan&);
template hipError_t lu_prepare<float>(const LUPlan&);

// Whether a step's trailing update is split between the two streams: below
// about 30 us of update (its CU time at the rate of the large updates) the two
// events of a split cost as much as the overlap with the next panel gives.
static bool lu_lookahead_pays(int elem_bytes, int64_t nr, int nbatch) {
  return (double)nr * (double)nr * nbatch * (elem_bytes / 4) > 2.5e6;
}

template <typename T>
hipError_t lu_factor(void* Av, int64_t ld, const LUPlan& plan, const LUWork& ws, int32_t* ipiv, hipStream_t st,
                     Prof* prof, hipStream_t side, int64_t sA, int64_t sipiv) {
  Prof noprof;
  Prof& P = prof ? *prof : noprof;
  using CT = cplx<T>;
  CT* A = static_cast<CT*>(Av);
  const int64_t n = plan.n;
  const int nb = plan.nb;
  const int nblk = (int)plan.blocks.size();
  const int NB = ws.nbatch;
  const double fb = (double)NB;
  hipError_t e;
  if (NB < 1 || NB > 65535 || !lu_plan_fits(plan) || plan.max_wg * NB > ws.gmax || plan.max_wg > ws.gitem ||
      plan.pb > ws.pb || (plan.split && !ws.split))
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(init_err_kernel, dim3(1), dim3(64), 0, st, ws.err);
  // exchange buffers start from zero (epoch 0 is never used), so epochs 1, 2, ...
  // of this factorisation are unique
  // (and the moved-row counters of every block, which the panels fill)
  {
    const size_t nc = (size_t)NB * ws.s_cand, nr = (size_t)NB * ws.s_rows, np = (size_t)NB * ws.s_npairs;
    const size_t nmax = std::max(std::max(nc, nr), np);
    hipLaunchKernelGGL(zero_u64_kernel, dim3((unsigned)((nmax + 255) / 256)), dim3(256), 0, st, ws.cand, nc, ws.rows, nr,
                       ws.npairs, np);
  }
  uint32_t epoch = 1;
  if ((e = lu_prepare<T>(plan)) != hipSuccess) return e;
  // Look-ahead: the main stream runs the panels, the triangular solves and the
  // update of the next panel's columns; the side stream runs the bulk of each
  // trailing update, overlapping the next panel.  (U12 in one launch: its columns
  // past the next panel's on the side stream, as a launch of their own before the
  // bulk, cost n = 12 000 in FP32 1.9 ms of 42.3, n = 3001 in FP64 0.5 of 11.6.)
  const bool la = side != nullptr && side != st && ws.events != nullptr;
  // events come from a pool owned by the caller and reused across calls (the
  // caller synchronises the stream before the next factorisation)
  size_t ev_used = 0;
  auto new_event = [&](hipEvent_t& ev) -> hipError_t {
    if (!ws.events) return hipErrorInvalidValue;
    if (ev_used == ws.events->size()) {
      hipEvent_t x;
      hipError_t r = hipEventCreateWithFlags(&x, hipEventDisableTiming);
      if (r != hipSuccess) return r;
      ws.events->push_back(x);
    }
    ev = (*ws.events)[ev_used++];
    return hipSuccess;
  };
#define LUCHK(x)                   \
  do {                             \
    if ((e = (x)) != hipSuccess) { \
      return e;                    \
    }                              \
  } while (0)
  CT* tinv0 = static_cast<CT*>(ws.tinv);
  const int64_t btinv = tinv_block_elems(nb);
  hipEvent_t bulk_done = nullptr;  // side stream finished the previous block's bulk update
  for (int bi = 0; bi < nblk; ++bi) {
    const LUBlock& b = plan.blocks[bi];
    const int64_t k0 = b.k0;
    const int w = b.w;
    const size_t lds = panel_lds_bytes(w, b.R, sizeof(CT), plan.pb);
    CT* tinv = tinv0 + bi * btinv;
    LUCHK(P.begin(st, PROF_PANEL, (double)w * fb));
    int32_t* dst = ws.pairs + bi * 4 * (size_t)nb;  // moved rows: destinations, then sources 2 nb later
    int32_t* src = dst + 2 * nb;
    int32_t* npr = ws.npairs + bi;
    int32_t* flag = ws.spec + bi;
    if (plan.spec) {
      LUCHK(launch_diag_lu<T>(A, ld, nb, k0, w, ipiv, flag, tinv, st, NB, sA, sipiv, ws.s_npairs, ws.s_tinv));
    } else {
      launch_panel<T>(plan.pb, panel_in_wave<T>(plan, b, ws.gitem), b, NB, lds, st, A, ld, n, ipiv, ws, epoch, sA, sipiv, dst, src, npr, 2 * nb);
      epoch += (uint32_t)w;
      LUCHK(hipGetLastError());
      LUCHK(launch_tile_inv<T>(A, ld, nb, k0, w, tinv, st, NB, sA, ws.s_tinv));
    }
    LUCHK(P.end(st));
    const int64_t c1 = k0 + w;
    const int64_t nr = n - c1;
    if (nr <= 0) break;
    // columns [c1, c1 + wa) on the main stream, [c1 + wa, n) on the side stream;
    // once the trailing matrix is small, all of it on the main stream
    const bool split = la && nr > nb && lu_lookahead_pays((int)sizeof(T), nr, NB);
    const int64_t wa = split ? nb : nr;
    // one block's interchanges on ncols columns from cb on (a speculative panel moves no rows)
    auto permute = [&](hipStream_t s, int64_t cb, int64_t ncols) -> hipError_t {
      if (plan.spec) return hipSuccess;
      hipError_t r;
      if ((r = P.begin(s, PROF_PERM, 0.0)) != hipSuccess) return r;
      hipLaunchKernelGGL(row_permute_kernel<T>, dim3((unsigned)ncols, NB), dim3(256), 0, s, A, ld, cb, dst, src, npr, sA,
                         ws.s_pairs, ws.s_npairs);
      if ((r = hipGetLastError()) != hipSuccess) return r;
      return P.end(s);
    };
    // split operands: L21's planes alternate between two buffers (the next panel
    // writes its own while this step's bulk update still reads), U12's columns go
    // to disjoint parts of one
    const bool split_ops = plan.split && w == nb;
    const int64_t ssplit = 3 * ws.s_split, pl_bytes = split_planes_bytes(plan.n - nb + 128, nb);
    SplitOut lout, uout;
    if (split_ops) {
      lout.planes = ws.split + (bi & 1) * ws.s_split;
      lout.scales = reinterpret_cast<float*>(lout.planes + pl_bytes);
      uout.planes = ws.split + 2 * ws.s_split;
      uout.scales = reinterpret_cast<float*>(uout.planes + pl_bytes);
    }
    auto u_at = [&](int64_t cb) {  // the part of U12 from column cb on
      SplitOut o = uout;
      if (split_ops) {
        o.planes += (cb - c1) / 32 * (int64_t)(nb / 16) * 4096;
        o.scales += cb - c1;
      }
      return o;
    };
    // L21 = A21 U11^-1 (speculative panels) and U12 = L11^-1 A12 of ncols columns
    auto tri = [&](hipStream_t s, int tag, int64_t nrows, int64_t cb, int64_t ncols) -> hipError_t {
      hipError_t r;
      if ((r = P.begin(s, tag, 8.0 * (double)(nrows + ncols) * w * w * fb)) != hipSuccess) return r;
      if ((r = launch_tri_panel<T>(A, ld, nb, k0, w, nrows, cb, ncols, tinv, flag, s, NB, sA, ws.s_tinv, ws.s_npairs,
                                   lout, u_at(cb), ssplit)) != hipSuccess)
        return r;
      return P.end(s);
    };
    // A22[:, cols] -= L21 U12[:, cols]
    auto update = [&](hipStream_t s, int tag, int64_t cb, int64_t ncols) -> hipError_t {
      hipError_t r;
      if ((r = P.begin(s, tag, 8.0 * (double)nr * (double)ncols * w * fb)) != hipSuccess) return r;
      if constexpr (sizeof(T) == 4) {
        if (split_ops) {
          const SplitOut uo = u_at(cb);
          if ((r = launch_update_split(nr, ncols, w, lout.planes, uo.planes, lout.scales, uo.scales, A + c1 + cb * ld, ld, s,
                                       ws.gmax, NB, ssplit, sA)) != hipSuccess)
            return r;
          return P.end(s);
        }
      }
      if ((r = launch_gemm_update<T>(nr, ncols, w, A + c1 + k0 * ld, ld, A + k0 + cb * ld, ld, A + c1 + cb * ld, ld, s, NB,
                                     sA, sA, sA)) != hipSuccess)
        return r;
      return P.end(s);
    };
    // L21 needs the panel alone: while the previous block's bulk update still
    // runs it goes ahead of the wait, else it shares the U12 block's launch
    const int64_t lrows = plan.spec ? nr : 0;
    if constexpr (sizeof(T) == 4) {
      if (!plan.spec && split_ops) LUCHK(launch_split_rows(A + c1 + k0 * ld, ld, nr, w, lout, st, NB, sA, ssplit));
    }
    if (bulk_done) {
      if (lrows > 0) LUCHK(tri(st, PROF_PANEL_L21, lrows, c1, 0));
      LUCHK(hipStreamWaitEvent(st, bulk_done, 0));  // columns of this step were in the bulk
      bulk_done = nullptr;
      LUCHK(permute(st, c1, nr));
      LUCHK(tri(st, PROF_TRSM, 0, c1, nr));
    } else {
      LUCHK(permute(st, c1, nr));
      LUCHK(tri(st, PROF_PANEL_L21, lrows, c1, nr));
    }
    // (a launch that reaches past the next panel's columns counts as bulk)
    LUCHK(update(st, wa <= nb ? PROF_LOOKAHEAD : PROF_UPDATE, c1, wa));
    if (!split) continue;
    // The side stream starts after the look-ahead product, so that the next
    // diagonal block's workgroup finds a free CU before the bulk update takes
    // them all.
    hipEvent_t main_updated = nullptr;
    LUCHK(new_event(main_updated));
    LUCHK(hipEventRecord(main_updated, st));
    LUCHK(hipStreamWaitEvent(side, main_updated, 0));
    LUCHK(update(side, PROF_UPDATE, c1 + wa, nr - wa));
    LUCHK(new_event(bulk_done));
    LUCHK(hipEventRecord(bulk_done, side));
  }
  if (bulk_done) LUCHK(hipStreamWaitEvent(st, bulk_done, 0));
  // the solve-ready form of all blocks at once
  LUCHK(P.begin(st, PROF_TRSM, 0.0));
  LUCHK(launch_finish<T>(A, ld, n, nb, tinv0, st, NB, sA, ws.s_tinv));
  LUCHK(P.end(st));
  return hipGetLastError();
#undef LUCHK
}

// Whether a transposed sweep pushes a block's part into the later columns
// (skinny_push_kernel) or gathers each block's sum (skinny_t_kernel).  Pushing
// saves a launch and the partial sums per block (n = 3000 speculative, time of a
// push over a gather: 0.40 for one column in FP32, 0.46 in FP64), but starts with
// the diagonal blocks, one workgroup each, whose time only several blocks make up
// for: n = 120 1.1 to 1.9 in FP32 and 1.4 to 3.0 in FP64, n = 420 0.61 to 0.88 and
// 0.79 (1 column), 1.00 (2), 1.30 (3, 4), 0.93 (5 and more), n = 1029 0.48 to 0.89
// and 0.57 to 0.99.  And its reductions over 128 rows, where a gather's run over
// 256, bound it once the launches are full: FP64 n = 6000 0.78 at 16 columns, 0.99
// at 32, 1.16 at 66, n = 2100 0.98 at 66, 1.05 at 130; FP32 n = 6000 0.98 at 66, 1.07
// at 130.
static bool lu_solve_pushes(int elem_bytes, int64_t n, int nblk, int64_t nr, int nbatch) {
  if (elem_bytes == 4) return nblk >= (nr == 1 ? 2 : 3) && n * nr * nbatch <= 450000;
  return nblk >= (nr == 1 ? 3 : nr == 2 ? 5 : nr <= 4 ? 8 : 4) && n * nr * nbatch <= 190000;
}

template <typename T>
hipError_t lu_solve(int trans, const void* Av, int64_t ld, const LUPlan& plan, const LUWork& ws, void* Bv,
                    int64_t ldb, int64_t nrhs, hipStream_t st, int64_t sA, int64_t sB) {
  using CT = cplx<T>;
  const CT* A = static_cast<const CT*>(Av);
  CT* Ball = static_cast<CT*>(Bv);
  const int64_t n = plan.n;
  const int nb = plan.nb;
  const int nblk = (int)plan.blocks.size();
  const int NB = ws.nbatch;
  CT* X = static_cast<CT*>(ws.tmp);
  const int64_t sX = ws.s_tmp;
  hipError_t e;
  if (nrhs <= 0) return hipSuccess;
  // RHS columns per pass: the plain solve keeps n per column in tmp; the
  // transposed steps need (chunks of the longest product) x nb partial sums per column.
  const int64_t chunk = ws.tmp_elems / (trans ? skinny_t_chunks(n, nb) * nb : n);
  if (chunk < 1) return hipErrorInvalidValue;
  const int64_t part_elems = (int64_t)NB * sX;  // the transposed partial sums of all items
  // factors left by a speculative plan have no interchanges (a failed check
  // repeats the factorisation with a pivoting plan), so their lists are empty
  const bool perm = !plan.spec;
  for (int64_t r0 = 0; r0 < nrhs; r0 += chunk) {
    const int64_t nr = nrhs - r0 < chunk ? nrhs - r0 : chunk;
    CT* B = Ball + r0 * ldb;
    const bool small = nr <= SKINNY_MAX_RHS;
    if (trans == 0) {
      // The forward result goes to tmp (Y, n x nr, leading dimension n), so that
      // every block step reads its operand rows in place: the step's product
      // writes those rows to the other buffer (the forward into Y, the backward
      // back into B), and no step needs a copy of them.
      CT* Y = X;
      // forward: P_b, then rows [k0, n) -= [I - L11^-1 ; L21 L11^-1] B_b, rows [k0, k0 + w) into Y
      for (int bi = 0; bi < nblk; ++bi) {
        const LUBlock& b = plan.blocks[bi];
        const int64_t k0 = b.k0;
        const int32_t* dst = ws.pairs + bi * 4 * (size_t)nb;
        const int32_t* src = dst + 2 * nb;
        if (perm) {
          hipLaunchKernelGGL(row_permute_kernel<T>, dim3((unsigned)nr, NB), dim3(256), 0, st, B, ldb, (int64_t)0, dst,
                             src, ws.npairs + bi, sB, ws.s_pairs, ws.s_npairs);
          if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        GemmMask m;
        m.akind = GEMM_MASK_STRICT_LOWER;
        m.ar0 = 0;
        m.adw = b.w;
        m.c2 = Y + k0;
        m.ldc2 = n;
        m.sc2 = sX;
        e = small ? launch_skinny_n<T>(n - k0, b.w, A + k0 + k0 * ld, ld, B + k0, ldb, B + k0, ldb, nr, st, m, NB, sA,
                                       sB, sB)
                  : launch_solve_step<T>(n - k0, b.w, A + k0 + k0 * ld, ld, B + k0, ldb, B + k0, ldb, nr, st, m, NB, sA,
                                         sB, sB);
        if (e != hipSuccess) return e;
      }
      // backward on Y: rows [0, k0 + w) -= [U01 U11^-1 ; I - U11^-1] Y_b, rows [k0, k0 + w) into B
      for (int bi = nblk - 1; bi >= 0; --bi) {
        const LUBlock& b = plan.blocks[bi];
        const int64_t k0 = b.k0;
        GemmMask m;
        m.akind = GEMM_MASK_UPPER;
        m.ar0 = k0;
        m.adw = b.w;
        m.c2 = B + k0;
        m.ldc2 = ldb;
        m.sc2 = sB;
        e = small ? launch_skinny_n<T>(k0 + b.w, b.w, A + k0 * ld, ld, Y + k0, n, Y, n, nr, st, m, NB, sA, sX, sX)
                  : launch_solve_step<T>(k0 + b.w, b.w, A + k0 * ld, ld, Y + k0, n, Y, n, nr, st, m, NB, sA, sX, sX);
        if (e != hipSuccess) return e;
      }
    } else {
      const bool push = lu_solve_pushes((int)sizeof(T), n, nblk, nr, NB);
      // M^T = U^T L_k^T P_k ... L_1^T P_1.  U^T forward, with V = U01 U11^-1 stored above the diagonal:
      //   z_b = U11^-T g_b - V_b^T z_above, the first term of all blocks at once
      if (push && (e = launch_skinny_diag_t<T>(false, n, nb, A, ld, B, ldb, nr, st, NB, sA, sB)) != hipSuccess) return e;
      // (or gathered, z_b = g_b - V_b^T z_above - (I - U11^-1)^T g_b: both products read g_b)
      for (int bi = 0; !push && bi < nblk; ++bi) {
        const LUBlock& b = plan.blocks[bi];
        const int64_t k0 = b.k0;
        if ((e = launch_skinny_t<T>(b.w, nr, A + k0 * ld, ld, B, ldb, k0, A + k0 + k0 * ld, ld, B + k0, ldb, b.w,
                                    GEMM_MASK_LOWER, X, part_elems, B + k0, ldb, st, NB, sA, sB, sB)) != hipSuccess)
          return e;
      }
      for (int bi = 0; push && bi + 1 < nblk; ++bi) {
        const LUBlock& b = plan.blocks[bi];
        const int64_t k0 = b.k0, c1 = k0 + b.w;
        if ((e = launch_skinny_push<T>(b.w, n - c1, A + k0 + c1 * ld, ld, B + k0, B + c1, ldb, nr, st, NB, sA, sB)) !=
            hipSuccess)
          return e;
      }
      // then for b = k..1: z_b = L11^-T z_b - (L21 L11^-1)^T z_below, and z = P_b^T z
      if (push && !perm) {
        if ((e = launch_skinny_diag_t<T>(true, n, nb, A, ld, B, ldb, nr, st, NB, sA, sB)) != hipSuccess) return e;
        for (int bi = nblk - 1; bi > 0; --bi) {
          const LUBlock& b = plan.blocks[bi];
          if ((e = launch_skinny_push<T>(b.w, b.k0, A + b.k0, ld, B + b.k0, B, ldb, nr, st, NB, sA, sB)) != hipSuccess)
            return e;
        }
        continue;
      }
      // (interchanges move rows between a block's sum and the next: gathered block by block)
      for (int bi = nblk - 1; bi >= 0; --bi) {
        const LUBlock& b = plan.blocks[bi];
        const int64_t k0 = b.k0, c1 = k0 + b.w;
        if ((e = launch_skinny_t<T>(b.w, nr, A + c1 + k0 * ld, ld, B + c1, ldb, n - c1, A + k0 + k0 * ld, ld, B + k0,
                                    ldb, b.w, GEMM_MASK_STRICT_UPPER, X, part_elems, B + k0, ldb, st, NB, sA, sB, sB)) !=
            hipSuccess)
          return e;
        if (!perm) continue;
        const int32_t* dst = ws.pairs + bi * 4 * (size_t)nb;
        const int32_t* src = dst + 2 * nb;
        hipLaunchKernelGGL(row_permute_inv_kernel<T>, dim3((unsigned)nr, NB), dim3(256), 0, st, B, ldb, (int64_t)0, dst,
                           src, ws.npairs + bi, sB, ws.s_pairs, ws.s_npairs);
      }
    }
  }
  return hipGetLastError();
}

template hipError_t lu_factor<double>(void*, int64_t, const LUPlan&, const LUWork&, int32_t*, hipStream_t, Prof*,
                                      hipStream_t, int64_t, int64_t);
template hipError_t lu_factor<float>(void*, int64_t, const LUPlan&, const LUWork&, int32_t*, hipStream_t, Prof*,
                                     hipStream_t, int64_t, int64_t);
template hipError_t lu_solve<double>(int, const void*, int64_t, const LUPlan&, const LUWork&, void*, int64_t, int64_t,
                                     hipStream_t, int64_t, int64_t);
template hipError_t lu_solve<float>(int, const void*, int64_t, const LUPlan&, const LUWork&, void*, int64_t, int64_t,
                                    hipStream_t, int64_t, int64_t);

}  // namespace gdm
