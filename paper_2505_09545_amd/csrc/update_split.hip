// FP32 trailing update C -= L U of the blocked LU (arXiv:2505.09545, Sec.
// "Numerical solution") on the f16 matrix cores, for factors whose solutions are
// refined in FP64.  Every row of L and every column of U is scaled by a power of
// two (exact, undone in the epilogue) so that its largest entry lies in [2^13,
// 2^14), and every scaled entry is the sum of two f16 numbers h + l: off by at most
// 2^-23 of the entry, or 2^-38 of the row's largest if that is more (below 2^-15
// of it).  Of the four products of two such sums h h' + (h l' + l h') are kept,
// accumulated in FP32.  So the error of an entry of C has, beside that of an FP32
// product, up to 2^-38 (max_k |l_ik| sum_k |u_kj| + max_k |u_kj| sum_k |l_ik|).
// That stays below FP32 rounding unless the rows of the matrix differ in size by
// 2^15 and more within a block (scales of whole rows or columns of C do not
// matter, scales along k do): a coupling matrix (A^-1 - G) A has its scales on the
// columns, a caller's matrix may have them anywhere and takes FP32 products.
// The f16 cores do 16 times the FP32 ones' rate, so the three products of each of
// the four real products of a complex one cost a quarter of the 3M form in FP32
// matrix instructions, which this replaces.  Error against 64 bits: see the
// comment at launch_update_split.
//
// The operands come split and in MFMA order from the triangular solves that
// form them (tiles.hip), so the product's loop has no conversions: a fragment
// is 32 rows (columns) x 16 k of one of the four planes (re h, re l, im h, im l),
// 64 lanes x 16 bytes, stored as [tile of 32][k / 16][plane].  L rows are the
// second MFMA operand, so a lane's results are one row of C in 16 columns and a
// wave's C accesses are 256-byte runs of a column.
#include <algorithm>

#include "gdm_common.hpp"
#include "gdm_kernels.hpp"
#include "lu_common.hpp"

namespace gdm {

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ inline f32x16 mfma_f16(u32x4 a, u32x4 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// acc += x y over one k step of 16: x, y the two planes of two operands
__device__ inline void mac3(f32x16& acc, const u32x4 (&x)[2], const u32x4 (&y)[2]) {
  acc = mfma_f16(x[1], y[0], acc);
  acc = mfma_f16(x[0], y[1], acc);
  acc = mfma_f16(x[0], y[0], acc);
}

// re, im += the complex product of one k step of 16 (l: rows, u: columns)
__device__ inline void mac_complex(f32x16& re, f32x16& im, const u32x4 (&l)[4], const u32x4 (&u)[4]) {
  const u32x4 lr[2] = {l[0], l[1]}, li[2] = {l[2], l[3]};
  const u32x4 ur[2] = {u[0], u[1]}, ui[2] = {u[2], u[3]};
  const u32x4 nui[2] = {u[2] ^ 0x80008000u, u[3] ^ 0x80008000u};
  mac3(re, ur, lr);
  mac3(im, ui, lr);
  mac3(re, nui, li);
  mac3(im, ur, li);
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
// entries of a C past the last-level cache, used once per launch: not kept in the caches
template <bool NT> __device__ inline float2 load_c(const float2* p) {
  if constexpr (!NT) return *p;
  const f32x2 v = __builtin_nontemporal_load(reinterpret_cast<const f32x2*>(p));
  return make_float2(v.x, v.y);
}
template <bool NT> __device__ inline void store_c(float2* p, float2 x) {
  if constexpr (NT) __builtin_nontemporal_store(f32x2{x.x, x.y}, reinterpret_cast<f32x2*>(p));
  else *p = x;
}

// Tile order of gemm.hip: each XCD takes a contiguous range of tiles, walked by
// groups of GM tile rows over a block of tile columns, so that the group's
// fragments and the block's stay in that XCD's L2.
template <int GM, int NBLK>
__device__ inline void grouped_tile(int t, int tiles_m, int tiles, int& tm, int& tn) {
  const int tiles_n = tiles / tiles_m;
  const int cbw = (tiles_n + NBLK - 1) / NBLK;
  const int per_blk = tiles_m * cbw;
  const int blk = t / per_blk;
  const int within = t - blk * per_blk;
  const int cols = min(cbw, tiles_n - blk * cbw);
  const int per_grp = GM * cols;
  const int grp = within / per_grp;
  const int w2 = within - grp * per_grp;
  const int rows = min(GM, tiles_m - grp * GM);
  tm = grp * GM + w2 % rows;
  tn = blk * cbw + w2 / rows;
}

}  // namespace

// 64 x 64 tiles: 2 x 2 waves of one 32 x 32 MFMA tile each.  Per 16 k the
// workgroup's fragments go through one of two LDS buffers (loaded into registers
// a step ahead), one barrier per step; C is loaded during the k loop, an equal
// part per step.  Three or four workgroups fit a CU, which overlaps one's
// epilogue with another's products.  NKT: k / 16 (8 or 4).
// m = n = 3000, k = 128: 47 us, 195 TFLOP/s by 8 m n k (128 x 128 tiles of 8
// waves 52-58 us); the 3M form in FP32 instructions took 94 us.
template <int NKT>
__global__ void __launch_bounds__(256)
update_split_kernel(int64_t m, int64_t n, const u32x4* __restrict__ L, const u32x4* __restrict__ U,
                    const float* __restrict__ sl, const float* __restrict__ su, float2* __restrict__ C, int64_t ldc,
                    int tiles_m, int tiles, int64_t sL, int64_t sC) {
  constexpr int NF = 16, FW = 4;             // fragments per step (8 of the rows, 8 of the columns), per wave
  constexpr int CE = 16 / NKT;               // entries of C loaded per step
  L += (int64_t)blockIdx.y * (sL / 16);
  U += (int64_t)blockIdx.y * (sL / 16);
  sl += (int64_t)blockIdx.y * (sL / 4);
  su += (int64_t)blockIdx.y * (sL / 4);
  C += (int64_t)blockIdx.y * sC;
  __shared__ u32x4 lds[2][NF * 64];
  const int bid = blockIdx.x;
  const int xcd = bid & 7, loc = bid >> 3;
  const int per = tiles >> 3, rem = tiles & 7;
  const int tile = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + loc;
  int tm, tn;
  grouped_tile<8, 8>(tile, tiles_m, tiles, tm, tn);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave & 1, wc = wave >> 1;
  // this wave's fragments of a step: plane `wave` of each of the four 32-row and 32-column tiles
  const u32x4* src[FW];
#pragma unroll
  for (int i = 0; i < FW; ++i)
    src[i] = (i < 2 ? L + (int64_t)(2 * tm + i) * NKT * 256 : U + (int64_t)(2 * tn + i - 2) * NKT * 256) + wave * 64;
  u32x4 st[FW];
  auto gload = [&](int kt) {
#pragma unroll
    for (int i = 0; i < FW; ++i) st[i] = src[i][kt * 256 + lane];
  };
  auto sstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < FW; ++i) lds[buf][(4 * i + wave) * 64 + lane] = st[i];
  };
  f32x16 re, im;
#pragma unroll
  for (int q = 0; q < 16; ++q) re[q] = im[q] = 0;
  const int64_t row = (int64_t)(2 * tm + wr) * 32 + (lane & 31);
  const int64_t col0 = (int64_t)(2 * tn + wc) * 32 + 4 * (lane >> 5);
  const bool full = (int64_t)(tm + 1) * 64 <= m && (int64_t)(tn + 1) * 64 <= n;
  auto col_of = [&](int q) { return col0 + (q & 3) + 8 * (q >> 2); };
  auto inside = [&](int q) { return full || (row < m && col_of(q) < n); };
  float2 c[16];
  auto cload = [&](int q) {
    c[q] = make_float2(0.f, 0.f);
    if (inside(q)) c[q] = C[row + col_of(q) * ldc];
  };
  auto mma = [&](int buf) {
    u32x4 l[4], u[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) l[p] = lds[buf][(4 * wr + p) * 64 + lane];
#pragma unroll
    for (int p = 0; p < 4; ++p) u[p] = lds[buf][(8 + 4 * wc + p) * 64 + lane];
    mac_complex(re, im, l, u);
  };
  gload(0);
  sstore(0);
  __syncthreads();
  auto step = [&](int kt) {
    if (kt + 1 < NKT) gload(kt + 1);
#pragma unroll
    for (int e = 0; e < CE; ++e) cload(CE * kt + e);
    __builtin_amdgcn_sched_barrier(0);
    mma(kt & 1);
    if (kt + 1 < NKT) sstore((kt + 1) & 1);
    __syncthreads();
  };
  static_for<NKT>([&](auto kt) { step(kt); });
  // C -= (acc 2^a) 2^b
  const float fr = sl[row];
#pragma unroll
  for (int q = 0; q < 16; ++q) {
    const float fc = su[col_of(q)];
    if (inside(q)) C[row + col_of(q) * ldc] = make_float2(fmaf(-re[q] * fr, fc, c[q].x), fmaf(-im[q] * fr, fc, c[q].y));
  }
}

// Large updates, k = 128: one workgroup of 8 waves per CU (its registers keep a
// second one out) walks its share of the 128 x 128 tiles as one stream of k
// steps.  The fragments of a step are loaded into registers two steps ahead,
// across tile ends; a tile's entries of C are loaded during its first steps and
// its results stored while the next tile's products start.  Two limits that
// overlap badly: the traffic of C (16 bytes per entry at 128 k: 465 us alone at m =
// n = 11 872) and the LDS reads with the products (450 us alone); neither is
// reached.  m = n = 11 872: 723 us, 200 TFLOP/s by 8 m n k (one workgroup per tile 850 us; without the non-temporal
// accesses 750-780; the 3M form in FP32 instructions 1365); m = n = 6000: 172 us
// (64 x 64 tiles 200-250).
template <bool NT>
__global__ void __launch_bounds__(512)
update_split_stream_kernel(int64_t m, int64_t n, const u32x4* __restrict__ L, const u32x4* __restrict__ U,
                           const float* __restrict__ sl, const float* __restrict__ su, float2* __restrict__ C, int64_t ldc,
                           int tiles_m, int tiles, int64_t sL, int64_t sC) {
  constexpr int PD = 2;                    // steps that the fragments are loaded ahead
  constexpr int NKT = 8, NF = 32, FW = 4;  // k steps; fragments (16 of the rows, 16 of the columns); per wave
  static_assert(NKT % PD == 0, "the register ring wraps at tile ends");
  L += (int64_t)blockIdx.y * (sL / 16);
  U += (int64_t)blockIdx.y * (sL / 16);
  sl += (int64_t)blockIdx.y * (sL / 4);
  su += (int64_t)blockIdx.y * (sL / 4);
  C += (int64_t)blockIdx.y * sC;
  __shared__ u32x4 lds[2][NF * 64];
  __shared__ float scl[2][256];
  // workgroup b of XCD b % 8 takes every (gridDim.x / 8)-th tile of that XCD's range
  const int xcd = blockIdx.x & 7, stride = gridDim.x >> 3;
  const int per = tiles >> 3, rem = tiles & 7;
  const int first = xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per;
  const int last = first + per + (xcd < rem ? 1 : 0);
  int t = first + (int)(blockIdx.x >> 3);
  if (t >= last) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave & 1, wc = wave >> 1;
  // fragments of a step: f = wave + 8 i; i < 2 are of the rows
  const int ft = wave >> 2, fp = wave & 3;
  const u32x4 *lsrc, *usrc, *lnext, *unext;
  int tm, tn;
  auto locate = [&](int tile, const u32x4*& l, const u32x4*& u) {
    grouped_tile<8, 8>(tile, tiles_m, tiles, tm, tn);
    l = L + ((int64_t)(4 * tm + ft) * NKT * 4 + fp) * 64;
    u = U + ((int64_t)(4 * tn + ft) * NKT * 4 + fp) * 64;
  };
  u32x4 st[PD][FW];
  auto gload = [&](int slot, const u32x4* l, const u32x4* u, int kt) {
    st[slot][0] = l[kt * 256 + lane];
    st[slot][1] = l[kt * 256 + lane + 2 * NKT * 256];
    st[slot][2] = u[kt * 256 + lane];
    st[slot][3] = u[kt * 256 + lane + 2 * NKT * 256];
  };
  auto sstore = [&](int buf, int slot) {
#pragma unroll
    for (int i = 0; i < FW; ++i) lds[buf][(wave + 8 * i) * 64 + lane] = st[slot][i];
  };
  f32x16 re[2], im[2];
  float2 c[32];
  auto mma = [&](int buf) {
    u32x4 l[2][4], u[4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int p = 0; p < 4; ++p) l[i][p] = lds[buf][(4 * (2 * wr + i) + p) * 64 + lane];
#pragma unroll
    for (int p = 0; p < 4; ++p) u[p] = lds[buf][(16 + 4 * wc + p) * 64 + lane];
#pragma unroll
    for (int i = 0; i < 2; ++i) mac_complex(re[i], im[i], l[i], u);
  };
  locate(t, lsrc, usrc);
#pragma unroll
  for (int k = 0; k < PD; ++k) gload(k, lsrc, usrc, k);
  sstore(0, 0);
  __syncthreads();
  for (int par = 0;; par ^= 1) {
    const int cm = tm, cn = tn;
    const int64_t row0 = (int64_t)(cm * 4 + wr * 2) * 32 + (lane & 31);
    const int64_t col0 = (int64_t)(cn * 4 + wc) * 32 + 4 * (lane >> 5);
    const bool full = (int64_t)(cm + 1) * 128 <= m && (int64_t)(cn + 1) * 128 <= n;
    float2* const cb = C + (int64_t)(cm * 4 + wr * 2) * 32 + (int64_t)(cn * 4 + wc) * 32 * ldc;  // uniform
    const uint32_t coff = (uint32_t)((lane & 31) * 8 + 4 * (lane >> 5) * (ldc * 8));
    auto entry = [&](int e) -> float2& {  // e: row tile e / 16, column (e % 4) + 8 (e / 4 % 4)
      return *reinterpret_cast<float2*>(reinterpret_cast<char*>(cb + 32 * (e >> 4) + ((e & 3) + 8 * ((e >> 2) & 3)) * ldc) +
                                        coff);
    };
    auto inside = [&](int e) { return full || (row0 + 32 * (e >> 4) < m && col0 + (e & 3) + 8 * ((e >> 2) & 3) < n); };
    const int tnext = t + stride < last ? t + stride : t;
    locate(tnext, lnext, unext);
    const float scale = threadIdx.x < 256
                            ? (threadIdx.x < 128 ? sl[(int64_t)cm * 128 + threadIdx.x] : su[(int64_t)cn * 128 + threadIdx.x - 128])
                            : 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        re[i][q] = 0;
        im[i][q] = 0;
      }
    static_for<NKT>([&](auto K) {
      constexpr int kt = decltype(K)::value;
      // slot of step kt + PD: the one whose fragments went to LDS a step ago
      if constexpr (kt + PD < NKT) gload((kt + PD) % PD, lsrc, usrc, kt + PD);
      else gload((kt + PD) % PD, lnext, unext, kt + PD - NKT);
      if constexpr (kt < 4) {
#pragma unroll
        for (int e = 8 * kt; e < 8 * kt + 8; ++e) {
          c[e] = make_float2(0.f, 0.f);
          if (inside(e)) c[e] = load_c<NT>(&entry(e));
        }
      }
      if constexpr (kt == 2)
        if (threadIdx.x < 256) scl[par][threadIdx.x] = scale;
      __builtin_amdgcn_sched_barrier(0);
      mma(kt & 1);
      sstore((kt + 1) & 1, (kt + 1) % PD);
      __syncthreads();
    });
    const float fr[2] = {scl[par][64 * wr + (lane & 31)], scl[par][64 * wr + 32 + (lane & 31)]};
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const float fc = scl[par][128 + 32 * wc + 4 * (lane >> 5) + (q & 3) + 8 * (q >> 2)];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int e = 16 * i + q;
        if (inside(e))
          store_c<NT>(&entry(e), make_float2(fmaf(-re[i][q] * fr[i], fc, c[e].x), fmaf(-im[i][q] * fr[i], fc, c[e].y)));
      }
    }
    if (t + stride >= last) break;
    t += stride;
    lsrc = lnext;
    usrc = unext;
  }
}

// planes of 32-row tiles, then one scale per row
int64_t split_bytes(int64_t rows, int k) { return split_planes_bytes(rows, k) + ((rows + 127) / 128) * 128 * 4; }
int64_t split_planes_bytes(int64_t rows, int k) { return ((rows + 127) / 128) * 4 * (int64_t)((k + 15) / 16) * 4096; }

// Error against 64 bits (of one update, relative to sum |l| |u| per entry; L and U
// Gaussian, the same with entries spread over e^(2 N), and with rows of L and columns
// of U, not k, spread over e^(3 N) on top): rms 1.3e-8, 6.0e-8, 6.1e-8, largest of 6000 7.1e-8,
// 3.2e-7, 3.7e-7; the 3M form in FP32 instructions 2.0e-8, 9.2e-8, 9.3e-8 and
// 1.1e-7, 7.2e-7, 6.0e-7.
//
// The stream of large tiles from 2e7 entries of C on (m = n = 3000: 52 us against
// 47 for the 64 x 64 tiles; 6000: 172 against 200), with non-temporal accesses to
// C once it exceeds the 256 MB of the last-level cache (6000: the same; 3000: 56
// against 52).  Its grid leaves 32 CUs (one per shader
// engine, which dispatch in order) to the panel kernels that run beside it.
hipError_t launch_update_split(int64_t m, int64_t n, int k, const void* L, const void* U, const float* sl, const float* su,
                               float2* C, int64_t ldc, hipStream_t st, int num_cu, int nbatch, int64_t sL, int64_t sC) {
  if (m <= 0 || n <= 0 || k <= 0 || nbatch <= 0) return hipSuccess;
  if (nbatch > 65535 || (k != 128 && k != 64) || sL % 16) return hipErrorInvalidValue;
  const auto* l = static_cast<const u32x4*>(L);
  const auto* u = static_cast<const u32x4*>(U);
  const int64_t entries = m * n;
  if (k == 128 && entries >= 20000000) {
    const int64_t tm = (m + 127) / 128, tn = (n + 127) / 128;
    if (tm * tn > INT32_MAX) return hipErrorInvalidValue;
    const int g = std::max(8, (num_cu - 32) / nbatch / 8 * 8);  // a multiple of the 8 XCDs
    const dim3 grid((unsigned)g, (unsigned)nbatch);
    if (entries * 8 * nbatch > ((int64_t)256 << 20))
      hipLaunchKernelGGL(update_split_stream_kernel<true>, grid, dim3(512), 0, st, m, n, l, u, sl, su, C, ldc, (int)tm,
                         (int)(tm * tn), sL, sC);
    else
      hipLaunchKernelGGL(update_split_stream_kernel<false>, grid, dim3(512), 0, st, m, n, l, u, sl, su, C, ldc, (int)tm,
                         (int)(tm * tn), sL, sC);
    return hipGetLastError();
  }
  const int64_t tm = (m + 63) / 64, tn = (n + 63) / 64;
  if (tm * tn > INT32_MAX) return hipErrorInvalidValue;
  const dim3 grid((unsigned)(tm * tn), (unsigned)nbatch);
#define GDM_SPLIT(NKT)                                                                                                 \
  hipLaunchKernelGGL(update_split_kernel<NKT>, grid, dim3(256), 0, st, m, n, l, u, sl, su, C, ldc, (int)tm,      \
                     (int)(tm * tn), sL, sC)
  if (k == 128) GDM_SPLIT(8);
  else GDM_SPLIT(4);
#undef GDM_SPLIT
  return hipGetLastError();
}

}  // namespace gdm
