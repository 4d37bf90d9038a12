// Block steps of the triangular solves for the factors of lu_factor when the
// right-hand sides are few, and for every transposed solve.
//
// The forward/backward steps update many rows from one 128-wide block (an
// m x k product with k <= 256); with 1-8 right-hand sides a 64 x 64 matrix-core
// tile would be almost empty, so a plain VALU kernel streams the block once:
// one row per lane, the k range split over the eight waves of a workgroup (at k =
// 128 every load of a wave is in flight at once, before the right-hand sides are
// staged in LDS), the waves' partial sums combined in LDS.  Bound by latency:
// k = 128, FP32, one column, m = 3000 on average 5.4 us (four waves, X first: 7.7); FP64,
// eight columns, m = 1500 9.9 us (14.6).
//
// A transposed solve subtracts a block's part from the later columns as soon as it
// is known (skinny_push_kernel).  For few blocks or many columns, and where
// interchanges come between the blocks (L^T of a pivoting panel's factors), a step
// instead gathers its 128-row block from a long product (k up to n): C[w x nr] -=
// op(A)^T B, and the transposed refinement residual is the same shape with w = n.  Each output is the dot product of a
// stored column of A with B: one wave per column, lanes along k (coalesced
// column reads), the k range split into chunks of KC rows, one partial sum per
// (chunk, column) reduced across the wave; the masked diagonal block is one
// more chunk.  A second kernel adds the partials to C in a fixed order
// (deterministic).  Right-hand sides are processed NR at a time (NR = 1, 2, 4
// or 8 picked from their count; blockIdx.y walks the groups).
#include "gdm_common.hpp"
#include "gdm_kernels.hpp"

namespace gdm {

constexpr int SK_KMAX = 256; // max k of the column-form kernel
constexpr int SK_KC = 256;   // k rows per chunk of the transposed form
constexpr int SK_TCOLS = 16; // output columns per workgroup of the transposed form (4 per wave)

__device__ inline bool sk_keep(int kind, int64_t r, int64_t c) {
  switch (kind) {
    case GEMM_MASK_STRICT_LOWER: return r > c;
    case GEMM_MASK_UPPER: return r <= c;
    case GEMM_MASK_LOWER: return r >= c;
    case GEMM_MASK_STRICT_UPPER: return r < c;
    default: return true;
  }
}

template <typename T>
__device__ inline void cfma_t(cplx<T>& acc, const cplx<T>& a, const cplx<T>& b) {
  acc.x += a.x * b.x - a.y * b.y;
  acc.y += a.x * b.y + a.y * b.x;
}

// C[m x nr] -= A[m x k] X[k x nr]; rows [ar0, ar0 + adw) of A are a square
// block of which only the `akind` triangle is read.  64 rows per workgroup, the
// k range split over its eight waves.
// With PART, blockIdx.z selects the k chunk [z SK_KMAX, (z + 1) SK_KMAX) of a
// longer product and the sums go to part[(z * nrhs + r) * m + row] instead.
// Batch: blockIdx.z = item (x nchunk + chunk with PART); item z reads A + z sA,
// X + z sX and writes C + z sC (PART: its own nchunk x nrhs x m partials).
template <typename T, int NR, bool PART>
__global__ void __launch_bounds__(512) skinny_n_kernel(int64_t m, int64_t k, const cplx<T>* __restrict__ A,
                                                        int64_t lda, const cplx<T>* __restrict__ X, int64_t ldx,
                                                        cplx<T>* __restrict__ C, int64_t ldc, int64_t nrhs,
                                                        GemmMask mk, int nchunk, int64_t sA, int64_t sX, int64_t sC) {
  using CT = cplx<T>;
  constexpr int NWV = 8;
  // X (SK_KMAX x NR), then the waves' sums
  constexpr int LE = SK_KMAX * NR > NWV * 64 * NR ? SK_KMAX * NR : NWV * 64 * NR;
  __shared__ CT lds[LE];
  const int64_t item = PART ? blockIdx.z / nchunk : blockIdx.z;
  const int64_t chunk = PART ? blockIdx.z - item * nchunk : 0;
  A += item * sA;
  X += item * sX;
  C += PART ? item * nchunk * nrhs * m : item * sC;
  if (PART) {
    const int64_t kc0 = chunk * SK_KMAX;
    A += kc0 * lda;
    X += kc0;
    k = k - kc0 < SK_KMAX ? k - kc0 : SK_KMAX;
  }
  const int64_t r0 = (int64_t)blockIdx.y * NR;
  const int nr = (int)(nrhs - r0 < NR ? nrhs - r0 : NR);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t row0 = (int64_t)blockIdx.x * 64;
  const int64_t row = row0 + lane < m ? row0 + lane : m - 1;  // (rows past the end: not stored)
  const int kn = (int)k, kq = (kn + NWV - 1) / NWV;
  const int ka = wave * kq, kb = ka + kq < kn ? ka + kq : kn;
  // the first KB (for k = 128 all) of the wave's columns are in flight before X is staged
  constexpr int KB = 16;
  CT a[KB];
  auto load = [&](int k0) {
#pragma unroll
    for (int u = 0; u < KB; ++u) a[u] = A[row + (int64_t)(k0 + u < kn ? k0 + u : kn - 1) * lda];
  };
  load(ka);
  for (int t = threadIdx.x; t < kn * NR; t += 512) {
    const int kk = t / NR, r = t % NR;
    CT v;
    v.x = 0;
    v.y = 0;
    if (r < nr) v = X[kk + (r0 + r) * ldx];
    lds[kk * NR + r] = v;
  }
  __syncthreads();
  CT acc[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) acc[r].x = acc[r].y = 0;
  // the masked triangle is stored, so it is read and replaced by zero
  const bool masked = mk.akind && row >= mk.ar0 && row < mk.ar0 + mk.adw;
  for (int k0 = ka; k0 < kb; k0 += KB) {
    if (k0 != ka) load(k0);
#pragma unroll
    for (int u = 0; u < KB; ++u) {
      const int kk = k0 + u;
      if (kk < kb) {
        CT v = a[u];
        if (masked && !sk_keep(mk.akind, row - mk.ar0, kk)) v.x = v.y = 0;
#pragma unroll
        for (int r = 0; r < NR; ++r) cfma_t<T>(acc[r], v, lds[kk * NR + r]);
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < NR; ++r) lds[(r * NWV + wave) * 64 + lane] = acc[r];
  __syncthreads();
  // wave r of the workgroup finishes right-hand side r
  const int r = wave;
  if (r >= nr || row0 + lane >= m) return;
  CT s = lds[r * NWV * 64 + lane];
#pragma unroll
  for (int w = 1; w < NWV; ++w) {
    s.x += lds[(r * NWV + w) * 64 + lane].x;
    s.y += lds[(r * NWV + w) * 64 + lane].y;
  }
  if (PART) {
    C[(chunk * nrhs + r0 + r) * m + row] = s;
  } else {
    // rows [ar0, ar0 + adw) optionally to the second destination mk.c2
    CT c = C[row + (r0 + r) * ldc];
    c.x -= s.x;
    c.y -= s.y;
    if (mk.c2 && row >= mk.ar0 && row < mk.ar0 + mk.adw)
      static_cast<CT*>(mk.c2)[item * mk.sc2 + (row - mk.ar0) + (r0 + r) * mk.ldc2] = c;
    else
      C[row + (r0 + r) * ldc] = c;
  }
}

struct SkSeg {
  const void* A;  // stored k x mo block (column-major, lda): op(A)[i][kk] = A[kk + i lda]
  int64_t lda;
  const void* B;  // k x nrhs (column-major, ldb)
  int64_t ldb;
  int64_t k;
  int kind;       // triangle kept of the square block (row i, column kk), 0 = all
  int nchunk;
};

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// part[(chunk * nrhs + r) * mo + i] = sum_{kk in chunk} op(A)[i][kk] B[kk][r];
// blockIdx.x = chunk * ngroups + column group (16 columns, 4 per wave).
template <typename T, int NR>
__global__ void __launch_bounds__(256) skinny_t_kernel(SkSeg s0, SkSeg s1, int64_t mo, int64_t nrhs, int ngroups,
                                                        cplx<T>* __restrict__ part, int64_t sA, int64_t sB) {
  using CT = cplx<T>;
  __shared__ CT bs[SK_KC][NR];
  const int64_t item = blockIdx.z;  // batch item: A + item sA, B + item sB, own partials
  part += item * (int64_t)(s0.nchunk + s1.nchunk) * nrhs * mo;
  const int chunk = blockIdx.x / ngroups, grp = blockIdx.x - chunk * ngroups;
  const bool second = chunk >= s0.nchunk;
  const SkSeg& s = second ? s1 : s0;
  const int64_t kc0 = (int64_t)(second ? chunk - s0.nchunk : chunk) * SK_KC;
  const int64_t kc1 = kc0 + SK_KC < s.k ? kc0 + SK_KC : s.k;
  const int64_t r0 = (int64_t)blockIdx.y * NR;
  const int nr = (int)(nrhs - r0 < NR ? nrhs - r0 : NR);
  const CT* A = static_cast<const CT*>(s.A) + item * sA;
  const CT* B = static_cast<const CT*>(s.B) + item * sB;
  for (int t = threadIdx.x; t < (kc1 - kc0) * NR; t += 256) {
    const int kk = t % (int)(kc1 - kc0), r = t / (int)(kc1 - kc0);
    CT v;
    v.x = 0;
    v.y = 0;
    if (r < nr) v = B[kc0 + kk + (r0 + r) * s.ldb];
    bs[kk][r] = v;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // all of this wave's loads (CPW columns x KS steps of 64 rows) in flight at
  // once, then the products column by column; masked entries are stored, so
  // they are read and replaced by zero
  constexpr int CPW = SK_TCOLS / 4, KS = SK_KC / 64;
  const int64_t i0 = (int64_t)grp * SK_TCOLS + wave * CPW;
  CT a[CPW][KS];
#pragma unroll
  for (int c = 0; c < CPW; ++c)
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      const int64_t kk = kc0 + lane + 64 * q;
      a[c][q].x = 0;
      a[c][q].y = 0;
      if (i0 + c < mo && kk < kc1) a[c][q] = A[kk + (i0 + c) * s.lda];
    }
#pragma unroll
  for (int c = 0; c < CPW; ++c) {
    const int64_t i = i0 + c;
    if (i >= mo) break;
    CT acc[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) acc[r].x = acc[r].y = 0;
#pragma unroll
    for (int q = 0; q < KS; ++q) {
      const int64_t kk = kc0 + lane + 64 * q;
      if (kk < kc1) {
        CT v = a[c][q];
        if (s.kind && !sk_keep(s.kind, i, kk)) v.x = v.y = 0;
#pragma unroll
        for (int r = 0; r < NR; ++r) cfma_t<T>(acc[r], v, bs[kk - kc0][r]);
      }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const T re = wave_sum(acc[r].x), im = wave_sum(acc[r].y);
      if (lane == 0 && r < nr) {
        CT v;
        v.x = re;
        v.y = im;
        part[((int64_t)chunk * nrhs + r0 + r) * mo + i] = v;
      }
    }
  }
}

// C[i + r ldc] -= sum_chunk part[(chunk * nrhs + r) * mo + i], chunks in order
template <typename T>
__global__ void skinny_reduce_kernel(const cplx<T>* __restrict__ part, int nchunk, int64_t mo, int64_t nrhs,
                                     cplx<T>* __restrict__ C, int64_t ldc, int64_t sC) {
  using CT = cplx<T>;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= mo * nrhs) return;
  // batch item blockIdx.y: its partials follow those of the previous items
  part += (int64_t)blockIdx.y * nchunk * nrhs * mo;
  C += (int64_t)blockIdx.y * sC;
  const int64_t r = t / mo, i = t - r * mo;
  CT s;
  s.x = 0;
  s.y = 0;
  for (int c = 0; c < nchunk; ++c) {
    const CT v = part[((int64_t)c * nrhs + r) * mo + i];
    s.x += v.x;
    s.y += v.y;
  }
  CT* p = C + i + r * ldc;
  CT c = *p;
  c.x -= s.x;
  c.y -= s.y;
  *p = c;
}

// Transposed solves, block by block downwards (upwards): once a block's unknowns
// z are known their part of every later column is subtracted,
//   y[c] -= sum_k A[k + c lda] z[k], k < w <= 128,
// one launch per block and no partial sums (gathering a block's own sum from all
// known unknowns took a product and a reduction: 11.5 us and two launches per
// block at n = 6000, this 4.2).  A wave takes four columns, lanes along k.
// Bound by latency: the block row is 3 MB on average.
template <typename T, int NR>
__global__ void __launch_bounds__(256) skinny_push_kernel(int w, int64_t ncols, const cplx<T>* __restrict__ A, int64_t lda,
                                                           const cplx<T>* __restrict__ z, cplx<T>* __restrict__ y,
                                                           int64_t ldb, int64_t nrhs, int64_t sA, int64_t sB) {
  using CT = cplx<T>;
  constexpr int CPW = 4;
  A += blockIdx.z * sA;
  z += blockIdx.z * sB;
  y += blockIdx.z * sB;
  const int64_t r0 = (int64_t)blockIdx.y * NR;
  const int nr = (int)(nrhs - r0 < NR ? nrhs - r0 : NR);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t c0 = ((int64_t)blockIdx.x * 4 + wave) * CPW;
  if (c0 >= ncols) return;
  CT a[CPW][2], b[2][NR], zero;
  zero.x = zero.y = 0;
#pragma unroll
  for (int c = 0; c < CPW; ++c)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int k = lane + 64 * h;
      a[c][h] = A[(k < w ? k : w - 1) + (c0 + c < ncols ? c0 + c : ncols - 1) * lda];
    }
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      b[h][r] = zero;
      if (lane + 64 * h < w && r < nr) b[h][r] = z[lane + 64 * h + (r0 + r) * ldb];
    }
#pragma unroll
  for (int h = 0; h < 2; ++h)
    if (lane + 64 * h >= w)
#pragma unroll
      for (int c = 0; c < CPW; ++c) a[c][h] = zero;
  // lane c + CPW r keeps column c of right-hand side r
  static_assert(CPW * NR <= 64, "one lane per result");
  CT sum = zero;
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int c = 0; c < CPW; ++c) {
      CT s = zero;
      cfma_t<T>(s, a[c][0], b[0][r]);
      cfma_t<T>(s, a[c][1], b[1][r]);
      s.x = wave_sum(s.x);
      s.y = wave_sum(s.y);
      if (lane == c + CPW * r) sum = s;
    }
  const int c = lane % CPW, r = lane / CPW;
  if (r < nr && c0 + c < ncols) {
    CT* p = y + c0 + c + (r0 + r) * ldb;
    CT v = *p;
    v.x -= sum.x;
    v.y -= sum.y;
    *p = v;
  }
}

// x_b = x_b - tri(D_b)^T x_b for every diagonal block b (LOWER false: its upper
// triangle with the diagonal, I - U11^-1; true: its strict lower one, I - L11^-1):
// one workgroup of 16 waves per block, in place.
template <typename T, int NR, bool LOWER>
__global__ void __launch_bounds__(1024) skinny_diag_t_kernel(int64_t n, int nb, const cplx<T>* __restrict__ A, int64_t lda,
                                                              cplx<T>* __restrict__ x, int64_t ldb, int64_t nrhs,
                                                              int64_t sA, int64_t sB) {
  using CT = cplx<T>;
  const int64_t k0 = (int64_t)blockIdx.x * nb;
  const int w = (int)(n - k0 < nb ? n - k0 : nb);
  A += blockIdx.z * sA + k0 + k0 * lda;
  x += blockIdx.z * sB + k0;
  const int64_t r0 = (int64_t)blockIdx.y * NR;
  const int nr = (int)(nrhs - r0 < NR ? nrhs - r0 : NR);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  CT b[2][NR], zero;
  zero.x = zero.y = 0;
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      b[h][r] = zero;
      if (lane + 64 * h < w && r < nr) b[h][r] = x[lane + 64 * h + (r0 + r) * ldb];
    }
  CT a[8][2];
#pragma unroll
  for (int u = 0; u < 8; ++u)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int c = 8 * wave + u, k = lane + 64 * h;
      a[u][h] = A[(k < w ? k : w - 1) + (int64_t)(c < w ? c : w - 1) * lda];
      if (k >= w || (LOWER ? k <= c : k > c)) a[u][h] = zero;
    }
  __syncthreads();  // every wave has read x
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int c = 8 * wave + u;
      CT s = zero;
      cfma_t<T>(s, a[u][0], b[0][r]);
      cfma_t<T>(s, a[u][1], b[1][r]);
      s.x = wave_sum(s.x);
      s.y = wave_sum(s.y);
      // (column c is a row of x that lane c % 64 holds)
      if (lane == c % 64 && c < w && r < nr) {
        CT v = c < 64 ? b[0][r] : b[1][r];
        v.x -= s.x;
        v.y -= s.y;
        x[c + (r0 + r) * ldb] = v;
      }
    }
}

static int pick_nr(int64_t nrhs) { return nrhs <= 1 ? 1 : nrhs <= 2 ? 2 : nrhs <= 4 ? 4 : 8; }

template <typename T>
hipError_t launch_skinny_n(int64_t m, int64_t k, const void* A, int64_t lda, const void* X, int64_t ldx, void* C,
                           int64_t ldc, int64_t nrhs, hipStream_t st, GemmMask mk, int nbatch, int64_t sA, int64_t sX,
                           int64_t sC) {
  if (m <= 0 || nrhs <= 0 || k <= 0 || nbatch <= 0) return hipSuccess;
  if (k > SK_KMAX || nbatch > 65535) return hipErrorInvalidValue;
  const int NRp = pick_nr(nrhs);
  const dim3 grid((unsigned)((m + 63) / 64), (unsigned)((nrhs + NRp - 1) / NRp), (unsigned)nbatch);
  const auto* a = static_cast<const cplx<T>*>(A);
  const auto* x = static_cast<const cplx<T>*>(X);
  auto* c = static_cast<cplx<T>*>(C);
  switch (NRp) {
    case 1: hipLaunchKernelGGL((skinny_n_kernel<T, 1, false>), grid, dim3(512), 0, st, m, k, a, lda, x, ldx, c, ldc, nrhs, mk, 1, sA, sX, sC); break;
    case 2: hipLaunchKernelGGL((skinny_n_kernel<T, 2, false>), grid, dim3(512), 0, st, m, k, a, lda, x, ldx, c, ldc, nrhs, mk, 1, sA, sX, sC); break;
    case 4: hipLaunchKernelGGL((skinny_n_kernel<T, 4, false>), grid, dim3(512), 0, st, m, k, a, lda, x, ldx, c, ldc, nrhs, mk, 1, sA, sX, sC); break;
    default: hipLaunchKernelGGL((skinny_n_kernel<T, 8, false>), grid, dim3(512), 0, st, m, k, a, lda, x, ldx, c, ldc, nrhs, mk, 1, sA, sX, sC); break;
  }
  return hipGetLastError();
}

int64_t skinny_n_long_parts(int64_t m, int64_t k, int64_t nrhs) {
  return (k + SK_KMAX - 1) / SK_KMAX * nrhs * m;
}

template <typename T>
hipError_t launch_skinny_n_long(int64_t m, int64_t k, const void* A, int64_t lda, const void* X, int64_t ldx, void* C,
                                int64_t ldc, int64_t nrhs, void* part, int64_t part_elems, hipStream_t st, int nbatch,
                                int64_t sA, int64_t sX, int64_t sC) {
  if (m <= 0 || nrhs <= 0 || k <= 0 || nbatch <= 0) return hipSuccess;
  const int64_t nchunk = (k + SK_KMAX - 1) / SK_KMAX;
  if (nbatch * skinny_n_long_parts(m, k, nrhs) > part_elems || nchunk * nbatch > 65535 || nbatch > 65535)
    return hipErrorInvalidValue;
  const int NRp = pick_nr(nrhs);
  const dim3 grid((unsigned)((m + 63) / 64), (unsigned)((nrhs + NRp - 1) / NRp), (unsigned)(nchunk * nbatch));
  const auto* a = static_cast<const cplx<T>*>(A);
  const auto* x = static_cast<const cplx<T>*>(X);
  auto* p = static_cast<cplx<T>*>(part);
  const GemmMask mk{};
  const int nc = (int)nchunk;
  switch (NRp) {
    case 1: hipLaunchKernelGGL((skinny_n_kernel<T, 1, true>), grid, dim3(512), 0, st, m, k, a, lda, x, ldx, p, m, nrhs, mk, nc, sA, sX, (int64_t)0); break;
    case 2: hipLaunchKernelGGL((skinny_n_kernel<T, 2, true>), grid, dim3(512), 0, st, m, k, a, lda, x, ldx, p, m, nrhs, mk, nc, sA, sX, (int64_t)0); break;
    case 4: hipLaunchKernelGGL((skinny_n_kernel<T, 4, true>), grid, dim3(512), 0, st, m, k, a, lda, x, ldx, p, m, nrhs, mk, nc, sA, sX, (int64_t)0); break;
    default: hipLaunchKernelGGL((skinny_n_kernel<T, 8, true>), grid, dim3(512), 0, st, m, k, a, lda, x, ldx, p, m, nrhs, mk, nc, sA, sX, (int64_t)0); break;
  }
  const int64_t tot = m * nrhs;
  hipLaunchKernelGGL(skinny_reduce_kernel<T>, dim3((unsigned)((tot + 255) / 256), (unsigned)nbatch), dim3(256), 0, st, p,
                     nc, m, nrhs, static_cast<cplx<T>*>(C), ldc, sC);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_partial_reduce(const void* part, int nchunk, int64_t mo, int64_t nrhs, void* C, int64_t ldc,
                                 hipStream_t st) {
  if (mo <= 0 || nrhs <= 0 || nchunk <= 0) return hipSuccess;
  const int64_t tot = mo * nrhs;
  hipLaunchKernelGGL(skinny_reduce_kernel<T>, dim3((unsigned)((tot + 255) / 256), 1), dim3(256), 0, st,
                     static_cast<const cplx<T>*>(part), nchunk, mo, nrhs, static_cast<cplx<T>*>(C), ldc, (int64_t)0);
  return hipGetLastError();
}
template hipError_t launch_partial_reduce<double>(const void*, int, int64_t, int64_t, void*, int64_t, hipStream_t);
template hipError_t launch_partial_reduce<float>(const void*, int, int64_t, int64_t, void*, int64_t, hipStream_t);

template <typename T>
hipError_t launch_skinny_push(int w, int64_t ncols, const void* A, int64_t lda, const void* z, void* y, int64_t ldb,
                              int64_t nrhs, hipStream_t st, int nbatch, int64_t sA, int64_t sB) {
  if (w <= 0 || ncols <= 0 || nrhs <= 0 || nbatch <= 0) return hipSuccess;
  if (w > 128 || nbatch > 65535) return hipErrorInvalidValue;
  const int NRp = pick_nr(nrhs);
  if ((nrhs + NRp - 1) / NRp > 65535) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((ncols + 15) / 16), (unsigned)((nrhs + NRp - 1) / NRp), (unsigned)nbatch);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, w, ncols, static_cast<const cplx<T>*>(A), lda,
                       static_cast<const cplx<T>*>(z), static_cast<cplx<T>*>(y), ldb, nrhs, sA, sB);
  };
  switch (NRp) {
    case 1: go(skinny_push_kernel<T, 1>); break;
    case 2: go(skinny_push_kernel<T, 2>); break;
    case 4: go(skinny_push_kernel<T, 4>); break;
    default: go(skinny_push_kernel<T, 8>); break;
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_skinny_diag_t(bool lower, int64_t n, int nb, const void* A, int64_t lda, void* x, int64_t ldb,
                                int64_t nrhs, hipStream_t st, int nbatch, int64_t sA, int64_t sB) {
  if (n <= 0 || nrhs <= 0 || nbatch <= 0) return hipSuccess;
  if (nb <= 0 || nb > 128 || nbatch > 65535) return hipErrorInvalidValue;
  const int NRp = nrhs <= 1 ? 1 : nrhs <= 2 ? 2 : 4;  // (8 right-hand sides would spill in FP64)
  if ((nrhs + NRp - 1) / NRp > 65535) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((n + nb - 1) / nb), (unsigned)((nrhs + NRp - 1) / NRp), (unsigned)nbatch);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(1024), 0, st, n, nb, static_cast<const cplx<T>*>(A), lda,
                       static_cast<cplx<T>*>(x), ldb, nrhs, sA, sB);
  };
  if (lower) {
    if (NRp == 1) go(skinny_diag_t_kernel<T, 1, true>);
    else if (NRp == 2) go(skinny_diag_t_kernel<T, 2, true>);
    else go(skinny_diag_t_kernel<T, 4, true>);
  } else {
    if (NRp == 1) go(skinny_diag_t_kernel<T, 1, false>);
    else if (NRp == 2) go(skinny_diag_t_kernel<T, 2, false>);
    else go(skinny_diag_t_kernel<T, 4, false>);
  }
  return hipGetLastError();
}
#define GDM_INST(T)                                                                                                       \
  template hipError_t launch_skinny_push<T>(int, int64_t, const void*, int64_t, const void*, void*, int64_t, int64_t,    \
                                            hipStream_t, int, int64_t, int64_t);                                          \
  template hipError_t launch_skinny_diag_t<T>(bool, int64_t, int, const void*, int64_t, void*, int64_t, int64_t,         \
                                              hipStream_t, int, int64_t, int64_t);
GDM_INST(double)
GDM_INST(float)
#undef GDM_INST

int64_t skinny_t_chunks(int64_t k0, int64_t k1) {
  return (k0 + SK_KC - 1) / SK_KC + (k1 + SK_KC - 1) / SK_KC;
}

template <typename T>
hipError_t launch_skinny_t(int64_t mo, int64_t nrhs, const void* A0, int64_t lda0, const void* B0, int64_t ldb0,
                           int64_t k0, const void* A1, int64_t lda1, const void* B1, int64_t ldb1, int64_t k1,
                           int kind1, void* part, int64_t part_elems, void* C, int64_t ldc, hipStream_t st, int nbatch,
                           int64_t sA, int64_t sB, int64_t sC) {
  if (mo <= 0 || nrhs <= 0 || nbatch <= 0) return hipSuccess;
  SkSeg s0{A0, lda0, B0, ldb0, k0, 0, (int)((k0 + SK_KC - 1) / SK_KC)};
  SkSeg s1{A1, lda1, B1, ldb1, k1, kind1, (int)((k1 + SK_KC - 1) / SK_KC)};
  const int nchunk = s0.nchunk + s1.nchunk;
  if (nchunk == 0) return hipSuccess;
  if ((int64_t)nbatch * nchunk * nrhs * mo > part_elems || nbatch > 65535) return hipErrorInvalidValue;
  const int64_t ngroups = (mo + SK_TCOLS - 1) / SK_TCOLS;
  if ((int64_t)nchunk * ngroups > INT32_MAX) return hipErrorInvalidValue;
  const int NRp = pick_nr(nrhs);
  const dim3 grid((unsigned)(nchunk * ngroups), (unsigned)((nrhs + NRp - 1) / NRp), (unsigned)nbatch);
  auto* p = static_cast<cplx<T>*>(part);
  const int ng = (int)ngroups;
  switch (NRp) {
    case 1: hipLaunchKernelGGL((skinny_t_kernel<T, 1>), grid, dim3(256), 0, st, s0, s1, mo, nrhs, ng, p, sA, sB); break;
    case 2: hipLaunchKernelGGL((skinny_t_kernel<T, 2>), grid, dim3(256), 0, st, s0, s1, mo, nrhs, ng, p, sA, sB); break;
    case 4: hipLaunchKernelGGL((skinny_t_kernel<T, 4>), grid, dim3(256), 0, st, s0, s1, mo, nrhs, ng, p, sA, sB); break;
    default: hipLaunchKernelGGL((skinny_t_kernel<T, 8>), grid, dim3(256), 0, st, s0, s1, mo, nrhs, ng, p, sA, sB); break;
  }
  const int64_t tot = mo * nrhs;
  hipLaunchKernelGGL(skinny_reduce_kernel<T>, dim3((unsigned)((tot + 255) / 256), (unsigned)nbatch), dim3(256), 0, st, p,
                     nchunk, mo, nrhs, static_cast<cplx<T>*>(C), ldc, sC);
  return hipGetLastError();
}

template hipError_t launch_skinny_n<double>(int64_t, int64_t, const void*, int64_t, const void*, int64_t, void*,
                                            int64_t, int64_t, hipStream_t, GemmMask, int, int64_t, int64_t, int64_t);
template hipError_t launch_skinny_n<float>(int64_t, int64_t, const void*, int64_t, const void*, int64_t, void*,
                                           int64_t, int64_t, hipStream_t, GemmMask, int, int64_t, int64_t, int64_t);
template hipError_t launch_skinny_n_long<double>(int64_t, int64_t, const void*, int64_t, const void*, int64_t, void*,
                                                 int64_t, int64_t, void*, int64_t, hipStream_t, int, int64_t, int64_t,
                                                 int64_t);
template hipError_t launch_skinny_n_long<float>(int64_t, int64_t, const void*, int64_t, const void*, int64_t, void*,
                                                int64_t, int64_t, void*, int64_t, hipStream_t, int, int64_t, int64_t,
                                                int64_t);
template hipError_t launch_skinny_t<double>(int64_t, int64_t, const void*, int64_t, const void*, int64_t, int64_t,
                                            const void*, int64_t, const void*, int64_t, int64_t, int, void*, int64_t,
                                            void*, int64_t, hipStream_t, int, int64_t, int64_t, int64_t);
template hipError_t launch_skinny_t<float>(int64_t, int64_t, const void*, int64_t, const void*, int64_t, int64_t,
                                           const void*, int64_t, const void*, int64_t, int64_t, int, void*, int64_t,
                                           void*, int64_t, hipStream_t, int, int64_t, int64_t, int64_t);

}  // namespace gdm
