// Block steps of the triangular solves with more than a few right-hand sides
// (and the small trailing updates of FP64 and caller's FP32 factorisations): C[m x nr] -= A[m x k]
// X[k x nr] with k <= 128, rows [ar0, ar0 + adw) of A a triangle.  A solve is a
// chain of these products, each a few microseconds of matrix-core work, so what
// bounds it is the latency inside a launch: loads, products, one reduction,
// stores.  A workgroup takes 16 rows and 16 NCT columns; its four waves
// split k, each with all of its operands loaded at once straight into the
// matrix-core layout (A is used once, so there is nothing to share in LDS; k
// is numbered so that a lane's entries of X are 8 (4) consecutive ones), and add
// their sums through LDS, one barrier in all.  16 rows per workgroup keep the
// chip filled down to m = 4096, and 16-wide column tiles pad 66 columns to 80.
// Solve of 66 columns at n = 12 000 in FP32 (188 steps): 2.26 ms, 32 x 32 tiles
// staged through LDS 3.41; n = 2000: 0.26 and 0.44; n = 6000 with 128 columns in
// FP64: 1.94 and 2.34.
#include <type_traits>

#include "gdm_common.hpp"
#include "gdm_kernels.hpp"
#include "lu_common.hpp"

namespace gdm {

// KS: k per lane and wave (8: k <= 128, 4: k <= 64)
template <typename T, int NCT, int KS>
__global__ void __launch_bounds__(256) solve_step_kernel(int64_t m, int nr, int k, const cplx<T>* __restrict__ A,
                                                          int64_t lda, const cplx<T>* __restrict__ X, int64_t ldx,
                                                          cplx<T>* C, int64_t ldc, GemmMask mk, int64_t sA, int64_t sX,
                                                          int64_t sC) {
  using CT = cplx<T>;
  using ACC = typename acc_of<T>::type;
  __shared__ CT red[4][NCT][4][64];  // [wave][column tile][register][lane]
  A += (int64_t)blockIdx.z * sA;
  X += (int64_t)blockIdx.z * sX;
  C += (int64_t)blockIdx.z * sC;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lr = lane & 15, lk = lane >> 4;
  const int64_t row = (int64_t)blockIdx.x * 16 + lr;
  const int64_t lrow = row < m ? row : m - 1;  // rows and columns past the end: loads repeat the last one
  const int c0 = blockIdx.y * 16 * NCT;
  // this wave's results after the reduction: register `wave` of every tile, row lane % 16
  const int oc = sizeof(T) == 8 ? lk + 4 * wave : 4 * lk + wave;
  CT cold[NCT];
#pragma unroll
  for (int t = 0; t < NCT; ++t) {
    const int col = c0 + 16 * t + oc;
    cold[t] = C[lrow + (int64_t)(col < nr ? col : nr - 1) * ldc];
  }
  ACC re[NCT], im[NCT];
#pragma unroll
  for (int t = 0; t < NCT; ++t) re[t] = im[t] = ACC{0, 0, 0, 0};
  const int kw = wave * 4 * KS;     // the wave's k range, a lane's first k
  const int kl = kw + KS * lk;
  // the lane's row of A keeps k in [kmin, kmax)
  int kmin = 0, kmax = k;
  if (mk.akind && lrow >= mk.ar0 && lrow < mk.ar0 + mk.adw) {
    const int r = (int)(lrow - mk.ar0);
    if (mk.akind == GEMM_MASK_STRICT_LOWER) kmax = r < k ? r : k;
    else kmin = r;  // GEMM_MASK_UPPER
  }
  auto product = [&](auto whole) __attribute__((always_inline)) {
    constexpr bool WHOLE = decltype(whole)::value;  // the wave's range lies below k
    auto at = [&](int s) { return WHOLE || kl + s < k ? kl + s : k - 1; };
    CT a[KS], x[NCT][KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) a[s] = A[lrow + (int64_t)at(s) * lda];
#pragma unroll
    for (int t = 0; t < NCT; ++t) {
      const int col = c0 + 16 * t + lr;
      const CT* xp = X + (int64_t)(col < nr ? col : nr - 1) * ldx;
#pragma unroll
      for (int s = 0; s < KS; ++s) x[t][s] = xp[at(s)];
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const bool keep = kl + s >= kmin && kl + s < kmax;
      a[s].x = keep ? a[s].x : 0;
      a[s].y = keep ? a[s].y : 0;
      if constexpr (!WHOLE) {
#pragma unroll
        for (int t = 0; t < NCT; ++t) {
          x[t][s].x = kl + s < k ? x[t][s].x : 0;
          x[t][s].y = kl + s < k ? x[t][s].y : 0;
        }
      }
    }
#pragma unroll
    for (int t = 0; t < NCT; ++t)
#pragma unroll
      for (int s = 0; s < KS; ++s) {
        re[t] = mfma16(x[t][s].x, a[s].x, re[t]);
        im[t] = mfma16(x[t][s].x, a[s].y, im[t]);
        re[t] = mfma16(-x[t][s].y, a[s].y, re[t]);
        im[t] = mfma16(x[t][s].y, a[s].x, im[t]);
      }
  };
  if (kw + 4 * KS <= k) product(std::true_type{});
  else if (kw < k) product(std::false_type{});
#pragma unroll
  for (int t = 0; t < NCT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      CT v;
      v.x = re[t][q];
      v.y = im[t][q];
      red[wave][t][q][lane] = v;
    }
  __syncthreads();
  if (row >= m) return;
  const bool second = mk.c2 && row >= mk.ar0 && row < mk.ar0 + mk.adw;
  CT* const out = second ? static_cast<CT*>(mk.c2) + (int64_t)blockIdx.z * mk.sc2 + (row - mk.ar0) : C + row;
  const int64_t ldo = second ? mk.ldc2 : ldc;
#pragma unroll
  for (int t = 0; t < NCT; ++t) {
    const int col = c0 + 16 * t + oc;
    if (col >= nr) break;
    CT s = red[0][t][wave][lane];
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      s.x += red[w][t][wave][lane].x;
      s.y += red[w][t][wave][lane].y;
    }
    CT v = cold[t];
    v.x -= s.x;
    v.y -= s.y;
    out[(int64_t)col * ldo] = v;
  }
}

template <typename T>
hipError_t launch_solve_step(int64_t m, int64_t k, const void* A, int64_t lda, const void* X, int64_t ldx, void* C,
                             int64_t ldc, int64_t nrhs, hipStream_t st, GemmMask mk, int nbatch, int64_t sA, int64_t sX,
                             int64_t sC) {
  if (m <= 0 || nrhs <= 0 || k <= 0 || nbatch <= 0) return hipSuccess;
  // Two column tiles per workgroup (66 columns, n = 12 000, FP32: 2.26 ms per solve; three 2.44,
  // five 2.53): twice the rows of A are read from L2, but a wave needs fewer registers.
  constexpr int MAXT = 2;
  const int64_t tiles = (nrhs + 15) / 16, chunks = (tiles + MAXT - 1) / MAXT;
  if (k > 128 || nbatch > 65535 || chunks > 65535 || nrhs > INT32_MAX - 256) return hipErrorInvalidValue;
  const int nct = (int)((tiles + chunks - 1) / chunks);
  const dim3 grid((unsigned)((m + 15) / 16), (unsigned)chunks, (unsigned)nbatch);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, m, (int)nrhs, (int)k, static_cast<const cplx<T>*>(A), lda,
                       static_cast<const cplx<T>*>(X), ldx, static_cast<cplx<T>*>(C), ldc, mk, sA, sX, sC);
  };
  auto pick = [&](auto ks) {
    constexpr int KS = decltype(ks)::value;
    if (nct == 1) go(solve_step_kernel<T, 1, KS>);
    else go(solve_step_kernel<T, MAXT, KS>);
  };
  if (k > 64) pick(std::integral_constant<int, 8>{});
  else pick(std::integral_constant<int, 4>{});
  return hipGetLastError();
}
template hipError_t launch_solve_step<double>(int64_t, int64_t, const void*, int64_t, const void*, int64_t, void*,
                                              int64_t, int64_t, hipStream_t, GemmMask, int, int64_t, int64_t, int64_t);
template hipError_t launch_solve_step<float>(int64_t, int64_t, const void*, int64_t, const void*, int64_t, void*,
                                             int64_t, int64_t, hipStream_t, GemmMask, int, int64_t, int64_t, int64_t);

}  // namespace gdm
