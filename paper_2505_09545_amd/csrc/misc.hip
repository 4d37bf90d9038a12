// Small kernels around the hot path: cubic-cell polarisability, incident plane
// wave, q = A F, the FP64 cross-section reductions, the exact far-field
// scattering double sum, and the helpers of FP64 iterative refinement.
//
// Physics (arXiv:2505.09545):
//  * alpha_pE = chi_ee d^3 / (4 pi), chi_ee = eps - eps_env (Sec. "Volume
//    discretization polarizabilities");
//  * plane-wave illumination (Appendix, 3D illuminations): E0 = e0 exp(i k
//    khat.r), H0 = n_env khat x E0 (Gaussian units, mu = 1);
//  * dipole moments (p, m) = alpha (E, H) (Eq. after LPS_6by6_discrete);
//  * extinction / absorption / scattering cross sections (Sec. "Observables"):
//    the kernels return the raw FP64 sums, the prefactor C = 4 pi k0 /
//    (n_env |E0|^2) is applied on the host.
#include <algorithm>
#include <type_traits>

#include "gdm_common.hpp"
#include "gdm_dyad.hpp"
#include "gdm_kernels.hpp"
#include "gdm_misc.hpp"

namespace gdm {

__global__ void cell_alpha_kernel(const double2* eps, int64_t nc, double eps_env, double f, double2* alpha) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nc) alpha[i] = make_double2((eps[i].x - eps_env) * f, eps[i].y * f);
}

hipError_t launch_cell_alpha(const double2* eps, int64_t nc, double eps_env, double step, double2* alpha,
                             hipStream_t st) {
  if (nc <= 0) return hipSuccess;
  const double f = step * step * step / (4.0 * 3.14159265358979323846);
  hipLaunchKernelGGL(cell_alpha_kernel, dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, st, eps, nc, eps_env, f,
                     alpha);
  return hipGetLastError();
}

__device__ inline double2 expi(double ph) {
  double s, c;
  sincos(ph, &s, &c);
  return make_double2(c, s);
}

__global__ void incident_kernel(DipoleView d, Wave w, double n_env, int64_t n_pw, const double* khat,
                                const double2* e0, double2* f0, int64_t n) {
  const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t r = blockIdx.y;
  if (u >= n || r >= n_pw) return;
  const int64_t N = d.N;
  const bool magnetic = u >= 3 * N;
  const int64_t dip = magnetic ? d.nc + (u - 3 * N) / 3 : u / 3;
  const int a = (int)(magnetic ? (u - 3 * N) % 3 : u % 3);
  const double kx = khat[3 * r], ky = khat[3 * r + 1], kz = khat[3 * r + 2];
  const double2 ph = expi(w.k * (kx * d.pos[3 * dip] + ky * d.pos[3 * dip + 1] + kz * d.pos[3 * dip + 2]));
  const double2* e = e0 + 3 * r;
  double2 v;
  if (!magnetic) {
    v = cmul(e[a], ph);
  } else {
    // (khat x e)_a
    const int b = (a + 1) % 3, c = (a + 2) % 3;
    const double kb = b == 0 ? kx : (b == 1 ? ky : kz);
    const double kc = c == 0 ? kx : (c == 1 ? ky : kz);
    const double2 cr = csub(cscale(e[c], kb), cscale(e[b], kc));
    v = cscale(cmul(cr, ph), n_env);
  }
  f0[r * n + u] = v;
}

hipError_t launch_incident(const DipoleView& d, const Wave& w, double n_env, int64_t n_pw, const double* khat,
                           const double2* e0, double2* f0, int64_t n, hipStream_t st) {
  if (n_pw <= 0 || n <= 0) return hipSuccess;
  hipLaunchKernelGGL(incident_kernel, dim3((unsigned)((n + 255) / 256), (unsigned)n_pw), dim3(256), 0, st, d, w, n_env,
                     n_pw, khat, e0, f0, n);
  return hipGetLastError();
}

// ACC: add the plane wave to E (and H) instead of writing it (total field at
// probes = incident + scattered).
template <bool ACC>
__global__ void planewave_points_kernel(Wave w, double n_env, int64_t n_pw, const double* khat, const double2* e0,
                                        const double* rp, int64_t P, double2* E, double2* H) {
  const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t r = blockIdx.y;
  if (p >= P) return;
  const double kx = khat[3 * r], ky = khat[3 * r + 1], kz = khat[3 * r + 2];
  const double2 ph = expi(w.k * (kx * rp[3 * p] + ky * rp[3 * p + 1] + kz * rp[3 * p + 2]));
  const double2* e = e0 + 3 * r;
  const double2 ex = cmul(e[0], ph), ey = cmul(e[1], ph), ez = cmul(e[2], ph);
  double2* oe = E + (r * P + p) * 3;
  oe[0] = ACC ? cadd(oe[0], ex) : ex;
  oe[1] = ACC ? cadd(oe[1], ey) : ey;
  oe[2] = ACC ? cadd(oe[2], ez) : ez;
  if (H) {
    double2* oh = H + (r * P + p) * 3;
    const double2 hx = cscale(csub(cscale(ez, ky), cscale(ey, kz)), n_env);
    const double2 hy = cscale(csub(cscale(ex, kz), cscale(ez, kx)), n_env);
    const double2 hz = cscale(csub(cscale(ey, kx), cscale(ex, ky)), n_env);
    oh[0] = ACC ? cadd(oh[0], hx) : hx;
    oh[1] = ACC ? cadd(oh[1], hy) : hy;
    oh[2] = ACC ? cadd(oh[2], hz) : hz;
  }
}

hipError_t launch_planewave_points(const Wave& w, double n_env, int64_t n_pw, const double* khat, const double2* e0,
                                   const double* r, int64_t P, double2* E, double2* H, hipStream_t st,
                                   bool accumulate) {
  if (n_pw <= 0 || P <= 0) return hipSuccess;
  const dim3 grid((unsigned)((P + 255) / 256), (unsigned)n_pw);
  if (accumulate)
    hipLaunchKernelGGL(planewave_points_kernel<true>, grid, dim3(256), 0, st, w, n_env, n_pw, khat, e0, r, P, E, H);
  else
    hipLaunchKernelGGL(planewave_points_kernel<false>, grid, dim3(256), 0, st, w, n_env, n_pw, khat, e0, r, P, E, H);
  return hipGetLastError();
}

// |E0|^2 = sum_a |e0[r][a]|^2 per plane wave
__global__ void pw_intensity_kernel(int64_t n_pw, const double2* __restrict__ e0, double* __restrict__ out) {
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_pw) return;
  double s = 0;
  for (int a = 0; a < 3; ++a) s += e0[3 * r + a].x * e0[3 * r + a].x + e0[3 * r + a].y * e0[3 * r + a].y;
  out[r] = s;
}

hipError_t launch_pw_intensity(int64_t n_pw, const double2* e0, double* out, hipStream_t st) {
  if (n_pw <= 0) return hipSuccess;
  hipLaunchKernelGGL(pw_intensity_kernel, dim3((unsigned)((n_pw + 255) / 256)), dim3(256), 0, st, n_pw, e0, out);
  return hipGetLastError();
}

// one thread per (dipole, rhs)
__global__ void apply_alpha_kernel(DipoleView d, const double2* F, int64_t ldf, double2* q, int64_t ldq,
                                   int64_t nrhs) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t r = blockIdx.y;
  if (i >= d.N) return;
  const double2* f = F + r * ldf;
  double2* o = q + r * ldq;
  if (i < d.nc) {
    const double2 a = d.alpha_c[i];
    for (int c = 0; c < 3; ++c) o[3 * i + c] = cmul(a, f[3 * i + c]);
  } else {
    const int64_t e = i - d.nc;
    double2 v[6];
    for (int c = 0; c < 3; ++c) {
      v[c] = f[3 * i + c];
      v[3 + c] = f[3 * d.N + 3 * e + c];
    }
    const double2* a = d.alpha6 + e * 36;
    for (int rr = 0; rr < 6; ++rr) {
      double2 s = make_double2(0, 0);
      for (int c = 0; c < 6; ++c) cfma(s, a[rr * 6 + c], v[c]);
      if (rr < 3) o[3 * i + rr] = s;
      else o[3 * d.N + 3 * e + (rr - 3)] = s;
    }
  }
}

hipError_t launch_apply_alpha(const DipoleView& d, const double2* F, int64_t ldf, double2* q, int64_t ldq,
                              int64_t nrhs, hipStream_t st) {
  if (d.N <= 0 || nrhs <= 0) return hipSuccess;
  hipLaunchKernelGGL(apply_alpha_kernel, dim3((unsigned)((d.N + 255) / 256), (unsigned)nrhs), dim3(256), 0, st, d, F,
                     ldf, q, ldq, nrhs);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_gpm_apply(d, F, ldf, q, ldq, nrhs, st);  // members of GPM groups (overwrites their q)
}

// one workgroup (1024 threads) per RHS, FP64 tree reduction in LDS
__global__ void __launch_bounds__(1024) cs_sums_kernel(DipoleView d, const double2* f0, const double2* q,
                                                       const double2* f, int64_t n, double* out) {
  const int64_t r = blockIdx.x;
  const double2* a0 = f0 + r * n;
  const double2* aq = q + r * n;
  const double2* af = f + r * n;
  double s[5] = {0, 0, 0, 0, 0};
  const int64_t ncE = 3 * d.nc, NE = 3 * d.N;
  for (int64_t u = threadIdx.x; u < n; u += blockDim.x) {
    const double2 qq = aq[u];
    const double2 x0 = a0[u], xf = af[u];
    s[0] += x0.x * qq.y - x0.y * qq.x;  // Im(conj(F0) q)
    s[1] += xf.x * qq.y - xf.y * qq.x;  // Im(conj(F) q)
    const double q2 = qq.x * qq.x + qq.y * qq.y;
    if (u < ncE) s[2] += q2;
    else if (u < NE) s[3] += q2;
    else s[4] += q2;
  }
  __shared__ double red[5][1024];
  for (int k = 0; k < 5; ++k) red[k][threadIdx.x] = s[k];
  __syncthreads();
  for (int off = 512; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off)
      for (int k = 0; k < 5; ++k) red[k][threadIdx.x] += red[k][threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x < 5) out[r * 5 + threadIdx.x] = red[threadIdx.x][0];
}

hipError_t launch_cs_sums(const DipoleView& d, const double2* f0, const double2* q, const double2* f, int64_t n,
                          int64_t nrhs, double* sums5, hipStream_t st) {
  if (nrhs <= 0) return hipSuccess;
  hipLaunchKernelGGL(cs_sums_kernel, dim3((unsigned)nrhs), dim3(1024), 0, st, d, f0, q, f, n, sums5);
  return hipGetLastError();
}

// Im sum_{i != j} q_i^H G6(r_i - r_j) q_j, NR right-hand sides per workgroup (the
// dyad of a pair once for all of them): a thread sums the field of the sources of
// its split at dipole i, then takes it against q_i.  blockIdx.x: (256 targets,
// split of the sources), blockIdx.y: right-hand sides.  Bound by the FP64 vector
// rate.  N = 2431, 24 right-hand sides: 0.44 ms (2.3 ms with a dyad matrix and its
// quadratic form per pair and right-hand side, one workgroup per 256 targets).
constexpr int FFT = 64;  // sources per LDS tile

template <int NR>
__global__ void __launch_bounds__(256) sca_ff_kernel(DipoleView d, Wave w, const double2* q, int64_t ldq, int64_t nrhs,
                                                     int nsplit, int64_t jps, double* partial, int64_t nblk) {
  __shared__ double spos[FFT][3];
  __shared__ double2 sq[FFT][NR][6];  // P = p / n, then m
  __shared__ double red[256];
  const int64_t r0 = (int64_t)blockIdx.y * NR;
  const int64_t i = (int64_t)(blockIdx.x / nsplit) * 256 + threadIdx.x;
  const int split = (int)(blockIdx.x % nsplit);
  const int64_t N = d.N, nc = d.nc;
  const int64_t j0 = split * jps, j1 = j0 + jps < N ? j0 + jps : N;
  const bool live = i < N, eff_t = live && i >= nc;
  const bool any_eff_t = __any(eff_t);
  const double inv_n = w.k0 / w.k;
  double x = 0, y = 0, z = 0;
  if (live) {
    x = d.pos[3 * i];
    y = d.pos[3 * i + 1];
    z = d.pos[3 * i + 2];
  }
  double2 E[NR][3], H[NR][3];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int a = 0; a < 3; ++a) E[r][a] = H[r][a] = make_double2(0, 0);
  for (int64_t t0 = j0; t0 < j1; t0 += FFT) {
    const int nt = (int)(j1 - t0 < FFT ? j1 - t0 : FFT);
    __syncthreads();
    for (int t = threadIdx.x; t < nt * NR; t += 256) {
      const int64_t j = t0 + t / NR;
      const int r = t % NR;
      const double2* qc = q + (r0 + r) * ldq;
      const bool rv = r0 + r < nrhs;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const double2 p = rv ? qc[3 * j + a] : make_double2(0, 0);
        sq[t / NR][r][a] = cscale(p, inv_n);
        sq[t / NR][r][3 + a] = rv && j >= nc ? qc[3 * N + 3 * (j - nc) + a] : make_double2(0, 0);
        if (r == 0) spos[t / NR][a] = d.pos[3 * j + a];
      }
    }
    __syncthreads();
    if (!live) continue;
    const int ncell_in_tile = (int)(nc - t0 > 0 ? (nc - t0 < nt ? nc - t0 : nt) : 0);
    auto sweep = [&](auto hs, auto ht, int ta, int tb) __attribute__((always_inline)) {
      constexpr bool HS = decltype(hs)::value, HT = decltype(ht)::value;
      for (int t = ta; t < tb; ++t) {
        if (t0 + t == i) continue;
        const double R[3] = {x - spos[t][0], y - spos[t][1], z - spos[t][2]};
        const Dyad g = dyad_at<HS || HT>(fma(R[2], R[2], fma(R[1], R[1], R[0] * R[0])), w.k);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          dyad_electric(E[r], g, R, sq[t][r][0], sq[t][r][1], sq[t][r][2]);
          if (HT) dyad_magnetic<1>(H[r], g, R, sq[t][r][0], sq[t][r][1], sq[t][r][2]);
          if (HS) {
            dyad_magnetic<-1>(E[r], g, R, sq[t][r][3], sq[t][r][4], sq[t][r][5]);
            if (HT) dyad_electric(H[r], g, R, sq[t][r][3], sq[t][r][4], sq[t][r][5]);
          }
        }
      }
    };
    const std::true_type yes;
    const std::false_type no;
    if (any_eff_t) {
      sweep(no, yes, 0, ncell_in_tile);
      sweep(yes, yes, ncell_in_tile, nt);
    } else {
      sweep(no, no, 0, ncell_in_tile);
      sweep(yes, no, ncell_in_tile, nt);
    }
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    // Im conj(P_i) . N + Im conj(m_i) . H
    double acc = 0;
    if (live && r0 + r < nrhs) {
      const double2* qc = q + (r0 + r) * ldq;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        const double2 p = cscale(qc[3 * i + a], inv_n);
        acc += p.x * E[r][a].y - p.y * E[r][a].x;
        if (eff_t) {
          const double2 m = qc[3 * N + 3 * (i - nc) + a];
          acc += m.x * H[r][a].y - m.y * H[r][a].x;
        }
      }
    }
    __syncthreads();
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
      if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
      __syncthreads();
    }
    if (threadIdx.x == 0 && r0 + r < nrhs) partial[(r0 + r) * nblk + blockIdx.x] = red[0];
  }
}

// splits of the sources: about 256 workgroups per group of right-hand sides, at
// least one LDS tile each
static int sca_ff_splits(int64_t N) {
  const int64_t tb = (N + 255) / 256;
  return (int)std::max<int64_t>(1, std::min<int64_t>((N + FFT - 1) / FFT, 256 / tb));
}
int64_t sca_ff_blocks(int64_t N, int splits) { return (N + 255) / 256 * (splits > 0 ? splits : sca_ff_splits(N)); }

hipError_t launch_sca_ff(const DipoleView& d, const Wave& w, const double2* q, int64_t ldq, int64_t nrhs,
                         double* partial, int64_t nblk, hipStream_t st) {
  if (nrhs <= 0 || d.N <= 0) return hipSuccess;
  const int ns = (int)(nblk / ((d.N + 255) / 256));
  const int64_t jps = ((d.N + ns - 1) / ns + FFT - 1) / FFT * FFT;  // trailing splits may be empty (partial sum 0)
  if (nrhs == 1)
    hipLaunchKernelGGL(sca_ff_kernel<1>, dim3((unsigned)nblk, 1), dim3(256), 0, st, d, w, q, ldq, nrhs, ns, jps, partial,
                       nblk);
  else
    hipLaunchKernelGGL(sca_ff_kernel<4>, dim3((unsigned)nblk, (unsigned)((nrhs + 3) / 4)), dim3(256), 0, st, d, w, q, ldq,
                       nrhs, ns, jps, partial, nblk);
  return hipGetLastError();
}

// ---- refinement helpers ------------------------------------------------------
__global__ void convert_d2f_kernel(const double2* a, int64_t lda, float2* b, int64_t ldb, int64_t m) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t c = blockIdx.y;
  if (i < m) {
    const double2 v = a[i + c * lda];
    b[i + c * ldb] = make_float2((float)v.x, (float)v.y);
  }
}
__global__ void convert_f2d_kernel(const float2* a, int64_t lda, double2* b, int64_t ldb, int64_t m) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t c = blockIdx.y;
  if (i < m) {
    const float2 v = a[i + c * lda];
    b[i + c * ldb] = make_double2(v.x, v.y);
  }
}
template <typename CT> __global__ void copy_kernel(const CT* a, int64_t lda, CT* b, int64_t ldb, int64_t m) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t c = blockIdx.y;
  if (i < m) b[i + c * ldb] = a[i + c * lda];
}

// large 2D grids: columns in blockIdx.y up to 65535, so split very wide matrices
template <typename K, typename... Args>
static hipError_t launch_cols(K kernel, int64_t m, int64_t n, hipStream_t st, Args... args) {
  if (m <= 0 || n <= 0) return hipSuccess;
  hipLaunchKernelGGL(kernel, dim3((unsigned)((m + 255) / 256), (unsigned)n), dim3(256), 0, st, args..., m);
  return hipGetLastError();
}

hipError_t launch_convert_d2f(const double2* a, int64_t lda, float2* b, int64_t ldb, int64_t m, int64_t n,
                              hipStream_t st) {
  for (int64_t c0 = 0; c0 < n; c0 += 65535) {
    const int64_t nc = n - c0 < 65535 ? n - c0 : 65535;
    hipError_t e = launch_cols(convert_d2f_kernel, m, nc, st, a + c0 * lda, lda, b + c0 * ldb, ldb);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
hipError_t launch_convert_f2d(const float2* a, int64_t lda, double2* b, int64_t ldb, int64_t m, int64_t n,
                              hipStream_t st) {
  for (int64_t c0 = 0; c0 < n; c0 += 65535) {
    const int64_t nc = n - c0 < 65535 ? n - c0 : 65535;
    hipError_t e = launch_cols(convert_f2d_kernel, m, nc, st, a + c0 * lda, lda, b + c0 * ldb, ldb);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
template <typename CT>
static hipError_t launch_copy(const CT* a, int64_t lda, CT* b, int64_t ldb, int64_t m, int64_t n, hipStream_t st) {
  for (int64_t c0 = 0; c0 < n; c0 += 65535) {
    const int64_t nc = n - c0 < 65535 ? n - c0 : 65535;
    hipError_t e = launch_cols(copy_kernel<CT>, m, nc, st, a + c0 * lda, lda, b + c0 * ldb, ldb);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
hipError_t launch_copy_d(const double2* a, int64_t lda, double2* b, int64_t ldb, int64_t m, int64_t n, hipStream_t st) {
  return launch_copy(a, lda, b, ldb, m, n, st);
}
hipError_t launch_copy_f(const float2* a, int64_t lda, float2* b, int64_t ldb, int64_t m, int64_t n, hipStream_t st) {
  return launch_copy(a, lda, b, ldb, m, n, st);
}

// one workgroup per column: x += c, cmax[col] = max |c|
__global__ void __launch_bounds__(256) axpy_f2d_kernel(const float2* c, int64_t ldc, double2* x, int64_t ldx,
                                                       int64_t m, double* cmax) {
  const int64_t col = blockIdx.x;
  double mx = 0;
  for (int64_t i = threadIdx.x; i < m; i += 256) {
    const float2 v = c[i + col * ldc];
    double2 xv = x[i + col * ldx];
    xv.x += (double)v.x;
    xv.y += (double)v.y;
    x[i + col * ldx] = xv;
    const double a = sqrt((double)v.x * v.x + (double)v.y * v.y);
    mx = a > mx ? a : mx;
  }
  __shared__ double red[256];
  red[threadIdx.x] = mx;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + off]);
    __syncthreads();
  }
  if (threadIdx.x == 0) cmax[col] = red[0];
}

hipError_t launch_axpy_f2d(const float2* c, int64_t ldc, double2* x, int64_t ldx, int64_t m, int64_t n,
                           double* cmax, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(axpy_f2d_kernel, dim3((unsigned)n), dim3(256), 0, st, c, ldc, x, ldx, m, cmax);
  return hipGetLastError();
}

__global__ void __launch_bounds__(256) colmax_kernel(const double2* a, int64_t lda, int64_t m, double* out) {
  const int64_t col = blockIdx.x;
  double mx = 0;
  for (int64_t i = threadIdx.x; i < m; i += 256) {
    const double2 v = a[i + col * lda];
    const double t = sqrt(v.x * v.x + v.y * v.y);
    mx = t > mx ? t : mx;
  }
  __shared__ double red[256];
  red[threadIdx.x] = mx;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + off]);
    __syncthreads();
  }
  if (threadIdx.x == 0) out[col] = red[0];
}

hipError_t launch_colmax(const double2* a, int64_t lda, int64_t m, int64_t n, double* out, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(colmax_kernel, dim3((unsigned)n), dim3(256), 0, st, a, lda, m, out);
  return hipGetLastError();
}

// cols[j] = sum_i |M_ij| (one workgroup per column, fixed-order reduction)
__global__ void __launch_bounds__(256) colsum_abs_kernel(const double2* M, int64_t ld, int64_t n, double* cols) {
  const int64_t col = blockIdx.x;
  double s = 0;
  for (int64_t i = threadIdx.x; i < n; i += 256) {
    const double2 v = M[i + col * ld];
    s += sqrt(v.x * v.x + v.y * v.y);
  }
  __shared__ double red[256];
  red[threadIdx.x] = s;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) cols[col] = red[0];
}

hipError_t launch_colsum_abs(const double2* M, int64_t ld, int64_t n, double* cols, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(colsum_abs_kernel, dim3((unsigned)n), dim3(256), 0, st, M, ld, n, cols);
  return hipGetLastError();
}

// rows[z n + i] = sum_j |M_z[i, j]|: 64 rows and cw columns (grid y) per workgroup,
// an eighth of the columns per wave, eight loads in flight per lane; one FP64
// atomic per row and column chunk when there are several, else a store.  Bound by
// the read of M: n = 12 000: 0.43 ms (5.3 TB/s), n = 6000: 0.154, n = 2916: 0.020; one row per
// thread and one load in flight took 0.47, 0.33 and 0.16 ms, and 2.42 instead of
// 0.90 ms for a batch of 16 matrices of n = 4500.
constexpr int RS_CHUNK = 256;
__global__ void __launch_bounds__(512) rowsum_abs_kernel(const double2* __restrict__ M, int64_t ld, int64_t n, int64_t sM,
                                                          int64_t cw, double* __restrict__ rows) {
  __shared__ double red[8][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t i = (int64_t)blockIdx.x * 64 + lane;
  const int64_t c0 = (int64_t)blockIdx.y * cw, c1 = c0 + cw < n ? c0 + cw : n;
  const double2* m = M + (int64_t)blockIdx.z * sM + (i < n ? i : n - 1);
  double s = 0;
  constexpr int U = 8;
  for (int64_t j = c0 + wave * U; j < c1; j += 8 * U) {
    double2 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = m[(j + u < c1 ? j + u : c1 - 1) * ld];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (j + u < c1) s += sqrt(v[u].x * v[u].x + v[u].y * v[u].y);
  }
  red[wave][lane] = s;
  __syncthreads();
  if (wave > 0 || i >= n) return;
#pragma unroll
  for (int w = 1; w < 8; ++w) s += red[w][lane];
  double* o = rows + (int64_t)blockIdx.z * n + i;
  if (gridDim.y > 1) atomicAdd(o, s);
  else *o = s;
}
__global__ void zero_d_kernel(double* a, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) a[i] = 0;
}

hipError_t launch_rowsum_abs(const double2* M, int64_t ld, int64_t n, double* rows, hipStream_t st, int nbatch,
                             int64_t sM) {
  if (n <= 0) return hipSuccess;
  // a batch has workgroups enough without a split of the columns (and no atomics: its order is fixed)
  const int64_t cw = nbatch > 0 ? n : RS_CHUNK, ny = (n + cw - 1) / cw;
  if (ny > 1)
    hipLaunchKernelGGL(zero_d_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, rows, n);
  hipLaunchKernelGGL(rowsum_abs_kernel, dim3((unsigned)((n + 63) / 64), (unsigned)ny, (unsigned)std::max(nbatch, 1)),
                     dim3(512), 0, st, M,
                     ld, n, sM, cw, rows);
  return hipGetLastError();
}

// ---- per-launch event timing -------------------------------------------------
hipError_t Prof::begin(hipStream_t st, int t, double w) {
  open = ((mask >> t) & 1u) != 0;
  if (!open) return hipSuccess;
  if (2 * used + 2 > ev.size()) {
    for (int i = 0; i < 2; ++i) {
      hipEvent_t e;
      hipError_t r = hipEventCreate(&e);
      if (r != hipSuccess) return r;
      ev.push_back(e);
    }
    tag.push_back(0);
    work.push_back(0);
  }
  tag[used] = t;
  work[used] = w;
  return hipEventRecord(ev[2 * used], st);
}
hipError_t Prof::end(hipStream_t st) {
  if (!open) return hipSuccess;
  open = false;
  hipError_t r = hipEventRecord(ev[2 * used + 1], st);
  ++used;
  return r;
}
void Prof::collect() {
  for (size_t i = 0; i < used; ++i) {
    float t = 0.f;
    if (hipEventElapsedTime(&t, ev[2 * i], ev[2 * i + 1]) == hipSuccess) {
      ms[tag[i]] += t;
      wsum[tag[i]] += work[i];
      cnt[tag[i]] += 1;
    }
  }
  used = 0;
}
void Prof::reset() {
  used = 0;
  for (int i = 0; i < PROF_NTAGS; ++i) ms[i] = wsum[i] = cnt[i] = 0;
}
Prof::~Prof() {
  for (hipEvent_t e : ev) (void)hipEventDestroy(e);
}


}  // namespace gdm
