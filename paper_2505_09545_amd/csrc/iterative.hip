// Step (b) without a stored matrix: the linear system M F = F0, M = I - G~ A,
// solved by a Krylov method whose matrix-vector product re-evaluates the
// coupling sum from the dyad on every call (arXiv:2505.09545, Sec. "Discrete
// Dipole Approximation - iterative solver": the DDA route past the size where
// the dense inversion no longer fits, cf. Sec. "Benchmarks", runtime and
// memory; the paper's own solver is the dense LU of Sec. "Numerical solution").
//
// Product: y = M x = x - G~ (A x).  q = A x (the dipole moments of the field
// x), then for every dipole i, as a target, the field of all other dipoles,
// sum_{j != i} G(r_i, r_j) q_j, plus the self-term S_i q_i of a cell; the 6x6
// dyad of every pair is recomputed in registers (gdm_dyad.hpp) and never stored;
// the product is bound by the FP64 vector rate (N = 3300: 49 us; 86 with the dyad
// as a 6x6 matrix and the library sincos).
// Sources are swept in LDS tiles, the sum split over several workgroups when
// there are few targets, the partial sums added in a fixed order by the kernel
// that forms y (deterministic).
//
// Preconditioner: block Jacobi over near-field blocks -- consecutive dipoles in
// groups of PC_DIP (spatial neighbours for the cubic grids and lattices of the
// workloads, which are laid out in grid order).  Each block's rows and columns
// of M (its E unknowns, then the H unknowns of its effective dipoles, at most
// PC_MAXD) are assembled in FP64 with the same block formula as the dense
// assembly and inverted by Gauss-Jordan elimination with partial pivoting.
//
// Krylov method: restarted GMRES with right preconditioning (so the residual
// it minimises is that of the original system), classical Gram-Schmidt with
// one re-orthogonalisation, Givens rotations of the small Hessenberg matrix on
// the host; one small device-to-host copy per iteration.  All arithmetic FP64.
#include <algorithm>
#include <cmath>
#include <complex>
#include <type_traits>
#include <vector>

#include "gdm_common.hpp"
#include "gdm_dyad.hpp"
#include "gdm_kernels.hpp"
#include "gdm_misc.hpp"
#include "gdm_iterative.hpp"

namespace gdm {

constexpr int CT = 256;  // source dipoles per LDS tile

// Partial coupling sums of the sources [split * jps, (split + 1) * jps): one
// thread per target dipole i; E_i for every target, H_i for effective targets,
// written to part[split][r][u] in the unknown layout (u = 3i + a for E, 3N +
// 3(i - nc) + a for H).  The pair j == i is skipped.
template <int NR>
__global__ void __launch_bounds__(256) coupling_kernel(DipoleView d, Wave w, const double2* __restrict__ q, int64_t n,
                                                        int64_t nrhs, int r0, int64_t jps,
                                                        double2* __restrict__ part) {
  __shared__ double spos[CT][3];
  __shared__ double2 sp[CT][NR][3];
  __shared__ double2 sm[CT][NR][3];
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int split = blockIdx.y;
  const int64_t N = d.N, nc = d.nc;
  const int64_t j0 = split * jps;
  const int64_t j1 = j0 + jps < N ? j0 + jps : N;
  const bool live = i < N;
  const bool eff_t = live && i >= nc;
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
    for (int a = 0; a < 3; ++a) {
      E[r][a] = make_double2(0, 0);
      H[r][a] = make_double2(0, 0);
    }
  for (int64_t t0 = j0; t0 < j1; t0 += CT) {
    const int nt = (int)(j1 - t0 < CT ? j1 - t0 : CT);
    __syncthreads();
    for (int t = threadIdx.x; t < nt; t += 256) {
      const int64_t j = t0 + t;
      double pv[3];
      double2 qv[NR][3], mv[NR][3];
#pragma unroll
      for (int a = 0; a < 3; ++a) pv[a] = d.pos[3 * j + a];
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const bool rv = r0 + r < nrhs;
        const double2* qc = q + (int64_t)(r0 + r) * n;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          qv[r][a] = rv ? qc[3 * j + a] : make_double2(0, 0);
          mv[r][a] = (rv && j >= nc) ? qc[3 * N + 3 * (j - nc) + a] : make_double2(0, 0);
        }
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) spos[t][a] = pv[a];
#pragma unroll
      for (int r = 0; r < NR; ++r)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          sp[t][r][a] = cscale(qv[r][a], inv_n);  // P = p / n
          sm[t][r][a] = mv[r][a];
        }
    }
    __syncthreads();
    if (!live) continue;
    const int ncell_in_tile = (int)(nc - t0 > 0 ? (nc - t0 < nt ? nc - t0 : nt) : 0);
    // sources [ta, tb) of the tile; HS: effective sources, HT: some lane of the
    // wave has an effective target
    auto sweep = [&](auto hs, auto ht, int ta, int tb) __attribute__((always_inline)) {
      constexpr bool HS = decltype(hs)::value, HT = decltype(ht)::value;
      for (int t = ta; t < tb; ++t) {
        if (t0 + t == i) continue;
        const double R[3] = {x - spos[t][0], y - spos[t][1], z - spos[t][2]};
        const Dyad g = dyad_at<HS || HT>(fma(R[2], R[2], fma(R[1], R[1], R[0] * R[0])), w.k);
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          dyad_electric(E[r], g, R, sp[t][r][0], sp[t][r][1], sp[t][r][2]);
          if (HT) dyad_magnetic<1>(H[r], g, R, sp[t][r][0], sp[t][r][1], sp[t][r][2]);
          if (HS) {
            dyad_magnetic<-1>(E[r], g, R, sm[t][r][0], sm[t][r][1], sm[t][r][2]);
            if (HT) dyad_electric(H[r], g, R, sm[t][r][0], sm[t][r][1], sm[t][r][2]);
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
  if (!live) return;
  const int64_t stride = nrhs * n;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    if (r0 + r >= nrhs) break;
    double2* o = part + split * stride + (int64_t)(r0 + r) * n;
#pragma unroll
    for (int a = 0; a < 3; ++a) o[3 * i + a] = cscale(E[r][a], inv_n);
    if (eff_t)
#pragma unroll
      for (int a = 0; a < 3; ++a) o[3 * N + 3 * (i - nc) + a] = H[r][a];
  }
}

// y = x - sum_s part[s] - (cell E unknowns) S q, over nrhs * n entries
__global__ void coupling_finish_kernel(const double2* __restrict__ part, int nsplit, int64_t stride,
                                       const double2* __restrict__ x, const double2* __restrict__ q, double2 self_c,
                                       int64_t ncell3, int64_t n, double2* __restrict__ y, int64_t count) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= count) return;
  double2 s = part[idx];
  for (int k = 1; k < nsplit; ++k) s = cadd(s, part[k * stride + idx]);
  double2 v = csub(x[idx], s);
  if (idx % n < ncell3) v = csub(v, cmul(self_c, q[idx]));
  y[idx] = v;
}

// ---------------------------------------------------------------------------
// block Jacobi preconditioner
// ---------------------------------------------------------------------------
// Block b: dipoles [b PC_DIP, min((b + 1) PC_DIP, N)).  Local unknowns: the E
// slots of its dipoles (3 each), then the H slots of its effective dipoles.
struct PcBlock {
  int64_t d0;  // first dipole
  int nd;      // dipoles
  int ne;      // effective dipoles among them (the last ne, since cells come first)
  int D;       // local unknowns 3 (nd + ne)
};
__device__ inline PcBlock pc_block(const DipoleView& d, int64_t b) {
  PcBlock p;
  p.d0 = b * PC_DIP;
  const int64_t d1 = p.d0 + PC_DIP < d.N ? p.d0 + PC_DIP : d.N;
  p.nd = (int)(d1 - p.d0);
  const int64_t e0 = p.d0 > d.nc ? p.d0 : d.nc;
  p.ne = d1 > e0 ? (int)(d1 - e0) : 0;
  p.D = 3 * (p.nd + p.ne);
  return p;
}
// global unknown of local unknown l of block p
__device__ inline int64_t pc_unknown(const DipoleView& d, const PcBlock& p, int l) {
  const int slot = l / 3, a = l % 3;
  if (slot < p.nd) return 3 * (p.d0 + slot) + a;
  const int64_t dip = p.d0 + p.nd - p.ne + (slot - p.nd);  // effective dipole
  return 3 * d.N + 3 * (dip - d.nc) + a;
}

// One workgroup per block: its D x D block of M in LDS next to the identity,
// Gauss-Jordan with partial pivoting (largest modulus in the column), the
// inverse written column-major to inv[b] (leading dimension PC_MAXD).  A zero
// pivot leaves the identity for that block (no preconditioning there).
__global__ void __launch_bounds__(256) precond_build_kernel(DipoleView d, Wave w, double2* __restrict__ inv) {
  __shared__ double2 T[PC_MAXD][2 * PC_MAXD + 1];  // augmented rows [block | identity]
  __shared__ int piv_row;
  __shared__ int singular;
  const int64_t b = blockIdx.x;
  const PcBlock p = pc_block(d, b);
  const int D = p.D, tid = threadIdx.x;
  if (tid == 0) singular = 0;
  for (int idx = tid; idx < PC_MAXD * (2 * PC_MAXD + 1); idx += 256)
    T[idx / (2 * PC_MAXD + 1)][idx % (2 * PC_MAXD + 1)] = make_double2(0.0, 0.0);
  __syncthreads();
  for (int r = tid; r < D; r += 256) T[r][PC_MAXD + r] = make_double2(1.0, 0.0);
  // blocks of M: (row slot, column dipole) pairs
  const int nslots = p.nd + p.ne;
  for (int item = tid; item < nslots * p.nd; item += 256) {
    const int rs = item / p.nd, cj = item % p.nd;
    const int64_t jdip = p.d0 + cj;
    const int f = rs < p.nd ? 0 : 1;
    const int64_t dr = f == 0 ? p.d0 + rs : p.d0 + p.nd - p.ne + (rs - p.nd);
    const int ce = jdip >= d.nc ? (int)(jdip - (p.d0 + p.nd - p.ne)) : -1;  // local effective index of the column dipole
    if (jdip < d.nc) {
      double2 v[3][3];
      m_block<false>(d, w, dr, f, jdip, v);
#pragma unroll
      for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int a = 0; a < 3; ++a) T[3 * rs + a][3 * cj + c] = v[c][a];
    } else {
      double2 v[6][3];
      m_block<true>(d, w, dr, f, jdip, v);
#pragma unroll
      for (int c = 0; c < 6; ++c)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const int col = c < 3 ? 3 * cj + c : 3 * (p.nd + ce) + (c - 3);
          T[3 * rs + a][col] = v[c][a];
        }
    }
  }
  __syncthreads();
  for (int k = 0; k < D; ++k) {
    if (tid < 64) {
      double best = -1.0;
      int br = k;
      for (int r = k + tid; r < D; r += 64) {
        const double m = fabs(T[r][k].x) + fabs(T[r][k].y);
        if (m > best) {
          best = m;
          br = r;
        }
      }
      // wave argmax (lowest row on ties)
      for (int off = 32; off >= 1; off >>= 1) {
        const double ob = __shfl_xor(best, off);
        const int orow = __shfl_xor(br, off);
        if (ob > best || (ob == best && orow < br)) {
          best = ob;
          br = orow;
        }
      }
      if (tid == 0) {
        piv_row = br;
        if (!(best > 0.0)) singular = 1;
      }
    }
    __syncthreads();
    if (singular) break;
    const int pr = piv_row;
    if (pr != k)
      for (int c = tid; c < 2 * PC_MAXD; c += 256) {
        const double2 t = T[k][c];
        T[k][c] = T[pr][c];
        T[pr][c] = t;
      }
    __syncthreads();
    const double2 pv = T[k][k];
    const double den = pv.x * pv.x + pv.y * pv.y;
    const double2 ip = make_double2(pv.x / den, -pv.y / den);
    __syncthreads();
    for (int c = tid; c < 2 * PC_MAXD; c += 256) T[k][c] = cmul(T[k][c], ip);
    __syncthreads();
    for (int idx = tid; idx < D * 2 * PC_MAXD; idx += 256) {
      const int r = idx / (2 * PC_MAXD), c = idx % (2 * PC_MAXD);
      if (r == k) continue;
      const double2 f = T[r][k];
      if (c == k) continue;  // column k of the other rows is cleared below
      T[r][c] = csub(T[r][c], cmul(f, T[k][c]));
    }
    __syncthreads();
    for (int r = tid; r < D; r += 256)
      if (r != k) T[r][k] = make_double2(0.0, 0.0);
    __syncthreads();
  }
  double2* o = inv + b * (int64_t)PC_MAXD * PC_MAXD;
  for (int idx = tid; idx < D * D; idx += 256) {
    const int r = idx % D, c = idx / D;
    const double2 v = singular ? make_double2(r == c ? 1.0 : 0.0, 0.0) : T[r][PC_MAXD + c];
    o[r + (int64_t)c * PC_MAXD] = v;
  }
}

// z = P v: one workgroup per (block, RHS); the block's unknowns of v gathered
// into LDS, multiplied by the block's inverse, scattered into z.
__global__ void __launch_bounds__(64) precond_apply_kernel(DipoleView d, const double2* __restrict__ inv, int64_t n,
                                                            const double2* __restrict__ v, double2* __restrict__ z) {
  __shared__ double2 vl[PC_MAXD];
  const int64_t b = blockIdx.x;
  const int64_t r = blockIdx.y;
  const PcBlock p = pc_block(d, b);
  const int tid = threadIdx.x;
  if (tid < p.D) vl[tid] = v[r * n + pc_unknown(d, p, tid)];
  __syncthreads();
  if (tid >= p.D) return;
  const double2* A = inv + b * (int64_t)PC_MAXD * PC_MAXD;
  double2 s = make_double2(0, 0);
  for (int c = 0; c < p.D; ++c) cfma(s, A[tid + (int64_t)c * PC_MAXD], vl[c]);
  z[r * n + pc_unknown(d, p, tid)] = s;
}

// ---------------------------------------------------------------------------
// Krylov vector kernels on [nrhs][n] arrays (basis vector i at V + i vs)
// ---------------------------------------------------------------------------
// An Arnoldi step after the product is three launches of arnoldi_kernel and one
// of scale_precond_kernel, each a pass over the basis or over W that also begins
// the next reduction: workgroup c of a right-hand side owns the entries
// [c E, (c + 1) E), leaves its part of every scalar product in hp (norm: np), and
// the next launch's workgroups add the parts in a fixed order.  Bound by the
// traffic of the basis from 10^4 unknowns on, below by launches and latency.
// Per step (15 basis vectors, the mean of a cycle of 30): n = 9900 24 us, n = 69 000
// 57 us; as ten kernels (one workgroup per product and norm) 74 and 268 us and two
// copies to the host.
constexpr int AR_T = 512;  // threads: 4 groups of 128 entries in sums, 8 waves in products
constexpr int AR_G = 4;

// entries of a workgroup's part (at most AR_EMAX, about 128 parts below that)
constexpr int AR_EMAX = 1024;
static int arnoldi_entries(int64_t n) {
  const int64_t e = (n + 128 * 128 - 1) / (128 * 128) * 128;
  return (int)(e < AR_EMAX ? e : AR_EMAX);
}

__device__ inline double2 wave_sum(double2 s) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    s.x += __shfl_xor(s.x, off);
    s.y += __shfl_xor(s.y, off);
  }
  return s;
}
__device__ inline double wave_sum(double s) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
  return s;
}

struct ArnoldiArgs {
  const double2* V;     // basis, vector i of right-hand side r at V + i vs + r n
  double2* W;           // the new vector (not scaled yet)
  int64_t vs, n;
  int m1, j1, E, C;     // rows of hp (restart + 1), basis vectors, entries per part, parts
  const double2* hin;   // [nrhs][m1][C]: the products that W is to lose
  double2* hout;        // [nrhs][m1][C]: products with the W formed here
  double* np;           // [nrhs][C]: parts of ||W||^2
  double2* host;        // [nrhs][m1] totals of hin, in host memory
  // the coupling product (as in coupling_finish_kernel)
  const double2 *part, *x, *q;
  int nsplit;
  int64_t stride, ncell3;
  double2 self_c;
};

enum { AR_PRODUCT = 0, AR_AGAIN = 1, AR_NORM = 2 };

// AR_PRODUCT: W = x - sum_s part[s] - S q, products with the basis
// AR_AGAIN:   W -= sum_i h_i V_i, products with the basis
// AR_NORM:    W -= sum_i h_i V_i, parts of the norm
template <int MODE>
__global__ void __launch_bounds__(AR_T) arnoldi_kernel(ArnoldiArgs A) {
  extern __shared__ double2 ar_lds[];
  double2* const wl = ar_lds;             // [E] this part of W
  double2* const red = ar_lds + A.E;      // [AR_G][128]
  double2* const h = red + AR_G * 128;    // [j1]
  const int c = blockIdx.x, r = blockIdx.y, tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int g = tid >> 7, l = tid & 127;
  const int64_t k0 = (int64_t)c * A.E;
  const int ne = (int)(A.n - k0 < A.E ? A.n - k0 : A.E);
  const double2* const V = A.V + (int64_t)r * A.n + k0;
  double2* const W = A.W + (int64_t)r * A.n + k0;
  if constexpr (MODE != AR_PRODUCT) {
    const double2* hi = A.hin + (int64_t)r * A.m1 * A.C;
    for (int i = wave; i < A.j1; i += AR_T / 64) {
      double2 s = make_double2(0, 0);
      for (int b = lane; b < A.C; b += 64) s = cadd(s, hi[(int64_t)i * A.C + b]);
      s = wave_sum(s);
      if (lane == 0) {
        h[i] = s;
        if (c == 0) A.host[(int64_t)r * A.m1 + i] = s;
      }
    }
    __syncthreads();
  }
  // the sum over splits or basis vectors, a contiguous range of them per group of 128 threads
  const int ns = MODE == AR_PRODUCT ? A.nsplit : A.j1;
  const int per = (ns + AR_G - 1) / AR_G;
  const int s0 = g * per < ns ? g * per : ns, s1 = s0 + per < ns ? s0 + per : ns;
  double nn = 0;
  for (int e0 = 0; e0 < ne; e0 += 128) {
    const int e = e0 + l;
    double2 s = make_double2(0, 0);
    if (e < ne) {
      if constexpr (MODE == AR_PRODUCT) {
        const double2* p = A.part + (int64_t)r * A.n + k0 + e;
#pragma unroll 8
        for (int t = s0; t < s1; ++t) s = cadd(s, p[(int64_t)t * A.stride]);
      } else {
#pragma unroll 8
        for (int t = s0; t < s1; ++t) cfma(s, h[t], V[(int64_t)t * A.vs + e]);
      }
    }
    red[g * 128 + l] = s;
    __syncthreads();
    if (g == 0 && e < ne) {
#pragma unroll
      for (int t = 1; t < AR_G; ++t) s = cadd(s, red[t * 128 + l]);
      double2 v;
      if constexpr (MODE == AR_PRODUCT) {
        const int64_t u = k0 + e;
        v = csub(A.x[(int64_t)r * A.n + u], s);
        if (u < A.ncell3) v = csub(v, cmul(A.self_c, A.q[(int64_t)r * A.n + u]));
      } else {
        v = csub(W[e], s);
      }
      W[e] = v;
      if constexpr (MODE == AR_NORM) nn += v.x * v.x + v.y * v.y;
      else wl[e] = v;
    }
    __syncthreads();
  }
  if constexpr (MODE == AR_NORM) {
    double* const rn = reinterpret_cast<double*>(red);
    nn = wave_sum(nn);
    if (lane == 0 && wave < 2) rn[wave] = nn;
    __syncthreads();
    if (tid == 0) A.np[(int64_t)r * A.C + c] = rn[0] + rn[1];
  } else {
    // products: wave w takes the vectors w, w + 8, ..., four at a time
    double2* ho = A.hout + (int64_t)r * A.m1 * A.C + c;
    constexpr int NWV = AR_T / 64, U = 4;
    for (int i0 = wave; i0 < A.j1; i0 += NWV * U) {
      double2 s[U];
#pragma unroll
      for (int u = 0; u < U; ++u) s[u] = make_double2(0, 0);
      for (int e = lane; e < ne; e += 64) {
        const double2 b = wl[e];
        double2 a[U];
#pragma unroll
        for (int u = 0; u < U; ++u) a[u] = i0 + NWV * u < A.j1 ? V[(int64_t)(i0 + NWV * u) * A.vs + e] : make_double2(0, 0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          s[u].x += a[u].x * b.x + a[u].y * b.y;
          s[u].y += a[u].x * b.y - a[u].y * b.x;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (i0 + NWV * u >= A.j1) break;
        const double2 t = wave_sum(s[u]);
        if (lane == 0) ho[(int64_t)(i0 + NWV * u) * A.C] = t;
      }
    }
  }
}

// V_0 = b - y (y null: b) and the parts of its norm
__global__ void __launch_bounds__(AR_T) residual_kernel(const double2* __restrict__ b, const double2* __restrict__ y,
                                                         double2* __restrict__ V0, int64_t n, int E, int C,
                                                         double* __restrict__ np) {
  __shared__ double red[AR_T / 64];
  const int c = blockIdx.x;
  const int64_t base = (int64_t)blockIdx.y * n;
  const int64_t k1 = (int64_t)(c + 1) * E < n ? (int64_t)(c + 1) * E : n;
  double s = 0;
  for (int64_t k = (int64_t)c * E + threadIdx.x; k < k1; k += AR_T) {
    double2 v = b[base + k];
    if (y) v = csub(v, y[base + k]);
    V0[base + k] = v;
    s += v.x * v.x + v.y * v.y;
  }
  s = wave_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < AR_T / 64; ++i) s += red[i];
    np[(int64_t)blockIdx.y * C + c] = s;
  }
}

// One wave per preconditioner block and right-hand side: v = v / ||v|| (0 if the
// norm is 0), z = P v and the moments q = A z of the block's dipoles.
__global__ void __launch_bounds__(64) scale_precond_kernel(DipoleView d, const double2* __restrict__ inv, int64_t n,
                                                            const double* __restrict__ np, int C, double2* __restrict__ v,
                                                            double2* __restrict__ z, double2* __restrict__ q,
                                                            double* __restrict__ host) {
  __shared__ double2 vl[PC_MAXD], zl[PC_MAXD];
  const int64_t b = blockIdx.x;
  const int64_t r = blockIdx.y;
  const PcBlock p = pc_block(d, b);
  const int tid = threadIdx.x;
  const int64_t u = r * n + (tid < p.D ? pc_unknown(d, p, tid) : 0);
  double2 x = make_double2(0, 0);
  if (tid < p.D) x = v[u];
  double s = 0;
  for (int c = tid; c < C; c += 64) s += np[r * C + c];
  const double nrm = sqrt(wave_sum(s));
  if (b == 0 && tid == 0) host[r] = nrm;
  const double f = nrm > 0 ? 1.0 / nrm : 0.0;
  x = cscale(x, f);
  if (tid < p.D) vl[tid] = x;
  __syncthreads();
  if (tid < p.D) {
    v[u] = x;
    const double2* A = inv + b * (int64_t)PC_MAXD * PC_MAXD + tid;
    double2 t = make_double2(0, 0);
#pragma unroll 12
    for (int c = 0; c < p.D; ++c) cfma(t, A[(int64_t)c * PC_MAXD], vl[c]);
    z[u] = t;
    zl[tid] = t;
  }
  __syncthreads();
  if (tid < p.D) {
    const int slot = tid / 3, a = tid % 3;
    const int ncell = p.nd - p.ne;
    if (slot < ncell) {
      q[u] = cmul(d.alpha_c[p.d0 + slot], zl[tid]);
    } else {
      const bool mag = slot >= p.nd;
      const int e = mag ? slot - p.nd : slot - ncell;  // effective dipole of the block
      const double2* al = d.alpha6 + (p.d0 + ncell + e - d.nc) * 36 + (a + (mag ? 3 : 0)) * 6;
      double2 t = make_double2(0, 0);
#pragma unroll
      for (int c = 0; c < 6; ++c) cfma(t, al[c], zl[c < 3 ? 3 * (ncell + e) + c : 3 * (p.nd + e) + c - 3]);
      q[u] = t;
    }
  }
}

// out[r][k] = beta out[r][k] + sgn sum_{i < m} c[i][r] V_i[r][k]
__global__ void mcomb_kernel(const double2* __restrict__ V, int64_t vs, const double2* __restrict__ c, int m,
                             double sgn, double beta, double2* __restrict__ out, int64_t n, int nrhs) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx >= (int64_t)nrhs * n) return;
  const int r = (int)(idx / n);
  double2 s = make_double2(0, 0);
  for (int i = 0; i < m; ++i) cfma(s, c[(int64_t)i * nrhs + r], V[i * vs + idx]);
  const double2 o = out[idx];
  out[idx] = make_double2(beta * o.x + sgn * s.x, beta * o.y + sgn * s.y);
}

// a[i] += b[i]
__global__ void add_kernel(double2* __restrict__ a, const double2* __restrict__ b, int64_t count) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < count) a[idx] = cadd(a[idx], b[idx]);
}

__global__ void zero_kernel(double2* __restrict__ a, int64_t count) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (idx < count) a[idx] = make_double2(0.0, 0.0);
}

static unsigned nblocks(int64_t count) { return (unsigned)((count + 255) / 256); }

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
int coupling_num_splits(int64_t N, int num_cu) {
  const int64_t tblocks = (N + 255) / 256;
  int64_t want = (4 * (int64_t)num_cu + tblocks - 1) / tblocks;
  const int64_t maxs = (N + 31) / 32;
  want = std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(want, maxs), 64));
  const int64_t len = ((N + want - 1) / want + 31) / 32 * 32;
  return (int)((N + len - 1) / len);
}

size_t iter_workspace_bytes(int64_t N, int64_t n, int64_t nrhs, int restart, int num_cu, bool tight) {
  IterWork w;
  iter_workspace_carve(nullptr, N, n, nrhs, restart, num_cu, tight, w);
  return w.bytes;
}

void iter_workspace_carve(void* base, int64_t N, int64_t n, int64_t nrhs, int restart, int num_cu, bool tight,
                          IterWork& w) {
  char* p = static_cast<char*>(base);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    char* r = p ? p + off : nullptr;
    off += (bytes + 255) / 256 * 256;
    return r;
  };
  const size_t vec = (size_t)nrhs * n * sizeof(double2);
  w.nsplit = coupling_num_splits(N, num_cu);
  w.nblk = (N + PC_DIP - 1) / PC_DIP;
  w.V = reinterpret_cast<double2*>(take((size_t)(restart + 1) * vec));
  w.z = reinterpret_cast<double2*>(take(vec));
  w.q = reinterpret_cast<double2*>(take(vec));
  // the parts of the scalar products (two passes) share the scratch vector, which
  // is used between cycles only
  w.E = arnoldi_entries(n);
  if (tight) {
    // so few parts that they fit the scratch vector, and the norm's parts 32 bytes per
    // basis vector (as far as a part of W fits the LDS of arnoldi_kernel)
    const int64_t c = std::max<int64_t>(1, std::min<int64_t>(n / (2 * (restart + 1)), 4 * (restart + 1)));
    const int64_t e = ((n + c - 1) / c + 127) / 128 * 128, emax = (4096 - AR_G * 128 - (restart + 1)) / 128 * 128;
    w.E = (int)std::max<int64_t>(w.E, std::min(e, emax));
  }
  w.C = (int)((n + w.E - 1) / w.E);
  const size_t hp = (size_t)nrhs * (restart + 1) * w.C * sizeof(double2);
  w.t = reinterpret_cast<double2*>(take(std::max(vec, 2 * hp)));
  w.hp = w.t;
  w.part = reinterpret_cast<double2*>(take((size_t)w.nsplit * vec));
  w.inv = reinterpret_cast<double2*>(take((size_t)w.nblk * PC_MAXD * PC_MAXD * sizeof(double2)));
  w.np = reinterpret_cast<double*>(take((size_t)nrhs * w.C * sizeof(double)));
  w.y = reinterpret_cast<double2*>(take((size_t)(restart + 1) * nrhs * sizeof(double2)));
  w.bytes = off + 256;
}

hipError_t launch_precond_build(const DipoleView& d, const Wave& w, const IterWork& iw, hipStream_t st) {
  hipLaunchKernelGGL(precond_build_kernel, dim3((unsigned)iw.nblk), dim3(256), 0, st, d, w, iw.inv);
  return hipGetLastError();
}

// the partial coupling sums of the moments iw.q into iw.part
static hipError_t launch_coupling(const DipoleView& d, const Wave& w, const IterWork& iw, int64_t n, int64_t nrhs,
                                  hipStream_t st) {
  const int64_t jps = ((d.N + iw.nsplit - 1) / iw.nsplit + 31) / 32 * 32;
  const dim3 grid((unsigned)((d.N + 255) / 256), (unsigned)iw.nsplit);
  for (int r0 = 0; r0 < nrhs; r0 += 2) {
    if (nrhs - r0 >= 2)
      hipLaunchKernelGGL(coupling_kernel<2>, grid, dim3(256), 0, st, d, w, iw.q, n, nrhs, r0, jps, iw.part);
    else
      hipLaunchKernelGGL(coupling_kernel<1>, grid, dim3(256), 0, st, d, w, iw.q, n, nrhs, r0, jps, iw.part);
  }
  return hipGetLastError();
}

// y = M x for nrhs vectors (x, y: [nrhs][n]; y may not alias x)
hipError_t launch_matvec(const DipoleView& d, const Wave& w, const IterWork& iw, int64_t n, int64_t nrhs,
                         const double2* x, double2* y, hipStream_t st) {
  hipError_t e = launch_apply_alpha(d, x, n, iw.q, n, nrhs, st);
  if (e != hipSuccess) return e;
  if ((e = launch_coupling(d, w, iw, n, nrhs, st)) != hipSuccess) return e;
  const int64_t count = nrhs * n;
  hipLaunchKernelGGL(coupling_finish_kernel, dim3(nblocks(count)), dim3(256), 0, st, iw.part, iw.nsplit, count, x,
                     iw.q, d.self_c, 3 * d.nc, n, y, count);
  return hipGetLastError();
}

hipError_t launch_precond_apply(const DipoleView& d, const IterWork& iw, int64_t n, int64_t nrhs, const double2* v,
                                double2* z, hipStream_t st) {
  hipLaunchKernelGGL(precond_apply_kernel, dim3((unsigned)iw.nblk, (unsigned)nrhs), dim3(64), 0, st, d, iw.inv, n, v,
                     z);
  return hipGetLastError();
}

size_t gmres_host_bytes(int64_t nrhs, int restart) {
  return (size_t)nrhs * (2 * (restart + 1) * sizeof(double2) + sizeof(double));
}

hipError_t gmres_solve(const DipoleView& d, const Wave& w, const IterWork& iw, int64_t n, int64_t nrhs,
                       const double2* B, double2* X, double tol, int max_iter, int restart, hipStream_t st,
                       GmresStats& gs, void* host, Prof* prof) {
  typedef std::complex<double> cd;
  hipError_t e;
#define GCHK(x)                        \
  do {                                 \
    if ((e = (x)) != hipSuccess) return e; \
  } while (0)
  const int64_t vs = nrhs * n;
  const int64_t count = vs;
  const int m = restart;
  gs = GmresStats{};
  GCHK(launch_precond_build(d, w, iw, st));
  hipLaunchKernelGGL(zero_kernel, dim3(nblocks(count)), dim3(256), 0, st, X, count);
  // scalar results, which the kernels write to host memory: products of both
  // passes [2][nrhs][m + 1], then norms [nrhs]
  const double2* const hh = static_cast<const double2*>(host);
  double2* const hdev = static_cast<double2*>(host);
  const int64_t hs = nrhs * (m + 1);
  const double* const hn = reinterpret_cast<const double*>(hh + 2 * hs);
  double* const ndev = reinterpret_cast<double*>(hdev + 2 * hs);
  struct Event {
    hipEvent_t e = nullptr;
    ~Event() {
      if (e) (void)hipEventDestroy(e);
    }
  } ready;
  GCHK(hipEventCreateWithFlags(&ready.e, hipEventDisableTiming));
  const dim3 agrid((unsigned)iw.C, (unsigned)nrhs);
  auto scale_precond = [&](double2* v) -> hipError_t {  // v / ||v||, z, q; the norm to the host
    hipLaunchKernelGGL(scale_precond_kernel, dim3((unsigned)iw.nblk, (unsigned)nrhs), dim3(64), 0, st, d, iw.inv, n, iw.np,
                       iw.C, v, iw.z, iw.q, ndev);
    hipError_t r = hipGetLastError();
    return r != hipSuccess ? r : hipEventRecord(ready.e, st);
  };
  auto coupling = [&]() -> hipError_t {
    hipError_t r;
    if (prof && (r = prof->begin(st, PROF_ITER_MATVEC, (double)d.N * (double)d.N * (double)nrhs)) != hipSuccess) return r;
    if ((r = launch_coupling(d, w, iw, n, nrhs, st)) != hipSuccess) return r;
    return prof ? prof->end(st) : hipSuccess;
  };
  std::vector<double> bn(nrhs), rn(nrhs);
  std::vector<std::vector<cd>> H(nrhs), G(nrhs);
  std::vector<std::vector<cd>> cs(nrhs), sn(nrhs);
  std::vector<double> relres(nrhs, 1.0);
  bool first = true;
  while (true) {
    // r = b - M x (x = 0 at the start: r = b), V_0 = r / ||r||
    double2* V0 = iw.V;
    if (!first) {
      if (prof) GCHK(prof->begin(st, PROF_ITER_MATVEC, (double)d.N * (double)d.N * (double)nrhs));
      GCHK(launch_matvec(d, w, iw, n, nrhs, X, iw.t, st));
      if (prof) GCHK(prof->end(st));
    }
    hipLaunchKernelGGL(residual_kernel, agrid, dim3(AR_T), 0, st, B, first ? nullptr : iw.t, V0, n, iw.E, iw.C, iw.np);
    GCHK(scale_precond(V0));
    GCHK(hipEventSynchronize(ready.e));
    std::copy(hn, hn + nrhs, rn.begin());
    if (first) bn = rn;
    first = false;
    bool done = true;
    for (int64_t r = 0; r < nrhs; ++r) {
      relres[r] = bn[r] > 0 ? rn[r] / bn[r] : 0.0;
      done = done && relres[r] <= tol;
    }
    gs.relres = *std::max_element(relres.begin(), relres.end());
    if (done || gs.iters >= max_iter) break;
    for (int64_t r = 0; r < nrhs; ++r) {
      H[r].assign((size_t)(m + 1) * m, cd(0, 0));
      G[r].assign(m + 1, cd(0, 0));
      G[r][0] = cd(rn[r], 0);
      cs[r].assign(m, cd(0, 0));
      sn[r].assign(m, cd(0, 0));
    }
    GCHK(coupling());
    int jdone = 0;
    double res_prev = gs.relres, res_now = gs.relres;  // largest residual after the last two steps
    for (int j = 0; j < m && gs.iters < max_iter; ++j) {
      // W = M P V_j; classical Gram-Schmidt, twice: h = V^H W, W -= V h
      ArnoldiArgs A;
      A.V = iw.V;
      A.W = iw.V + (j + 1) * vs;
      A.vs = vs;
      A.n = n;
      A.m1 = m + 1;
      A.j1 = j + 1;
      A.E = iw.E;
      A.C = iw.C;
      A.hin = nullptr;
      A.hout = iw.hp;
      A.np = iw.np;
      A.host = nullptr;
      A.part = iw.part;
      A.x = iw.z;
      A.q = iw.q;
      A.nsplit = iw.nsplit;
      A.stride = count;
      A.ncell3 = 3 * d.nc;
      A.self_c = d.self_c;
      const size_t lds = sizeof(double2) * (size_t)(iw.E + AR_G * 128 + j + 1);
      hipLaunchKernelGGL(arnoldi_kernel<AR_PRODUCT>, agrid, dim3(AR_T), lds, st, A);
      A.hin = iw.hp;
      A.hout = iw.hp + hs * iw.C;
      A.host = hdev;
      hipLaunchKernelGGL(arnoldi_kernel<AR_AGAIN>, agrid, dim3(AR_T), lds, st, A);
      A.hin = A.hout;
      A.hout = nullptr;
      A.host = hdev + hs;
      hipLaunchKernelGGL(arnoldi_kernel<AR_NORM>, agrid, dim3(AR_T), lds, st, A);
      GCHK(scale_precond(A.W));
      // the next product starts while the host works on this step, unless the
      // residual, falling as in the last step, would then have converged
      const bool more = j + 1 < m && gs.iters + 1 < max_iter;
      const bool ahead = more && res_now * res_now > 0.5 * tol * res_prev;
      if (ahead) GCHK(coupling());
      GCHK(hipEventSynchronize(ready.e));
      ++gs.iters;
      jdone = j + 1;
      bool all = true;
      double res = 0.0;
      for (int64_t r = 0; r < nrhs; ++r) {
        // Hessenberg column j: h of both passes, then ||W||
        std::vector<cd> col(j + 2);
        for (int i = 0; i <= j; ++i) {
          const double2 h1 = hh[r * (m + 1) + i], h2 = hh[hs + r * (m + 1) + i];
          col[i] = cd(h1.x + h2.x, h1.y + h2.y);
        }
        col[j + 1] = cd(hn[r], 0);
        // earlier rotations
        for (int i = 0; i < j; ++i) {
          const cd t0 = cs[r][i] * col[i] + sn[r][i] * col[i + 1];
          const cd t1 = -std::conj(sn[r][i]) * col[i] + std::conj(cs[r][i]) * col[i + 1];
          col[i] = t0;
          col[i + 1] = t1;
        }
        // new rotation zeroing col[j + 1]
        const double a = std::abs(col[j]), bb = std::abs(col[j + 1]);
        if (bb == 0.0) {
          cs[r][j] = cd(1, 0);
          sn[r][j] = cd(0, 0);
        } else {
          const double den = std::hypot(a, bb);
          const cd ph = a > 0 ? col[j] / a : cd(1, 0);
          cs[r][j] = cd(a / den, 0);
          sn[r][j] = ph * std::conj(col[j + 1]) / den;
          col[j] = ph * den;
          col[j + 1] = cd(0, 0);
        }
        for (int i = 0; i <= j; ++i) H[r][(size_t)i * m + j] = col[i];
        const cd g0 = G[r][j];
        G[r][j] = cs[r][j] * g0;
        G[r][j + 1] = -std::conj(sn[r][j]) * g0;
        relres[r] = bn[r] > 0 ? std::abs(G[r][j + 1]) / bn[r] : 0.0;
        res = std::max(res, relres[r]);
        all = all && relres[r] <= 0.5 * tol;
      }
      if (all) break;
      res_prev = res_now;
      res_now = res;
      if (more && !ahead) GCHK(coupling());
    }
    // y = H^-1 g (upper triangular, jdone x jdone), then x += P V y
    std::vector<double2> yh((size_t)(m + 1) * nrhs, make_double2(0, 0));
    for (int64_t r = 0; r < nrhs; ++r) {
      std::vector<cd> y(jdone);
      for (int i = jdone - 1; i >= 0; --i) {
        cd s = G[r][i];
        for (int k = i + 1; k < jdone; ++k) s -= H[r][(size_t)i * m + k] * y[k];
        const cd hd = H[r][(size_t)i * m + i];
        y[i] = hd != cd(0, 0) ? s / hd : cd(0, 0);
      }
      for (int i = 0; i < jdone; ++i) yh[(size_t)i * nrhs + r] = make_double2(y[i].real(), y[i].imag());
    }
    GCHK(hipMemcpyAsync(iw.y, yh.data(), sizeof(double2) * (size_t)jdone * nrhs, hipMemcpyHostToDevice, st));
    hipLaunchKernelGGL(mcomb_kernel, dim3(nblocks(count)), dim3(256), 0, st, iw.V, vs, iw.y, jdone, 1.0, 0.0, iw.t, n,
                       (int)nrhs);
    GCHK(launch_precond_apply(d, iw, n, nrhs, iw.t, iw.z, st));
    hipLaunchKernelGGL(add_kernel, dim3(nblocks(count)), dim3(256), 0, st, X, iw.z, count);
    GCHK(hipGetLastError());
    ++gs.cycles;
  }
  return hipGetLastError();
#undef GCHK
}

}  // namespace gdm
