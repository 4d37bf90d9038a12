// Triangular block operations of the blocked LU (arXiv:2505.09545, Sec.
// "Numerical solution") on 16 x 16 matrix-core tiles:
//   diag_lu_kernel    the w x w diagonal block (w <= 128) of a speculative
//                     panel, factored without interchanges, and the inverses of
//                     its 16 x 16 diagonal triangles;
//   tile_inv_kernel   those inverses alone, for a block factored by a
//                     pivoting panel;
//   tri_rows_kernel   X U11 = B (rows below or above the block; with the pivot
//                     check of the speculative panel) and X L11 = B;
//   tri_panel_kernel  L21 U11 = A21 and L11 U12 = A12 in one launch;
//   diag_finish_kernel  the solve-ready form of the diagonal blocks.
//
// Every triangular solve is a blocked substitution over tiles, X_s = (B_s -
// sum_k X_k U_ks) U_ss^-1, one wave per 16 rows (or columns) of B.  A lane's
// results of a 16 x 16 x 4 MFMA are the k values it has to supply as the next
// product's second operand when the k index of step q is taken as rof(q) below,
// so X stays in registers over the whole block: no LDS, no barrier, in place,
// and the 128-wide inverses (whose 128-step substitution took 30 us per block)
// and the operand copies of the products with them are not needed.  L21 of a
// block with few rows takes 13 us in FP32 and 28 us in FP64, where inverse, copy,
// product and check took 50 and 70.
#include "gdm_common.hpp"
#include "gdm_kernels.hpp"
#include "lu_common.hpp"

namespace gdm {

namespace {

// Tile row (0..15) of accumulator register q in lane group lk = lane / 16: the
// FP32 MFMA returns rows 4 lk + q, the FP64 one rows lk + 4 q.
template <typename T> __device__ inline int rof(int lk, int q) { return sizeof(T) == 8 ? lk + 4 * q : 4 * lk + q; }

// A 16 x 16 complex tile as accumulators: register q holds (row rof(q), column lane % 16).
template <typename T> struct Tile {
  typename acc_of<T>::type re, im;
};
// A first operand: register q holds (row lane % 16, k = rof(q)).
template <typename T> struct Frag {
  T re[4], im[4];
};

template <typename T> __device__ inline Tile<T> tile_zero() {
  Tile<T> t;
  t.re = typename acc_of<T>::type{0, 0, 0, 0};
  t.im = typename acc_of<T>::type{0, 0, 0, 0};
  return t;
}

// acc += F X, X a tile as it was accumulated (k = rof(q) in register q)
template <typename T> __device__ inline void tile_mac(Tile<T>& acc, const Frag<T>& f, const Tile<T>& x) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    acc.re = mfma16(f.re[q], x.re[q], acc.re);
    acc.im = mfma16(f.re[q], x.im[q], acc.im);
    acc.re = mfma16(-f.im[q], x.im[q], acc.re);
    acc.im = mfma16(f.im[q], x.re[q], acc.im);
  }
}

// Number of 16-wide tiles of a block of width w.
__device__ inline int tiles_of(int w) { return (w + 15) >> 4; }

// The element at byte offset `off` (of this lane) from a uniform base.
template <typename CT> __device__ inline CT& at_off(const CT* base, uint32_t off) {
  return *reinterpret_cast<CT*>(reinterpret_cast<char*>(const_cast<CT*>(base)) + off);
}

// First operands out of the diagonal block D: TR false: row lane % 16 of the
// tile, k along its columns (L_sk); true: the transposed tile, row = tile
// column, k along the rows (U_ks^T, L_ks^T).  Addresses are a uniform part
// (tile, q) and one 32-bit lane offset for all tiles.  FULL: the block is a
// whole number of tiles, else entries past w read as zero.
template <typename T, bool TR, bool FULL> struct BlockFrags {
  using CT = cplx<T>;
  static constexpr int QS = sizeof(T) == 8 ? 4 : 1;  // step of rof in q
  const CT* D;
  int64_t ld;
  int w, lr, lk;
  uint32_t off;
  __device__ BlockFrags(const CT* D_, int64_t ld_, int w_, int lr_, int lk_) : D(D_), ld(ld_), w(w_), lr(lr_), lk(lk_) {
    const int64_t o = TR ? rof<T>(lk, 0) + lr * ld : lr + rof<T>(lk, 0) * ld;
    off = (uint32_t)(o * (int64_t)sizeof(CT));
  }
  __device__ Frag<T> tile(int tr, int tc) const {
    Frag<T> f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const CT* base = D + 16 * tr + 16 * (int64_t)tc * ld + (TR ? q * QS : q * QS * ld);
      CT v;
      if (FULL) {
        v = at_off(base, off);
      } else {
        const int r = 16 * tr + (TR ? rof<T>(lk, q) : lr), c = 16 * tc + (TR ? lr : rof<T>(lk, q));
        v.x = 0;
        v.y = 0;
        if (r < w && c < w) v = at_off(base, off);
      }
      f.re[q] = v.x;
      f.im[q] = v.y;
    }
    return f;
  }
};

// Tile inverses of a block: tiles_of(nb) column-major 16 x 16 inverses of L_ss,
// then as many of U_ss (tinv_block_elems complex per block).
template <typename T, bool TR>
__device__ inline Frag<T> load_inv(const cplx<T>* __restrict__ ti, int s, int lr, int lk) {
  constexpr int QS = sizeof(T) == 8 ? 4 : 1;
  const uint32_t off = (uint32_t)((TR ? rof<T>(lk, 0) + 16 * lr : lr + 16 * rof<T>(lk, 0)) * sizeof(cplx<T>));
  Frag<T> f;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const cplx<T> v = at_off(ti + s * 256 + (TR ? q * QS : 16 * q * QS), off);
    f.re[q] = v.x;
    f.im[q] = v.y;
  }
  return f;
}

// Rows (columns) r0 .. r0 + 15 into the split planes of the trailing update
// (update_split.hip), k = 16 NT of each in tiles x: scaled so that the largest
// |re|, |im| of a row lies in [2^13, 2^14), then h + l with both rounded to f16;
// fragments [r / 32][k / 16][plane] of 64 lanes x 8 f16, lane = r % 32 + 32 (k %
// 16 / 8); the row's inverse scale to scales[r].  Every lane of the wave calls it.
template <int NT>
__device__ inline void put_planes(unsigned char* planes, float* scales, const Tile<float> (&x)[NT], int64_t r0, bool rv,
                                  int lr, int lk) {
  float big = 0.f;
  static_for<NT>([&](auto s) {
#pragma unroll
    for (int q = 0; q < 4; ++q) big = fmaxf(big, fmaxf(fabsf(x[s].re[q]), fabsf(x[s].im[q])));
  });
  big = fmaxf(big, __shfl_xor(big, 16));
  big = fmaxf(big, __shfl_xor(big, 32));
  int ex = 14 - __builtin_amdgcn_frexp_expf(big);
  // the scale and its inverse are both normal numbers
  ex = big > 0.f ? min(max(ex, -113), 126) : 0;
  const float sc = ldexpf(1.f, ex);
  if (!rv) return;
  if (lk == 0) scales[r0 + lr] = ldexpf(1.f, -ex);
  unsigned char* f = planes + (r0 >> 5) * NT * 4096 + ((int)(r0 & 16) + lr + 32 * (lk >> 1)) * 16 + 8 * (lk & 1);
  typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
  static_for<NT>([&](auto s) {
    f16x4 p[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float a = x[s].re[q] * sc, b = x[s].im[q] * sc;
      p[0][q] = (_Float16)a;
      p[1][q] = (_Float16)(a - (float)p[0][q]);
      p[2][q] = (_Float16)b;
      p[3][q] = (_Float16)(b - (float)p[2][q]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<f16x4*>(f + 4096 * s + 1024 * i) = p[i];
  });
}

// One wave's blocked substitution on 16 rows (RIGHT) or columns of X, in place.
enum { TRI_RIGHT_UPPER = 0, TRI_LEFT_LOWER = 1, TRI_RIGHT_LOWER = 2 };

// NT: number of tiles of the block.  CHECK (TRI_RIGHT_UPPER): returns whether an
// entry fails |l u_jj| <= |u_jj|.  planes (FP32, may be null): X also goes there
// split, as the trailing update reads it.
template <typename T, int KIND, int NT, bool FULL, bool CHECK>
__device__ inline bool tri_wave(const cplx<T>* __restrict__ D, int64_t ld, int w, const cplx<T>* __restrict__ linv,
                                const cplx<T>* __restrict__ uinv, cplx<T>* __restrict__ X, int64_t ldx, int64_t r0,
                                int64_t cnt, unsigned char* planes, float* scales) {
  using CT = cplx<T>;
  constexpr bool TR = KIND != TRI_LEFT_LOWER;
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  const bool rv = r0 + lr < cnt;
  // lanes past the end work on the last row (not stored)
  const int64_t r = rv ? r0 + lr : cnt - 1;
  const CT* ti = KIND == TRI_RIGHT_UPPER ? uinv : linv;
  constexpr int QS = sizeof(T) == 8 ? 4 : 1;
  X += KIND == TRI_LEFT_LOWER ? r0 * ldx : r0;  // uniform
  const int64_t lane_o = KIND == TRI_LEFT_LOWER ? rof<T>(lk, 0) + (r - r0) * ldx : (r - r0) + rof<T>(lk, 0) * ldx;
  const uint32_t xoff = (uint32_t)(lane_o * (int64_t)sizeof(CT));
  auto at = [&](int s, int q) -> CT& {
    const int c = 16 * s + QS * q;
    return at_off<CT>(KIND == TRI_LEFT_LOWER ? X + c : X + c * ldx, xoff);
  };
  const BlockFrags<T, TR, FULL> bf(D, ld, w, lr, lk);
  auto frag = [&](int s, int k) { return TR ? bf.tile(k, s) : bf.tile(s, k); };
  Tile<T> x[NT];
  static_for<NT>([&](auto s) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      CT v;
      v.x = 0;
      v.y = 0;
      if (FULL || 16 * s + rof<T>(lk, q) < w) v = at(s, q);
      x[s].re[q] = v.x;
      x[s].im[q] = v.y;
    }
  });
  bool bad = false;
  // tile of step i: ascending, TRI_RIGHT_LOWER descending
  auto tl = [](int i) { return KIND == TRI_RIGHT_LOWER ? NT - 1 - i : i; };
  // (tiles past w have no inverse: nothing is read there, and zeros keep them out of
  // the tiles that TRI_RIGHT_LOWER takes after them)
  auto tile_inv = [&](int s) {
    Frag<T> f;
    if (FULL || 16 * s < w) return load_inv<T, TR>(ti, s, lr, lk);
#pragma unroll
    for (int q = 0; q < 4; ++q) f.re[q] = f.im[q] = 0;
    return f;
  };
  constexpr int PRE = sizeof(T) == 8 ? 1 : 2;
  Frag<T> pre[PRE];  // operands of the next step's first products, loaded a step ahead
  Frag<T> inv = tile_inv(tl(0));
  static_for<NT>([&](auto step) {
    constexpr int S = decltype(step)::value;
    const int s = tl(S);
    CT d[4];
    if constexpr (CHECK) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = 16 * s + rof<T>(lk, q);
        d[q] = D[FULL || c < w ? c + (int64_t)c * ld : 0];
      }
    }
    Tile<T> acc = tile_zero<T>();
    static_for<S>([&](auto p) {
      constexpr int P = decltype(p)::value;
      if constexpr (P < PRE) tile_mac<T>(acc, pre[P], x[tl(P)]);
      else tile_mac<T>(acc, frag(s, tl(P)), x[tl(P)]);
    });
    Tile<T> b;
    b.re = x[s].re - acc.re;
    b.im = x[s].im - acc.im;
    Tile<T> y = tile_zero<T>();
    const Frag<T> iv = inv;
    if constexpr (S + 1 < NT) {
      inv = tile_inv(tl(S + 1));
      static_for<(S + 1 < PRE ? S + 1 : PRE)>([&](auto p) { pre[p] = frag(tl(S + 1), tl(p)); });
    }
    tile_mac<T>(y, iv, b);
    x[s] = y;
    if constexpr (CHECK) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        CT l;
        l.x = y.re[q];
        l.y = y.im[q];
        if ((FULL || 16 * s + rof<T>(lk, q) < w) && !(cabs1_f(cmul_t(l, d[q])) <= cabs1_f(d[q]))) bad = true;
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      CT v;
      v.x = y.re[q];
      v.y = y.im[q];
      if (rv && (FULL || 16 * s + rof<T>(lk, q) < w)) at(s, q) = v;
    }
    __builtin_amdgcn_sched_barrier(0);  // operands of a later step are not hoisted past here (registers)
  });
  if constexpr (sizeof(T) == 4 && FULL && KIND != TRI_RIGHT_LOWER)
    if (planes) put_planes<NT>(planes, scales, x, r0, rv, lr, lk);
  return CHECK && bad && rv;
}

// A block of any width: blocks of 128 or 64 columns unrolled without
// masks, else the smallest masked form that holds it (no planes: split updates
// follow whole blocks of 128 or 64 only).
template <typename T, int KIND, bool CHECK>
__device__ inline bool tri_wave_any(const cplx<T>* __restrict__ D, int64_t ld, int w, const cplx<T>* __restrict__ linv,
                                    const cplx<T>* __restrict__ uinv, cplx<T>* __restrict__ X, int64_t ldx, int64_t r0,
                                    int64_t cnt, unsigned char* planes = nullptr, float* scales = nullptr) {
  if (w == 128) return tri_wave<T, KIND, 8, true, CHECK>(D, ld, w, linv, uinv, X, ldx, r0, cnt, planes, scales);
  if (w == 64) return tri_wave<T, KIND, 4, true, CHECK>(D, ld, w, linv, uinv, X, ldx, r0, cnt, planes, scales);
  if (w <= 64) return tri_wave<T, KIND, 4, false, CHECK>(D, ld, w, linv, uinv, X, ldx, r0, cnt, nullptr, nullptr);
  return tri_wave<T, KIND, 8, false, CHECK>(D, ld, w, linv, uinv, X, ldx, r0, cnt, nullptr, nullptr);
}

__device__ inline float lane_of(float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); }
__device__ inline double lane_of(double v, int l) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
template <typename CT> __device__ inline CT lane_of_c(const CT& v, int l) {
  CT r;
  r.x = lane_of(v.x, l);
  r.y = lane_of(v.y, l);
  return r;
}

}  // namespace

// 1 / p of a pivot from one reciprocal of |p|^2 (Newton steps on the hardware's
// approximation, to about an ulp).  bits collects the largest exponent-field
// pattern of the reciprocals, from the smallest normal one on: a zero, NaN,
// overflowing or underflowing |p|^2 brings it to 0x7e000000 or more, and the
// speculative factorisation is repeated with the pivot search, whose reciprocals
// are scaled.
__device__ inline float2 pivot_inv(float2 p, uint32_t& bits) {
  const float d = fmaf(p.x, p.x, p.y * p.y);
  float r = __builtin_amdgcn_rcpf(d);
  r = fmaf(fmaf(-d, r, 1.f), r, r);
  bits = max(bits, __float_as_uint(r) - 0x00800000u);
  return make_float2(p.x * r, -p.y * r);
}
__device__ inline double2 pivot_inv(double2 p, uint32_t& bits) {
  const double d = fma(p.x, p.x, p.y * p.y);
  double r = __builtin_amdgcn_rcp(d);
  r = fma(fma(-d, r, 1.0), r, r);
  r = fma(fma(-d, r, 1.0), r, r);
  bits = max(bits, (uint32_t)(__double_as_longlong(r) >> 32) - 0x00800000u);
  return make_double2(p.x * r, -p.y * r);
}

// LDS of diag_lu_kernel, in complex: the column panel of two steps (128 rows of
// 16, stride 17), then 16 x 16 tiles (stride 17): the diagonal tile before and
// after its factorisation, an identity, and the inverses of two steps.
constexpr int DLU_S = 17, DLU_PANEL = 128 * DLU_S, DLU_TILE = 16 * DLU_S;
size_t diag_lu_lds_bytes(int elem_bytes) { return (size_t)(2 * DLU_PANEL + 7 * DLU_TILE) * 2 * elem_bytes; }

// The diagonal block of a speculative panel: 8 waves, wave c holding the 8
// tiles of tile column c as accumulators.  Per 16-wide step s:
//   the owner puts the diagonal tile into LDS; wave 0 factors it with one row
//   per lane (16 elimination steps in registers, the pivot row broadcast by
//   readlane, rows of the identity in lanes 16-31 turning into U_ss^-1) and
//   wave 1 the same by columns (giving L_ss^-1), while the other waves apply
//   the rest of the previous step's update;
//   wave j > s forms L_js = A_js U_ss^-1 (from LDS, back to LDS) and U_sj =
//   L_ss^-1 A_sj (its own registers), then updates the next diagonal tile first.
// What bounds it is the chain of 128 pivots (reciprocal, broadcast, update:
// 16 to 18 dependent operations each) on one wave; the matrix-core work beside
// it takes less.  One 128 x 128 block alone: 51 us in FP32 and 87 us in FP64
// (one workgroup with rank-1 updates of the whole block on its vector units and
// a barrier per column took 139-165 and 190-220).  The entries below each pivot are checked as the speculative
// panel requires: in the tile by wave 0, below it here as |l u| <= |u|.
// Columns and rows past w are an identity block; ipiv = identity.
template <typename T>
__global__ void __launch_bounds__(512) diag_lu_kernel(cplx<T>* __restrict__ A, int64_t ld, int64_t k0, int w,
                                                      int32_t* __restrict__ ipiv, int32_t* __restrict__ flag,
                                                      cplx<T>* __restrict__ tinv, int uoff, int64_t sA, int64_t sipiv,
                                                      int64_t sflag, int64_t stinv) {
  using CT = cplx<T>;
  extern __shared__ __align__(16) unsigned char dlu_smem[];
  CT* const lds = reinterpret_cast<CT*>(dlu_smem);
  CT* const Dg = lds + 2 * DLU_PANEL;  // tiles as [row][column]
  CT* const Do = Dg + DLU_TILE;
  CT* const Id = Do + DLU_TILE;
  CT* const Inv = Id + DLU_TILE;  // L_ss^-1, U_ss^-1 of even steps, then of odd ones
  A += (int64_t)blockIdx.y * sA;  // batch item blockIdx.y
  ipiv += (int64_t)blockIdx.y * sipiv;
  flag += (int64_t)blockIdx.y * sflag;
  tinv += (int64_t)blockIdx.y * stinv;
  __builtin_amdgcn_s_setprio(3);  // a serial chain beside throughput kernels
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lk = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nt = tiles_of(w);
  const bool full = w == 16 * nt;
  CT* D = A + k0 + k0 * ld;
  constexpr int QS = sizeof(T) == 8 ? 4 : 1;
  const uint32_t doff = (uint32_t)((rof<T>(lk, 0) + lr * ld) * (int64_t)sizeof(CT));
  const int toff = rof<T>(lk, 0) * DLU_S + lr;  // LDS tiles: register q at toff + q QS DLU_S
  const int foff = lr * DLU_S + rof<T>(lk, 0);  // the same tile as first operand: + q QS
  Tile<T> a[8];
  static_for<8>([&](auto i) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = 16 * i + rof<T>(lk, q), c = 16 * wv + lr;
      CT v;
      v.x = r == c ? 1 : 0;
      v.y = 0;
      if (r < w && c < w) v = at_off(D + 16 * i + QS * q + 16 * wv * ld, doff);
      a[i].re[q] = v.x;
      a[i].im[q] = v.y;
    }
  });
  auto put = [&](CT* t, const Tile<T>& x) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      CT v;
      v.x = x.re[q];
      v.y = x.im[q];
      t[toff + q * QS * DLU_S] = v;
    }
  };
  auto get = [&](const CT* t) {
    Tile<T> x;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const CT v = t[toff + q * QS * DLU_S];
      x.re[q] = v.x;
      x.im[q] = v.y;
    }
    return x;
  };
  auto frag = [&](const CT* t, T sign) {
    Frag<T> f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const CT v = t[foff + q * QS];
      f.re[q] = sign * v.x;
      f.im[q] = sign * v.y;
    }
    return f;
  };
  // tile (ti, tj) of the block to memory
  auto store = [&](const Tile<T>& x, int ti, int tj) {
    CT* base = D + 16 * ti + 16 * tj * ld;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      CT v;
      v.x = x.re[q];
      v.y = x.im[q];
      if (full || (16 * ti + rof<T>(lk, q) < w && 16 * tj + lr < w)) at_off(base + QS * q, doff) = v;
    }
  };
  if (tid < 256) {
    CT v;
    v.x = (tid & 15) == (tid >> 4) ? 1 : 0;
    v.y = 0;
    Id[(tid >> 4) * DLU_S + (tid & 15)] = v;
  }
  int bad = 0;
  uint32_t idbits = 0;
  Tile<T> u = tile_zero<T>();  // U_s,wv of the last step
  // wave wv's tiles of step s to memory, with the check of L_wv,s (its entries
  // times their column's pivot, U_ss[c][c] = 1 / U_ss^-1[c][c], against it):
  // left to the next step's chain, which the other waves wait for
  auto settle = [&](int s, const CT* Lq) {
    const CT ud = cinv_t(Inv[(2 * (s & 1) + 1) * DLU_TILE + lr * DLU_S + lr]);
    const float pk = cabs1_f(ud);
    const Tile<T> l = get(Lq + 16 * wv * DLU_S);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      CT v;
      v.x = l.re[q];
      v.y = l.im[q];
      bad |= (int)!(cabs1_f(cmul_t(v, ud)) <= pk);
    }
    store(l, wv, s);
    store(u, s, wv);
  };
  for (int s = 0; s < nt; ++s) {
    CT* const Lp = lds + (s & 1) * DLU_PANEL;
    CT* const Li = Inv + 2 * (s & 1) * DLU_TILE;
    CT* const Ui = Li + DLU_TILE;
    const CT* const Lq = lds + (~s & 1) * DLU_PANEL;  // the previous step's column panel
    if (wv == s)
      static_for<8>([&](auto i) {
        if (i == s) {
          if (s > 0) tile_mac<T>(a[i], frag(Lq + 16 * i * DLU_S, -1), u);
          put(Dg, a[i]);
        }
      });
    __syncthreads();
    // lanes 0-15 of the panel waves: rows (columns) of the tile, 16-31 of the identity
    const int ln = lane & 31, li = ln & 15;
    if (wv == 0) {
      const CT* src = (ln < 16 ? Dg : Id) + li * DLU_S;
      CT x[16];
      static_for<16>([&](auto c) { x[c] = src[c]; });
      CT piv = lane_of_c(x[0], 0);
      CT inv = pivot_inv(piv, idbits);
      static_for<16>([&](auto j) {
        constexpr int J = decltype(j)::value;
        const bool below = __builtin_amdgcn_inverse_ballot_w64(~0ull << (J + 1));
        const bool diag = __builtin_amdgcn_inverse_ballot_w64((0xffffull << (J + 1)) & 0xffffull);
        // an entry below the pivot in the tile larger than it (bit patterns of
        // non-negative floats order as integers, NaN above all)
        const int over = __float_as_int(cabs1_f(x[J])) - __float_as_int(cabs1_f(piv));
        bad = max(bad, diag ? over : 0);
        asm volatile("" : "+v"(bad), "+v"(idbits));  // taken now, not collected for later
        CT l = cmul_t(x[J], inv);
        x[J].x = below ? l.x : x[J].x;
        x[J].y = below ? l.y : x[J].y;
        l.x = below ? l.x : 0;
        l.y = below ? l.y : 0;
        // all broadcasts before the first update (a scalar read right after its
        // readlane stalls the wave)
        CT uj[16];
        static_for<15 - J>([&](auto d) {
          constexpr int c = J + 1 + decltype(d)::value;
          uj[c] = lane_of_c(x[c], J);
        });
        __builtin_amdgcn_sched_barrier(0);
        static_for<15 - J>([&](auto d) {
          constexpr int c = J + 1 + decltype(d)::value;
          x[c] = r1_upd(x[c], l, uj[c]);
          // the next pivot's reciprocal beside the rest of this step's updates
          if constexpr (c == J + 1) {
            piv = lane_of_c(x[c], c);
            inv = pivot_inv(piv, idbits);
          }
        });
        __builtin_amdgcn_sched_barrier(0);  // one step's broadcasts in scalar registers at a time
      });
      CT* out = (ln < 16 ? Do : Ui) + li * DLU_S;
      if (lane < 32) static_for<16>([&](auto c) { out[c] = x[c]; });
    }
    if (wv == 1) {
      const CT* src = (ln < 16 ? Dg : Id) + li;
      CT x[16];
      static_for<16>([&](auto r) { x[r] = src[r * DLU_S]; });
      CT inv = pivot_inv(lane_of_c(x[0], 0), idbits);
      static_for<16>([&](auto j) {
        constexpr int J = decltype(j)::value;
        // x_r -= a_rj (u_j / piv) for the rows r below j of the tile's column j
        const CT uj = cmul_t(x[J], inv);
        CT lj[16];
        static_for<15 - J>([&](auto d) {
          constexpr int r = J + 1 + decltype(d)::value;
          lj[r] = lane_of_c(x[r], J);
        });
        __builtin_amdgcn_sched_barrier(0);
        static_for<15 - J>([&](auto d) {
          constexpr int r = J + 1 + decltype(d)::value;
          x[r] = r1_upd(x[r], uj, lj[r]);
          if constexpr (r == J + 1) inv = pivot_inv(lane_of_c(x[r], r), idbits);
        });
        __builtin_amdgcn_sched_barrier(0);
      });
      if (lane >= 16 && lane < 32) static_for<16>([&](auto r) { Li[r * DLU_S + li] = x[r]; });
    }
    // the rest of the previous step's update (its owner's diagonal tile is done),
    // then the owner of column s puts the tiles below the diagonal into LDS
    if (s > 0 && wv >= s && wv < nt) {
      settle(s - 1, Lq);
      static_for<8>([&](auto i) {
        if (i >= s && i < nt && !(i == s && wv == s)) tile_mac<T>(a[i], frag(Lq + 16 * i * DLU_S, -1), u);
      });
    }
    if (wv == s)
      static_for<8>([&](auto i) {
        if (i > s && i < nt) put(Lp + 16 * i * DLU_S, a[i]);
      });
    __syncthreads();
    if (wv == s) {  // the finished diagonal tile and the inverses to memory
      store(get(Do), s, s);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int e = 4 * lane + q, c = e >> 4, r = e & 15;  // column-major
        tinv[s * 256 + e] = Li[r * DLU_S + c];
        tinv[uoff + s * 256 + e] = Ui[r * DLU_S + c];
      }
    }
    if (wv > s && wv < nt) {
      Tile<T> l = tile_zero<T>();
      tile_mac<T>(l, frag(Lp + 16 * wv * DLU_S, 1), get(Ui));
      const Frag<T> lf = frag(Li, 1);
      u = tile_zero<T>();
      static_for<8>([&](auto i) {
        if (i == s) tile_mac<T>(u, lf, a[i]);
      });
      put(Lp + 16 * wv * DLU_S, l);
    }
    __syncthreads();
  }
  if (tid < w) ipiv[k0 + tid] = (int32_t)(k0 + tid);
  if (__syncthreads_or(bad > 0 || idbits >= 0x7e000000u) && tid == 0) atomicOr(flag, 1);
}

// The inverses of the 16 x 16 diagonal triangles of a factored block (pivoting
// panels): one wave per tile, lane c < 16 substitutes column c of the identity
// with the tile's L, lane 16 + r row r of the identity with its U.
template <typename T>
__global__ void __launch_bounds__(64) tile_inv_kernel(const cplx<T>* __restrict__ A, int64_t ld, int64_t k0, int w,
                                                      cplx<T>* __restrict__ tinv, int uoff, int64_t sA, int64_t stinv) {
  using CT = cplx<T>;
  A += (int64_t)blockIdx.y * sA;
  tinv += (int64_t)blockIdx.y * stinv;
  __shared__ CT t[16][17];
  const int lane = threadIdx.x, s = blockIdx.x;
  const CT* D = A + k0 + k0 * ld;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int r = lane & 15, c = (lane >> 4) + 4 * q;
    CT v;
    v.x = r == c ? 1 : 0;
    v.y = 0;
    if (16 * s + r < w && 16 * s + c < w) v = D[16 * s + r + (int64_t)(16 * s + c) * ld];
    t[r][c] = v;
  }
  __syncthreads();
  const int i = lane & 15;
  CT x[16];
  static_for<16>([&](auto c) {
    x[c].x = i == c ? 1 : 0;
    x[c].y = 0;
  });
  if (lane < 16) {
    static_for<16>([&](auto j) {
      static_for<15 - decltype(j)::value>([&](auto d) {
        constexpr int r = decltype(j)::value + 1 + decltype(d)::value;
        x[r] = r1_upd(x[r], t[r][j], x[j]);
      });
    });
    static_for<16>([&](auto r) { tinv[s * 256 + i * 16 + r] = x[r]; });
  } else if (lane < 32) {
    static_for<16>([&](auto j) {
      x[j] = cmul_t(x[j], cinv_t(t[j][j]));
      static_for<15 - decltype(j)::value>([&](auto d) {
        constexpr int c = decltype(j)::value + 1 + decltype(d)::value;
        x[c] = r1_upd(x[c], x[j], t[j][c]);
      });
    });
    static_for<16>([&](auto c) { tinv[uoff + s * 256 + c * 16 + i] = x[c]; });
  }
}

// L21 U11 = A21 (nrows rows below the block, with the pivot check) and L11 U12 =
// A12 (ncols columns from column cu on), either of them possibly empty: one
// wave per 16 rows or columns, the columns first.
template <typename T>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 3)))
tri_panel_kernel(cplx<T>* __restrict__ A, int64_t ld, int64_t k0, int w, int64_t nrows, int64_t cu, int64_t ncols,
                 int cblocks, const cplx<T>* __restrict__ tinv, int uoff, int32_t* __restrict__ flag,
                 SplitOut lout, SplitOut uout, int64_t sA, int64_t stinv, int64_t sflag, int64_t ssplit) {
  using CT = cplx<T>;
  A += (int64_t)blockIdx.y * sA;
  tinv += (int64_t)blockIdx.y * stinv;
  flag += (int64_t)blockIdx.y * sflag;
  const CT* D = A + k0 + k0 * ld;
  const int b = blockIdx.x;
  const int64_t po = (int64_t)blockIdx.y * ssplit;  // bytes per item
  if (b < cblocks) {
    tri_wave_any<T, TRI_LEFT_LOWER, false>(D, ld, w, tinv, tinv + uoff, A + k0 + cu * ld, ld, 16 * (int64_t)b, ncols,
                                           uout.planes ? uout.planes + po : nullptr, uout.scales + po / 4);
  } else {
    const bool bad = tri_wave_any<T, TRI_RIGHT_UPPER, true>(D, ld, w, tinv, tinv + uoff, A + (k0 + w) + k0 * ld, ld,
                                                            16 * (int64_t)(b - cblocks), nrows,
                                                            lout.planes ? lout.planes + po : nullptr,
                                                            lout.scales + po / 4);
    if (__ballot(bad) != 0 && threadIdx.x == 0) atomicOr(flag, 1);
  }
}

// The split planes of an L21 that a pivoting panel has formed (16 NT columns).
template <int NT>
__global__ void __launch_bounds__(64) split_rows_kernel(const float2* __restrict__ X, int64_t ld, int64_t nrows,
                                                        SplitOut out, int64_t sX, int64_t ssplit) {
  X += (int64_t)blockIdx.y * sX;
  const int64_t po = (int64_t)blockIdx.y * ssplit;
  const int lane = threadIdx.x, lr = lane & 15, lk = lane >> 4;
  const int64_t r0 = 16 * (int64_t)blockIdx.x;
  const bool rv = r0 + lr < nrows;
  X += rv ? r0 + lr : nrows - 1;
  Tile<float> x[NT];
  static_for<NT>([&](auto s) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float2 v = X[(int64_t)(16 * s + rof<float>(lk, q)) * ld];
      x[s].re[q] = v.x;
      x[s].im[q] = v.y;
    }
  });
  put_planes<NT>(out.planes + po, out.scales + po / 4, x, r0, rv, lr, lk);
}

// Solve-ready block columns, all blocks in one launch: rows above block
// blockIdx.y become U01 U11^-1, rows below it L21 L11^-1 (blockIdx.x: 16 rows of
// the block column without its diagonal block).
template <typename T>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 3)))
tri_rows_kernel(cplx<T>* __restrict__ A, int64_t ld, int64_t n, int nb,
                                                      const cplx<T>* __restrict__ tinv, int64_t btinv, int uoff,
                                                      int64_t sA, int64_t stinv) {
  using CT = cplx<T>;
  A += (int64_t)blockIdx.z * sA;
  const int64_t k0 = (int64_t)blockIdx.y * nb;
  const int w = (int)(n - k0 < nb ? n - k0 : nb);
  tinv += (int64_t)blockIdx.z * stinv + (int64_t)blockIdx.y * btinv;
  const CT* D = A + k0 + k0 * ld;
  CT* X = A + k0 * ld;
  const int64_t above = (k0 + 15) / 16, b = blockIdx.x;
  if (b < above) {
    tri_wave_any<T, TRI_RIGHT_UPPER, false>(D, ld, w, tinv, tinv + uoff, X, ld, 16 * b, k0);
  } else {
    const int64_t r0 = 16 * (b - above), cnt = n - k0 - w;
    if (r0 < cnt) tri_wave_any<T, TRI_RIGHT_LOWER, false>(D, ld, w, tinv, tinv + uoff, X + k0 + w, ld, r0, cnt);
  }
}

// Solve-ready diagonal blocks (after tri_rows_kernel, which reads the triangles):
// strict lower part I - L11^-1 (blockIdx.z even), upper part I - U11^-1 (odd).
// Wave j substitutes tile column j (L) or tile row j (U) of the identity; the
// block is written once every wave has read it.
template <typename T>
__global__ void __launch_bounds__(512) diag_finish_kernel(cplx<T>* __restrict__ A, int64_t ld, int64_t n, int nb,
                                                          const cplx<T>* __restrict__ tinv, int64_t btinv, int uoff,
                                                          int64_t sA, int64_t stinv) {
  using CT = cplx<T>;
  const int item = blockIdx.z >> 1;
  const bool upper = blockIdx.z & 1;
  A += (int64_t)item * sA;
  const int64_t k0 = (int64_t)blockIdx.x * nb;
  const int w = (int)(n - k0 < nb ? n - k0 : nb);
  tinv += (int64_t)item * stinv + (int64_t)blockIdx.x * btinv;
  CT* D = A + k0 + k0 * ld;
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = lane >> 4;
  const int j = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nt = tiles_of(w);
  Tile<T> x[8];
  static_for<8>([&](auto s) {
    if (s < j || s >= nt) return;
    Tile<T> acc = tile_zero<T>();
    static_for<decltype(s)::value>([&](auto k) {
      if (k < j) return;
      tile_mac<T>(acc, upper ? BlockFrags<T, true, false>(D, ld, w, lr, lk).tile(k, s)
                             : BlockFrags<T, false, false>(D, ld, w, lr, lk).tile(s, k),
                  x[k]);
    });
    Tile<T> b;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      b.re[q] = (s == j && rof<T>(lk, q) == lr ? 1 : 0) - acc.re[q];
      b.im[q] = -acc.im[q];
    }
    const Frag<T> inv = upper ? load_inv<T, true>(tinv + uoff, s, lr, lk) : load_inv<T, false>(tinv, s, lr, lk);
    x[s] = tile_zero<T>();
    tile_mac<T>(x[s], inv, b);
  });
  __syncthreads();
  static_for<8>([&](auto s) {
    if (s < j || s >= nt) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = 16 * s + rof<T>(lk, q), o = 16 * j + lr;  // along the substitution, and the identity's index
      const int r = upper ? o : i, c = upper ? i : o;
      if (r >= w || c >= w || (upper ? r > c : r <= c)) continue;
      CT v;
      v.x = (r == c ? 1 : 0) - x[s].re[q];
      v.y = -x[s].im[q];
      D[r + (int64_t)c * ld] = v;
    }
  });
}

// ---------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------
int64_t tinv_block_elems(int nb) { return (int64_t)((nb + 15) / 16) * 512; }
static int tinv_uoff(int nb) { return (nb + 15) / 16 * 256; }

template <typename T>
hipError_t prepare_diag_lu() {
  // more than the default 64 KB of LDS in FP64 (a host-side setting)
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&diag_lu_kernel<T>), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)diag_lu_lds_bytes(sizeof(T)));
}
template hipError_t prepare_diag_lu<double>();
template hipError_t prepare_diag_lu<float>();

template <typename T>
hipError_t launch_diag_lu(cplx<T>* A, int64_t ld, int nb, int64_t k0, int w, int32_t* ipiv, int32_t* flag,
                          cplx<T>* tinv, hipStream_t st, int nbatch, int64_t sA, int64_t sipiv, int64_t sflag,
                          int64_t stinv) {
  if (w < 1 || w > 128 || w > nb || ld > tiles_max_ld(sizeof(T))) return hipErrorInvalidValue;
  hipLaunchKernelGGL(diag_lu_kernel<T>, dim3(1, (unsigned)nbatch), dim3(512), diag_lu_lds_bytes(sizeof(T)), st, A, ld, k0,
                     w, ipiv, flag, tinv, tinv_uoff(nb), sA, sipiv, sflag, stinv);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_tile_inv(const cplx<T>* A, int64_t ld, int nb, int64_t k0, int w, cplx<T>* tinv, hipStream_t st,
                           int nbatch, int64_t sA, int64_t stinv) {
  if (w < 1 || w > 128 || w > nb) return hipErrorInvalidValue;
  hipLaunchKernelGGL(tile_inv_kernel<T>, dim3((unsigned)((w + 15) / 16), (unsigned)nbatch), dim3(64), 0, st, A, ld, k0, w,
                     tinv, tinv_uoff(nb), sA, stinv);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_tri_panel(cplx<T>* A, int64_t ld, int nb, int64_t k0, int w, int64_t nrows, int64_t cu, int64_t ncols,
                            const cplx<T>* tinv, int32_t* flag, hipStream_t st, int nbatch, int64_t sA, int64_t stinv,
                            int64_t sflag, SplitOut lout, SplitOut uout, int64_t ssplit) {
  const int64_t cb = (ncols + 15) / 16, rb = (nrows + 15) / 16;
  if (cb + rb <= 0) return hipSuccess;
  if (w < 1 || w > 128 || w > nb || cb + rb > INT32_MAX || ld > tiles_max_ld(sizeof(T))) return hipErrorInvalidValue;
  if ((lout.planes || uout.planes) && w != 128 && w != 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(tri_panel_kernel<T>, dim3((unsigned)(cb + rb), (unsigned)nbatch), dim3(64), 0, st, A, ld, k0, w,
                     nrows, cu, ncols, (int)cb, tinv, tinv_uoff(nb), flag, lout, uout, sA, stinv, sflag, ssplit);
  return hipGetLastError();
}

hipError_t launch_split_rows(const float2* X, int64_t ld, int64_t nrows, int w, SplitOut out, hipStream_t st, int nbatch,
                             int64_t sX, int64_t ssplit) {
  if (nrows <= 0) return hipSuccess;
  if ((w != 128 && w != 64) || (nrows + 15) / 16 > INT32_MAX) return hipErrorInvalidValue;
  const dim3 g((unsigned)((nrows + 15) / 16), (unsigned)nbatch);
  if (w == 128) hipLaunchKernelGGL(split_rows_kernel<8>, g, dim3(64), 0, st, X, ld, nrows, out, sX, ssplit);
  else hipLaunchKernelGGL(split_rows_kernel<4>, g, dim3(64), 0, st, X, ld, nrows, out, sX, ssplit);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_finish(cplx<T>* A, int64_t ld, int64_t n, int nb, const cplx<T>* tinv, hipStream_t st, int nbatch,
                         int64_t sA, int64_t stinv) {
  const int64_t nblk = (n + nb - 1) / nb;
  if (nblk > 65535 || 2 * (int64_t)nbatch > 65535 || ld > tiles_max_ld(sizeof(T))) return hipErrorInvalidValue;
  if (nblk > 1) {
    // rows of a block column outside its diagonal block, in 16s (at most one more than n / 16)
    hipLaunchKernelGGL(tri_rows_kernel<T>, dim3((unsigned)((n + 15) / 16 + 1), (unsigned)nblk, (unsigned)nbatch), dim3(64),
                       0, st, A, ld, n, nb, tinv, tinv_block_elems(nb), tinv_uoff(nb), sA, stinv);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(diag_finish_kernel<T>, dim3((unsigned)nblk, 1, (unsigned)(2 * nbatch)), dim3(512), 0, st, A, ld, n, nb,
                     tinv, tinv_block_elems(nb), tinv_uoff(nb), sA, stinv);
  return hipGetLastError();
}

#define GDM_TILES(T)                                                                                                    \
  template hipError_t launch_diag_lu<T>(cplx<T>*, int64_t, int, int64_t, int, int32_t*, int32_t*, cplx<T>*, hipStream_t, \
                                        int, int64_t, int64_t, int64_t, int64_t);                                      \
  template hipError_t launch_tile_inv<T>(const cplx<T>*, int64_t, int, int64_t, int, cplx<T>*, hipStream_t, int,       \
                                         int64_t, int64_t);                                                            \
  template hipError_t launch_tri_panel<T>(cplx<T>*, int64_t, int, int64_t, int, int64_t, int64_t, int64_t,             \
                                          const cplx<T>*, int32_t*, hipStream_t, int, int64_t, int64_t, int64_t,       \
                                          SplitOut, SplitOut, int64_t);                                                \
  template hipError_t launch_finish<T>(cplx<T>*, int64_t, int64_t, int, const cplx<T>*, hipStream_t, int, int64_t,     \
                                       int64_t);
GDM_TILES(double)
GDM_TILES(float)
#undef GDM_TILES

}  // namespace gdm
