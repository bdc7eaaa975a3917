// Screened-interaction elements from one reduction of the transition matrix
// (FP64).
//
// With V[P][ia] = 2 Delta_ia^1/2 M^P_ia and C = diag(Delta^2) + V^T V (the RPA
// matrix in its symmetric form, frequency independent), the Woodbury identity
// turns W^c_nm(z) = b^T [(1 - Pi(z))^-1 - 1] b into
//
//        W^c_nm(z) = u^T (z^2 - C)^-1 u,      u = V^T b_nm,
//
// so every frequency of a call is a shift of the same real symmetric matrix.
// C is brought once to block-tridiagonal form by an orthogonal transformation H
// that is applied to the rows of V as well (V H, from which u = (V H)^T b_nm);
// each W is then a banded complex symmetric elimination of order n_ov and
// half-bandwidth SB = 32 instead of an N_aux x N_aux Pi build (2 N^2 n_ov flops)
// and a factorisation (4/3 N^3): about 8 32^2 n_ov flops.  The reduction costs
// 4/3 n_ov^3 + 2 n_ov^2 N_aux flops, once a call.
//
// The reduction rounds C by eps |C|, of which the Delta^2 of the core levels are
// the largest, and a residue W lies within 2 x eta of the poles: by the
// elimination alone Sigma is off by up to 5e-13 and Im Sigma^dec by 4e-12 of
// their largest values (n_ov 175 and 1026), 25 to 160 times what the Pi builds
// give.  So W of a residue is taken from
//
//        W = w^T Pi w - y^T y,   w = b + y,   w^T Pi w = sum_ia (V^T w)_ia^2 / (z^2 - Delta_ia^2),
//
// which is b^T [(1 - Pi)^-1 - 1] b for y = (1 - Pi)^-1 b - b and stationary there
// (with 1 - Pi between y and its error twice): y = V x from the band's solution
// x = (z^2 - T)^-1 u has the reduction's error e, W its square.  Every Delta_ia
// enters by itself, as in a Pi build, and V is the untransformed one.  The band's
// own W, off by e to first order, tells how large e is.  On the imaginary axis
// nothing is near a pole and the elimination's W is as exact as the Pi builds'.
//
// Reduction (indices ordered by Delta; SB - n_ov % SB decoupled rows in front,
// with diagonal elements taken from the Delta^2, make the order a multiple of SB).
// It starts with a reflection that turns the first SB coordinates into SB
// pseudo-random directions: a band grown from single transitions runs out of
// directions in one irreducible block of a symmetric molecule before the others
// (at order 567 with two to eight blocks panel 6 to 14 of 16 is singular), random
// ones only where an eigenvalue is SB-fold (smallest pivot there 1e-5 of its
// diagonal element).  It costs one panel more, 1/32 of the reduction at order
// 1026.  Per panel P of SB columns with the m rows below its diagonal block, five
// dependent launches:
//   panel_q        Q = P L1^-T by rows, with G = P^T P = L1 L1^T from the launch
//                  before, and partial sums of G2 = Q^T Q = 1 + E;
//   panel_x        Xq = A22 Q (and u^T Q), the product that reads the matrix; one
//                  more workgroup meanwhile sums G2, orthonormalises Q1 =
//                  Q (1 - Phi) and reconstructs the Householder form of Q1:
//                  Phi = the upper triangle of E, its diagonal halved (1 - Phi
//                  inverts the Cholesky factor R2 = 1 + Phi of 1 + E to O(E^2);
//                  where |E| > 1e-8, as in a last square panel, it is factored);
//                  Q1_top - S = Y1 U without pivoting, S_jj = -sign, T = -U S
//                  Y1^-T, so that H = 1 - Y T Y^T with Y = (Q1 - [S; 0]) U^-1
//                  has H^T P = [S R2 L1^T; 0];
//   panel_xsum     Y = Q M2 - [SU; 0] and X = A22 Y = Xq M2 - A22[:, :SB] SU with
//                  M2 = (1 - Phi) U^-1, SU = S U^-1, Xq summed over its splits;
//                  Y^T X, and in the last workgroup E2 = T^T (Y^T X) T / 2;
//   panel_w        W = X T - Y E2;
//   panel_update   A22 -= Y W^T + W Y^T, u -= Y (u^T Y T)^T; the tiles that
//                  hold the next panel also form its G, and the last of them
//                  the Cholesky factor, while the others go on.
// Of the matrix only the 32 x 32 blocks on and above the diagonal are kept up to
// date; panels are read as rows, and panel_x takes A22's columns below the
// diagonal from its rows.  (With the mirrors written and read instead: update
// 84 -> 71 ms of a reduction of order 16524, panel_x 94 -> 87; 7.4 -> 6.0 ms and
// no change at 5859.)
// Panels go in pairs: after the first of a pair only the columns of the second
// (and u's rows beside them) are updated, the second takes what is missing of
// A22 in its products (A22 Y = A Y - Ya (Wa^T Y) - Wa (Ya^T Y)), and one update
// with both halves its passes over the matrix.
// Two Cholesky passes orthogonalise a panel of condition up to 3e6; beyond that
// (dependent columns) a flag is raised and the caller screens by Pi builds.
#include <algorithm>
#include <utility>

#include "gwc_internal.h"

namespace gwc {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef double d2 __attribute__((ext_vector_type(2)));

constexpr int SB = SPECTRAL_BAND;
constexpr int SLD = SB + 1;   // LDS row stride of 32-wide rows
constexpr int PROWS = 256;    // panel rows per workgroup of panel_gram
constexpr int XROWS = 128;    // rows per workgroup of panel_xsum
constexpr int XTHREADS = 1024;
constexpr int UT = 64;        // tile of the rank update and the transition matrix
constexpr int ULD = SB + 2;   // LDS row stride of its operands (no bank conflicts)
// Rows from which panels go in pairs: the second panel's own products cost about
// 40 us, half a pass over the matrix more than that from here on (a call of order
// 16524 in pairs down to 10240, 7168 and 3072 rows: 210.5, 208.1 and 209.0 ms;
// one of 5859 without pairs 22.5 ms, with pairs down to 3072 rows 23.5).
constexpr int PAIR_ROWS = 7168;
constexpr int Q_PART = 768, Q_PART2 = 768 + 2 * SB * SB;  // partial sums of panel_q

// 32 x 32 matrices and 32-vectors one panel step hands to the next.
struct PanelSmall {
  double R1[SB * SB], rd1[SB];    // L1^T, reciprocal diagonal
  double M2[SB * SB], SU[SB * SB];
  double T[SB * SB], E2[SB * SB];
  double V1[SB * SB], V2[SB * SB];  // Wa^T Y, Ya^T Y of a pair's second panel
};

__device__ __forceinline__ d4 mfma(double a, double b, d4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ double bcast(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

// The value of lane C of each row of 16 lanes.
template <int C>
__device__ __forceinline__ double row_bcast(double v) {
  return __longlong_as_double(__builtin_amdgcn_update_dpp(0ll, __double_as_longlong(v), 0x150 + C, 0xf, 0xf, true));
}
template <int I>
struct Index {
  static constexpr int value = I;
};
template <class F, int... I>
__device__ __forceinline__ void for_each_index(F &&f, std::integer_sequence<int, I...>) {
  (f(Index<I>{}), ...);
}
// f(Index<0>) ... f(Index<N - 1>)
template <int N, class F>
__device__ __forceinline__ void for_each_index(F &&f) {
  for_each_index(f, std::make_integer_sequence<int, N>{});
}

// The sum over the four rows of 16 lanes.
__device__ __forceinline__ double row_sum(double v) {
  auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
  auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
  v = __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
  lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
  hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

// Orders a wave's LDS accesses across its lanes.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Values that the workgroups of one launch hand to the last of them: written
// through to memory and read past the caches of the reader's XCD, so that no
// cache has to be flushed or invalidated around them.
__device__ __forceinline__ void put_through(double *p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double get_through(const double *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// True in exactly one workgroup of `count`, the one that arrives last: what the
// others wrote through is then in memory.  The ticket is left at 0.
// This relies on two properties of gfx950 rather than on the language's rule, which
// would ask for a release and an acquire at agent scope around the ticket: an
// agent-scope atomic store is issued with sc1, is performed at the point where the
// device's XCDs agree, and leaves the wave's vmcnt only then, so that the wait for
// 0 below, in every wave before the workgroup's barrier and thread 0's arrival, is
// all that a release at that scope does for such stores (the rest of it writes
// back other dirty lines of the L2, 2 us a launch here); and an agent-scope atomic
// load (sc1) is served from there, past lines that the reader's caches still hold.
// Only put_through and get_through may carry values across it.
__device__ __forceinline__ bool last_arrival(int *ticket, int count, int *shared_flag) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  if (threadIdx.x == 0) {
    const int old = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *shared_flag = old == count - 1;
    if (old == count - 1) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
  return *shared_flag != 0;
}

// 1 / x and 1 / sqrt(x) by Newton steps from the hardware's estimates (2^-24):
// two steps reach rounding, and their chain is short.
__device__ __forceinline__ double fast_rcp(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = fma(fma(-x, r, 1.0), r, r);
  return fma(fma(-x, r, 1.0), r, r);
}
__device__ __forceinline__ double fast_rsqrt(double x) {
  double r = __builtin_amdgcn_rsq(x);
  r = fma(0.5 * r, fma(-x * r, r, 1.0), r);
  return fma(0.5 * r, fma(-x * r, r, 1.0), r);
}

// Tile (wave / 2, wave % 2) of the 32 x 32 product op(A) op(B) of matrices in
// LDS; element r of the result is [4 r + lk][li] of the tile.
template <bool TA, bool TB>
__device__ __forceinline__ d4 prod32(const double (*A)[SLD], const double (*B)[SLD], int wave, int li, int lk) {
  const int i = 16 * (wave >> 1) + li, j = 16 * (wave & 1) + li;
  d4 x{0.0, 0.0, 0.0, 0.0}, y = x;
#pragma unroll
  for (int s = 0; s < 8; s += 2) {
    const int k = 4 * s + lk;
    x = mfma(TA ? A[k][i] : A[i][k], TB ? B[j][k] : B[k][j], x);
    y = mfma(TA ? A[k + 4][i] : A[i][k + 4], TB ? B[j][k + 4] : B[k + 4][j], y);
  }
  return x + y;
}

// sum_w p[w stride + e], in order, for the N values e = first, first + step, ...,
// with up to 16 loads of each in flight.
template <int N>
__device__ __forceinline__ void ordered_sums(const double *p, int first, int step, long long stride, int count,
                                             double (&x)[N]) {
#pragma unroll
  for (int n = 0; n < N; ++n) x[n] = 0.0;
  for (int w0 = 0; w0 < count; w0 += 16) {
    double v[N][16];
#pragma unroll
    for (int w = 0; w < 16; ++w)
#pragma unroll
      for (int n = 0; n < N; ++n) v[n][w] = get_through(p + (long long)min(w0 + w, count - 1) * stride + first + n * step);
#pragma unroll
    for (int w = 0; w < 16; ++w)
#pragma unroll
      for (int n = 0; n < N; ++n) x[n] += w0 + w < count ? v[n][w] : 0.0;
  }
}

// The 32 x 32 factorisations below are chains of 32 dependent pivots on one
// wave, 16 at a time: a lane of each row of 16 holds a column of the 16 x 16
// diagonal block (the four rows copies of it), so that a pivot's column reaches
// the others by DPP in the instruction that uses it, and the off-diagonal block
// is split over the rows; the trailing block takes one MFMA product.  (Rows in
// lanes, eight columns at a time and readlane broadcasts before: Cholesky 8.4 ->
// 3.4 us, LU 9.0 -> 4.5, U^-1 and T 6.8 -> 2.7 us.)

// Cholesky factor of the symmetric 32 x 32 G in place (lower triangle), by one
// wave, and its reciprocal diagonal.  True when a pivot is not above 1e-13 of
// its diagonal element.
__device__ __forceinline__ bool chol32(double (*G)[SLD], double *rd, int lane) {
  const int li = lane & 15, lk = lane >> 4;
  const double g0 = G[li][li], g1 = G[16 + li][16 + li];
  bool bad = false;
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    const int o = 16 * h;
    double p[16], q[4], dg = 1.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) p[i] = G[o + i][o + li];
#pragma unroll
    for (int k = 0; k < 4; ++k) q[k] = G[16 + 4 * k + lk][o + li];
    for_each_index<16>([&](auto ic) {
      constexpr int c = decltype(ic)::value;
      const double d = row_bcast<c>(p[c]);
      if (li == c) dg = d;
      const double t = li > c ? -p[c] * fast_rcp(d) : 0.0;
#pragma unroll
      for (int i = c + 1; i < 16; ++i) p[i] = fma(row_bcast<c>(p[i]), t, p[i]);
#pragma unroll
      for (int k = 0; k < 4; ++k) q[k] = fma(row_bcast<c>(q[k]), t, q[k]);
    });
    bad = bad || !(dg > 1e-13 * (h ? g1 : g0));
    const double r = fast_rsqrt(dg);
    if (lane < 16) {
#pragma unroll
      for (int i = 0; i < 16; ++i) G[o + i][o + li] = i >= li ? p[i] * r : 0.0;
      rd[o + li] = r;
    }
    if (h) break;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      G[16 + 4 * k + lk][li] = q[k] * r;
      G[4 * k + lk][16 + li] = 0.0;
    }
    wave_sync();
    d4 x;
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = G[16 + 4 * k + lk][16 + li];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const double l = G[16 + li][4 * s + lk];
      x = mfma(-l, l, x);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) G[16 + 4 * k + lk][16 + li] = x[k];
    wave_sync();
  }
  return __any(bad);
}

// X = L^-1 (lower triangular) of a Cholesky factor, by one wave: lane i holds
// row i of X^T, i.e. column i of X, and takes L's rows by broadcast.
__device__ __forceinline__ void invert_lower32(const double (*L)[SLD], const double *rd, double (*XT)[SLD], int lane) {
  const int i = lane & (SB - 1);
#pragma unroll 1
  for (int j = 0; j < SB; ++j) {
    double x = i == j ? 1.0 : 0.0;
    for (int k = 0; k < j; ++k) x = fma(-L[j][k], XT[i][k], x);
    if (lane < SB) XT[i][j] = j >= i ? x * rd[j] : 0.0;
    wave_sync();
  }
}

// H - S = Y1 U without pivoting, S_jj = -sign of the pivot (so |U_jj| >= 1 for
// orthonormal columns), in place by one wave; S_jj to sg, 1 / U_jj to rdu.
__device__ __forceinline__ void lu32(double (*H)[SLD], double *rdu, double *sg, int lane) {
  const int li = lane & 15, lk = lane >> 4;
#pragma unroll 1
  for (int h = 0; h < 2; ++h) {
    const int o = 16 * h;
    // the diagonal block, the block below it (a quarter a row of lanes), the block beside it
    double p[16], q[4], w[16], sign = 1.0, rp = 1.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      p[i] = H[o + i][o + li];
      w[i] = H[i][16 + li];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) q[k] = H[16 + 4 * k + lk][o + li];
    for_each_index<16>([&](auto ic) {
      constexpr int c = decltype(ic)::value;
      const double x = row_bcast<c>(p[c]), s = x >= 0.0 ? -1.0 : 1.0, d = x - s, inv = fast_rcp(d);
      if (li == c) {
        sign = s;
        rp = inv;
        p[c] = d;
      }
      const double t = li > c ? -p[c] * inv : 0.0, u = -w[c] * inv;
#pragma unroll
      for (int i = c + 1; i < 16; ++i) {
        const double l = row_bcast<c>(p[i]);
        p[i] = fma(l, t, p[i]);
        w[i] = fma(l, u, w[i]);
        asm volatile("" : "+v"(w[i]));  // now, or every l stays in registers for later
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) q[k] = fma(row_bcast<c>(q[k]), t, q[k]);
    });
    if (lane < 16) {
#pragma unroll
      for (int i = 0; i < 16; ++i) H[o + i][o + li] = i > li ? p[i] * rp : p[i];
      rdu[o + li] = rp;
      sg[o + li] = sign;
    }
    if (h) break;
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (lk == 1) H[i][16 + li] = w[i];
#pragma unroll
    for (int k = 0; k < 4; ++k) H[16 + 4 * k + lk][li] = q[k] * rp;
    wave_sync();
    d4 x;
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = H[16 + 4 * k + lk][16 + li];
#pragma unroll
    for (int s = 0; s < 4; ++s) x = mfma(-H[16 + li][4 * s + lk], H[4 * s + lk][16 + li], x);
#pragma unroll
    for (int k = 0; k < 4; ++k) H[16 + 4 * k + lk][16 + li] = x[k];
    wave_sync();
  }
}

// X = U^-1 and Z = Y1^-1 from lu32's factors in H, by four waves: each inverts
// one 16 x 16 diagonal block (U's transposed), a column a lane, then two of them
// form the off-diagonal blocks.  Ends with a barrier.
__device__ __forceinline__ void invert_factors32(const double (*H)[SLD], const double *rdu, double (*X)[SLD], double (*Z)[SLD],
                                 int lane, int wave) {
  const int li = lane & 15, lk = lane >> 4, o = 16 * (wave & 1);
  const bool up = wave >> 1;
  double l[16], x[16];
  const double rp = up ? rdu[o + li] : 1.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    l[i] = up ? H[o + li][o + i] : H[o + i][o + li];
    x[i] = i == li ? 1.0 : 0.0;
  }
  for_each_index<16>([&](auto it) {
    constexpr int t = decltype(it)::value;
    x[t] *= row_bcast<t>(rp);
#pragma unroll
    for (int i = t + 1; i < 16; ++i) {
      x[i] = fma(row_bcast<t>(l[i]), -x[t], x[i]);
      asm volatile("" : "+v"(l[i]), "+v"(x[i]));  // in this order: later steps' broadcasts would fill the registers
    }
  });
  if (lane < 16) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (up) X[o + li][o + i] = x[i];
      else Z[o + i][o + li] = x[i];
    }
  } else if (lane < 32 && o) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (up) X[16 + i][li] = 0.0;
      else Z[i][16 + li] = 0.0;
    }
  }
  __syncthreads();
  if (wave < 2) {
    // X01 = -X00 (U01 X11), Z10 = -Z11 (L10 Z00), the inner product through its place
    double(*D)[SLD] = wave ? Z : X;
    const int ro = wave ? 16 : 0, co = 16 - ro;  // the block's first row and column
    d4 y{0.0, 0.0, 0.0, 0.0}, z = y;
#pragma unroll
    for (int s = 0; s < 4; ++s) y = mfma(H[ro + li][co + 4 * s + lk], D[co + 4 * s + lk][co + li], y);
#pragma unroll
    for (int r = 0; r < 4; ++r) D[ro + 4 * r + lk][co + li] = y[r];
    wave_sync();
#pragma unroll
    for (int s = 0; s < 4; ++s) z = mfma(-D[ro + li][ro + 4 * s + lk], D[ro + 4 * s + lk][co + li], z);
    wave_sync();
#pragma unroll
    for (int r = 0; r < 4; ++r) D[ro + 4 * r + lk][co + li] = z[r];
  }
  __syncthreads();
}

}  // namespace

// V[P][pad + k] = 2 sqrt(Delta_ia) M^P_ia, ia = perm[k]; zero for the `pad`
// columns in front.
__global__ void __launch_bounds__(256)
spectral_operand_kernel(const double *__restrict__ M_ov, const double *__restrict__ eps,
                        const int *__restrict__ perm, int n_aux, int n_occ, int n_virt, int pad,
                        int np, double *__restrict__ V) {
  const int n_ov = n_occ * n_virt;
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= np) return;
  int ia = 0;
  double sd = 0.0;
  if (k >= pad) {
    ia = perm[k - pad];
    const int i = ia / n_virt, a = ia - i * n_virt;
    sd = 2.0 * sqrt(eps[n_occ + a] - eps[i]);
  }
  for (int P = blockIdx.y; P < n_aux; P += gridDim.y)
    V[(long long)P * np + k] = k >= pad ? sd * M_ov[(long long)P * n_ov + ia] : 0.0;
}

// B[P][c n_basis + m] = M^P_nm for the c-th core state n, zero-padded to Rp columns.
__global__ void __launch_bounds__(256)
spectral_pairs_kernel(const double *__restrict__ M_oo, const double *__restrict__ M_ov, int n_aux, int n_occ,
                      int n_virt, const int *__restrict__ core, int R, int Rp, double *__restrict__ B) {
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= Rp) return;
  const int nb = n_occ + n_virt, c = r / nb, m = r - c * nb, n = r < R ? core[c] : 0;
  for (int P = blockIdx.y; P < n_aux; P += gridDim.y) {
    const long long row = (long long)P * n_occ + n;
    B[(long long)P * Rp + r] = r >= R ? 0.0 : (m < n_occ ? M_oo[row * n_occ + m] : M_ov[row * n_virt + m - n_occ]);
  }
}

// Workgroup -> tile (i, j), i <= j < nt, of a triangle of tiles: row a and row
// nt - 1 - a share nt + 1 consecutive workgroups.
__device__ __forceinline__ bool triangle_tile(int wg, int nt, int &i, int &j) {
  const int a = wg / (nt + 1), b = wg - a * (nt + 1);
  if (b < nt - a) {
    i = a;
    j = a + b;
  } else {
    i = nt - 1 - a;
    j = i + (b - (nt - a));
    if (i == a) return false;
  }
  return true;
}
static unsigned triangle_tiles(int nt) { return (unsigned)((nt + 1) / 2) * (unsigned)(nt + 1); }

// out[i][j] = sum_P A[P][i] B[P][j] on MFMA, a square of 16 W columns per wave,
// four waves a workgroup; the operands are rows of A and B (16 consecutive
// doubles a quarter wave), read through the L1 a batch of 32 / W rows ahead.
// SYM: A = B, tiles i <= j, and delta[i - pad]^2 is added on the diagonal (on the
// `pad` rows in front, where A is zero, elements spread over delta: distinct, so
// that no eigenvalue becomes SB-fold by them).  Sizes are multiples of 32.  Bound by the matrix cores where W = 4 (half the operand
// loads a product), which needs many tiles to fill the chip.
template <bool SYM, int W>
__global__ void __launch_bounds__(256, W == 4 ? 2 : 4)
spectral_gemm_kernel(const double *__restrict__ A, int lda, const double *__restrict__ B, int ldb,
                     int M, int N, int K, const double *__restrict__ delta, int pad,
                     double *__restrict__ out, long long ldo) {
  constexpr int WT = 16 * W, TILE = 2 * WT, S = 8 / W;
  int ti, tj;
  if (SYM) {
    if (!triangle_tile(blockIdx.x, (M + TILE - 1) / TILE, ti, tj)) return;
  } else {
    const int nj = (N + TILE - 1) / TILE;
    ti = blockIdx.x / nj;
    tj = blockIdx.x - ti * nj;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  const int i0 = ti * TILE + (wave >> 1) * WT, j0 = tj * TILE + (wave & 1) * WT;
  if (i0 >= M || j0 >= N || (SYM && i0 > j0)) return;  // the whole wave
  d4 acc[W][W];
#pragma unroll
  for (int a = 0; a < W; ++a)
#pragma unroll
    for (int b = 0; b < W; ++b) acc[a][b] = d4{0.0, 0.0, 0.0, 0.0};
  // columns of the wave's square beyond the matrix are read from its last 32
  int ca[W], cb[W];
#pragma unroll
  for (int a = 0; a < W; ++a) {
    ca[a] = min(i0 + 16 * a, M - 16) + li;
    cb[a] = min(j0 + 16 * a, N - 16) + li;
  }
  double va[2][S][W], vb[2][S][W];
  auto fetch = [&](int k, double(&x)[S][W], double(&y)[S][W]) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int r = k + 4 * s + lk;
      const bool in = r < K;
      const double *ra = A + (long long)(in ? r : 0) * lda, *rb = B + (long long)(in ? r : 0) * ldb;
#pragma unroll
      for (int a = 0; a < W; ++a) {
        const double p = ra[ca[a]], q = rb[cb[a]];
        x[s][a] = in ? p : 0.0;
        y[s][a] = in ? q : 0.0;
      }
    }
  };
  auto product = [&](const double(&x)[S][W], const double(&y)[S][W]) {
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
      for (int a = 0; a < W; ++a)
#pragma unroll
        for (int b = 0; b < W; ++b) acc[a][b] = mfma(x[s][a], y[s][b], acc[a][b]);
  };
  fetch(0, va[0], vb[0]);
  for (int k = 0; k < K; k += 8 * S) {
    fetch(k + 4 * S, va[1], vb[1]);
    product(va[0], vb[0]);
    fetch(k + 8 * S, va[0], vb[0]);
    product(va[1], vb[1]);
  }
#pragma unroll
  for (int a = 0; a < W; ++a)
#pragma unroll
    for (int b = 0; b < W; ++b) {
      if (i0 + 16 * a >= M || j0 + 16 * b >= N) continue;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = i0 + 16 * a + 4 * r + lk, j = j0 + 16 * b + li;
        double x = acc[a][b][r];
        if (SYM && i == j) {
          const double d = delta[i >= pad ? i - pad : (int)((long long)i * (M - pad) / SB)];
          x = fma(d, d, x);
        }
        out[(long long)i * ldo + j] = x;
      }
    }
}

// The panel of the first reflection: column c of P[c][row] is SB m pseudo-random
// numbers in (-1, 1) (the mixing function of splitmix64 on the element's index).
__global__ void __launch_bounds__(256)
panel_start_kernel(double *__restrict__ P, long long count) {
  const long long e = blockIdx.x * 256LL + threadIdx.x;
  if (e >= count) return;
  unsigned long long x = (unsigned long long)(e + 1) * 0x9e3779b97f4a7c15ull;
  x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
  x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
  x ^= x >> 31;
  P[e] = (double)(long long)x * 0x1p-63;
}

// Sum of the per-wave Gram tiles (0,0), (0,1), (1,1) through LDS: element
// q 256 + tid of the three tiles goes to out(q, value).
template <class F>
__device__ __forceinline__ void gram_combine(double *buf, const d4 &g00, const d4 &g01, const d4 &g11, F &&out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int o = wave * 768 + (4 * r + lk) * 16 + li;
    buf[o] = g00[r];
    buf[o + 256] = g01[r];
    buf[o + 512] = g11[r];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const int e = q * 256 + tid;
    out(e, ((buf[e] + buf[768 + e]) + buf[1536 + e]) + buf[2304 + e]);
  }
}

// The symmetric 32 x 32 matrix of `count` partial sums.
__device__ __forceinline__ void gram_collect(const double *part, int stride, int count, double (*G)[SLD]) {
  const int tid = threadIdx.x, i = tid >> 4, j = tid & 15;
  double s[3];
  ordered_sums(part, tid, 256, stride, count, s);
  G[i][j] = s[0];
  G[i][16 + j] = s[1];
  G[16 + j][i] = s[1];
  G[16 + i][16 + j] = s[2];
}

// G = L1 L1^T by one workgroup; buf holds SB SLD doubles.
__device__ __forceinline__ void panel_factor(const double *part, int count, double *buf, PanelSmall *sm, int *flag) {
  __shared__ double rdsh[SB];
  double(*G)[SLD] = reinterpret_cast<double(*)[SLD]>(buf);
  const int tid = threadIdx.x;
  gram_collect(part, 768, count, G);
  __syncthreads();
  if (tid < 64) {
    const bool bad = chol32(G, rdsh, tid);
    if (bad && tid == 0) *flag = 1;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = q * 256 + tid;
    sm->R1[e] = G[e % SB][e / SB];
  }
  if (tid < SB) sm->rd1[tid] = rdsh[tid];
}

// G of the first reflection's panel (m rows) and its factor: 256 rows per workgroup.
__global__ void __launch_bounds__(PROWS)
panel_gram_kernel(const double *__restrict__ P, long long ldp, int m, PanelSmall *__restrict__ sm,
                  double *part, int *__restrict__ ticket, int *__restrict__ flag) {
  __shared__ double buf[PROWS * SLD];
  __shared__ int last;
  double(*S)[SLD] = reinterpret_cast<double(*)[SLD]>(buf);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int row0 = blockIdx.x * PROWS;
  double q[SB];
#pragma unroll
  for (int c = 0; c < SB; ++c) q[c] = row0 + tid < m ? P[(long long)c * ldp + row0 + tid] : 0.0;
#pragma unroll
  for (int c = 0; c < SB; ++c) S[tid][c] = q[c];
  __syncthreads();
  d4 g00{0.0, 0.0, 0.0, 0.0}, g01 = g00, g11 = g00;
#pragma unroll 4
  for (int s = 0; s < 16; ++s) {
    const int k = 64 * wave + 4 * s + lk;
    const double a0 = S[k][li], a1 = S[k][16 + li];
    g00 = mfma(a0, a0, g00);
    g01 = mfma(a0, a1, g01);
    g11 = mfma(a1, a1, g11);
  }
  __syncthreads();
  gram_combine(buf, g00, g01, g11, [&](int e, double v) { put_through(part + (long long)blockIdx.x * 768 + e, v); });
  if (last_arrival(ticket, gridDim.x, &last)) panel_factor(part, gridDim.x, buf, sm, flag);
}

// Q = P L1^-T, one row per thread, and the partial sums of Q^T Q; for a pair's
// second panel also of Wa^T Q and Ya^T Q.  Latency: the panel and L1 are loaded
// in one batch and L1's elements reach the rows' threads by DPP, from registers
// (24 -> 10.3 us at 5859 rows; four batches and scalar loads of L1 before).
template <bool SECOND>
__global__ void __launch_bounds__(PROWS)
panel_q_kernel(const double *__restrict__ P, long long ldp, int m, const PanelSmall *__restrict__ sm,
               const double *__restrict__ Ya, const double *__restrict__ Wa, double *__restrict__ Q,
               double *__restrict__ part) {
  __shared__ double buf[PROWS * SLD];
  double(*S)[SLD] = reinterpret_cast<double(*)[SLD]>(buf);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int row0 = blockIdx.x * PROWS;
  // R1's row j at lane li: columns li (ra, j < 16) and 16 + li (rb)
  double q[SB], ra[16], rb[SB];
#pragma unroll
  for (int c = 0; c < SB; ++c) q[c] = row0 + tid < m ? P[(long long)c * ldp + row0 + tid] : 0.0;
#pragma unroll
  for (int j = 0; j < 16; ++j) ra[j] = sm->R1[j * SB + li];
#pragma unroll
  for (int j = 0; j < SB; ++j) rb[j] = sm->R1[j * SB + 16 + li];
  const double rda = sm->rd1[li], rdb = sm->rd1[16 + li];
  for_each_index<16>([&](auto ij) {
    constexpr int j = decltype(ij)::value;
    q[j] *= row_bcast<j>(rda);
    const double x = -q[j];
    for_each_index<15 - j>([&](auto ik) {
      constexpr int k = j + 1 + decltype(ik)::value;
      q[k] = fma(row_bcast<k>(ra[j]), x, q[k]);
    });
    for_each_index<16>([&](auto ik) {
      constexpr int k = decltype(ik)::value;
      q[16 + k] = fma(row_bcast<k>(rb[j]), x, q[16 + k]);
    });
  });
  for_each_index<16>([&](auto ij) {
    constexpr int j = decltype(ij)::value;
    q[16 + j] *= row_bcast<j>(rdb);
    const double x = -q[16 + j];
    for_each_index<15 - j>([&](auto ik) {
      constexpr int k = j + 1 + decltype(ik)::value;
      q[16 + k] = fma(row_bcast<k>(rb[16 + j]), x, q[16 + k]);
    });
  });
#pragma unroll
  for (int j = 0; j < SB; ++j) S[tid][j] = q[j];
  __syncthreads();
#pragma unroll 8
  for (int it = 0; it < SB; ++it) {
    const int e = it * PROWS + tid, r = e / SB, c = e % SB;
    if (row0 + r < m) Q[(long long)row0 * SB + e] = S[r][c];
  }
  d4 g00{0.0, 0.0, 0.0, 0.0}, g01 = g00, g11 = g00;
#pragma unroll 4
  for (int s = 0; s < 16; ++s) {
    const int k = 64 * wave + 4 * s + lk;
    const double a0 = S[k][li], a1 = S[k][16 + li];
    g00 = mfma(a0, a0, g00);
    g01 = mfma(a0, a1, g01);
    g11 = mfma(a1, a1, g11);
  }
  constexpr int PART = SECOND ? Q_PART2 : Q_PART;
  double *o = part + (long long)blockIdx.x * PART;
  d4 c[2][2][2];
  if (SECOND) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const double *Z = (p ? Ya : Wa) + (long long)row0 * SB;
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) c[p][a][b] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
      for (int s = 0; s < 16; ++s) {
        const int k = 64 * wave + 4 * s + lk;
        const bool in = row0 + k < m;
        const double *z = Z + (long long)(in ? k : 0) * SB + li;
        const double z0 = in ? z[0] : 0.0, z1 = in ? z[16] : 0.0, q0 = S[k][li], q1 = S[k][16 + li];
        c[p][0][0] = mfma(z0, q0, c[p][0][0]);
        c[p][0][1] = mfma(z0, q1, c[p][0][1]);
        c[p][1][0] = mfma(z1, q0, c[p][1][0]);
        c[p][1][1] = mfma(z1, q1, c[p][1][1]);
      }
    }
  }
  __syncthreads();
  gram_combine(buf, g00, g01, g11, [&](int e, double v) { o[e] = v; });
  if (SECOND) {
    double *red = buf + 4 * 768;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            red[wave * SB * SB + (16 * a + 4 * r + lk) * SB + 16 * b + li] = c[p][a][b][r];
      __syncthreads();
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int e = q * 256 + tid;
        o[768 + p * SB * SB + e] = ((red[e] + red[SB * SB + e]) + red[2 * SB * SB + e]) + red[3 * SB * SB + e];
      }
      __syncthreads();
    }
  }
}


// From G2's partial sums to M2, SU, T and the block's coupling Bk = S R2 L1^T
// (see the head of this file), by one workgroup, and V1, V2 of a pair's second
// panel; buf holds 4 SB SLD + SB doubles.
template <bool SECOND>
__device__ __forceinline__ void panel_reconstruct(const double *__restrict__ Q, const double *part, int count,
                                  const double *__restrict__ Ya, const double *__restrict__ Wa, double *buf,
                                  PanelSmall *__restrict__ sm, int *flag, double *__restrict__ Bk) {
  constexpr int PART = SECOND ? Q_PART2 : Q_PART;
  __shared__ double rdsh[SB];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
  double(*G)[SLD] = reinterpret_cast<double(*)[SLD]>(buf);
  double(*H)[SLD] = reinterpret_cast<double(*)[SLD]>(buf + SB * SLD);
  double(*T)[SLD] = reinterpret_cast<double(*)[SLD]>(buf + 2 * SB * SLD);
  double(*L)[SLD] = reinterpret_cast<double(*)[SLD]>(buf + 3 * SB * SLD);
  double *sg = buf + 4 * SB * SLD;
  double q0[4], r1[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = q * 256 + tid;
    q0[q] = Q[e];
    r1[q] = sm->R1[e];
  }
  gram_collect(part, PART, count, G);
  __syncthreads();
  int off = 0;
  double phi[4], r2[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = q * 256 + tid, i = e / SB, j = e % SB;
    const double x = G[i][j] - (i == j ? 1.0 : 0.0);
    off |= !(fabs(x) <= 1e-8);
    phi[q] = i < j ? x : (i == j ? 0.5 * x : 0.0);
    r2[q] = phi[q] + (i == j ? 1.0 : 0.0);
  }
  if (__syncthreads_or(off)) {
    if (wave == 0) {
      const bool bad = chol32(G, rdsh, lane);
      if (bad && lane == 0) *flag = 1;
      wave_sync();
      invert_lower32(G, rdsh, T, lane);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e = q * 256 + tid, i = e / SB, j = e % SB;
      phi[q] = (i == j ? 1.0 : 0.0) - T[i][j];  // T = L2^-T
      r2[q] = i <= j ? G[j][i] : 0.0;
    }
    __syncthreads();
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = q * 256 + tid, i = e / SB, j = e % SB;
    T[i][j] = phi[q];
    G[i][j] = r2[q];
    H[i][j] = q0[q];
    L[i][j] = r1[q];
  }
  __syncthreads();
  const int i0 = 16 * (wave >> 1) + lk, j0 = 16 * (wave & 1) + li;  // of this lane's product elements
  const d4 h = prod32<false, false>(H, T, wave, li, lk);
  const d4 b = prod32<false, false>(G, L, wave, li, lk);  // S times the coupling, S not yet known
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) H[i0 + 4 * r][j0] -= h[r];
  __syncthreads();
  if (wave == 0) lu32(H, rdsh, sg, lane);  // S, Y1 and U
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = q * 256 + tid;
    L[e / SB][e % SB] = phi[q];
  }
  __syncthreads();
  invert_factors32(H, rdsh, G, T, lane, wave);  // U^-1 and Y1^-1
  const d4 pu = prod32<false, false>(L, G, wave, li, lk);
  d4 tf{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int i = 16 * (wave >> 1) + li, k = 4 * s + lk;
    tf = mfma(k >= i ? -H[i][k] * sg[k] : 0.0, T[j0][k], tf);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = i0 + 4 * r, j = j0, e = i * SB + j;
    sm->M2[e] = G[i][j] - pu[r];
    sm->SU[e] = sg[i] * G[i][j];
    sm->T[e] = i <= j ? tf[r] : 0.0;
    Bk[e] = i <= j ? sg[i] * b[r] : 0.0;
  }
  if (SECOND) {
    // V = (Z^T Q) M2 - Z_top^T SU for Z = Wa, Ya: M2 in G, SU in H
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + 4 * r;
      H[i][j0] = sg[i] * G[i][j0];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) G[i0 + 4 * r][j0] -= pu[r];
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const double *Z = p ? Ya : Wa;
      double c[4];
      ordered_sums(part + 768 + p * SB * SB, tid, 256, PART, count, c);
      __syncthreads();
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int e = q * 256 + tid;
        T[e / SB][e % SB] = c[q];
        L[e / SB][e % SB] = Z[e];
      }
      __syncthreads();
      const d4 v = prod32<false, false>(T, G, wave, li, lk), w = prod32<true, false>(L, H, wave, li, lk);
      double *V = p ? sm->V2 : sm->V1;
#pragma unroll
      for (int r = 0; r < 4; ++r) V[(i0 + 4 * r) * SB + j0] = v[r] - w[r];
    }
  }
}

// Xq = A22^T Q over the columns from A (A22's own, then u's): workgroup
// (32 columns, split s), its four waves on consecutive parts of the split's
// rows, summed in order.  A's rows are read 16 doubles a quarter wave.
// Workgroup 0 does the panel's small matrices instead: about 13 us of
// dependent steps, hidden behind the product.  (Three workgroups a CU: its
// registers are bounded by what the product needs.)
template <bool SECOND>
__global__ void __launch_bounds__(256, 3)
panel_x_kernel(const double *__restrict__ A, long long lda, int m, int mx, int splits,
               const double *__restrict__ Q, double *__restrict__ Xpart, const double *__restrict__ part,
               int parts2, const double *__restrict__ Ya, const double *__restrict__ Wa,
               PanelSmall *__restrict__ sm, int *__restrict__ flag, double *__restrict__ Bk) {
  __shared__ double buf[4 * SB * SLD + SB];
  if (blockIdx.x == 0) {
    panel_reconstruct<SECOND>(Q, part, parts2, Ya, Wa, buf, sm, flag, Bk);
    return;
  }
  double(*red)[SB * SB] = reinterpret_cast<double(*)[SB * SB]>(buf);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int nx = mx / SB, split = (blockIdx.x - 1) / nx, c0 = (blockIdx.x - 1 - split * nx) * SB;
  const int nkb = m / SB, parts = 4 * splits, w = 4 * split + wave;
  const int k0 = (int)((long long)nkb * w / parts) * SB, k1 = (int)((long long)nkb * (w + 1) / parts) * SB;
  d4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = d4{0.0, 0.0, 0.0, 0.0};
  // rows above the columns' diagonal block and it: A[k][c0 + j]
  const int kd = min(k1, c0 + SB);
  const double *pa = A + (long long)(k0 + lk) * lda + c0 + li;
  const double *py = Q + (long long)(k0 + lk) * SB + li;
  for (int k = k0; k < kd; k += 32) {
    double a0[8], a1[8], y0[8], y1[8];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      a0[s] = pa[(long long)(4 * s) * lda];
      a1[s] = pa[(long long)(4 * s) * lda + 16];
      y0[s] = py[4 * s * SB];
      y1[s] = py[4 * s * SB + 16];
    }
    pa += 32 * lda;
    py += 32 * SB;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      acc[0][0] = mfma(a0[s], y0[s], acc[0][0]);
      acc[0][1] = mfma(a0[s], y1[s], acc[0][1]);
      acc[1][0] = mfma(a1[s], y0[s], acc[1][0]);
      acc[1][1] = mfma(a1[s], y1[s], acc[1][1]);
    }
  }
  // and below, from the stored triangle: A[c0 + j][k], two neighbours of k a lane
  const int kl = max(k0, c0 + SB);
  pa = A + (long long)(c0 + li) * lda + kl + 2 * lk;
  py = Q + (long long)(kl + 2 * lk) * SB + li;
  for (int k = kl; k < k1; k += 32) {
    d2 a0[4], a1[4];
    double y0[8], y1[8];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      a0[s] = *reinterpret_cast<const d2 *>(pa + 8 * s);
      a1[s] = *reinterpret_cast<const d2 *>(pa + 16 * lda + 8 * s);
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        y0[2 * s + e] = py[(8 * s + e) * SB];
        y1[2 * s + e] = py[(8 * s + e) * SB + 16];
      }
    }
    pa += 32;
    py += 32 * SB;
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      acc[0][0] = mfma(a0[s / 2][s % 2], y0[s], acc[0][0]);
      acc[0][1] = mfma(a0[s / 2][s % 2], y1[s], acc[0][1]);
      acc[1][0] = mfma(a1[s / 2][s % 2], y0[s], acc[1][0]);
      acc[1][1] = mfma(a1[s / 2][s % 2], y1[s], acc[1][1]);
    }
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][(16 * a + 4 * r + lk) * SB + 16 * b + li] = acc[a][b][r];
  __syncthreads();
  double *o = Xpart + ((long long)split * mx + c0) * SB;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = q * 256 + tid;
    o[e] = ((red[0][e] + red[1][e]) + red[2][e]) + red[3][e];
  }
}

// Y, X and E2 (see the head of this file), 128 rows per workgroup, a 16 x 16
// tile of both a wave, so that a workgroup's loads are one batch (16 waves:
// 19.9 us at 5859 rows; eight of 16 rows: 21; four of 32: 25).
template <bool SECOND>
__global__ void __launch_bounds__(XTHREADS)
panel_xsum_kernel(const double *__restrict__ Xpart, int splits, const double *__restrict__ A, long long lda, int m,
                  int mx, const double *__restrict__ Q, const double *__restrict__ Ya,
                  const double *__restrict__ Wa, const PanelSmall *__restrict__ sm_in, PanelSmall *__restrict__ sm,
                  double *__restrict__ X, double *__restrict__ Y, double *part,
                  int *__restrict__ ticket) {
  __shared__ double buf[2 * XROWS * SLD];
  __shared__ int last;
  double(*Xs)[SLD] = reinterpret_cast<double(*)[SLD]>(buf);
  double(*Ys)[SLD] = reinterpret_cast<double(*)[SLD]>(buf + XROWS * SLD);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int row0 = blockIdx.x * XROWS;
#pragma unroll
  for (int it = 0; it < XROWS * SB / XTHREADS; ++it) {
    const int e = it * XTHREADS + tid, r = e / SB, c = e % SB;
    const long long o = row0 + r < mx ? (long long)row0 * SB + e : 0;
    double v[SPECTRAL_MAX_SPLITS], x = 0.0;
#pragma unroll
    for (int s = 0; s < SPECTRAL_MAX_SPLITS; ++s) v[s] = Xpart[(long long)min(s, splits - 1) * mx * SB + o];
    const double y = Q[row0 + r < m ? o : 0];
#pragma unroll
    for (int s = 0; s < SPECTRAL_MAX_SPLITS; ++s) x += s < splits ? v[s] : 0.0;
    Xs[r][c] = x;
    Ys[r][c] = row0 + r < m ? y : 0.0;
  }
  // this wave's 16 x 16 tile of X and of Y: m, mx are multiples of 32
  const int wr = 16 * (wave >> 1), wc = 16 * (wave & 1), row = row0 + wr;
  const bool in = row < mx, mat = row < m;
  double st[8], m2[8], su[8];  // st: the first SB rows of A22 at the tile's rows
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    st[s] = in ? -A[(long long)(4 * s + lk) * lda + row + li] : 0.0;
    m2[s] = sm_in->M2[(4 * s + lk) * SB + wc + li];
    su[s] = sm_in->SU[(4 * s + lk) * SB + wc + li];
  }
  __syncthreads();
  d4 x{0.0, 0.0, 0.0, 0.0}, x2 = x, y = x;
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int i = wr + li, k = 4 * s + lk;
    x = mfma(Xs[i][k], m2[s], x);
    x2 = mfma(st[s], su[s], x2);
    y = mfma(Ys[i][k], m2[s], y);
  }
  if (SECOND) {
    // what the first panel's update would have taken from A22
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int k = 4 * s + lk;
      const long long o = (long long)(row + li) * SB + k;
      const double wa = in ? -Wa[o] : 0.0, ya = mat ? -Ya[o] : 0.0;
      x = mfma(wa, sm_in->V2[k * SB + wc + li], x);
      x2 = mfma(ya, sm_in->V1[k * SB + wc + li], x2);
    }
  }
  x += x2;
  if (row < SB) {
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] -= sm_in->SU[(row + 4 * r + lk) * SB + wc + li];
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = 4 * r + lk, j = wc + li;
    if (in) X[(long long)(row + i) * SB + j] = x[r];
    if (mat) Y[(long long)(row + i) * SB + j] = y[r];
    Xs[wr + i][j] = x[r];
    Ys[wr + i][j] = mat ? y[r] : 0.0;
  }
  if (row0 >= m) return;  // the whole workgroup: rows of u only
  __syncthreads();
  // Y^T X: tile wave % 4 over the rows 32 (wave / 4) ..
  d4 acc{0.0, 0.0, 0.0, 0.0};
  const int ta = 16 * ((wave >> 1) & 1);
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int k = 32 * (wave >> 2) + 4 * s + lk;
    acc = mfma(Ys[k][ta + li], Xs[k][wc + li], acc);
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < 4; ++r) buf[(wave >> 2) * SB * SB + (ta + 4 * r + lk) * SB + wc + li] = acc[r];
  __syncthreads();
  put_through(part + (long long)blockIdx.x * SB * SB + tid,
              ((buf[tid] + buf[SB * SB + tid]) + buf[2 * SB * SB + tid]) + buf[3 * SB * SB + tid]);
  const int count = (m + XROWS - 1) / XROWS;
  if (!last_arrival(ticket, count, &last)) return;
  double(*M)[SLD] = Xs;
  double(*T)[SLD] = reinterpret_cast<double(*)[SLD]>(buf + SB * SLD);
  double(*MT)[SLD] = reinterpret_cast<double(*)[SLD]>(buf + 2 * SB * SLD);
  static_assert(XTHREADS == SB * SB && XROWS == 128, "an element a thread, eight tiles of rows");
  double c[1];
  const double tv = sm_in->T[tid];
  ordered_sums(part, tid, 0, SB * SB, count, c);
  M[tid / SB][tid % SB] = c[0];
  T[tid / SB][tid % SB] = tv;
  __syncthreads();
  // a tile a wave for the first four
  const int i0 = 16 * (wave >> 1) + lk, j0 = 16 * (wave & 1) + li;
  if (wave < 4) {
    const d4 mt = prod32<false, false>(M, T, wave, li, lk);
#pragma unroll
    for (int r = 0; r < 4; ++r) MT[i0 + 4 * r][j0] = mt[r];
  }
  __syncthreads();
  if (wave < 4) {
    const d4 e2 = prod32<true, false>(T, MT, wave, li, lk);
#pragma unroll
    for (int r = 0; r < 4; ++r) sm->E2[(i0 + 4 * r) * SB + j0] = 0.5 * e2[r];
  }
}

// W = X T - Y E2 for the m matrix rows, W = X T for the rows of u; 16 rows a wave.
__global__ void __launch_bounds__(256)
panel_w_kernel(const double *__restrict__ X, const double *__restrict__ Y, int m, int mx,
               const PanelSmall *__restrict__ sm, double *__restrict__ W) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, lk = lane >> 4;
  const int row = (blockIdx.x * 4 + wave) * 16;
  if (row >= mx) return;
  d4 acc[2];
  acc[0] = d4{0.0, 0.0, 0.0, 0.0};
  acc[1] = acc[0];
  const bool mat = row < m;  // m is a multiple of 32
  double x[8], y[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    x[s] = X[(long long)(row + li) * SB + 4 * s + lk];
    y[s] = mat ? -Y[(long long)(row + li) * SB + 4 * s + lk] : 0.0;
  }
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int o = (4 * s + lk) * SB + li;
    acc[0] = mfma(x[s], sm->T[o], acc[0]);
    acc[1] = mfma(x[s], sm->T[o + 16], acc[1]);
  }
  if (mat) {
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int o = (4 * s + lk) * SB + li;
      acc[0] = mfma(y[s], sm->E2[o], acc[0]);
      acc[1] = mfma(y[s], sm->E2[o + 16], acc[1]);
    }
  }
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) W[(long long)(row + 4 * r + lk) * SB + 16 * b + li] = acc[b][r];
}

// A22 -= Y W^T + W Y^T for one panel or both of a pair, on 64 x 64 tiles on or
// above the diagonal; and u -= Y Wu^T on the columns behind the matrix (the
// workgroups from n_mat on).  m, mx multiples of 32.  STRIP: only the first SB
// rows (a pair's second panel).  The first row of tiles (the first workgroups)
// holds the next panel transposed, A22[:SB, SB:], and forms its G.  A wave owns
// a quadrant of the tile (idle below the diagonal) and loads its old values
// first.
template <bool STRIP>
__global__ void __launch_bounds__(256)
panel_update_kernel(double *__restrict__ A, long long lda, int m, int mx, const double *__restrict__ Ya,
                    const double *__restrict__ Wa, const double *__restrict__ Yb, const double *__restrict__ Wb,
                    int n_mat, PanelSmall *__restrict__ sm, double *part, int *__restrict__ ticket,
                    int *__restrict__ flag) {
  constexpr int PER = UT * SB / 2 / 256;
  __shared__ double Ls[UT * ULD], Rs[4 * 768 > UT * ULD ? 4 * 768 : UT * ULD];
  __shared__ int last;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
  const int nt = (m + UT - 1) / UT, mrow = STRIP ? SB : m;
  int i0, j0, jend;
  bool next = false;
  const bool mat = (int)blockIdx.x < n_mat;
  if (mat) {
    int ti = 0, tj = blockIdx.x;
    if (!STRIP && !triangle_tile(blockIdx.x, nt, ti, tj)) return;
    i0 = ti * UT;
    j0 = tj * UT;
    jend = m;
    next = ti == 0 && m > SB;
  } else {
    const int q = blockIdx.x - n_mat, tj = STRIP ? q : q / nt;
    i0 = STRIP ? 0 : (q - tj * nt) * UT;
    j0 = m + tj * UT;
    jend = mx;
  }
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  const bool in = i0 + wr < mrow && j0 + wc < jend && i0 + wr <= j0 + wc;  // the whole quadrant
  double *At = A + (long long)(i0 + wr) * lda + j0 + wc;
  double old[2][2][4];
  if (in) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) old[a][b][r] = At[(long long)(16 * a + 4 * r + lk) * lda + 16 * b + li];
  }
  d4 acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b) acc[a][b] = d4{0.0, 0.0, 0.0, 0.0};
  // Y W^T and W Y^T of each panel; u's columns take Y W^T only
  const int step = mat ? 1 : 2, parts = Yb ? 4 : 2;
  d2 lv[PER], rv[PER];
  auto fetch = [&](int h) {
    const double *Y = h < 2 ? Ya : Yb, *W = h < 2 ? Wa : Wb;
    const double *Lp = ((h & 1) ? W : Y) + (long long)i0 * SB, *Rp = ((h & 1) ? Y : W) + (long long)j0 * SB;
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      const int e = (it * 256 + tid) * 2, r = e / SB;
      lv[it] = d2{0.0, 0.0};
      rv[it] = d2{0.0, 0.0};
      if (i0 + r < mrow) lv[it] = *reinterpret_cast<const d2 *>(Lp + e);
      if (j0 + r < jend) rv[it] = *reinterpret_cast<const d2 *>(Rp + e);
    }
  };
  fetch(0);
  for (int h = 0; h < parts; h += step) {
    if (h) __syncthreads();
#pragma unroll
    for (int it = 0; it < PER; ++it) {
      const int e = (it * 256 + tid) * 2, r = e / SB, c = e % SB;
      *reinterpret_cast<d2 *>(&Ls[r * ULD + c]) = lv[it];
      *reinterpret_cast<d2 *>(&Rs[r * ULD + c]) = rv[it];
    }
    __syncthreads();
    if (h + step < parts) fetch(h + step);
    if (!in) continue;
#pragma unroll
    for (int s = 0; s < SB / 4; ++s) {
      const int k = 4 * s + lk;
      const double a0 = Ls[(wr + li) * ULD + k], a1 = Ls[(wr + 16 + li) * ULD + k];
      const double b0 = Rs[(wc + li) * ULD + k], b1 = Rs[(wc + 16 + li) * ULD + k];
      acc[0][0] = mfma(a0, b0, acc[0][0]);
      acc[0][1] = mfma(a0, b1, acc[0][1]);
      acc[1][0] = mfma(a1, b0, acc[1][0]);
      acc[1][1] = mfma(a1, b1, acc[1][1]);
    }
  }
  if (in) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const double x = old[a][b][r] - acc[a][b][r];
          At[(long long)(16 * a + 4 * r + lk) * lda + 16 * b + li] = x;
          old[a][b][r] = x;
        }
  }
  if (!next) return;  // the whole workgroup
  // Ls[c][j] = A22[c][j0 + j] for c < SB, zero outside the panel
  constexpr int PLD = UT + 2;
  static_assert(UT * ULD >= SB * PLD && UT * ULD >= 2 * SB * SLD, "the panel's tile fits");
  __syncthreads();
  if (wr == 0) {
    const bool panel = in && j0 + wc >= SB;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          Ls[(16 * a + 4 * r + lk) * PLD + wc + 16 * b + li] = panel ? old[a][b][r] : 0.0;
  }
  __syncthreads();
  d4 g00{0.0, 0.0, 0.0, 0.0}, g01 = g00, g11 = g00;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int k = 16 * wave + 4 * s + lk;
    const double a0 = Ls[li * PLD + k], a1 = Ls[(16 + li) * PLD + k];
    g00 = mfma(a0, a0, g00);
    g01 = mfma(a0, a1, g01);
    g11 = mfma(a1, a1, g11);
  }
  __syncthreads();
  gram_combine(Rs, g00, g01, g11, [&](int e, double v) { put_through(part + (long long)(j0 / UT) * 768 + e, v); });
  if (last_arrival(ticket, nt, &last)) panel_factor(part, nt, Ls, sm, flag);
}

// The band in 16 x 16 tiles, per 16-row block p: (p, p), (p, p + 1), (p, p + 2);
// two zero blocks behind the last.  Even p: diagonal block k = p / 2 holds the
// first two, the transposed coupling B_k the third; odd p: B_k both.
__global__ void __launch_bounds__(256)
spectral_band_kernel(const double *__restrict__ A, long long lda, const double *__restrict__ Bk,
                     int nblk, double *__restrict__ band) {
  const int p = blockIdx.x, k = p >> 1, h = p & 1;
  const int i = threadIdx.x >> 4, j = threadIdx.x & 15;
  double d = 0.0, e = 0.0, f = 0.0;
  if (k < nblk) {
    const double *D = A + (long long)k * SB * lda + (long long)k * SB;
    d = D[(long long)(16 * h + i) * lda + 16 * h + j];
    if (h == 0) e = D[(long long)i * lda + 16 + j];
    if (k + 1 < nblk) {
      const double *B = Bk + (long long)k * SB * SB;  // rows of block k + 1, columns of block k
      if (h == 0) {
        f = B[j * SB + i];
      } else {
        e = B[j * SB + 16 + i];
        f = B[(16 + j) * SB + 16 + i];
      }
    }
  }
  double *o = band + (long long)p * 768 + threadIdx.x;
  o[0] = d;
  o[256] = e;
  o[512] = f;
}

// out[c][r] = in[r][c] for c < cols and r < rows; zero for rows <= r < rows_out.
// 32 x 32 tiles through LDS.
__global__ void __launch_bounds__(256)
spectral_transpose_kernel(const double *__restrict__ in, long long ldi, int rows, int cols, double *__restrict__ out,
                          long long ldo, int rows_out) {
  __shared__ double t[32][33];
  const int r0 = blockIdx.x * 32, c0 = blockIdx.y * 32, x = threadIdx.x & 31, y = threadIdx.x >> 5;
#pragma unroll
  for (int q = 0; q < 32; q += 8)
    t[q + y][x] = r0 + q + y < rows && c0 + x < cols ? in[(long long)(r0 + q + y) * ldi + c0 + x] : 0.0;
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 32; q += 8)
    if (c0 + q + y < cols && r0 + x < rows_out) out[(long long)(c0 + q + y) * ldo + r0 + x] = t[x][q + y];
}

// W = u^T (z^2 - C)^-1 u of a task's one to 16 vectors u (one where COMPLEX) by
// elimination of the band, two waves per task: one from the first row down, the other from the
// last row up, to the two blocks in the middle, which the first finishes.
//
// A step eliminates 16 rows.  Their 48 columns inside the band and 16 vectors
// sit one column per lane (rows in registers); a pivot's multipliers are the
// pivot row scaled by 1/d (the matrix is symmetric), broadcast from the lanes
// that hold them.  z^2 - C has the imaginary part 2 x eta 1, or is definite on
// the imaginary axis, so no pivot vanishes.  What the step leaves on the next
// two blocks and their vectors is a product of the eliminated rows, on MFMA
// (accumulators initialised with the band itself); the layouts change through
// the wave's LDS.  COMPLEX = false is the imaginary axis (z^2 = -w^2, real).
// COMPLEX also solves for x = (z^2 - T)^-1 u: the eliminated rows over their pivots
// go to `factors`, SPECTRAL_ROWS values a step (per row the solved right-hand side
// and the 32 columns behind the diagonal), and each wave substitutes back from the
// middle over its own; x's planes go to row blockIdx.x (real parts) and gridDim.x +
// blockIdx.x of X, the elimination's W to W_out[blockIdx.x].  The way back reads
// 8.4 KB a step, loaded a step ahead, and takes 15 dependent products of it.
// Bound by the steps' chains where there are fewer tasks than fill the chip, by
// instructions beyond that (order 5859, 1024 complex tasks without the way back:
// 5.1 -> 1.8 ms a round of the device against one wave a task that updated sixteen
// columns of vectors, with it 2.6; 608 real tasks 1.15 -> 0.83).
template <bool COMPLEX>
__global__ void __launch_bounds__(128, COMPLEX ? 2 : 3)
spectral_w_kernel(const double *__restrict__ band, const double *__restrict__ Ut, int np, int nb16,
                  const SpectralTask *__restrict__ tasks, double2 *__restrict__ W_out, double2 *factors,
                  double *__restrict__ X) {
  constexpr int C2 = COMPLEX ? 2 : 1;
  __shared__ double rows[2][16 * 64 * C2];  // eliminated rows, [t][column]
  __shared__ double2 invs[2][16];           // 1/d_t
  const SpectralTask task = tasks[blockIdx.x];
  const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
  const bool up = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double *const row = rows[up];
  double2 *const dinv = invs[up];
  const double zr = (task.x - task.y) * (task.x + task.y), zi = COMPLEX ? 2.0 * task.x * task.y : 0.0;
  const double *u = Ut + (long long)(task.col + (COMPLEX ? 0 : min(li, task.nrhs - 1))) * np;
  const bool urow = li < task.nrhs;

  // Blocks p and p + `which` of the wave's order, in accumulator layout: element
  // r is [4 r + lk][li].  The upward wave's indices run backwards: its diagonal
  // tiles are turned by 180 degrees, the others transposed as well.
  auto tile_of = [&](bool back, int p, int which) {
    const double *b = band + (long long)(back ? nb16 - 1 - p - which : p) * 768 + which * 256 +
                      (!back ? lane : which ? 16 * (15 - li) + 15 - lk : 255 - lane);
    const int st = !back ? 64 : which ? -4 : -64;
    return d4{b[0], b[st], b[2 * st], b[3 * st]};
  };
  auto tile = [&](int p, int which) { return tile_of(up, p, which); };
  auto vec_of = [&](bool back, int p) {
    d4 v;
    const double *x = u + (back ? np - 1 - 16 * p - lk : 16 * p + lk);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const double y = x[back ? -4 * r : 4 * r];
      v[r] = urow ? y : 0.0;
    }
    return v;
  };
  auto vec = [&](int p) { return vec_of(up, p); };
  // COMPLEX: element li of the one vector's block p
  auto one_of = [&](bool back, int p) { return u[back ? np - 1 - 16 * p - li : 16 * p + li]; };
  auto shifted_diag = [&](const d4 &d, d4 &re, d4 &im) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const bool on = 4 * r + lk == li;
      re[r] = (on ? zr : 0.0) - d[r];
      im[r] = on ? zi : 0.0;
    }
  };
  auto put = [&](double *buf, int c, const d4 &re, const d4 &im) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      double *q = buf + ((4 * r + lk) * 64 + c + li) * C2;
      if (COMPLEX) *reinterpret_cast<double2 *>(q) = make_double2(re[r], im[r]);
      else *q = re[r];
    }
  };
  auto get = [&](const double *buf, int o, double &re, double &im) {
    if (COMPLEX) {
      const double2 v = *reinterpret_cast<const double2 *>(buf + o * C2);
      re = v.x;
      im = v.y;
    } else {
      re = buf[o];
      im = 0.0;
    }
  };
  const d4 zero{0.0, 0.0, 0.0, 0.0};
  const int half = nb16 / 2 - 1;  // steps of each wave; nb16 is even
  d4 s11r, s11i, s22r, s22i;
  shifted_diag(tile(0, 0), s11r, s11i);
  shifted_diag(tile(1, 0), s22r, s22i);
  d4 s12r = -tile(0, 1), s12i = zero, f = half > 0 ? -tile(0, 2) : zero;
  d4 y1 = zero, y2 = zero;
  double v1r = 0.0, v1i = 0.0, v2r = 0.0, v2i = 0.0;
  if (COMPLEX) {
    v1r = one_of(up, 0);
    v2r = one_of(up, 1);
    if (lk > 0) {  // the unused columns of the rows' fourth tile
#pragma unroll
      for (int t = 0; t < 16; t += 2) *reinterpret_cast<double2 *>(row + ((t + (lk & 1)) * 64 + 48 + li) * C2) = make_double2(0.0, 0.0);
    }
  } else {
    y1 = vec(0);
    y2 = vec(1);
  }
  auto put_one = [&](double *buf, int c, double re, double im) {
    if (lk == 0) *reinterpret_cast<double2 *>(buf + (li * 64 + c) * C2) = make_double2(re, im);
  };
  double wr = 0.0, wi = 0.0;
  // the factors of the wave's p-th block
  auto factor_of = [&](int p) { return factors + ((long long)blockIdx.x * nb16 + (up ? nb16 - 1 - p : p)) * SPECTRAL_ROWS; };

#pragma unroll 1
  for (int p = 0; p < half + 2; ++p) {
    if (p == half) {
      // the middle blocks: both waves' remainders less the matrix, which both hold
      if (up) {
        put(row, 0, s22r, s22i);
        put(row, 16, s12r, s12i);
        put(row, 32, s11r, s11i);
        if (COMPLEX) put_one(row, 48, v2r, v2i);
        else put(row, 48, y2, zero);
      }
      __syncthreads();
      if (up) {  // the other wave is through with its rows
        if (COMPLEX) put_one(rows[0], 0, v1r, v1i);
        else put(rows[0], 0, y1, zero);
        put(rows[0], 16, d4{wr, 0.0, 0.0, 0.0}, d4{wi, 0.0, 0.0, 0.0});  // not a tile: [lk][16 + li]
      }
      __syncthreads();
      if (up) break;
      d4 o11r, o11i, o22r, o22i;
      shifted_diag(tile_of(false, half, 0), o11r, o11i);
      shifted_diag(tile_of(false, half + 1, 0), o22r, o22i);
      const d4 o12 = -tile_of(false, half, 1);
      double ar, ai;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 15 - (4 * r + lk), j = 15 - li;  // where the upward wave has it
        get(rows[1], i * 64 + j, ar, ai);
        s11r[r] += ar - o11r[r];
        s11i[r] += ai - o11i[r];
        get(rows[1], j * 64 + 16 + i, ar, ai);
        s12r[r] += ar - o12[r];
        s12i[r] += ai;
        get(rows[1], i * 64 + 32 + j, ar, ai);
        s22r[r] += ar - o22r[r];
        s22i[r] += ai - o22i[r];
      }
      if (COMPLEX) {
        get(rows[1], (15 - li) * 64 + 48, ar, ai);
        v1r += ar - one_of(false, half);
        v1i += ai;
        get(rows[0], (15 - li) * 64, ar, ai);
        v2r += ar - one_of(false, half + 1);
        v2i += ai;
      } else {
        const d4 u1 = vec_of(false, half), u2 = vec_of(false, half + 1);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = 15 - (4 * r + lk);
          y1[r] += rows[1][i * 64 + 48 + li] - u1[r];
          y2[r] += rows[0][i * 64 + li] - u2[r];
        }
      }
      get(rows[0], lk * 64 + 16 + li, ar, ai);
      wr += ar;
      wi += ai;
      f = zero;
      wave_sync();
    }
    // the next step's fresh tiles
    d4 nd = zero, ne = zero, nf = zero, nu = zero;
    double nv = 0.0;
    if (p < half) {
      nd = tile(p + 2, 0);
      ne = tile(p + 1, 1);
      if (p + 1 < half) nf = tile(p + 1, 2);
      if (COMPLEX) nv = one_of(up, p + 2);
      else nu = vec(p + 2);
    }
    put(row, 0, s11r, s11i);
    put(row, 16, s12r, s12i);
    put(row, 32, f, zero);
    if (COMPLEX) put_one(row, 48, v1r, v1i);
    else put(row, 48, y1, zero);
    wave_sync();
    double mr[16], mi[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) get(row, t * 64 + lane, mr[t], mi[t]);
    wave_sync();
    double2 *const fac = COMPLEX ? factor_of(p) + (lane == 48 ? 0 : lane) : nullptr;
    const int keep_step = lane == 48 ? 33 : 32;  // the right-hand side's lane, or 32 t + lane
#pragma unroll
    for (int t = 0; t < 16; ++t) {
      const double dr = bcast(mr[t], t);
      double lr, lm;
      if (COMPLEX) {
        const double di = bcast(mi[t], t);
        const double q = fast_rcp(fma(dr, dr, di * di));
        const double ir = dr * q, ii = -di * q;
        if (lane == 0) dinv[t] = make_double2(ir, ii);
        lr = mr[t] * ir - mi[t] * ii;
        lm = mr[t] * ii + mi[t] * ir;
        wr += mr[t] * lr - mi[t] * lm;
        wi += mr[t] * lm + mi[t] * lr;
        if (lane == 48 || (unsigned)(lane - t - 1) < 32u) fac[t * keep_step] = make_double2(lr, lm);
#pragma unroll
        for (int i = t + 1; i < 16; ++i) {
          const double a = bcast(lr, i), b = bcast(lm, i);
          mr[i] = fma(b, mi[t], fma(-a, mr[t], mr[i]));
          mi[i] = fma(-b, mr[t], fma(-a, mi[t], mi[i]));
          asm volatile("" : "+v"(mr[i]), "+v"(mi[i]));  // now, or the broadcasts spill
        }
        *reinterpret_cast<double2 *>(row + (t * 64 + lane) * C2) = make_double2(mr[t], mi[t]);
      } else {
        const double q = fast_rcp(dr);
        if (lane == 0) dinv[t].x = q;
        lr = mr[t] * q;
        wr += mr[t] * lr;
#pragma unroll
        for (int i = t + 1; i < 16; ++i) {
          mr[i] = fma(-bcast(lr, i), mr[t], mr[i]);
          asm volatile("" : "+v"(mr[i]));
        }
        row[t * 64 + lane] = mr[t];
      }
    }
    wave_sync();
    // what is left on blocks p + 1, p + 2
    d4 n11r = s22r, n11i = s22i, n12r = -ne, n12i = zero, n22r, n22i, ny1 = y2, ny2 = nu;
    double m1r = 0.0, m1i = 0.0, m2r = 0.0, m2i = 0.0;
    shifted_diag(nd, n22r, n22i);
    auto add = [&](d4 &re, d4 &im, double ar, double ai, double br, double bi) {
      re = mfma(-ar, br, re);
      if (COMPLEX) {
        re = mfma(ai, bi, re);
        im = mfma(-ar, bi, im);
        im = mfma(-ai, br, im);
      }
    };
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int t = 4 * s + lk;
      double a1r, a1i, a2r, a2i, b1r, b1i, b2r, b2i, cr, ci;
      get(row, t * 64 + 16 + li, b1r, b1i);
      get(row, t * 64 + 32 + li, b2r, b2i);
      get(row, t * 64 + 48 + (COMPLEX ? 0 : li), cr, ci);
      const double2 q = dinv[t];
      if (COMPLEX) {
        a1r = b1r * q.x - b1i * q.y;
        a1i = b1r * q.y + b1i * q.x;
        a2r = b2r * q.x - b2i * q.y;
        a2i = b2r * q.y + b2i * q.x;
      } else {
        a1r = b1r * q.x;
        a2r = b2r * q.x;
        a1i = a2i = 0.0;
      }
      add(n11r, n11i, a1r, a1i, b1r, b1i);
      add(n12r, n12i, a1r, a1i, b2r, b2i);
      add(n22r, n22i, a2r, a2i, b2r, b2i);
      if (COMPLEX) {
        m1r = fma(a1r, cr, fma(-a1i, ci, m1r));
        m1i = fma(a1r, ci, fma(a1i, cr, m1i));
        m2r = fma(a2r, cr, fma(-a2i, ci, m2r));
        m2i = fma(a2r, ci, fma(a2i, cr, m2i));
      } else {
        ny1 = mfma(-a1r, cr, ny1);
        ny2 = mfma(-a2r, cr, ny2);
      }
    }
    wave_sync();
    s11r = n11r; s11i = n11i; s12r = n12r; s12i = n12i; s22r = n22r; s22i = n22i;
    if (COMPLEX) {
      v1r = v2r - row_sum(m1r);
      v1i = v2i - row_sum(m1i);
      v2r = nv - row_sum(m2r);
      v2i = -row_sum(m2i);
    } else {
      y1 = ny1;
      y2 = ny2;
    }
    f = -nf;
  }
  if (!COMPLEX) {
    if (!up && lane >= 48 && lane - 48 < task.nrhs)
      W_out[task.out_base + (long long)(lane - 48) * task.out_stride] = make_double2(wr, wi);
    return;
  }
  if (!up && lane == 48) W_out[blockIdx.x] = make_double2(wr, wi);
  // back: window[16 ..] holds x of the two blocks behind the one being solved
  __shared__ d2 windows[2][48];
  d2 *const window = windows[up], *const rowz = reinterpret_cast<d2 *>(row);
  constexpr int LOADS = (SPECTRAL_ROWS + 63) / 64;
  static_assert(SPECTRAL_ROWS == 16 * 33 && LOADS == 9, "16 rows of 33; the ninth load takes the last 16");
  auto load = [&](int p, d2(&v)[LOADS]) {
    const d2 *f = reinterpret_cast<const d2 *>(factor_of(p));
#pragma unroll
    for (int q = 0; q < LOADS; ++q) v[q] = f[min(64 * q + lane, SPECTRAL_ROWS - 1)];
  };
  // x of a block, element li in every lane
  auto solve = [&](const d2(&v)[LOADS], double &xr, double &xi) {
#pragma unroll
    for (int q = 0; q < LOADS - 1; ++q) rowz[64 * q + lane] = v[q];
    if (lane < 16) rowz[64 * (LOADS - 1) + lane] = v[LOADS - 1];
    wave_sync();
    const d2 *r = rowz + 33 * li;
    const d2 y = r[0];
    double sr = lk == 0 ? y.x : 0.0, si = lk == 0 ? y.y : 0.0;
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      const int k = 1 + lk + 4 * c;
      const d2 m = r[k], x = window[li + k];  // zero inside the block
      sr = fma(m.y, x.y, fma(-m.x, x.x, sr));
      si = fma(-m.y, x.x, fma(-m.x, x.y, si));
    }
    d2 m[16];
#pragma unroll
    for (int t = 1; t < 16; ++t) {
      m[t] = r[max(t - li, 0)];
      m[t] *= li < t ? 1.0 : 0.0;
    }
    sr = row_sum(sr);
    si = row_sum(si);
    for_each_index<15>([&](auto ic) {
      constexpr int t = 15 - decltype(ic)::value;
      const double a = row_bcast<t>(sr), b = row_bcast<t>(si);
      sr = fma(m[t].y, b, fma(-m[t].x, a, sr));
      si = fma(-m[t].y, a, fma(-m[t].x, b, si));
    });
    xr = sr;
    xi = si;
    wave_sync();
  };
  auto keep = [&](int p, double xr, double xi) {
    const int at = up ? np - 1 - 16 * p - li : 16 * p + li;
    if (lk < 2) X[((long long)blockIdx.x + (lk ? gridDim.x : 0)) * np + at] = lk ? xi : xr;
    if (lk == 0) {
      window[32 + li] = window[16 + li];
      window[16 + li] = d2{xr, xi};
    }
    wave_sync();
  };
  d2 v[LOADS], next[LOADS];
  double xr, xi;
  if (!up) {
    if (lane < 48) window[lane] = d2{0.0, 0.0};
    load(half + 1, v);
    load(half, next);
    wave_sync();
    solve(v, xr, xi);
    keep(half + 1, xr, xi);
    if (lk == 0) windows[1][16 + 15 - li] = d2{xr, xi};  // the upward wave's order
    solve(next, xr, xi);
    keep(half, xr, xi);
    if (lk == 0) {
      windows[1][32 + 15 - li] = d2{xr, xi};
      windows[1][li] = d2{0.0, 0.0};
    }
  }
  if (half > 0) load(half - 1, v);
  __syncthreads();
#pragma unroll 1
  for (int p = half - 1; p >= 0; --p) {
    if (p > 0) load(p - 1, next);
    solve(v, xr, xi);
    keep(p, xr, xi);
#pragma unroll
    for (int q = 0; q < LOADS; ++q) v[q] = next[q];
  }
}

// w = b + y in the place of y (real parts of the T tasks, then imaginary ones),
// and by blocks of YROWS rows the sums of y^2 (complex) and of b^2.
constexpr int YROWS = 32, GROWS = 64;
__global__ void __launch_bounds__(64)
spectral_shift_kernel(double *__restrict__ Y, int ldy, int n_aux, const double *__restrict__ B, int ldb,
                      const SpectralTask *__restrict__ tasks, int T, double *__restrict__ part) {
  const int t = blockIdx.x * 64 + threadIdx.x;
  if (t >= T) return;
  const double *b = B + tasks[t].col;
  const int P0 = blockIdx.y * YROWS, P1 = min(n_aux, P0 + YROWS);
  double sr = 0.0, si = 0.0, sb = 0.0;
#pragma unroll 8
  for (int P = P0; P < P1; ++P) {
    double *y = Y + (long long)P * ldy + t;
    const double yr = y[0], yi = y[T], bp = b[(long long)P * ldb];
    sr = fma(yr, yr, fma(-yi, yi, sr));
    si = fma(2.0 * yr, yi, si);
    sb = fma(bp, bp, sb);
    y[0] = bp + yr;
  }
  double *o = part + (long long)blockIdx.y * 3 * T + t;
  o[0] = sr;
  o[T] = si;
  o[2 * T] = sb;
}

// By blocks of GROWS transitions the sums of g^2 / (z^2 - Delta^2), g = V^T w.
__global__ void __launch_bounds__(64)
spectral_poles_kernel(const double *__restrict__ G, int ldg, int np, int pad, const double *__restrict__ delta,
                      const SpectralTask *__restrict__ tasks, int T, double *__restrict__ part) {
  const int t = blockIdx.x * 64 + threadIdx.x;
  if (t >= T) return;
  const double x = tasks[t].x, y = tasks[t].y, y2 = y * y, im = 2.0 * x * y;
  const int k0 = max(pad, (int)blockIdx.y * GROWS), k1 = min(np, ((int)blockIdx.y + 1) * GROWS);
  double sr = 0.0, si = 0.0;
#pragma unroll 4
  for (int k = k0; k < k1; ++k) {
    const double d = delta[k - pad], re = (x - d) * (x + d) - y2, q = 1.0 / fma(re, re, im * im);
    const double gr = G[(long long)k * ldg + t], gi = G[(long long)k * ldg + T + t];
    const double ar = fma(gr, gr, -gi * gi) * q, ai = 2.0 * gr * gi * q;
    sr = fma(ar, re, fma(ai, im, sr));
    si = fma(ai, re, fma(-ar, im, si));
  }
  double *o = part + (long long)blockIdx.y * 2 * T + t;
  o[0] = sr;
  o[T] = si;
}

// W = w^T Pi w - y^T y.  The band's own W is off by the first-order error e of
// the reduction, this one by its square times |1 - Pi| (up to some hundreds next
// to a pole): where they differ by more than 1e-8, that may be above rounding,
// and the flag sends the call to the Pi builds.  (Measured differences: up to
// 1e-11.  The second term is rounding of W where it cancels against b^T b.)
__global__ void __launch_bounds__(64)
spectral_finish_kernel(const double *__restrict__ part_y, int ny, const double *__restrict__ part_g, int ng,
                       const double2 *__restrict__ W_band, const SpectralTask *__restrict__ tasks, int T,
                       double2 *__restrict__ W_out, int *__restrict__ flag) {
  const int t = blockIdx.x * 64 + threadIdx.x;
  if (t >= T) return;
  double yr = 0.0, yi = 0.0, bb = 0.0, gr = 0.0, gi = 0.0;
#pragma unroll 4
  for (int k = 0; k < ny; ++k) {
    const double *o = part_y + (long long)k * 3 * T + t;
    yr += o[0];
    yi += o[T];
    bb += o[2 * T];
  }
#pragma unroll 8
  for (int k = 0; k < ng; ++k) {
    const double *o = part_g + (long long)k * 2 * T + t;
    gr += o[0];
    gi += o[T];
  }
  const double wr = gr - yr, wi = gi - yi;
  const double2 w0 = W_band[t];
  const double off = fmax(fabs(wr - w0.x), fabs(wi - w0.y));
  if (!(off <= 1e-8 * fmax(fabs(wr), fabs(wi)) + 1e-13 * bb)) atomicOr(flag, 1);
  W_out[tasks[t].out_base] = make_double2(wr, wi);
}

size_t spectral_small_bytes() { return sizeof(PanelSmall); }
int spectral_gram_parts(int np) { return (np + UT - 1) / UT * 768; }
int spectral_xsum_parts(int np) {
  return std::max((np + XROWS - 1) / XROWS * SB * SB, (np + PROWS - 1) / PROWS * Q_PART2);
}

void launch_spectral_operand(const double *M_ov, const double *eps, const int *perm, int n_aux, int n_occ,
                             int n_virt, int pad, int np, double *V, hipStream_t s) {
  dim3 grid((np + 255) / 256, std::min(n_aux, 256));
  spectral_operand_kernel<<<grid, 256, 0, s>>>(M_ov, eps, perm, n_aux, n_occ, n_virt, pad, np, V);
}

void launch_spectral_pairs(const double *M_oo, const double *M_ov, int n_aux, int n_occ, int n_virt,
                           const int *core, int R, int Rp, double *B, hipStream_t s) {
  dim3 grid((Rp + 255) / 256, std::min(n_aux, 256));
  spectral_pairs_kernel<<<grid, 256, 0, s>>>(M_oo, M_ov, n_aux, n_occ, n_virt, core, R, Rp, B);
}

static void transpose(const double *in, long long ldi, int rows, int cols, double *out, long long ldo, int rows_out,
                      hipStream_t s) {
  spectral_transpose_kernel<<<dim3((rows_out + 31) / 32, (cols + 31) / 32), 256, 0, s>>>(in, ldi, rows, cols, out, ldo, rows_out);
}

// out[i][j] = sum_P A[P][i] B[P][j]: 128 x 128 tiles where they nearly fill the 512
// that run at once, else 64 x 64 (1216 x 5888 products for 1680 to 3072 tasks: 270
// large tiles 1.66 ms against 1.49, 370 1.71 against 1.56, 480 1.59 against 2.7).
static void product(const double *A, int lda, const double *B, int ldb, int M, int N, int K, double *out, long long ldo,
                    hipStream_t s) {
  auto tiles = [&](int t) { return ((M + t - 1) / t) * ((N + t - 1) / t); };
  if (tiles(2 * UT) >= 384)
    spectral_gemm_kernel<false, 4><<<tiles(2 * UT), 256, 0, s>>>(A, lda, B, ldb, M, N, K, nullptr, 0, out, ldo);
  else
    spectral_gemm_kernel<false, 2><<<tiles(UT), 256, 0, s>>>(A, lda, B, ldb, M, N, K, nullptr, 0, out, ldo);
}

void launch_spectral_matrix(const double *V, int np, int Np, int n_aux, const double *delta, int pad, double *A,
                            long long lda, hipStream_t s) {
  const int nt = (np + UT - 1) / UT, nt2 = (np + 2 * UT - 1) / (2 * UT);
  // 128 x 128 tiles from where they are twice what runs at once (512): at order
  // 16544 15.5 -> 11.0 ms, at 5888 1.03 -> 0.85 ms, at 1056 0.053 against 0.079.
  if (np >= 4096)
    spectral_gemm_kernel<true, 4><<<triangle_tiles(nt2), 256, 0, s>>>(V, np, V, np, np, np, n_aux, delta, pad, A, lda);
  else
    spectral_gemm_kernel<true, 2><<<triangle_tiles(nt), 256, 0, s>>>(V, np, V, np, np, np, n_aux, delta, pad, A, lda);
  transpose(V, np, n_aux, np, A + np, lda, Np, s);
}

void launch_spectral_reduce(double *A, long long lda, int np, int Rp, const SpectralWork &w, hipStream_t s) {
  PanelSmall *sm = static_cast<PanelSmall *>(w.small);
  const int panels = np / SB - 1;
  if (panels < 1) return;
  // One reflection: of the matrix A22 (m rows, u's columns behind) by the panel P
  // (transposed); `second`: of a pair; `strip`: the pair's first, whose update of
  // all but the next panel waits for the second's.
  auto reflect = [&](const double *P, long long ldp, double *A22, int m, double *Bk, bool second, bool strip) {
    // rows of the first panel's Y and W from this panel's first row on
    const double *Ya = w.Y[0] + SB * SB, *Wa = w.W[0] + SB * SB;
    double *Y = w.Y[second], *W = w.W[second];
    const int mx = m + Rp, ng = (m + PROWS - 1) / PROWS, nx = mx / SB;
    // splits of the rows: about eight workgroups a CU, a wave's part at least 32 rows
    const int splits = std::max(1, std::min({SPECTRAL_MAX_SPLITS, 2048 / nx, m / 128}));
    const unsigned gx = 1 + nx * splits, gs = (mx + XROWS - 1) / XROWS;
    if (second) {
      panel_q_kernel<true><<<ng, PROWS, 0, s>>>(P, ldp, m, sm, Ya, Wa, w.Q, w.part);
      panel_x_kernel<true><<<gx, 256, 0, s>>>(A22, lda, m, mx, splits, w.Q, w.Xpart, w.part, ng, Ya, Wa, sm, w.flag, Bk);
      panel_xsum_kernel<true><<<gs, XTHREADS, 0, s>>>(w.Xpart, splits, A22, lda, m, mx, w.Q, Ya, Wa, sm, sm, w.X, Y, w.part, w.ticket);
    } else {
      panel_q_kernel<false><<<ng, PROWS, 0, s>>>(P, ldp, m, sm, nullptr, nullptr, w.Q, w.part);
      panel_x_kernel<false><<<gx, 256, 0, s>>>(A22, lda, m, mx, splits, w.Q, w.Xpart, w.part, ng, nullptr, nullptr, sm, w.flag, Bk);
      panel_xsum_kernel<false><<<gs, XTHREADS, 0, s>>>(w.Xpart, splits, A22, lda, m, mx, w.Q, nullptr, nullptr, sm, sm, w.X, Y, w.part, w.ticket);
    }
    panel_w_kernel<<<(mx + 63) / 64, 256, 0, s>>>(w.X, Y, m, mx, sm, W);
    const double *y0 = second ? Ya : Y, *w0 = second ? Wa : W, *y1 = second ? Y : nullptr, *w1 = second ? W : nullptr;
    const int nt = (m + UT - 1) / UT, nu = (Rp + UT - 1) / UT;
    const unsigned tri = triangle_tiles(nt);
    if (strip) panel_update_kernel<true><<<nt + nu, 256, 0, s>>>(A22, lda, m, mx, y0, w0, y1, w1, nt, sm, w.part, w.ticket, w.flag);
    else panel_update_kernel<false><<<tri + nt * nu, 256, 0, s>>>(A22, lda, m, mx, y0, w0, y1, w1, (int)tri, sm, w.part, w.ticket, w.flag);
  };
  // the first coordinates, pseudo-random: their panel in X, which is written only
  // after the panel has been read; its coupling goes to Bk's last block, which no
  // pair of diagonal blocks uses
  const long long count = (long long)SB * np;
  panel_start_kernel<<<(unsigned)((count + 255) / 256), 256, 0, s>>>(w.X, count);
  panel_gram_kernel<<<(np + PROWS - 1) / PROWS, PROWS, 0, s>>>(w.X, np, np, sm, w.part, w.ticket, w.flag);
  reflect(w.X, np, A, np, w.Bk + (long long)panels * SB * SB, false, false);
  bool pair = false, second = false;
  for (int k = 0; k < panels; ++k) {
    const int c0 = k * SB, r0 = c0 + SB, m = np - r0;
    second = (k & 1) && pair;
    // a pair saves a pass over A22 and costs products of its own
    pair = !(k & 1) && k + 1 < panels && m >= PAIR_ROWS;
    reflect(A + (long long)c0 * lda + r0, lda, A + (long long)r0 * lda + r0, m, w.Bk + (long long)k * SB * SB, second, pair);
  }
}

void launch_spectral_pack(const double *A, long long lda, int np, int Np, int n_aux, const double *Bk, const double *Bp,
                          int Rp, double *band, double *Vt, double *Vh, double *Ut, hipStream_t s) {
  spectral_band_kernel<<<np / 16 + 2, 256, 0, s>>>(A, lda, Bk, np / SB, band);
  transpose(A + np, lda, np, n_aux, Vt, np, np, s);
  transpose(Vt, np, n_aux, np, Vh, Np, Np, s);
  product(Bp, Rp, Vt, np, Rp, np, n_aux, Ut, np, s);
}

void launch_spectral_w(const double *band, const double *Ut, int np, const SpectralTask *tasks, int n_tasks,
                       double2 *W_out, hipStream_t s) {
  spectral_w_kernel<false><<<n_tasks, 128, 0, s>>>(band, Ut, np, np / 16, tasks, W_out, nullptr, nullptr);
}

int spectral_columns(int T) { return (2 * T + SB - 1) / SB * SB; }
size_t spectral_residue_parts(int n_aux, int np, int T) {
  return (size_t)T * (3 * ((n_aux + YROWS - 1) / YROWS) + 2 * ((np + GROWS - 1) / GROWS));
}

void launch_spectral_residues(const double *band, const double *Ut, int np, int pad, const double *V, int n_aux,
                              const double *Vh, int Np, const double *Bp, int Rp, const double *delta,
                              const SpectralTask *tasks, int T, const SpectralResidueWork &w, double2 *W_out, int *flag,
                              hipStream_t s) {
  const int C = spectral_columns(T), tb = (T + 63) / 64;
  const int ny = (n_aux + YROWS - 1) / YROWS, ng = (np + GROWS - 1) / GROWS;
  double *part_y = w.part, *part_g = part_y + (size_t)3 * ny * T;
  spectral_w_kernel<true><<<T, 128, 0, s>>>(band, Ut, np, np / 16, tasks, w.W, w.factors, w.X);
  transpose(w.X, np, 2 * T, np, w.XG, C, C, s);
  product(Vh, Np, w.XG, C, Np, C, np, w.Y, C, s);  // y = V H x
  spectral_shift_kernel<<<dim3(tb, ny), 64, 0, s>>>(w.Y, C, n_aux, Bp, Rp, tasks, T, part_y);
  product(V, np, w.Y, C, np, C, n_aux, w.XG, C, s);  // g = V^T w
  spectral_poles_kernel<<<dim3(tb, ng), 64, 0, s>>>(w.XG, C, np, pad, delta, tasks, T, part_g);
  spectral_finish_kernel<<<tb, 64, 0, s>>>(part_y, ny, part_g, ng, w.W, tasks, T, W_out, flag);
}

}  // namespace gwc
