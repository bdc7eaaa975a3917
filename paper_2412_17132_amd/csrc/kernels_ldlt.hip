// Screened-interaction elements from a bordered LDL^T factorisation without
// pivoting (FP64 complex symmetric).
//
// 1 - Pi(z) is complex symmetric (Pi = L diag(chi) L^T).  On the real axis,
// z = x + i eta with x > 0, every Im chi_ia < 0, so Im(1 - Pi) = L |Im chi| L^T
// is positive semidefinite; on the imaginary axis 1 - Pi is real symmetric
// positive definite.  Then v^T (1 - Pi) v has a positive imaginary (or real)
// part for every real nonzero v restricted to a leading block, so every
// leading principal minor is nonsingular and the elimination needs no
// pivoting.  The bordered matrix
//
//        [ 1 - Pi(z)   B ]
//   M =  [ B^T         0 ]      (symmetric, order n = N + R)
//
// is factored L D L^T over its first N columns; the border block then holds
// the Schur complement -B^T (1 - Pi)^-1 B, and W^c = -S_rr - b^T b as for the
// LU (launch_bordered_finish).  Only the lower triangle is read.
//
// Right-looking, 64-column steps, per step and batch of matrices:
//   D  one workgroup per matrix: the 64 x 64 diagonal block A11 = L11 D1 L11^T
//      and L11^-1 (unit lower, to the scratch), 16 pivots at a time in one
//      wave's registers; D1^-1 to the matrix's row of pivots' inverses;
//   T  one workgroup per (matrix, 64-row block below the panel): W = A21 L11^-T
//      on MFMA from the block staged in LDS, stored transposed in the row part
//      (the upper triangle, otherwise unused): W^T = D1 L21^T, so that
//   G  the trailing update A22 -= L21 (W^T) = L21 D1 L21^T is the LU's
//      trailing kernel restricted to the tiles on or below the diagonal
//      (half the tiles; border-border tiles off the diagonal skipped), both
//      operands read from the row part (L21[r][k] = W^T[k][r] / D[k]: the
//      left operand's loads are coalesced along r and no column part is
//      written).
// Up to LDLT_GROUP panels share one trailing update (K = 64 LDLT_GROUP), a
// later panel of a group first receiving the group's earlier panels on its own
// 64 columns.  Against the partial-pivoting LU this halves the trailing flops
// and removes the pivot searches, interchanges and row moves.
#include "gwc_internal.h"

namespace gwc {

namespace {

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int NB = 64;
constexpr int NXCD = 8;
constexpr int LDLT_GROUP = 4;

// Workgroup -> (matrix, item), all items of a matrix on one XCD.
__device__ __forceinline__ bool xcd_item(int wg, int items, int F, int &f, int &item) {
  const int x = wg % NXCD, j = wg / NXCD;
  f = (j / items) * NXCD + x;
  item = j - (j / items) * items;
  return f < F;
}

__device__ __forceinline__ double bcast(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

// 1/d, scaled by a power of two against overflow; the reciprocal by Newton
// steps from the hardware's estimate (short dependent chain).
__device__ __forceinline__ double2 zinv_fast(double2 d) {
  const int e = __builtin_amdgcn_frexp_exp(fmax(fabs(d.x), fabs(d.y)));
  const double x = ldexp(d.x, -e), y = ldexp(d.y, -e), q = fma(x, x, y * y);
  double r = __builtin_amdgcn_rcp(q);
  r = fma(fma(-q, r, 1.0), r, r);
  r = fma(fma(-q, r, 1.0), r, r);
  r = fma(fma(-q, r, 1.0), r, r);
  return make_double2(ldexp(x * r, -e), ldexp(-y * r, -e));
}

// C -= M^T B of 16 x 16 tiles (C = -M^T B where `clear`), complex, on MFMA:
// rows t of M (stride NB) and B (stride ldb), C row-major.
__device__ __forceinline__ void rank_tile(double2 *C, bool clear, const double2 *M, const double2 *B, int ldb, int li,
                                          int lk) {
  d4 cr, ci;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const double2 x = clear ? make_double2(0.0, 0.0) : C[(4 * r + lk) * 16 + li];
    cr[r] = x.x;
    ci[r] = x.y;
  }
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int t = 4 * s + lk;
    const double2 x = M[t * NB + li], y = B[t * ldb + li];
    cr = __builtin_amdgcn_mfma_f64_16x16x4f64(-x.x, y.x, cr, 0, 0, 0);
    cr = __builtin_amdgcn_mfma_f64_16x16x4f64(x.y, y.y, cr, 0, 0, 0);
    ci = __builtin_amdgcn_mfma_f64_16x16x4f64(-x.x, y.y, ci, 0, 0, 0);
    ci = __builtin_amdgcn_mfma_f64_16x16x4f64(-x.y, y.x, ci, 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) C[(4 * r + lk) * 16 + li] = make_double2(cr[r], ci[r]);
}

// D: one workgroup (4 waves) per matrix.  The kb x kb diagonal block (identity
// beyond kb) as 16 x 16 tiles of its upper triangle in LDS.  Stage h: wave 0
// takes the rows of block h into registers, one column per lane, and
// eliminates their 16 pivots; a pivot's multipliers are its row over d (the
// block is symmetric), broadcast from the lanes that hold them.  The lanes left
// of the block hold the rows of L11^-1 found so far (they take the same row
// operations).  Then wave 0 inverts the block's unit lower triangle while the
// others subtract the rows' product from the tiles below, on MFMA; the tiles of
// L11^-1 move into the slots of the eliminated row, and its finished rows go to
// the scratch.  D1^-1 goes to dinv_g[f N + K0 + t].  Bound by the pivots' chain
// of dependent steps.  (64 steps with a barrier each, twice, before.)
__global__ void __launch_bounds__(256, 2)
ldlt_diag_kernel(const double2 *__restrict__ G, long long gs, int ldg, int N, int K0,
                 double2 *__restrict__ linv_g, double2 *__restrict__ dinv_g, int *__restrict__ status) {
  constexpr int TB = 16, NT = NB / TB;
  __shared__ double2 X[NT * (NT + 1) / 2][TB * TB];
  __shared__ double2 U[TB][NB], Mul[TB][NB], Ek[TB][TB];
  const int f = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, li = lane & 15, lk = lane >> 4;
  const double2 *A = G + (long long)f * gs;
  const int kb = min(NB, N - K0);
  // slot of the tile of blocks i <= j (and of L11^-1's tile (j, i))
  auto slot = [](int i, int j) { return i * NT - i * (i - 1) / 2 + j - i; };
  {
    // all of a thread's loads in flight before its first LDS store; every load
    // from an element inside the block, of the stored lower triangle
    constexpr int PER = NT * (NT + 1) / 2;
    double2 v[PER];
    const int r = tid >> 4, c = tid & 15;
    int q = 0;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = i; j < NT; ++j, ++q) {
        const int row = min(max(TB * i + r, TB * j + c), kb - 1), col = min(min(TB * i + r, TB * j + c), kb - 1);
        v[q] = A[(long long)(K0 + row) * ldg + K0 + col];
      }
    q = 0;
#pragma unroll
    for (int i = 0; i < NT; ++i)
#pragma unroll
      for (int j = i; j < NT; ++j, ++q) {
        const int gi = TB * i + r, gj = TB * j + c;
        X[q][tid] = gi < kb && gj < kb ? v[q] : make_double2(gi == gj ? 1.0 : 0.0, 0.0);
      }
  }
  double2 *Li = linv_g + (long long)f * NB * NB;
  const int stages = (kb + TB - 1) / TB;
  for (int e = stages * TB * NB + tid; e < NB * NB; e += 256) Li[e] = make_double2(0.0, 0.0);
  bool zero = false;
  for (int h = 0; h < stages; ++h) {
    __syncthreads();
    if (wave == 0) {
      const int jb = lane >> 4, p0 = TB * h;
      const double2 *src = X[jb < h ? slot(jb, h) : slot(h, jb)] + li;
      double mr[TB], mi[TB];
      double2 dv = make_double2(0.0, 0.0);
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        const double2 x = src[t * TB];
        mr[t] = x.x;
        mi[t] = x.y;
      }
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        const double2 d = make_double2(bcast(mr[t], p0 + t), bcast(mi[t], p0 + t));
        const bool dz = d.x == 0.0 && d.y == 0.0;
        zero = zero || dz;
        double2 inv = zinv_fast(d);
        if (dz) inv = make_double2(0.0, 0.0);
        if (lane == t) dv = inv;
        const double lr = mr[t] * inv.x - mi[t] * inv.y, lm = mr[t] * inv.y + mi[t] * inv.x;
        U[t][lane] = make_double2(mr[t], mi[t]);
        Mul[t][lane] = make_double2(lr, lm);
#pragma unroll
        for (int i = t + 1; i < TB; ++i) {
          const double a = bcast(lr, p0 + i), b = bcast(lm, p0 + i);
          mr[i] = fma(b, mi[t], fma(-a, mr[t], mr[i]));
          mi[i] = fma(-b, mr[t], fma(-a, mi[t], mi[i]));
        }
      }
      if (lane < TB && p0 + lane < kb) dinv_g[(long long)f * N + K0 + p0 + lane] = dv;
    }
    __syncthreads();
    if (wave == 0) {
      // the diagonal tile of L11^-1, a column per lane (four copies)
      double er[TB], ei[TB];
#pragma unroll
      for (int t = 0; t < TB; ++t) {
        er[t] = li == t ? 1.0 : 0.0;
        ei[t] = 0.0;
      }
#pragma unroll
      for (int t = 0; t < TB - 1; ++t)
#pragma unroll
        for (int i = t + 1; i < TB; ++i) {
          const double2 l = Mul[t][TB * h + i];
          er[i] = fma(l.y, ei[t], fma(-l.x, er[t], er[i]));
          ei[i] = fma(-l.y, er[t], fma(-l.x, ei[t], ei[i]));
        }
#pragma unroll
      for (int t = 0; t < TB; ++t)
        if (lane < TB) Ek[t][lane] = make_double2(er[t], ei[t]);
    } else {
      // rows below: tiles (i, j), i > h, with j >= i of the block and j < h of L11^-1
      int q = 0;
      for (int i = h + 1; i < NT; ++i)
        for (int j = 0; j < NT; ++j) {
          if (j >= h && j < i) continue;
          if (q++ % 3 != wave - 1) continue;
          rank_tile(X[j < i ? slot(j, i) : slot(i, j)], false, &Mul[0][TB * i], &U[0][TB * j], NB, li, lk);
        }
    }
    __syncthreads();
    // and j = h, with the rows of L11^-1 that are now final
    for (int i = h + 1 + wave; i < NT; i += 4) rank_tile(X[slot(h, i)], true, &Mul[0][TB * i], &Ek[0][0], TB, li, lk);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = 4 * q + wave, row = TB * h + r, c = lane;
      const double2 x = c < TB * h ? U[r][c] : Ek[r][c & 15];
      Li[row * NB + c] = row < kb && c <= row ? x : make_double2(0.0, 0.0);
    }
  }
  if (tid == 0 && zero) status[f] = 1;
}

// T: one workgroup (4 waves) per (matrix, 64-row block of rows r0.. below the
// panel).  The A21 block is staged through LDS (coalesced rows); each wave
// forms 16 rows of W = A21 L11^-T on MFMA (L11^-1 from L2, shared by the
// matrix's workgroups on its XCD); W goes back to LDS and is stored
// transposed into the row part, A[K0 + k][r] = W[r][k], along contiguous
// rows.  Columns >= kb of the block are zero in LDS, rows >= n are not
// stored.  MFMA layouts: A[l%16][l/16], B[l/16][l%16], D[4r + l/16][l%16].
__global__ void __launch_bounds__(256)
ldlt_trsm_kernel(double2 *__restrict__ G, long long gs, int ldg, int N, int R, int K0, int F,
                 int nblk, const double2 *__restrict__ linv_g) {
  __shared__ double2 S[NB][NB + 1];
  int f, blk;
  if (!xcd_item(blockIdx.x, nblk, F, f, blk)) return;
  const int n = N + R;
  const int kb = min(NB, N - K0);
  const int r0 = K0 + kb + NB * blk;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  double2 *A = G + (long long)f * gs;
  const double2 *Li = linv_g + (long long)f * NB * NB;
  // all of a thread's loads in flight before its first LDS store
  constexpr int PER = NB * NB / 256;
  double2 v[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int idx = q * 256 + tid, r = idx / NB, k = idx - r * NB;
    v[q] = (r0 + r < n && k < kb) ? A[(long long)(r0 + r) * ldg + K0 + k] : make_double2(0.0, 0.0);
  }
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int idx = q * 256 + tid;
    S[idx / NB][idx % NB] = v[q];
  }
  __syncthreads();
  d4 re[4], im[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    re[b] = d4{0.0, 0.0, 0.0, 0.0};
    im[b] = d4{0.0, 0.0, 0.0, 0.0};
  }
  const int wr = 16 * wave;
  // the whole K of 64 unrolled (S and L11^-1 are zero beyond kb), so that the
  // L11^-1 loads of later steps are issued ahead of the products
#pragma unroll
  for (int kk = 0; kk < NB; kk += 4) {
    const int k = kk + lk;
    // A operand: rows wr + li of the block, column k; B operand:
    // L11^-T [k][c] = L11^-1 [c][k] (zero for k >= kb), c = 16 b + li.
    // Column block b needs k <= 16 b + 15 only: L11^-1 is lower triangular.
    const double2 av = S[wr + li][k];
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      if (kk < 16 * b + 16) {
        const double2 bv = Li[(16 * b + li) * NB + k];
        re[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.x, bv.x, re[b], 0, 0, 0);
        re[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(-av.y, bv.y, re[b], 0, 0, 0);
        im[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.x, bv.y, im[b], 0, 0, 0);
        im[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(av.y, bv.x, im[b], 0, 0, 0);
      }
    }
  }
  __syncthreads();  // every wave has read its A21 rows
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) S[wr + 4 * r + lk][16 * b + li] = make_double2(re[b][r], im[b][r]);
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int idx = q * 256 + tid, k = idx / NB, r = idx - k * NB;
    if (k < kb && r0 + r < n) A[(long long)(K0 + k) * ldg + r0 + r] = S[r][k];
  }
}

struct LdltLaunch {
  double2 *G;
  long long gs;
  int ldg, N, R, F, fgroups;
  double2 *linv, *dinv;
  int *status;
  bool real;
  hipStream_t s;

  void diag_trsm(int K0) const {
    const int n = N + R;
    const int kb = min(NB, N - K0);
    ldlt_diag_kernel<<<F, 256, 0, s>>>(G, gs, ldg, N, K0, linv, dinv, status);
    const int nblk = (n - K0 - kb + NB - 1) / NB;
    if (nblk > 0)
      ldlt_trsm_kernel<<<NXCD * fgroups * nblk, 256, 0, s>>>(G, gs, ldg, N, R, K0, F, nblk, linv);
  }
  // rows [r0, n) x columns [c0, c1) -= L[.., K range] W^T[K range, ..]
  void trailing(int r0, int c0, int c1, int kstart, int klen, bool lower) const {
    launch_trailing_update_sym(G, gs, ldg, N, R, F, r0, c0, c1, kstart, klen, lower, real, dinv, N, s);
  }
};

}  // namespace

// L11^-1 of the current panel per matrix, then every pivot's D^-1 per matrix.
size_t ldlt_scratch_bytes(int F, int N) {
  return (size_t)F * ((size_t)NB * NB + (size_t)N) * sizeof(double2) + 256;
}

hipError_t launch_ldlt_bordered(double2 *G, long long g_stride, int ldg, int N, int R, int F,
                                const double *bb, const long long *out_base, const int *out_stride,
                                double2 *W_out, int *status, void *scratch, bool real, hipStream_t stream) {
  const int n = N + R;
  double2 *linv = static_cast<double2 *>(scratch);
  double2 *dinv = linv + (size_t)F * NB * NB;
  launch_zero_status(status, F, stream);
  const LdltLaunch L{G, g_stride, ldg, N, R, F, (F + NXCD - 1) / NXCD, linv, dinv, status, real, stream};
  int K0 = 0;
  while (K0 < N) {
    const int g = min(LDLT_GROUP, (N - K0) / NB);
    if (g >= 2) {
      const int a = K0, e = K0 + g * NB;
      for (int p = 0; p < g; ++p) {
        const int b = a + p * NB;
        if (p > 0) L.trailing(b, b, b + NB, a, p * NB, false);
        L.diag_trsm(b);
      }
      L.trailing(e, e, n, a, g * NB, true);
      K0 = e;
    } else {
      const int kend = min(K0 + NB, N);
      L.diag_trsm(K0);
      L.trailing(kend, kend, n, K0, kend - K0, true);
      K0 = kend;
    }
  }
  launch_bordered_finish(G, g_stride, ldg, N, R, F, bb, out_base, out_stride, W_out, stream);
  return hipGetLastError();
}

}  // namespace gwc
