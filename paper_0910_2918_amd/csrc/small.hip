// The small problem of the sign approximation on gfx950: the k-vector z with
// sgn(A) x ~ ||x|| V_k z.
//
//  ell == 0 (non-nested, Eqs. (3)-(4)): z = sgn(H_k) e_1 by Roberts-Higham on
//  the dense k x k Ritz matrix.
//  ell  > 0 (nested, Sec. 3, Eqs. (5)-(6)): B = H_k + H_k^{-1}; an inner
//  Krylov space K_l(B, e_1) (Lanczos for Hermitian H_k, two-sided Lanczos
//  otherwise, full re-(bi)orthogonalisation); z = V_l sgn(H_l) e_1.
//
// H_k^{-1} comes from one LU factorisation of the tridiagonal H_k with
// partial pivoting (U has two super-diagonals), after which k threads solve
// H x = e_j for every column j at once and write B densely; the inner
// iteration then only needs dense mat-vecs with B (and B^dag), which spread
// over the whole GPU, instead of k-long sequential solves inside its loop.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

#include "hostbuf.h"
#include "nk_internal.h"
#include "wave.h"

namespace nk {

constexpr int LMAX = 512;  // largest inner size (LDS of k_in_sub)

// one inner problem
struct Inner {
  int k, herm, lmax;
  const C64 *al, *be, *de;  // H_k: diagonal, super- and sub-diagonal
  C64 *Lm, *U0i, *U1, *U2;  // its elimination
  int* Sw;
  int* out;      // host memory: receives the two flags at the last step
  C64* B;
  C64* BH;
  C64* V;
  C64* W;
  C64* uraw[2];  // ping-pong raw vectors (u side)
  C64* qraw[2];  // (q side)
  C64* part1;    // [2][nb1][lmax] partial projections from k_in_gemv
  C64* part2;    // [2][nb2][lmax] second-pass partial projections
  double* part3; // [4][nb2] normalisation partial sums
  int nb1, nb2;
  C64* a;
  C64* b;
  C64* d;
  // breakdown step (0: none), singular H_k, and the breakdown step from
  // k_in_gemv, which reads the first and writes this one, to k_in_sub, which
  // hands it on to the first: no launch reads what it writes
  int* flags;
  C64* hcol;     // [lmax][lmax] Arnoldi: column i of H_l at i * lmax (both passes summed)
  int arnoldi;   // 1: one-sided recurrence on a general B, every coefficient kept
};

__device__ __forceinline__ double cabs1s(C64 a) { return fabs(a.re) + fabs(a.im); }
// a b with the two ways to round the imaginary part
__device__ __forceinline__ C64 cmul_a(C64 a, C64 b) {
  return mk(fma(a.re, b.re, -(a.im * b.im)), fma(a.im, b.re, a.re * b.im));
}
__device__ __forceinline__ C64 cmul_b(C64 a, C64 b) {
  return mk(fma(a.re, b.re, -(a.im * b.im)), fma(a.re, b.im, a.im * b.re));
}
// c ? a : b by component (a select of two structs goes through scratch memory)
__device__ __forceinline__ C64 csel(bool c, C64 a, C64 b) { return mk(c ? a.re : b.re, c ? a.im : b.im); }
// 1 / b = conj(b) / |b|^2 with b first scaled by a power of two (exact) so
// that |b|^2 neither overflows nor underflows: one division on the
// recurrence's critical path
__device__ __forceinline__ C64 crecip(C64 b) {
  int e;
  (void)frexp(fmax(fabs(b.re), fabs(b.im)), &e);
  const double br = ldexp(b.re, -e), bi = ldexp(b.im, -e);
  const double q = 1.0 / (br * br + bi * bi);
  return mk(ldexp(br * q, -e), ldexp(-bi * q, -e));
}

// LU with partial pivoting of the tridiagonal H (diag alpha, super beta,
// sub delta).  Row i of U holds 1/U0i[i], U1[i], U2[i] on columns i, i+1, i+2;
// Lm[i] is the multiplier that eliminates column i of the row below the
// pivot row; Sw[i] says whether rows i and i+1 were exchanged.  The
// elimination is sequential (one thread) and bound by the latency of its
// dependent operations; the coefficients are first staged in LDS by the whole
// block and read a step ahead.  Up to TRI_REC_MAX the reciprocals of the
// sub-diagonal are staged too, which are the pivots' wherever rows are
// exchanged, and the results take the places of the consumed coefficients
// until the whole block writes them out.  Measured at k = 500: 98 us, 128 us
// with crecip on the chain and the coefficients of a step read in that step.
constexpr int TRI_LDS_MAX = 1365;  // 3 k complex in LDS (<= 64 KB of dynamic LDS)
constexpr int TRI_REC_MAX = 960;   // 4 k complex and k int

// where the factors go
struct TriLu {
  gp<C64> Lm, U0i, U1, U2;
  gp<int> Sw;
};

// The sequential elimination, with the coefficients read through al/be/de
// (LDS or global: one instantiation each, so every access has its own
// address space).  The products are rounded in a fixed order (the other one in
// a1's imaginary part): the inner recurrence can amplify a last bit of
// H^{-1}.  Returns 1 if a pivot vanishes.
template <class P>
__device__ __forceinline__ int tri_lu_seq(int k, P al, P be, P de, const TriLu& o) {
  const C64 z = mk(0.0, 0.0);
  C64 a0 = ldg(al), a1 = k > 1 ? ldg(be) : z, a2 = z;
  int bad = 0;
  for (int i = 0; i + 1 < k; ++i) {
    const C64 b0 = ldg(de + i), b1 = ldg(al + i + 1), b2 = (i + 2 < k) ? ldg(be + i + 1) : z;
    const bool sw = cabs1s(a0) < cabs1s(b0);
    const C64 p0 = csel(sw, b0, a0), p1 = csel(sw, b1, a1), p2 = csel(sw, b2, a2);
    const C64 o0 = csel(sw, a0, b0), o1 = csel(sw, a1, b1), o2 = csel(sw, a2, b2);
    if (!(cabs1s(p0) > 0.0)) bad = 1;
    const C64 inv = crecip(p0);
    const C64 m = cmul_a(o0, inv);
    stg(o.U0i + i, inv);
    stg(o.U1 + i, p1);
    stg(o.U2 + i, p2);
    stg(o.Lm + i, m);
    o.Sw[i] = sw ? 1 : 0;
    a0 = o1 - cmul_a(m, p1);
    a1 = o2 - cmul_b(m, p2);
    a2 = z;
  }
  if (!(cabs1s(a0) > 0.0)) bad = 1;
  stg(o.U0i + k - 1, crecip(a0));
  stg(o.U1 + k - 1, z);
  stg(o.U2 + k - 1, z);
  if (k >= 2) stg(o.U2 + k - 2, z);
  return bad;
}

// The same in LDS, with the same bits, for pivots between 2^-200 and 2^200
// (returns 2, with nothing else of use, if one is not).  sm holds al, be, de,
// the reciprocals of de (k each, zeros past the end of be and de); the
// factors of step i take the places of the coefficients that it consumes: U0i
// al[i], U1 be[i], U2 de[i], Lm the reciprocal's, Sw behind them.  Bound by the
// number of instructions and their latency: no selects (a branch per step,
// whose two sides drop the products with the zero of row i), no scaling in
// the reciprocal (exact, so it only guards the range); the coefficients of four
// steps are read together, in the four before.
__device__ __forceinline__ int tri_lu_mid(int k, C64* sm) {
  C64 *s0 = sm, *s1 = sm + k, *s2 = sm + 2 * k, *s3 = sm + 3 * k;
  int* ssw = reinterpret_cast<int*>(sm + 4 * k);
  constexpr int NS = 4;  // steps whose coefficients are read together
  struct Row {
    C64 b0, b1, b2, rb;
  };
  Row c[NS], nx[NS];
  auto fetch = [&](Row(&v)[NS], int i) {
#pragma unroll
    for (int r = 0; r < NS; ++r) {
      const int j = min(i + r, k - 1), j1 = min(i + r + 1, k - 1);
      v[r].b0 = s2[j];
      v[r].b1 = s0[j1];
      v[r].b2 = s1[j1];
      v[r].rb = s3[j];
    }
  };
  C64 a0 = s0[0], a1 = s1[0];
  double lo = 1.0, hi = 1.0;  // the pivots' range
  auto step = [&](int i, const Row& w) {
    const C64 b0 = w.b0, b1 = w.b1, b2 = w.b2, rb = w.rb;
    const double n = fma(a0.re, a0.re, a0.im * a0.im);
    double y = __builtin_amdgcn_rcp(n);
    y = fma(y, fma(-n, y, 1.0), y);
    y = fma(y, fma(-n, y, 1.0), y);
    y = fma(fma(-n, y, 1.0), y, y);
    const double na = cabs1s(a0), nb = cabs1s(b0);
    const double np = fmax(na, nb);
    lo = fmin(lo, np);
    hi = fmax(hi, np);
    if (__builtin_amdgcn_ballot_w64(na < nb) != 0) {
      const C64 m = cmul_a(a0, rb);
      s0[i] = rb;
      s1[i] = b1;
      s2[i] = b2;
      s3[i] = m;
      ssw[i] = 1;
      a0 = a1 - cmul_a(m, b1);
      a1 = mk(0.0, 0.0) - cmul_b(m, b2);
    } else {
      const C64 inv = mk(a0.re * y, y * -a0.im);
      const C64 m = cmul_a(b0, inv);
      s0[i] = inv;
      s1[i] = a1;
      s2[i] = mk(0.0, 0.0);
      s3[i] = m;
      ssw[i] = 0;
      a0 = b1 - cmul_a(m, a1);
      a1 = b2;
    }
  };
  fetch(c, 0);
  int i = 0;
  for (; i + NS < k; i += NS) {
    fetch(nx, i + NS);
#pragma unroll
    for (int r = 0; r < NS; ++r) step(i + r, c[r]);
#pragma unroll
    for (int r = 0; r < NS; ++r) c[r] = nx[r];
  }
#pragma unroll
  for (int r = 0; r < NS; ++r)
    if (i + r + 1 < k) step(i + r, c[r]);
  const double last = cabs1s(a0);
  s0[k - 1] = crecip(a0);
  s1[k - 1] = mk(0.0, 0.0);
  s2[k - 1] = mk(0.0, 0.0);
  if (k >= 2) s2[k - 2] = mk(0.0, 0.0);
  if (!(lo > 0x1p-200 && hi < 0x1p200)) return 2;
  return last > 0.0 ? 0 : 1;
}

// dynamic LDS for problems of order up to kmax
static size_t tri_lu_lds(int kmax) {
  const size_t r = std::min(kmax, TRI_REC_MAX) * (4 * sizeof(C64) + sizeof(int));
  return kmax > TRI_REC_MAX ? std::max(r, std::min(kmax, TRI_LDS_MAX) * 3 * sizeof(C64)) : r;
}

// one workgroup per problem (s0 for one, SS for a batch); the state of the
// inner recurrence starts here too
__global__ void __launch_bounds__(256) k_tri_lu(const Inner s0, const Inner* __restrict__ SS) {
  extern __shared__ C64 sm[];
  const Inner& s = SS ? SS[blockIdx.x] : s0;
  const int k = s.k;
  gp<const C64> alpha = as_global(s.al), beta = as_global(s.be), delta = as_global(s.de);
  const C64 z = mk(0.0, 0.0);
  for (int j = threadIdx.x; j < s.lmax; j += blockDim.x) {
    stg(as_global(s.a) + j, z);
    stg(as_global(s.b) + j, z);
    stg(as_global(s.d) + j, z);
  }
  gp<int> flags = as_global(s.flags);
  if (threadIdx.x == 0) flags[0] = flags[2] = 0;
  const bool lds = k <= TRI_LDS_MAX, rec = k <= TRI_REC_MAX;
  if (lds) {
    for (int i = threadIdx.x; i < k; i += blockDim.x) {
      const int p = i + 1 < k ? i : 0;
      const C64 be = ldg(beta + p), dv = ldg(delta + p), de = csel(i + 1 < k, dv, z);
      sm[i] = ldg(alpha + i);
      sm[k + i] = csel(i + 1 < k, be, z);
      sm[2 * k + i] = de;
      if (rec) sm[3 * k + i] = crecip(de);
    }
    __syncthreads();
  }
  const C64* l = sm;
  const TriLu o{as_global(s.Lm), as_global(s.U0i), as_global(s.U1), as_global(s.U2), as_global(s.Sw)};
  __shared__ int s_bad;
  if (threadIdx.x == 0) {
    int bad = rec ? tri_lu_mid(k, sm) : 2;
    s_bad = bad;
    if (bad == 2)
      bad = lds && !rec ? tri_lu_seq(k, l, l + k, l + 2 * k, o) : tri_lu_seq(k, alpha, beta, delta, o);
    flags[1] = bad;
  }
  if (!rec) return;
  __syncthreads();
  if (s_bad == 2) return;
  for (int i = threadIdx.x; i < k; i += blockDim.x) {
    stg(o.U0i + i, sm[i]);
    stg(o.U1 + i, sm[k + i]);
    stg(o.U2 + i, sm[2 * k + i]);
    stg(o.Lm + i, sm[3 * k + i]);
    o.Sw[i] = reinterpret_cast<const int*>(sm + 4 * k)[i];
  }
}

// column j of H^{-1} (solve H x = e_j), then B = H + H^{-1}; B row-major k x k.
// The factors are staged in LDS when they fit.  The forward sweep of e_j is
// zero before row j - 1, so a wave starts before its first column.  The backward sweep reads eight
// rows of the forward result at a time, sixteen rows ahead of the recurrence
// at most (rows below the one being written, so the reads never see a row of
// this sweep): their round trip passes behind the eight rows before.  Bound by
// the latency of the 2 k dependent steps: k = 500 66 us (88 with a round trip
// per eight rows and lanes that started at their own rows).
struct TriF {
  C64 lm, u0i, u1, u2;
};
constexpr int TRI_INV_LDS_MAX = 960;  // k x (64 + 4) B in LDS (<= 64 KB of dynamic LDS)

template <bool LDS>
__device__ __forceinline__ void tri_inv_col(int j, int k, const TriF* sf, const int* ssw, gp<const C64> Lm,
                                            gp<const int> Sw, gp<const C64> U0i, gp<const C64> U1,
                                            gp<const C64> U2, gp<C64> B) {
  const C64 z = mk(0.0, 0.0);
  // rows in step over the wave, from its first column's first nonzero row (the others hold zeros until theirs)
  const int i0 = max((int)(blockIdx.x * 64) - 1, 0);
  for (int i = 0; i < i0; ++i) stg(B + (size_t)i * k + j, z);
  C64 fc = mk(j == 0 ? 1.0 : 0.0, 0.0);
#pragma unroll 8
  for (int i = i0; i < k - 1; ++i) {
    const C64 fn = mk(i + 1 == j ? 1.0 : 0.0, 0.0);
    const int sw = LDS ? ssw[i] : Sw[i];
    const C64 lm = LDS ? sf[i].lm : ldg(Lm + i);
    const C64 piv = csel(sw, fn, fc), oth = csel(sw, fc, fn);
    stg(B + (size_t)i * k + j, piv);
    fc = oth - cmul(lm, piv);
  }
  stg(B + (size_t)(k - 1) * k + j, fc);
  C64 x1 = z, x2 = z;
  auto step = [&](int i, C64 y) {
    const C64 u1 = LDS ? sf[i].u1 : ldg(U1 + i), u2 = LDS ? sf[i].u2 : ldg(U2 + i), u0 = LDS ? sf[i].u0i : ldg(U0i + i);
    const C64 xi = cmul(y - cmul(u1, x1) - cmul(u2, x2), u0);
    stg(B + (size_t)i * k + j, xi);
    x2 = x1;
    x1 = xi;
  };
  int i = k - 1;
  C64 y[8], yn[8];
  auto fetch = [&](C64(&v)[8], int i0) {  // rows i0 .. i0 - 7 (row 0 in the place of rows before it)
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = ldg(B + (size_t)max(i0 - u, 0) * k + j);
  };
  if (i >= 7) fetch(y, i);
  for (; i >= 7; i -= 8) {
    fetch(yn, i - 8);
#pragma unroll
    for (int u = 0; u < 8; ++u) step(i - u, y[u]);
#pragma unroll
    for (int u = 0; u < 8; ++u) y[u] = yn[u];
  }
  for (; i >= 0; --i) step(i, ldg(B + (size_t)i * k + j));
}

__global__ void __launch_bounds__(64) k_tri_inv(const Inner s0, const Inner* __restrict__ SS) {
  extern __shared__ TriF sf[];
  const Inner& s = SS ? SS[blockIdx.z] : s0;
  const int k = s.k;
  if ((int)(blockIdx.x * blockDim.x) >= k) return;
  gp<const C64> Lm = as_global((const C64*)s.Lm), U0i = as_global((const C64*)s.U0i),
                U1 = as_global((const C64*)s.U1), U2 = as_global((const C64*)s.U2);
  gp<const C64> alpha = as_global(s.al), beta = as_global(s.be), delta = as_global(s.de);
  gp<const int> Sw = as_global((const int*)s.Sw);
  gp<C64> B = as_global(s.B);
  int* ssw = reinterpret_cast<int*>(sf + (k <= TRI_INV_LDS_MAX ? k : 0));
  const bool lds = k <= TRI_INV_LDS_MAX;
  if (lds) {
    for (int i = threadIdx.x; i < k; i += blockDim.x) {
      sf[i].lm = ldg(Lm + i);
      sf[i].u0i = ldg(U0i + i);
      sf[i].u1 = ldg(U1 + i);
      sf[i].u2 = ldg(U2 + i);
      ssw[i] = Sw[i];
    }
    __syncthreads();
  }
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= k) return;
  if (lds)
    tri_inv_col<true>(j, k, sf, ssw, Lm, Sw, U0i, U1, U2, B);
  else
    tri_inv_col<false>(j, k, sf, ssw, Lm, Sw, U0i, U1, U2, B);
  auto add = [&](int i, C64 h) {
    gp<C64> o = B + (size_t)i * k + j;
    stg(o, ldg(o) + h);
  };
  add(j, ldg(alpha + j));
  if (j > 0) add(j - 1, ldg(beta + j - 1));
  if (j + 1 < k) add(j + 1, ldg(delta + j));
}

// BH = B^dag (tiled transpose through LDS)
__global__ void k_adjoint(const Inner s0, const Inner* __restrict__ SS) {
  __shared__ C64 t[32][33];
  const Inner& s = SS ? SS[blockIdx.z] : s0;
  const int k = s.k;
  gp<const C64> B = as_global((const C64*)s.B);
  gp<C64> BH = as_global(s.BH);
  const int bx = blockIdx.x * 32, by = blockIdx.y * 32;
  for (int yy = threadIdx.y; yy < 32; yy += 8) {
    const int r = by + yy, c = bx + threadIdx.x;
    if (r < k && c < k) t[yy][threadIdx.x] = ldg(B + (size_t)r * k + c);
  }
  __syncthreads();
  for (int yy = threadIdx.y; yy < 32; yy += 8) {
    const int r = bx + yy, c = by + threadIdx.x;
    if (r < k && c < k) stg(BH + (size_t)r * k + c, conj(t[threadIdx.x][yy]));
  }
}

// dense tridiagonal H (ld = k), row-major
__global__ void k_tri_dense(int k, const C64* __restrict__ alpha, const C64* __restrict__ beta,
                            const C64* __restrict__ delta, C64* __restrict__ H) {
  const size_t nn = (size_t)k * k;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < nn; e += (size_t)gridDim.x * blockDim.x) {
    const int i = (int)(e / k), j = (int)(e % k);
    C64 v = mk(0.0, 0.0);
    if (i == j) v = alpha[i];
    else if (j == i + 1) v = beta[i];
    else if (i == j + 1) v = delta[j];
    H[e] = v;
  }
}

// ---------------------------------------------------------------------------
// inner Krylov on dense B: three launches per step.
//  k_in_gemv : normalise the previous raw vectors (from partial sums), store
//              v_i / w_i, u = B v_i - beta v_{i-1}, q = B^dag w_i - delta w_{i-1}
//              (one wave per row), and the partial first-pass projections
//              W^dag u, V^dag q over the block's GR rows;
//  k_in_sub  : reduce the partial projections, subtract (u -= V c, q -= W d;
//              eight lanes per row), then emit either the partial projections
//              of the second Gram-Schmidt pass or the partial sums of
//              s = q^dag u, |u|^2, |q|^2 for the next normalisation.
// V, W column-major (column j at j*k).  Hermitian: one side, W = V, q = u.
// Arnoldi: the one-sided form on a general B, with every projection
// coefficient kept (column i of the Hessenberg H_l, both passes summed).
constexpr int GR = 16;  // rows per k_in_gemv block (one wave each, 1024 threads)
constexpr int SR = 32;  // rows per k_in_sub block (eight lanes each)

// the descriptor with its buffers seen as global memory (see as_global)
struct InnerG {
  int k, herm, lmax, nb1, nb2;
  gp<const C64> B, BH;
  gp<C64> V, W, u0, u1, q0, q1, part1, part2, a, b, d;  // u0/u1, q0/q1: the raw ping-pong vectors
  gp<double> part3;
  gp<int> flags;
  gp<C64> hcol;
  int arnoldi;
};

__device__ __forceinline__ InnerG inner_view(const Inner& s) {
  InnerG g;
  g.k = s.k;
  g.herm = s.herm;
  g.lmax = s.lmax;
  g.nb1 = s.nb1;
  g.nb2 = s.nb2;
  g.B = as_global(s.B);
  g.BH = as_global(s.BH);
  g.V = as_global(s.V);
  g.W = as_global(s.W);
  g.u0 = as_global(s.uraw[0]);
  g.u1 = as_global(s.uraw[1]);
  g.q0 = as_global(s.qraw[0]);
  g.q1 = as_global(s.qraw[1]);
  g.part1 = as_global(s.part1);
  g.part2 = as_global(s.part2);
  g.part3 = as_global(s.part3);
  g.a = as_global(s.a);
  g.b = as_global(s.b);
  g.d = as_global(s.d);
  g.flags = as_global(s.flags);
  g.hcol = as_global(s.hcol);
  g.arnoldi = s.arnoldi;
  return g;
}

// The descriptor of this block's problem: a kernel argument (read straight
// from the kernel-argument segment, one round trip less) for a single
// problem, entry z of a device array for a batch.
template <bool BATCH>
__device__ __forceinline__ const Inner& inner_desc(const Inner& s0, const Inner* SS, int z) {
  if constexpr (BATCH)
    return SS[z];
  else
    return s0;
}

// c ? a : b for two fields of a local descriptor.  A plain select of two
// fields lets the compiler turn it into one load through a selected address,
// which keeps the whole descriptor in scratch memory; passing both values
// through an empty asm first leaves a select of registers.
template <class T>
__device__ __forceinline__ T pick(bool c, T a, T b) {
  asm volatile("" : "+s"(a), "+s"(b));
  return c ? a : b;
}

// raw vector h (0/1) of the u side (q = 0) or the q side (q = 1)
__device__ __forceinline__ gp<C64> rawv(const InnerG& g, int q, int h) {
  return pick(q != 0, pick(h != 0, g.q1, g.q0), pick(h != 0, g.u1, g.u0));
}

// the sums of nb partial sums, thread t holding partial t (and t + NTH, ..):
// the waves' sums in a fixed order; when only the first wave holds any
// (nb <= 64), that wave alone reduces and shares them, which gives the same
// sums (the other waves would add zeros)
template <int NTH>
__device__ __forceinline__ void bsum_first(double (&v)[4], int nb) {
  __shared__ double sh[NTH / 64][4];
  const bool one = nb <= 64;
  if (!one || threadIdx.x < 64)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[q] = wave_xsum(v[q]);
      if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6][q] = v[q];
    }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = sh[0][q];
  if (!one)
    for (int w = 1; w < NTH / 64; ++w)
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] += sh[w][q];
}

// problem and workgroup within it: one problem's workgroups after the other,
// dealt over the XCDs.  (From eight problems on, each kept on one XCD, whose
// L2 then holds its B: 16 problems of k = 300 17.4 us a mat-vec, as here 15.8;
// 12 of k = 600 35.6 and 27.2, 32 of k = 600 81 and 72.)
template <bool BATCH>
__device__ __forceinline__ void inner_place(int nbmax, int* z, int* x) {
  *z = BATCH ? blockIdx.x / nbmax : 0;
  *x = BATCH ? blockIdx.x % nbmax : blockIdx.x;
}

// Every inner kernel serves a batch of independent problems: problem z is
// SS[z]; the grid is sized for the largest, and a workgroup beyond its own
// problem's size or steps returns at once.
// Everything a block loads except the normalisation scale is known at launch
// (the row of B, the previous raw vector, the old basis entry and the
// projection columns), so it is all issued before the partial sums of the
// previous step are reduced: one memory round trip instead of four.  Each
// wave multiplies its own row's new entry into the projection columns and
// leaves the products in LDS; they are summed over the block's rows in row
// order, as a single thread summing them would.  The new vector is scaled once
// per workgroup, into LDS (by every wave for itself it cost as many loads as
// the matrix): k = 500 6.9 us (8.9), 16 problems of k = 300 15.8 us (22).  The
// products are rounded in a fixed order, as in the elimination.
constexpr int XC = 512;  // columns of B staged at a time, eight per lane
constexpr int GP = 2;  // projection columns per lane loaded at launch (j < 128)

template <bool BATCH>
__global__ void __launch_bounds__(GR * 64) k_in_gemv(const Inner s0, const Inner* __restrict__ SS, int nbmax, int i) {
  extern __shared__ C64 s_p[];  // [GR][i + 1] per-row projection products
  __shared__ C64 s_x[XC];       // v_i (or w_i), a stretch of it
  int z, blk;
  inner_place<BATCH>(nbmax, &z, &blk);
  const Inner& S = inner_desc<BATCH>(s0, SS, z);
  const InnerG s = inner_view(S);
  const int side = BATCH ? blk >= s.nb1 : blockIdx.y;  // 0: u = B v, 1: q = B^dag w
  if (BATCH) blk -= side ? s.nb1 : 0;
  // a batch launch covers the largest problem; a single problem is launched
  // for exactly its own steps and blocks
  if (BATCH && (i >= s.lmax || blk >= s.nb1 || (side && s.herm))) return;
  const int k = s.k;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = blk * GR + wave;
  const bool live = r < k;
  const int rs = live ? r : 0;  // rows past k load row 0 and discard it
  // the previous step's normalisation partial sums (i > 0) and the breakdown
  // flag, first: what they decide does not wait for the matrix
  int flag = s.flags[0];
  double v[4] = {0, 0, 0, 0};
  if (i > 0) {
    gp<const double> p3 = s.part3;
    if ((int)threadIdx.x < s.nb2)
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] = p3[q * s.nb2 + threadIdx.x];
    for (int bb = threadIdx.x + GR * 64; bb < s.nb2; bb += GR * 64)
#pragma unroll
      for (int q = 0; q < 4; ++q) v[q] += p3[q * s.nb2 + bb];
  }
  // the side-dependent pointers come straight from the descriptor: selected
  // copies of the local view would keep that view in scratch memory
  const int h = i & 1;
  C64* const r0 = side ? S.qraw[0] : S.uraw[0];
  C64* const r1 = side ? S.qraw[1] : S.uraw[1];
  gp<const C64> src = as_global((const C64*)(h ? r1 : r0));
  gp<C64> dst = as_global(h ? r0 : r1);
  gp<const C64> M = as_global(side ? S.BH : S.B);
  gp<C64> basis = as_global(side ? S.W : S.V);
  const bool other = !s.herm;
  gp<const C64> proj = as_global((const C64*)(s.herm ? S.V : (side ? S.V : S.W)));
  gp<const C64> osrc = as_global((const C64*)(side ? (h ? S.uraw[1] : S.uraw[0]) : (h ? S.qraw[1] : S.qraw[0])));
  // loads issued at launch: eight columns of the row per lane (clamped to
  // column 0 past the end), an entry of the raw vector per thread, this row's
  // raw entries, the old basis entry and up to GP projection columns per lane
  C64 mv[8], xs;
  auto fetch = [&](int c0) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int c = c0 + lane + 64 * u, cc = c < k ? c : 0;
      mv[u] = ldg(M + (size_t)rs * k + cc);
    }
    const int c = c0 + (int)threadIdx.x;
    xs = ldg(src + (c < k ? c : 0));
  };
  fetch(0);
  const C64 xr_raw = ldg(src + rs);
  const C64 xo_raw = ldg(osrc + rs);
  const C64 vold = ldg(basis + (size_t)(i > 0 ? i - 1 : 0) * k + rs);
  C64 pj[GP];
#pragma unroll
  for (int m = 0; m < GP; ++m) {
    const int j = lane + 64 * m;
    pj[m] = ldg(proj + (size_t)(j < i ? j : 0) * k + rs);
  }
  // a breakdown at an earlier step ends the iteration; tested only now so that
  // the flag's latency overlaps the loads above (all in bounds)
  asm volatile("" : "+v"(flag));
  if (flag) return;
  C64 scal = mk(1.0, 0.0), sub = mk(0.0, 0.0);
  C64 scal_o = mk(1.0, 0.0);  // scale of the other side's new column
  if (i > 0) {
    bsum_first<GR * 64>(v, s.nb2);
    const C64 sd = s.herm ? mk(v[2], 0.0) : mk(v[0], v[1]);
    const double sabs = sqrt(fma(sd.re, sd.re, sd.im * sd.im));  // (rounded in this order in every build)
    if (!(sabs > 1e-14 * sqrt(v[2] * (s.herm ? v[2] : v[3])))) {
      if (blk == 0 && side == 0 && threadIdx.x == 0) s.flags[2] = i;
      return;
    }
    const double delta = sqrt(sabs);
    const C64 beta = (1.0 / delta) * sd;
    if (blk == 0 && side == 0 && threadIdx.x == 0) {
      stg(s.b + (i - 1), beta);
      stg(s.d + (i - 1), mk(delta, 0.0));
    }
    const C64 sv = mk(1.0 / delta, 0.0), sw = (1.0 / fma(beta.re, beta.re, beta.im * beta.im)) * beta;  // v = u / delta, w = q / conj(beta)
    scal = side ? sw : sv;
    scal_o = side ? sv : sw;
    sub = side ? mk(delta, 0.0) : beta;
  }
  // u_r = (B v_i)_r - sub * v_{i-1, r}, XC columns at a time: the workgroup
  // scales them once, into LDS, for all its rows
  C64 ac[4] = {mk(0.0, 0.0), mk(0.0, 0.0), mk(0.0, 0.0), mk(0.0, 0.0)};
  for (int c0 = 0; c0 < k; c0 += XC) {
    if (c0 > 0) {
      fetch(c0);
      __syncthreads();
    }
    if (threadIdx.x < XC) s_x[threadIdx.x] = (i > 0) ? cmul_a(scal, xs) : mk(c0 + threadIdx.x == 0 ? 1.0 : 0.0, 0.0);
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (c0 + lane + 64 * u < k) ac[u & 3] = ac[u & 3] + cmul_b(mv[u], s_x[lane + 64 * u]);
  }
  C64 acc = (ac[0] + ac[1]) + (ac[2] + ac[3]);
  acc = mk(wave_xsum(acc.re), wave_xsum(acc.im));
  const C64 xr = (i > 0) ? cmul_a(scal, xr_raw) : mk(r == 0 ? 1.0 : 0.0, 0.0);  // v_i (or w_i) at row r
  if (i > 0) acc = acc - cmul_b(sub, vold);
  if (live && lane == 0) {
    stg(basis + (size_t)i * k + r, xr);
    stg(dst + r, acc);
  }
  // this row's terms of the first-pass projections W^dag u (V^dag q): column
  // i of the other basis is being written by the other side's blocks in this
  // launch, so its entry is formed here from the raw vector (Hermitian: it
  // is this row's own new entry)
  const int ncol = i + 1;
  for (int m0 = 0; m0 * 64 < ncol; m0 += GP) {
#pragma unroll
    for (int m = 0; m < GP; ++m) {
      const int j = lane + 64 * (m0 + m);
      if (j < ncol) {
        C64 pv;
        if (j == i) pv = other ? ((i > 0) ? cmul_b(scal_o, xo_raw) : mk(r == 0 ? 1.0 : 0.0, 0.0)) : xr;
        else pv = (m0 == 0) ? pj[m] : ldg(proj + (size_t)j * k + rs);
        s_p[wave * ncol + j] = mk(fma(pv.im, acc.im, pv.re * acc.re), fma(pv.re, acc.im, -(pv.im * acc.re)));
      }
    }
  }
  __syncthreads();
  gp<C64> out = s.part1 + ((size_t)side * s.nb1 + blk) * s.lmax;
  for (int j = threadIdx.x; j < ncol; j += GR * 64) {
    C64 t = mk(0.0, 0.0), pw[GR];
#pragma unroll
    for (int w = 0; w < GR; ++w) pw[w] = s_p[w * ncol + j];
#pragma unroll
    for (int w = 0; w < GR; ++w) t = csel(blk * GR + w < k, t + pw[w], t);
    stg(out + j, t);
  }
}

// dynamic LDS of k_in_gemv at step i: GR x (i + 1) products (128 KB at the
// largest inner size)
static size_t gemv_lds(int i) { return (size_t)GR * (i + 1) * sizeof(C64); }

// pass 1 (last == 0): reduce part1, subtract, emit part2;
// pass 2 (last == 1): reduce part2, subtract, emit the normalisation sums.
// The partial-sum and projection phases give each (side, column) four
// consecutive lanes that split the terms and meet by DPP; the subtraction has
// a half of the workgroup per side, eight lanes per row.  What the three
// phases load of the partial sums and the bases (up to 64 columns) is known at
// launch and issued together: one memory round trip instead of three.
// Bound by the launch and that round trip: 5.2 us at k = 500 (6.5 when each
// phase loaded for itself), 6.2 us for 16 problems of k = 300 (8.9).
constexpr int ST = 512;
constexpr int TPJ = 4;  // lanes per (side, column) in the reduction phases

template <bool BATCH>
__global__ void __launch_bounds__(ST) k_in_sub(const Inner s0, const Inner* __restrict__ SS, int nbmax,
                                               int i, int last) {
  int z, blk;
  inner_place<BATCH>(nbmax, &z, &blk);
  const Inner& S = inner_desc<BATCH>(s0, SS, z);
  const InnerG s = inner_view(S);
  const bool report = blk == 0 && threadIdx.x == 0 && !last && i + 1 >= s.lmax;  // the problem's last launch
  if (BATCH && (i >= s.lmax || (last && i + 1 >= s.lmax) || blk >= s.nb2)) return;
  const int k = s.k;
  const int sides = s.herm ? 1 : 2;
  __shared__ C64 s_c[2][LMAX];
  __shared__ C64 s_u[2][SR];
  gp<const C64> pin = pick(last != 0, s.part2, s.part1);
  const int nbin = pick(last != 0, s.nb2, s.nb1);
  const int ncol = i + 1;
  const int l4 = threadIdx.x & (TPJ - 1);
  constexpr int NIT = ST / TPJ;  // items per sweep over the workgroup
  const int it1 = (int)threadIdx.x / TPJ;
  // item -> (side, column); past the end: (0, 0)
  auto item = [&](int it, int* side, int* j) {
    const bool ok = it < sides * ncol;
    *side = ok && it >= ncol ? 1 : 0;
    *j = ok ? it - *side * ncol : 0;
    return ok;
  };
  // this thread's side, row and columns in the subtraction
  const int side2 = (int)threadIdx.x / (ST / 2), rl = ((int)threadIdx.x & (ST / 2 - 1)) >> 3, jl = threadIdx.x & 7;
  const int r = blk * SR + rl, rs = r < k ? r : 0;
  const bool mine = side2 < sides;
  const int nr = min(SR, k - blk * SR);  // rows of this block (s_u is zero past them)
  // --- loads known at launch: the first sweep's partial sums, the first 64
  // columns of the subtraction, the first sweep's columns of the projections
  C64 pv[8], bv[8], qv[8];
  int side1, j1;
  const bool ok1 = item(it1, &side1, &j1);
  auto load_part = [&](int side, int j, int bb0) {
    gp<const C64> pp = pin + (size_t)side * nbin * s.lmax + j;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int bb = bb0 + u * TPJ;
      pv[u] = ldg(pp + (size_t)(bb < nbin ? bb : 0) * s.lmax);
    }
  };
  gp<const C64> basis = side2 ? s.W : s.V;
  auto load_basis = [&](int j0) {
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int j = j0 + 8 * m;
      bv[m] = ldg(basis + (size_t)(j <= i ? j : 0) * k + rs);
    }
  };
  auto load_proj = [&](int side, int j) {
    gp<const C64> pj = (s.herm || side ? s.V : s.W) + (size_t)j * k + blk * SR;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int w = l4 + m * TPJ;
      qv[m] = ldg(pj + (w < nr ? w : 0));
    }
  };
  static_assert(SR == 8 * TPJ, "one batch of loads covers the block's rows");
  int flag = s.flags[2];
  load_part(side1, j1, l4);
  load_basis(jl);
  gp<C64> x = rawv(s, side2, (i + 1) & 1);
  const C64 xr = ldg(x + rs);
  if (!last) load_proj(side1, j1);
  // reduce the partial projections: item = (side, j), TPJ lanes each
  for (int it0 = 0; it0 < sides * ncol; it0 += NIT) {
    int side, j;
    const bool ok = it0 == 0 ? (side = side1, j = j1, ok1) : item(it0 + it1, &side, &j);
    C64 t0 = mk(0.0, 0.0), t1 = t0;
    for (int bb0 = l4; bb0 < nbin; bb0 += 8 * TPJ) {
      if (it0 > 0 || bb0 > l4) load_part(side, j, bb0);
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (bb0 + u * TPJ < nbin) {
          if (u & 1)
            t1 = t1 + pv[u];
          else
            t0 = t0 + pv[u];
        }
    }
    C64 t = t0 + t1;
    t = mk(quad_xsum(t.re), quad_xsum(t.im));
    if (ok && l4 == 0) s_c[side][j] = t;
  }
  // a breakdown flagged at this or an earlier step ends the iteration; tested
  // only now so that the flag's latency overlaps the loads above (all in bounds)
  asm volatile("" : "+v"(flag));
  if (report) {
    gp<int> o = as_global(S.out);
    o[0] = flag;
    o[1] = s.flags[1];
  }
  if (flag) {
    if (blk == 0 && threadIdx.x == 0) s.flags[0] = flag;
    return;
  }
  __syncthreads();
  if (!last && blk == 0 && threadIdx.x == 0) stg(s.a + i, s.herm ? mk(s_c[0][i].re, 0.0) : s_c[0][i]);
  if (s.arnoldi && blk == 0)  // column i of H_l: the first pass stores, the second adds
    for (int j = threadIdx.x; j <= i; j += ST) {
      gp<C64> h = s.hcol + (size_t)i * s.lmax + j;
      stg(h, last ? ldg(h) + s_c[0][j] : s_c[0][j]);
    }
  // u -= V c, q -= W d: eight lanes per row, columns jl, jl + 8, ...
  C64 acc[2] = {mk(0.0, 0.0), mk(0.0, 0.0)};
  if (mine && r < k)
    for (int j0 = jl; j0 <= i; j0 += 8 * 8) {
      if (j0 > jl) load_basis(j0);
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const int j = j0 + 8 * m;
        if (j <= i) acc[m & 1] = acc[m & 1] + cmul(bv[m], s_c[side2][j]);
      }
    }
  C64 a = acc[0] + acc[1];
  a = mk(oct_xsum(a.re), oct_xsum(a.im));
  if (mine && jl == 0) {
    C64 nv = mk(0.0, 0.0);
    if (r < k) {
      nv = xr - a;
      stg(x + r, nv);
    }
    s_u[side2][rl] = nv;
  }
  __syncthreads();
  if (!last) {
    // second-pass partial projections over this block's rows: item = (side, j)
    for (int it0 = 0; it0 < sides * ncol; it0 += NIT) {
      int side, j;
      const bool ok = it0 == 0 ? (side = side1, j = j1, ok1) : item(it0 + it1, &side, &j);
      if (it0 > 0) load_proj(side, j);
      C64 t0 = mk(0.0, 0.0), t1 = t0;
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const int w = l4 + m * TPJ;
        if (w < nr) {
          if (m & 1)
            t1 = t1 + cmulc(qv[m], s_u[side][w]);
          else
            t0 = t0 + cmulc(qv[m], s_u[side][w]);
        }
      }
      C64 t = t0 + t1;
      t = mk(quad_xsum(t.re), quad_xsum(t.im));
      if (ok && l4 == 0) stg(s.part2 + ((size_t)side * s.nb2 + blk) * s.lmax + j, t);
    }
    return;
  }
  if (threadIdx.x >= 64) return;
  double v[4] = {0, 0, 0, 0};
  if (threadIdx.x < SR) {
    const C64 un = s_u[0][threadIdx.x];
    const C64 qn = s.herm ? un : s_u[1][threadIdx.x];
    const C64 t = cmulc(qn, un);
    v[0] = t.re;
    v[1] = t.im;
    v[2] = norm2(un);
    v[3] = norm2(qn);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) v[q] = wave_xsum(v[q]);
  if (threadIdx.x == 0)
#pragma unroll
    for (int q = 0; q < 4; ++q) s.part3[q * s.nb2 + blk] = v[q];
}

// dense upper Hessenberg H_l (ld = l, row-major) of the Arnoldi option.
// The recurrence subtracts b[c - 1] v_{c-1} from B v_c before it projects
// (the Lanczos form), so the stored coefficient of v_{c-1} lacks b[c - 1]:
// H[r][c] = hcol[c * lmax + r] (+ b[r] for r = c - 1) for r <= c,
// H[c + 1][c] = |u_c| = d[c], else 0
__global__ void k_hess_dense(int l, int lmax, const C64* __restrict__ hcol, const C64* __restrict__ b,
                             const C64* __restrict__ d, C64* __restrict__ H) {
  const size_t nn = (size_t)l * l;
  for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < nn; e += (size_t)gridDim.x * blockDim.x) {
    const int r = (int)(e / l), c = (int)(e % l);
    C64 v = mk(0.0, 0.0);
    if (r <= c) v = hcol[(size_t)c * lmax + r];
    if (r + 1 == c) v = v + b[r];
    if (r == c + 1) v = d[c];
    H[e] = v;
  }
}

// z = V y, y the first column of S (leading dimension ldy): 16 rows and 16
// groups of columns per workgroup, every load of 256 B, eight in flight (one
// thread per row waited for its l columns one after another)
constexpr int LT = 256, LR = 16;
__device__ __forceinline__ void lift_rows(int k, int l, const C64* __restrict__ V, const C64* __restrict__ y, int ldy,
                                          C64* __restrict__ z) {
  __shared__ C64 s_r[LT / 64][LR];
  const int t = threadIdx.x, rr = t & 15, grp = t >> 4, r = blockIdx.x * LR + rr, rs = min(r, k - 1);
  C64 acc = mk(0.0, 0.0);
  for (int j0 = grp; j0 < l; j0 += 8 * (LT / LR)) {
    C64 v[8], c[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int j = min(j0 + m * (LT / LR), l - 1);
      v[m] = V[(size_t)j * k + rs];
      c[m] = y[(size_t)j * ldy];
    }
#pragma unroll
    for (int m = 0; m < 8; ++m)
      if (j0 + m * (LT / LR) < l) acc = acc + cmul(v[m], c[m]);
  }
#pragma unroll
  for (int o = 16; o <= 32; o <<= 1) {
    acc.re += __shfl_xor(acc.re, o, 64);
    acc.im += __shfl_xor(acc.im, o, 64);
  }
  if ((t & 63) < LR) s_r[t >> 6][rr] = acc;
  __syncthreads();
  if (t < LR && r < k) z[r] = (s_r[0][rr] + s_r[1][rr]) + (s_r[2][rr] + s_r[3][rr]);
}

__global__ void __launch_bounds__(LT) k_in_lift(int k, int l, const C64* __restrict__ V, const C64* __restrict__ S,
                                                int lds, C64* __restrict__ z) {
  lift_rows(k, l, V, S, lds, z);
}

// the same for source blockIdx.y of a batch: order kv[s], lv[s] columns, its
// basis, matrix and result at multiples of vstride, ld * ld and zstride
__global__ void __launch_bounds__(LT) k_in_lift_batch(const int* __restrict__ kv, const int* __restrict__ lv,
                                                      const C64* __restrict__ V, size_t vstride,
                                                      const C64* __restrict__ S, int ld, C64* __restrict__ z,
                                                      int zstride) {
  const int s = blockIdx.y, k = kv[s];
  if ((int)blockIdx.x * LR >= k) return;
  lift_rows(k, lv[s], V + s * vstride, S + (size_t)s * ld * ld, ld, z + (size_t)s * zstride);
}

// z = column 0 of S (ld = k)
__global__ void k_col0(int k, const C64* __restrict__ S, C64* __restrict__ z) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r < k) z[r] = S[(size_t)r * k];
}

// ---------------------------------------------------------------------------
namespace {
DevBuf g_small, g_batch;
HostBuf g_small_pin;  // pinned readback of the inner iteration's flags
std::mutex g_coef_mu;
DevBuf g_coef;        // coefficients of small_sign_host, and
HostBuf g_coef_pin;   // their pinned staging, with the result

__global__ void k_zeros(int n, C64* __restrict__ z) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) z[i] = mk(0.0, 0.0);
}

__global__ void k_upload(int n, const C64* __restrict__ host, C64* __restrict__ dev) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) dev[i] = host[i];
}
}

// workspace of one inner problem of order k with ell steps, carved from base
// (base == nullptr: only the size); fills s.  The basis V and H_l may live
// elsewhere (vl, hl: diagonal, super- and sub-diagonal ldh apart).
static size_t inner_layout(int k, int ell, int hermitian, char* base, Inner* s, C64* vl = nullptr, C64* hl = nullptr,
                           int ldh = 0) {
  const int nb1 = (k + GR - 1) / GR, nb2 = (k + SR - 1) / SR;
  const size_t kk = (size_t)k * k;
  size_t bytes = 0;
  auto take = [&](size_t b) {
    size_t o = bytes;
    bytes += (b + 255) & ~(size_t)255;
    return o;
  };
  const size_t oB = take(kk * sizeof(C64));
  const size_t oBH = take(hermitian ? 0 : kk * sizeof(C64));
  const size_t oV = take(vl ? 0 : (size_t)k * ell * sizeof(C64));
  const size_t oW = take(hermitian ? 0 : (size_t)k * ell * sizeof(C64));
  const size_t oR = take((size_t)4 * k * sizeof(C64));
  const size_t oF = take((size_t)4 * k * sizeof(C64) + (size_t)k * sizeof(int));
  const size_t oC = take((size_t)3 * ell * sizeof(C64));
  const size_t oP1 = take((size_t)2 * nb1 * ell * sizeof(C64));
  const size_t oP2 = take((size_t)2 * nb2 * ell * sizeof(C64));
  const size_t oP3 = take((size_t)4 * nb2 * sizeof(double));
  const size_t oHc = take((size_t)ell * ell * sizeof(C64));
  const size_t oI = take(8 * sizeof(int));
  if (!base) return bytes;
  s->k = k;
  s->herm = hermitian;
  s->lmax = ell;
  s->B = (C64*)(base + oB);
  s->BH = hermitian ? s->B : (C64*)(base + oBH);
  s->V = vl ? vl : (C64*)(base + oV);
  s->W = hermitian ? s->V : (C64*)(base + oW);
  C64* R = (C64*)(base + oR);
  s->uraw[0] = R;
  s->uraw[1] = R + k;
  s->qraw[0] = R + 2 * k;
  s->qraw[1] = R + 3 * k;
  C64* F = (C64*)(base + oF);
  s->Lm = F;
  s->U0i = F + k;
  s->U1 = F + 2 * k;
  s->U2 = F + 3 * k;
  s->Sw = (int*)(F + 4 * k);
  if (!hl) {
    hl = (C64*)(base + oC);
    ldh = ell;
  }
  s->a = hl;
  s->b = hl + ldh;
  s->d = hl + 2 * ldh;
  s->part1 = (C64*)(base + oP1);
  s->part2 = (C64*)(base + oP2);
  s->part3 = (double*)(base + oP3);
  s->nb1 = nb1;
  s->nb2 = nb2;
  s->flags = (int*)(base + oI);
  s->hcol = (C64*)(base + oHc);
  s->arnoldi = 0;
  return bytes;
}

// B = H_k + H_k^{-1} (and B^dag), then the inner iteration of r problems (one:
// by value in s0; more: descriptors in device memory) of order up to kmax
// with up to lmax steps: one launch per kernel and step serves all of them
template <bool BATCH>
static void inner_launch(int r, const Inner& s0, const Inner* SS, int oneside, int kmax, int lmax, hipStream_t st) {
  const int kl = std::min(kmax, TRI_INV_LDS_MAX), kt = (kmax + 31) / 32;
  hipLaunchKernelGGL(k_tri_lu, dim3(r), dim3(256), tri_lu_lds(kmax), st, s0, SS);
  hipLaunchKernelGGL(k_tri_inv, dim3((kmax + 63) / 64, 1, r), dim3(64), (size_t)kl * (sizeof(TriF) + sizeof(int)), st,
                     s0, SS);
  if (!oneside) hipLaunchKernelGGL(k_adjoint, dim3(kt, kt, r), dim3(32, 8), 0, st, s0, SS);
  const int sides = oneside ? 1 : 2, nb1 = (kmax + GR - 1) / GR, nb2 = (kmax + SR - 1) / SR;
  const dim3 g1 = BATCH ? dim3(r * sides * nb1) : dim3(nb1, sides);
  const dim3 g2 = BATCH ? dim3(r * nb2) : dim3(nb2);
  for (int i = 0; i < lmax; ++i) {
    hipLaunchKernelGGL(k_in_gemv<BATCH>, g1, dim3(GR * 64), gemv_lds(i), st, s0, SS, sides * nb1, i);
    hipLaunchKernelGGL(k_in_sub<BATCH>, g2, dim3(ST), 0, st, s0, SS, nb2, i, 0);
    if (i + 1 < lmax) hipLaunchKernelGGL(k_in_sub<BATCH>, g2, dim3(ST), 0, st, s0, SS, nb2, i, 1);
  }
}

int small_sign_dev(int k, int ell, int hermitian, const C64* alpha, const C64* beta, const C64* delta,
                   int rh_scaling, int rh_maxit, double rh_tol, C64* z, SmallOut* out, hipStream_t st, int inner) {
  if (k <= 0) return NK_EINVAL;
  if (ell > k) ell = k;
  // Arnoldi runs the one-sided (Lanczos-form) recurrence on the general B and
  // keeps every coefficient; its H_l is upper Hessenberg
  const int arnoldi = inner == NK_INNER_ARNOLDI && ell > 0;
  const int oneside = hermitian || arnoldi;
  if (arnoldi && out && (out->hl_host || out->inner_only)) {
    set_error("the tridiagonal H_l export is for the outer level's family only");
    return NK_EINVAL;
  }
  if (ell <= 0) {
    // non-nested: RH on dense H_k
    if (g_small.ensure((size_t)k * k * sizeof(C64))) return NK_ENOMEM;
    C64* H = g_small.as<C64>();
    hipLaunchKernelGGL(k_tri_dense, dim3(1024), dim3(256), 0, st, k, alpha, beta, delta, H);
    NK_HIP(hipGetLastError());
    int it = 0;
    double res = 0;
    const TriIn tri{alpha, beta, delta, 0};
    int e = rh_sign_batched(1, k, &k, H, rh_scaling, rh_maxit, rh_tol, &it, &res, st, &tri);
    if (e < 0) return e;
    hipLaunchKernelGGL(k_col0, dim3((k + 255) / 256), dim3(256), 0, st, k, H, z);
    NK_HIP(hipGetLastError());
    if (out) {
      out->rh_iters = it;
      out->ell_used = 0;
      out->rh_residual = res;
    }
    return e;
  }
  // nested
  if (ell > LMAX) {
    set_error("inner Krylov size %d exceeds %d", ell, LMAX);
    return NK_EINVAL;
  }
  const size_t lay = inner_layout(k, ell, oneside, nullptr, nullptr);
  if (g_small.ensure(lay + (size_t)ell * ell * sizeof(C64)) || g_small_pin.ensure(2 * sizeof(int))) return NK_ENOMEM;
  char* base = g_small.as<char>();
  Inner s{};
  inner_layout(k, ell, oneside, base, &s);
  s.arnoldi = arnoldi;
  s.al = alpha;
  s.be = beta;
  s.de = delta;
  s.out = g_small_pin.dev<int>();
  C64* Hl = reinterpret_cast<C64*>(base + lay);
  inner_launch<false>(1, s, nullptr, oneside, k, ell, st);
  NK_HIP(hipGetLastError());
  NK_HIP(hipStreamSynchronize(st));
  const int* fl = g_small_pin.host<int>();
  const int brk = fl[0];
  if (fl[1]) {  // no result: zeros, not what the buffer held
    if (z) hipLaunchKernelGGL(k_zeros, dim3((k + 255) / 256), dim3(256), 0, st, k, z);
    NK_HIP(hipGetLastError());
    set_error("nested small problem: H_k is singular");
    return NK_WARN_NOTCONV;
  }
  const int lu = brk ? brk : ell;
  if (out && out->hl_host) {
    NK_HIP(hipMemcpyAsync(out->hl_host, s.a, lu * sizeof(C64), hipMemcpyDeviceToHost, st));
    NK_HIP(hipMemcpyAsync(out->hl_host + lu, s.b, lu * sizeof(C64), hipMemcpyDeviceToHost, st));
    NK_HIP(hipMemcpyAsync(out->hl_host + 2 * lu, s.d, lu * sizeof(C64), hipMemcpyDeviceToHost, st));
    NK_HIP(hipStreamSynchronize(st));
  }
  if (out && out->vl_dev)
    NK_HIP(hipMemcpyAsync(out->vl_dev, s.V, (size_t)k * lu * sizeof(C64), hipMemcpyDeviceToDevice, st));
  if (out && out->inner_only) {
    out->ell_used = lu;
    return brk ? NK_WARN_BREAKDOWN : NK_OK;
  }
  if (arnoldi)
    hipLaunchKernelGGL(k_hess_dense, dim3(256), dim3(256), 0, st, lu, ell, s.hcol, s.b, s.d, Hl);
  else
    hipLaunchKernelGGL(k_tri_dense, dim3(256), dim3(256), 0, st, lu, s.a, s.b, s.d, Hl);
  NK_HIP(hipGetLastError());
  int it = 0;
  double res = 0;
  const TriIn tri{s.a, s.b, s.d, 0};
  int e = rh_sign_batched(1, lu, &lu, Hl, rh_scaling, rh_maxit, rh_tol, &it, &res, st, arnoldi ? nullptr : &tri);
  if (e < 0) return e;
  hipLaunchKernelGGL(k_in_lift, dim3((k + LR - 1) / LR), dim3(LT), 0, st, k, lu, s.V, Hl, lu, z);
  NK_HIP(hipGetLastError());
  if (out) {
    out->rh_iters = it;
    out->ell_used = lu;
    out->rh_residual = res;
  }
  return e ? e : (brk ? NK_WARN_BREAKDOWN : NK_OK);
}

// The small problem on host coefficients, on the null stream.  The staging
// (4 k entries) is kept between calls and the coefficients are read from it by
// a kernel: an allocation, three copies of pageable memory and one back on
// every call were 45 of the plain method's 260 us at k = 500.
int small_sign_host(int k, int ell, int hermitian, const void* alpha, const void* beta, const void* delta,
                    int rh_scaling, int rh_maxit, double rh_tol, void* z, SmallOut* out, int inner) {
  std::lock_guard<std::mutex> lock(g_coef_mu);
  const size_t b = (size_t)k * sizeof(C64);
  if (g_coef.ensure(3 * b) || g_coef_pin.ensure(4 * b)) return NK_ENOMEM;
  char* h = g_coef_pin.host<char>();
  std::memcpy(h, alpha, b);
  std::memcpy(h + b, beta, b);
  std::memcpy(h + 2 * b, delta, b);
  std::memset(h + 3 * b, 0, b);  // a warning without a result (a singular H_k) leaves zeros
  C64* a = g_coef.as<C64>();
  hipLaunchKernelGGL(k_upload, dim3((3 * k + 255) / 256), dim3(256), 0, nullptr, 3 * k, g_coef_pin.dev<C64>(), a);
  const int e = small_sign_dev(k, ell, hermitian, a, a + k, a + 2 * k, rh_scaling, rh_maxit, rh_tol,
                               g_coef_pin.dev<C64>() + 3 * (size_t)k, out, nullptr, inner);
  // (also after a failure: nothing may still read the staging when the next call fills it)
  const hipError_t es = hipStreamSynchronize(nullptr);
  if (e < 0) return e;
  NK_HIP(es);
  std::memcpy(z, h + 3 * b, b);
  return e;
}

// The inner projections of r problems at once: one launch per kernel and
// step serves all of them.  Problem s has order k[s] and ell[s] steps; its
// H_ell (diagonal, super-, sub-diagonal, zero from its last step on) goes to
// hl_dev + s * 3 * ldh (rows of ldh) and its basis V_ell (column j at
// j * k[s]) to vl_dev + s * vl_stride; ell_used[s] < ell[s] after an
// invariant subspace or a breakdown, 0 where H_k is singular (the others are
// not concerned).
int small_inner_batch(int r, const int* k, const int* ell, int hermitian, const C64* alpha, const C64* beta,
                      const C64* delta, size_t cstride, C64* hl_dev, int ldh, C64* vl_dev, size_t vl_stride,
                      int* ell_used, hipStream_t st) {
  std::vector<size_t> off(r + 1, 0);
  for (int s = 0; s < r; ++s) {
    if (ell[s] < 1 || ell[s] > LMAX || ell[s] > k[s] || ell[s] > ldh) {
      set_error("inner problem %d: ell = %d outside [1, min(k = %d, %d)]", s, ell[s], k[s], LMAX);
      return NK_EINVAL;
    }
    off[s + 1] = off[s] + inner_layout(k[s], ell[s], hermitian, nullptr, nullptr, vl_dev);
  }
  // descriptors: written to pinned memory, read by the kernels from the device's copy
  const size_t dbytes = (size_t)r * sizeof(Inner);
  if (g_batch.ensure(off[r] + dbytes) || g_small_pin.ensure(dbytes + (size_t)2 * r * sizeof(int))) return NK_ENOMEM;
  char* base = g_batch.as<char>();
  Inner* S = g_small_pin.host<Inner>();
  int* fl = reinterpret_cast<int*>(g_small_pin.host<char>() + dbytes);
  int* fl_dev = reinterpret_cast<int*>(g_small_pin.dev<char>() + dbytes);
  int lmax = 0, kmax = 0;
  for (int s = 0; s < r; ++s) {
    Inner in{};
    inner_layout(k[s], ell[s], hermitian, base + off[s], &in, vl_dev + s * vl_stride, hl_dev + (size_t)s * 3 * ldh, ldh);
    in.al = alpha + s * cstride;
    in.be = beta + s * cstride;
    in.de = delta + s * cstride;
    in.out = fl_dev + 2 * s;
    S[s] = in;
    lmax = std::max(lmax, ell[s]);
    kmax = std::max(kmax, k[s]);
  }
  Inner* sdev = reinterpret_cast<Inner*>(base + off[r]);
  NK_HIP(hipMemcpyAsync(sdev, S, dbytes, hipMemcpyHostToDevice, st));
  inner_launch<true>(r, Inner{}, sdev, hermitian, kmax, lmax, st);
  NK_HIP(hipGetLastError());
  NK_HIP(hipStreamSynchronize(st));
  int warn = NK_OK;
  for (int s = 0; s < r; ++s) {
    if (fl[2 * s + 1]) {
      set_error("nested small problem %d: H_k is singular", s);
      ell_used[s] = 0;
      warn = NK_WARN_NOTCONV;
      continue;
    }
    ell_used[s] = fl[2 * s] ? fl[2 * s] : ell[s];
    if (fl[2 * s] && warn == NK_OK) warn = NK_WARN_BREAKDOWN;
  }
  return warn;
}

void small_lift_batch(int r, int kmax, const int* kv, const int* lv, const C64* V, size_t vstride, const C64* S,
                      int ld, C64* z, int zstride, hipStream_t st) {
  hipLaunchKernelGGL(k_in_lift_batch, dim3((kmax + LR - 1) / LR, r), dim3(LT), 0, st, kv, lv, V, vstride, S, ld, z,
                     zstride);
}

}  // namespace nk
