// The Roberts-Higham iteration of Eq. (4) from a tridiagonal start matrix H
// (the Ritz matrix H_k, or H_l of the inner Lanczos space), without
// inverting its dense iterates.
//
// Every iterate is a rational function of H, S_{n+1} = (mu_n S_n +
// (mu_n S_n)^{-1}) / 2 with S_0 = H (mu_n = 1 unscaled), and so is its inverse.
// S_n^{-1} has simple poles only, the 2^n zeros of S_n.  They lie on the
// imaginary axis: with S_n(i t) = i s_n(t), s_{n+1} = (mu s_n - 1/(mu s_n)) / 2,
// they are the preimages of 0, found backwards from y = 0 by
//   y <- (y +- sqrt(y^2 + 1)) / mu_m,  m = n - 1 .. 0,
// and the residue at a zero t is rho = 1 / s_n'(t), s_n'(t) = prod_m
// (mu_m + 1/(mu_m y_m^2)) / 2 along the same path (a product of positive terms).
// So
//   S_n^{-1} = sum over the 2^n zeros of  rho (H - i t)^{-1},
// a sum of inverses of tridiagonal matrices: O(2^n k^2) work with one
// dependent chain of length k, against the k dependent pivots of an O(k^3)
// elimination.  The iterates, the change that the stopping test looks at and
// the iteration count are those of Eq. (4).
//
// One inverse: with the leading minors N_i and the trailing ones M_i of
// H - i t (the three-term recurrences N_{i+1} = (a_i - i t) N_i - b_{i-1} d_{i-1}
// N_{i-1} and its mirror image; each computed minor is the exact one of a
// matrix whose entries a_i - i t and b d differ from H's by a few units in the
// last place) the pivots of the two eliminations are D_i = N_{i+1} / N_i and
// E_i = M_i / M_{i+1}, and
//   (M^{-1})_jj = 1 / g_j,  g_j = D_j - b_j d_j / E_{j+1},
//   (M^{-1})_ij = (M^{-1})_{i+1,j} u_i,  u_i = -b_i / D_i      for i < j,
//   (M^{-1})_ij = (M^{-1})_{i-1,j} l_i,  l_i = -d_{i-1} / E_i  for i > j
// (b, d the super- and sub-diagonal).  An exactly zero pivot is replaced by
// 1e-30 of the matrix's size.  Between two different blocks of 16 rows the
// inverse therefore has rank one per pole: for a block of rows c before the
// block of columns C,
//   rho (M^{-1})_ij = [u_i .. u_end(c)] [all u of the blocks between] [rho / g_j u_start(C) .. u_{j-1}],
// so a 16 x 16 tile of S_n^{-1} is a product of a 16 x 2^n and a 2^n x 16
// matrix, which the FP64 matrix cores form.  The tiles on the diagonal are cut
// the same way, into the pairs of halves of blocks of 16, 8, 4 and 2 rows and
// the diagonal itself: nine such products, each for its own entries.
//
// Against the oracle the result is as accurate as the iteration with explicit
// inverses or more (k = 300, condition 1.4e4: 1.2e-13 from the spectral sign
// against 4.2e-13).
//
// Where it does not apply, a matrix is flagged and goes back to the iteration
// with explicit inverses from S_0: when a last pivot vanishes (an iterate is
// singular), when a row is more than 2^50 below the largest entry (a pivot
// below 1e-30 could then be the true one), or when the minors leave 2^-900
// within a block of rows (the next one could underflow).  Entries of up to
// 2^50 of their neighbours are taken: the quotients of minors are formed of operands
// scaled by a power of two, since the minors of small rows fall by that factor
// row after row (order 64, diagonal +-2 with one entry of 1e12: 2e-16 of S_9 e_1
// from the explicit inverses; squares of unscaled minors underflowed from
// 1e10 on).
//
// Kernels, over a batch (grid z):
//   k_tri_chain (k_tri_chain_mu when scaled): the minors, one lane per pole and
//     direction, all poles of all steps at once (scaled: step by step, since
//     mu_n needs det S_n, a quotient of determinants of H - i t);
//   k_tri_mid, k_tri_between: the factors above;
//   k_tri_tile: S_1 .. S_L of the entries of a 16 x 16 tile in registers, and
//     the sums of the stopping test.
// Measured for k = 500, nine steps (511 poles): 37 + 29 + 8 + 53 us, where the
// blocked elimination and its Newton-Schulz tail took 5.2 ms; for k = 60, ten
// steps 9 + 18 + 3 + 28 us (the one-workgroup elimination: 455 to 600).
#include <algorithm>
#include <cmath>

#include "hostbuf.h"
#include "nk_internal.h"
#include "rhtri.h"
#include "wave.h"

namespace nk {

namespace {

constexpr int TB = 16;  // rows of a block, and poles of a step on the matrix cores
constexpr double TINYPIV = 1e-30, SINGPIV = 1e-28;
constexpr double ROWLOW = 0x1p-50;  // rows below this part of the matrix's largest entry: flagged
constexpr int MINLOW = -900;        // exponent of the minors of a block below which: flagged

typedef double nk_d4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ double abs1(C64 a) { return fabs(a.re) + fabs(a.im); }

// the exponent of a's larger component (2^e is above it)
__device__ __forceinline__ int expo(C64 a) {
  int e;
  (void)frexp(fmax(fabs(a.re), fabs(a.im)), &e);
  return e;
}
// 1 / a: one reciprocal with two Newton steps (of pivots, between 1e-30 and
// 1e30 by the replacement of smaller ones, and what they are combined to)
__device__ __forceinline__ C64 recip(C64 a) {
  const double n = fma(a.im, a.im, a.re * a.re);
  double y = __builtin_amdgcn_rcp(n);
  y = fma(y, fma(-n, y, 1.0), y);
  y = fma(y, fma(-n, y, 1.0), y);
  return mk(a.re * y, -a.im * y);
}

// the zero with index q = 2^n + j of S_n and its residue (mu == nullptr: unscaled)
__device__ __forceinline__ void zero_of(int q, const double* mu, double* t, double* rho) {
  double y = 0.0, f = 1.0;
  const int n = q > 0 ? 31 - __clz(q) : 0;
  for (int m = n - 1; m >= 0; --m) {
    const double s = (q >> m) & 1 ? -1.0 : 1.0;
    const double big = fabs(y) + sqrt(fma(y, y, 1.0));
    const double u = mu ? mu[m] : 1.0;
    y = (s * y >= 0.0 ? s * big : s / big) / u;
    f *= 0.5 * (u + 1.0 / (u * y * y));
  }
  *t = y;
  *rho = q > 0 ? 1.0 / f : 0.0;  // index 0 pads the first group
}

// workspace of a batch.  Minors: per matrix nch blocks of 18 rows of np poles (a
// lane of the recurrences is a pole).  The factors: np poles of ldp = 16 nch
// rows (a lane of the products is a row), so every load is of whole lines.
struct TriWs {
  int ld, np, nch, nsum;  // nch blocks of 16 rows; nsum workgroups of k_tri_tile
  C64* N;     // block c, entry r = 0 .. 16: N_{16 c + r}, up to one power of two per block, times kappa^i; entry 17:
              // N_{16 c - 1}
  C64* M;     // block c, entry r: M_{16 c + r} likewise; entry 17: M_{e + 1}, e the row after the block
  C64* au;    // u_i .. u_end of the row's block
  C64* ad;    // l_start .. l_i
  C64* bu;    // rho / g_j u_start .. u_{j-1}
  C64* bd;    // rho / g_j l_{j+1} .. l_end
  C64* gg;    // rho / g
  C64* fu[4]; // above the diagonal, splits into halves of 8, 4, 2, 1 rows: row in the first half: u up to the
              // split, in the second: rho / g times the u from the split
  C64* fd[4]; // below the diagonal: row in the first half: rho / g times the l up to the split, in the second: the
              // l from the split
  C64* rt;    // [batch][nch][2][np] products of all u, all l of a block
  C64* rr;    // [batch][nch (C)][nch (c)][np] products over the blocks between c and C
  double* rho;  // [batch][np] residues
  double* kap;  // [batch][np] each pole's kappa
  double* mu;   // [batch][L]
  double* sums; // [batch][2 L][nsum]
  int* sing;    // [batch]
};

// entry r of block c of matrix b's minors
__device__ __forceinline__ size_t mix(const TriWs& w, int b, int c, int r) {
  return (((size_t)b * w.nch + c) * (TB + 2) + r) * w.np;
}

// 64 rows of a matrix in LDS: the diagonal, and the product b d of the pair
// that couples a row to the one before it in the recurrence, both of the matrix
// over the power of two that brings its largest entry to one (exact; products
// of entries below 1e-154 would underflow)
struct Rows {
  C64 a[64], c[64];
};

// One recurrence by the lanes of one wave, each following its own pole q of
// the same matrix (lanes without one repeat another's): DIR 0 the leading
// minors from row 0 up, DIR 1 the trailing ones from the last row down.  Entries
// are scaled by kappa, the power of two that brings H - i t to entries of at
// most one, and the running pair by a power of two at every block of 16 rows.
// Bound by the latency of its k dependent steps (two dependent products each;
// carrying the pivots themselves, with a reciprocal per step, took 158 ns a
// step, this 74 ns at k = 500).  A minor may vanish: the recurrence does not divide.
// DIR 0 flags what the closed form does not cover (see above) and (LD) leaves
// log|det(H - i t)| in *ld; with rows, its rows are looked at too (one wave's
// work for the whole matrix).
template <bool LD, int DIR>
__device__ __forceinline__ void chain(const TriWs& w, const TriIn& h, int b, int n, int q, double t, Rows& sh,
                                      double* ld, bool rows = false) {
  const C64* a = h.a + b * h.stride;
  const C64* be = h.b + b * h.stride;
  const C64* de = h.d + b * h.stride;
  const int lane = threadIdx.x & 63;
  const int nblk = (n + TB - 1) / TB, nld = (n + 63) / 64;
  double sc = 0.0, low = INFINITY;  // the matrix's largest entry, and the least over the rows of a row's largest
#pragma unroll 8
  for (int k = 0; k < nld; ++k) {
    const int i = min(64 * k + lane, n - 1), j = min(i, max(n - 2, 0)), j1 = max(i - 1, 0);
    const double sb = n > 1 ? abs1(be[j]) : 0.0, sd = n > 1 ? abs1(de[j]) : 0.0, sa = abs1(a[i]);
    sc = fmax(sc, fmax(sa, fmax(sb, sd)));
    if (DIR == 0 && rows) {
      const double s1 = i > 0 ? abs1(de[j1]) : 0.0;
      low = fmin(low, fmax(sa, fmax(i + 1 < n ? sb : 0.0, s1)));
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    sc = fmax(sc, __shfl_xor(sc, o, 64));
    if (DIR == 0 && rows) low = fmin(low, __shfl_xor(low, o, 64));
  }
  int ks, ke;
  (void)frexp(sc, &ks);
  (void)frexp(sc + fabs(t), &ke);
  const double kt = ldexp(t, -ke), kap = ldexp(1.0, ks - ke), kap2 = kap * kap;  // kap: of the rows in LDS
  if (DIR == 0) w.kap[(size_t)b * w.np + q] = ldexp(1.0, -ke);
  auto sca = [&](C64 v) { return mk(ldexp(v.re, -ks), ldexp(v.im, -ks)); };
  C64 ra, rc;
  auto fetch = [&](int k) {  // rows 64 k ..
    const int i = 64 * k + lane;
    const bool in = i < n;
    const int j = DIR == 0 ? i - 1 : i;  // the pair that couples row i to the row before it
    const bool inb = j >= 0 && j + 1 < n;
    const C64 va = sca(a[in ? i : 0]), vc = cmul(sca(be[inb ? j : 0]), sca(de[inb ? j : 0]));
    ra = mk(in ? va.re : 0.0, in ? va.im : 0.0);
    rc = mk(inb ? vc.re : 0.0, inb ? vc.im : 0.0);
  };
  fetch(DIR == 0 ? 0 : nld - 1);
  C64 x = mk(1.0, 0.0), y = mk(0.0, 0.0);  // the minor before this row, and the one before that
  int ex = 0, least = 0;
  C64* out = DIR == 0 ? w.N : w.M;
  for (int kk = 0; kk < nld; ++kk) {
    const int k = DIR == 0 ? kk : nld - 1 - kk;
    __builtin_amdgcn_wave_barrier();
    sh.a[lane] = ra;
    sh.c[lane] = rc;
    __builtin_amdgcn_wave_barrier();
    if (kk + 1 < nld) fetch(DIR == 0 ? k + 1 : k - 1);
    for (int cc = 0; cc < 4; ++cc) {
      const int sub = DIR == 0 ? cc : 3 - cc, c = 4 * k + sub;
      if (c >= nblk) continue;
      const int nr = min(n - c * TB, TB);
      // the pair's power of two
      int e;
      (void)frexp(fmax(fmax(fabs(x.re), fabs(x.im)), fmax(fabs(y.re), fabs(y.im))), &e);
      least = min(least, e);
      x = mk(ldexp(x.re, -e), ldexp(x.im, -e));
      y = mk(ldexp(y.re, -e), ldexp(y.im, -e));
      if (LD) ex += e;
      C64* o = out + mix(w, b, c, 0) + q;
      o[(size_t)(DIR == 0 ? 0 : nr) * w.np] = x;
      o[(size_t)(TB + 1) * w.np] = y;
      auto step = [&](int r) {
        const C64 ai = sh.a[sub * TB + r], ci = sh.c[sub * TB + r];
        const C64 s = mk(kap * ai.re, fma(kap, ai.im, -kt)), p = mk(kap2 * ci.re, kap2 * ci.im);
        // s x - p y, the product with y first: it does not wait for x
        const C64 f = mk(fma(p.im, y.im, -(p.re * y.re)), -fma(p.re, y.im, p.im * y.re));
        const C64 nx = mk(fma(-s.im, x.im, fma(s.re, x.re, f.re)), fma(s.im, x.re, fma(s.re, x.im, f.im)));
        y = x;
        x = nx;
        o[(size_t)(DIR == 0 ? r + 1 : r) * w.np] = x;
      };
      if (nr == TB) {
#pragma unroll
        for (int r = 0; r < TB; ++r) step(DIR == 0 ? r : TB - 1 - r);
      } else {
        for (int r = 0; r < nr; ++r) step(DIR == 0 ? r : nr - 1 - r);
      }
    }
  }
  least = min(least, max(expo(x), expo(y)));
  if (q > 0 && least < MINLOW) w.sing[b] = 1;
  if (DIR == 0 && q > 0 && !(abs1(x) > SINGPIV * abs1(y) && low >= ROWLOW * sc)) w.sing[b] = 1;
  if (LD) {
    const int e = expo(x);
    const C64 s = mk(ldexp(x.re, -e), ldexp(x.im, -e));
    *ld = abs1(x) > 0.0 ? 0.5 * log(norm2(s)) + (ex + e + (double)n * ke) * 0.69314718055994530942 : -1e300;
  }
}

// unscaled: every pole's zero is known beforehand; one wave per 64 poles and direction
__global__ void __launch_bounds__(64) k_tri_chain(TriWs w, TriIn h, const int* __restrict__ nvec, int L) {
  __shared__ Rows sh;
  const int b = blockIdx.z, n = nvec[b];
  const int q = blockIdx.x * 64 + threadIdx.x;  // np is a multiple of 64
  if (q == 0 && blockIdx.y == 0)
    for (int m = 0; m < L; ++m) w.mu[(size_t)b * L + m] = 1.0;
  if (n <= 0) return;
  double t, rho;
  zero_of(q, nullptr, &t, &rho);
  if (blockIdx.y == 0) w.rho[(size_t)b * w.np + q] = q < (1 << L) ? rho : 0.0;
  if (blockIdx.y == 0)
    chain<false, 0>(w, h, b, n, q, t, sh, nullptr, blockIdx.x == 0);
  else
    chain<false, 1>(w, h, b, n, q, t, sh, nullptr);
}

// scaled: one workgroup per matrix, step by step.  log|det S_n| from the
// factored form S_n = C prod_zeros(S_n) (H - i t) / prod of the zeros of S_m,
// m < n, with C = prod mu_m / 2; then mu_n = |det S_n|^{-1/k}, times the
// learned correction where there is one.
__global__ void __launch_bounds__(512) k_tri_chain_mu(TriWs w, TriIn h, const int* __restrict__ nvec, int L,
                                                      const double* __restrict__ sched, int nsched) {
  __shared__ Rows sh[8];
  __shared__ double s_mu[16], s_red[8];
  const int b = blockIdx.z, n = nvec[b];
  if (n <= 0) return;
  const int j = threadIdx.x & 255;
  const int dir = __builtin_amdgcn_readfirstlane(threadIdx.x >> 8), wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double prevs = 0.0, logc = 0.0;  // sum of log|det| over the earlier steps' zeros, log C
  for (int s = 0; s < L; ++s) {
    const int half = 1 << s;  // 2^s <= 256 poles, the two directions in their own waves
    double v = 0.0;
    if ((j & ~63) < half) {
      const bool live = j < half;
      const int q = half + (live ? j : 0);
      double t, rho, ld = 0.0;
      zero_of(q, s_mu, &t, &rho);
      if (dir == 0) w.rho[(size_t)b * w.np + q] = rho;
      if (dir == 0)
        chain<true, 0>(w, h, b, n, q, t, sh[wv], &ld, s == 0);
      else
        chain<false, 1>(w, h, b, n, q, t, sh[wv], nullptr);
      if (dir == 0 && live) v = ld;
    }
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s_red[wv] = v;
    __syncthreads();
    double ld = 0.0;
    for (int k = 0; k < 8; ++k) ld += s_red[k];
    double mu = exp(-(ld - prevs + n * logc) / n);
    if (sched && s < nsched) {
      const double c = sched[(size_t)b * nsched + s];
      if (c > 0.0) mu *= c;
    }
    prevs += ld;
    logc += log(0.5 * mu);
    if (threadIdx.x == 0) {
      s_mu[s] = mu;
      w.mu[(size_t)b * L + s] = mu;
    }
    __syncthreads();
  }
  // the padding pole 0, and the poles of steps past L: any regular shift, with
  // a zero residue
  for (int q0 = 0; q0 < w.np; q0 += 256) {
    const int q = q0 + j;
    const bool pad = q == 0 || (q >= (1 << L) && q < w.np);
    if (!__any(pad)) continue;
    const int first = q0 == 0 ? 0 : 1 << L;  // lanes without a pole repeat one of the pads
    const int qq = pad ? q : (first == 0 ? 0 : first);
    if (dir == 0) w.rho[(size_t)b * w.np + qq] = 0.0;
    if (dir == 0)
      chain<false, 0>(w, h, b, n, qq, 1.0, sh[wv], nullptr);
    else
      chain<false, 1>(w, h, b, n, qq, 1.0, sh[wv], nullptr);
  }
}

__device__ __forceinline__ C64 quot(C64 a, C64 b) {
  return cmul(a, recip(b));
}
// the quotient of two minors, which may lie anywhere in the exponent range:
// both scaled by the power of two (exact) that brings b to one
__device__ __forceinline__ C64 quot_minors(C64 a, C64 b) {
  const int e = expo(b);
  return quot(mk(ldexp(a.re, -e), ldexp(a.im, -e)), mk(ldexp(b.re, -e), ldexp(b.im, -e)));
}
// rho / g and the products within a block of 16 rows: a lane per pole, a wave
// per block and direction (y = 2 block + direction); every load is known at
// the start, so the whole block costs about one memory round trip
__global__ void __launch_bounds__(64) k_tri_mid(TriWs w, TriIn h, const int* __restrict__ nvec) {
  const int b = blockIdx.z, n = nvec[b];
  const int q = blockIdx.x * 64 + threadIdx.x, c = blockIdx.y >> 1, dir = blockIdx.y & 1;
  const int lo = c * TB, nr = min(n - lo, TB);
  if (nr <= 0) return;  // (np is a multiple of 64)
  const C64* be = h.b + b * h.stride;
  const C64* de = h.d + b * h.stride;
  const double rho = w.rho[(size_t)b * w.np + q];
  const double kap = w.kap[(size_t)b * w.np + q];  // the minors are those of kappa (H - i t)
  // f: the direction's multipliers; g: rho / g_j
  C64 f[TB], g[TB];
  {
    const C64* N = w.N + mix(w, b, c, 0) + q;
    const C64* M = w.M + mix(w, b, c, 0) + q;
    C64 nv[TB + 1], mv[TB + 1];
#pragma unroll
    for (int k = 0; k <= TB; ++k) {
      nv[k] = N[(size_t)min(k, nr) * w.np];
      mv[k] = M[(size_t)min(k, nr) * w.np];
    }
    C64 np1 = N[(size_t)(TB + 1) * w.np], mp1 = M[(size_t)(TB + 1) * w.np];
    // the row after the block: l needs its pair of trailing minors, in that block's scale
    const bool more = lo + nr < n;
    const C64* M2 = w.M + mix(w, b, more ? c + 1 : c, 0) + q;
    C64 m0 = M2[0], m1 = M2[w.np];
    // vanishing minors replaced by TINYPIV of the one before them: the same
    // value, up to the block's power of two, wherever it is read
    auto fix = [](C64 v, C64 before) {
      const double low = TINYPIV * abs1(before);
      return abs1(v) < low ? mk(low, 0.0) : v;
    };
    nv[0] = fix(nv[0], np1);
#pragma unroll
    for (int k = 1; k <= TB; ++k) nv[k] = fix(nv[k], nv[k - 1]);
    {
      const bool one = n - (lo + nr) == 1;  // the next block is its last row alone: m1 = M_n = 1
      const C64 mm = M2[(size_t)(one ? TB + 1 : 2) * w.np];
      m1 = one ? m1 : fix(m1, mm);
      m0 = fix(m0, m1);
    }
    // l_{j+1} of the row below each row j
    C64 ln = mk(0.0, 0.0);
    if (more) {
      const C64 d = de[lo + nr - 1];
      ln = quot(mk(-kap * d.re, -kap * d.im), quot_minors(m0, m1));
    }
    if (nr == TB && more) mv[TB] = fix(mv[TB], mp1);  // (M_n = 1 needs none)
#pragma unroll
    for (int k = TB - 1; k >= 0; --k)
      if (k < nr) mv[k] = fix(mv[k], mv[k + 1]);
#pragma unroll
    for (int k = TB - 1; k >= 0; --k) {
      if (k < nr) {
        const int j = lo + k;
        const C64 D = quot_minors(nv[k + 1], nv[k]);  // kappa D_j
        const C64 bj = be[j + 1 < n ? j : 0];
        C64 gj = D;
        if (j + 1 < n) gj = gj + cmul(mk(kap * bj.re, kap * bj.im), ln);
        const C64 r = recip(gj);
        const double f0 = rho * kap;
        g[k] = mk(rho != 0.0 ? f0 * r.re : 0.0, rho != 0.0 ? f0 * r.im : 0.0);  // (rho = 0: padding)
        const C64 dj = de[j > 0 ? j - 1 : 0];
        const C64 l = j > 0 ? quot(mk(-kap * dj.re, -kap * dj.im), quot_minors(mv[k], mv[k + 1])) : mk(0.0, 0.0);
        f[k] = dir ? l : (j + 1 < n ? quot(mk(-kap * bj.re, -kap * bj.im), D) : mk(0.0, 0.0));
        ln = l;
      } else {
        f[k] = mk(0.0, 0.0);
        g[k] = mk(0.0, 0.0);
      }
    }
  }
  const size_t o0 = ((size_t)b * w.np + q) * w.nch * TB + lo;
  // products over a block of S rows (S = 16: the whole one): from its middle
  // outwards for the halves of the block, from its ends for the other blocks
  auto store = [&](C64* a, int k, C64 v) { a[o0 + k] = v; };  // (rows past the order: finite, never used)
  if (dir == 0) {
    C64 p = mk(1.0, 0.0);
#pragma unroll
    for (int k = 0; k < TB; ++k) {
      store(w.bu, k, cmul(g[k], p));
      if (k < nr) p = cmul(p, f[k]);
    }
    w.rt[(((size_t)b * w.nch + c) * 2 + dir) * w.np + q] = p;
    p = mk(1.0, 0.0);
#pragma unroll
    for (int k = TB - 1; k >= 0; --k) {
      if (k < nr) p = cmul(p, f[k]);
      store(w.au, k, p);
    }
#pragma unroll
    for (int hh = 0; hh < 4; ++hh) {
      const int H = 8 >> hh;
#pragma unroll
      for (int m = H; m < TB; m += 2 * H) {  // the split: rows m - H .. m - 1 and m .. m + H - 1
        p = mk(1.0, 0.0);
#pragma unroll
        for (int k = m - 1; k >= m - H; --k) store(w.fu[hh], k, p = cmul(p, f[k]));
        p = mk(1.0, 0.0);
#pragma unroll
        for (int k = m; k < m + H; ++k) {
          store(w.fu[hh], k, cmul(g[k], p));
          p = cmul(p, f[k]);
        }
      }
    }
  } else {
    C64 p = mk(1.0, 0.0);
#pragma unroll
    for (int k = TB - 1; k >= 0; --k) {
      store(w.bd, k, cmul(g[k], p));
      store(w.gg, k, g[k]);
      if (k < nr) p = cmul(p, f[k]);
    }
    w.rt[(((size_t)b * w.nch + c) * 2 + dir) * w.np + q] = p;
    p = mk(1.0, 0.0);
#pragma unroll
    for (int k = 0; k < TB; ++k) {
      if (k < nr) p = cmul(p, f[k]);
      store(w.ad, k, p);
    }
#pragma unroll
    for (int hh = 0; hh < 4; ++hh) {
      const int H = 8 >> hh;
#pragma unroll
      for (int m = H; m < TB; m += 2 * H) {
        p = mk(1.0, 0.0);
#pragma unroll
        for (int k = m - 1; k >= m - H; --k) {
          store(w.fd[hh], k, cmul(g[k], p));
          p = cmul(p, f[k]);
        }
        p = mk(1.0, 0.0);
#pragma unroll
        for (int k = m; k < m + H; ++k) store(w.fd[hh], k, p = cmul(p, f[k]));
      }
    }
  }
}

// products over the blocks strictly between c and C, for every pair: a lane
// per pole, a wave per C and direction
__global__ void __launch_bounds__(64) k_tri_between(TriWs w, const int* __restrict__ nvec) {
  const int b = blockIdx.z, n = nvec[b];
  const int q = blockIdx.x * 64 + threadIdx.x, C = blockIdx.y >> 1, dir = blockIdx.y & 1;
  const int nc = (n + TB - 1) / TB;
  if (C >= nc) return;
  C64* rr = w.rr + ((size_t)b * w.nch + C) * w.nch * w.np + q;
  const C64* rt = w.rt + ((size_t)b * w.nch * 2 + dir) * w.np + q;
  C64 p = mk(1.0, 0.0);
  if (dir == 0) {
#pragma unroll 4
    for (int c = C - 1; c >= 0; --c) {
      rr[(size_t)c * w.np] = p;
      p = cmul(p, rt[(size_t)c * 2 * w.np]);
    }
  } else {
#pragma unroll 4
    for (int c = C + 1; c < nc; ++c) {
      rr[(size_t)c * w.np] = p;
      p = cmul(p, rt[(size_t)c * 2 * w.np]);
    }
  }
}

// S_1 .. S_L of one 16 x 16 tile (rows of block c, columns of block C), or of
// one part of a tile on the diagonal.  Per step the waves share the
// poles, on the matrix cores (layout: lane l holds A[l % 16][l / 16],
// B[l / 16][l % 16] and D[4 i + l / 16][l % 16]); the partial sums meet in LDS, where
// every thread owns one entry of the tile, takes it from S_n to S_{n+1} and
// adds to the step's sums.  S holds S_0 = H and receives S_L.  Bound by the
// matrix cores' FP64 rate and the loads of the factors from L2; nothing of an
// inverse goes through memory (kept as partial sums per 16 poles, in an
// earlier form, they were 140 MB written and read at k = 500, 140 + 37 us).
// steps, if given: the steps of each matrix (at most Lw), none where it is not positive.
constexpr int TLMAX = 10;
constexpr int TPARTS = 9;  // parts of a diagonal tile: halves of 16, 8, 4, 2 rows above, then below, then the diagonal
template <int NW>
__global__ void __launch_bounds__(64 * NW, NW == 4 ? 3 : 4) k_tri_tile(TriWs w, const int* __restrict__ nvec, int Lw,
                                                                          const int* __restrict__ steps, C64* S_b) {
  __shared__ C64 red[2 * NW][TB][TB + 1];  // partial tiles: of the first six steps, later two sets, one per wave
  __shared__ double sred[4][2 * TLMAX];
  const int b = blockIdx.z, n = nvec[b], L = steps ? steps[b] : Lw;
  if (L <= 0) return;
  // workgroups: the parts of the diagonal tiles, then the other tiles row by row
  const int nd = w.nch * TPARTS;
  int c, C, part = -1;
  if ((int)blockIdx.x < nd) {
    c = C = blockIdx.x / TPARTS;
    part = blockIdx.x % TPARTS;
  } else {
    const int t = blockIdx.x - nd;
    c = t / (w.nch - 1);
    C = t % (w.nch - 1);
    C += C >= c ? 1 : 0;
  }
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l16 = lane & 15, lq = lane >> 4;
  const int er = (threadIdx.x >> 4) & 15, ec = threadIdx.x & 15;  // the entry this thread (of the first four waves) owns
  bool own = wv < 4 && c * TB + er < n && C * TB + ec < n;
  const int ldp = w.nch * TB;
  const C64 *A, *B;
  const C64* R = nullptr;
  bool ones = false;
  if (part < 0) {
    A = c < C ? w.au : w.ad;
    B = c < C ? w.bu : w.bd;
    R = w.rr + (((size_t)b * w.nch + C) * w.nch + c) * w.np;
  } else if (part < 8) {
    const int hh = part & 3, H = 8 >> hh;
    const bool below = part >= 4;
    A = B = below ? (hh == 0 ? w.fd[0] : hh == 1 ? w.fd[1] : hh == 2 ? w.fd[2] : w.fd[3])
                  : (hh == 0 ? w.fu[0] : hh == 1 ? w.fu[1] : hh == 2 ? w.fu[2] : w.fu[3]);
    own = own && (er ^ ec) < 2 * H && ((er & H) != 0) == below && ((ec & H) != 0) != below;
  } else {
    A = B = w.gg;
    ones = true;
    own = own && er == ec;
  }
  double ds[TLMAX], ns[TLMAX];
#pragma unroll
  for (int m = 0; m < TLMAX; ++m) ds[m] = ns[m] = 0.0;
  if (c * TB < n && C * TB < n) {
    const size_t so = (size_t)b * w.ld * w.ld + (size_t)(own ? c * TB + er : 0) * w.ld + (own ? C * TB + ec : 0);
    C64 s = S_b[so];
    const double* mu = w.mu + (size_t)b * Lw;
    // this lane's row of the left and column of the right factor
    A += (size_t)b * w.np * ldp + c * TB + l16;
    B += (size_t)b * w.np * ldp + C * TB + l16;
    struct Ops {
      C64 x[4], b[4];
    };
    // the operands of 16 poles, the left one times the blocks between
    auto load = [&](int g) {
      Ops o;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int q = g + 4 * u + lq;
        o.x[u] = A[(size_t)q * ldp];
        o.b[u] = B[(size_t)q * ldp];
        if (R) o.x[u] = cmul(R[q], o.x[u]);
        if (ones) o.x[u] = mk(1.0, 0.0);
      }
      return o;
    };
    nk_d4 re, im;
    auto zero = [&]() { re = im = nk_d4{0.0, 0.0, 0.0, 0.0}; };
    auto mac = [&](C64 x, C64 y) {
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(x.re, y.re, re, 0, 0, 0);
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(-x.im, y.im, re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.re, y.im, im, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(x.im, y.re, im, 0, 0, 0);
    };
    auto put = [&](int slot) {
#pragma unroll
      for (int i = 0; i < 4; ++i) red[slot][4 * i + lq][l16] = mk(re[i], im[i]);
    };
    auto update = [&](int m, C64 T) {
      const double u = mu[m];
      const C64 xs = u * s;
      s = 0.5 * (xs + (1.0 / u) * T);
      if (own) {
        ds[m] = norm2(s - xs);
        ns[m] = norm2(s);
      }
    };
    // the first six steps, whole steps to a wave: 0 to 3 share one group of 16
    // poles (wave 0), then 4 (wave 1) and 5 (wave 2)
    if (wv == 0) {
      const Ops o = load(0);
#pragma unroll
      for (int m = 0; m < 4; ++m) {
        zero();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int q = 4 * u + lq;
          const bool in = q >= 1 << m && q < 2 << m;
          if (4 * u < 2 << m && 4 * u + 4 > 1 << m) mac(mk(in ? o.x[u].re : 0.0, in ? o.x[u].im : 0.0), o.b[u]);
        }
        put(m);
      }
    } else if (wv < 3 && 3 + wv < L) {
      zero();
      for (int g = 16 * wv; g < 32 * wv; g += 16) {
        const Ops o = load(g);
#pragma unroll
        for (int u = 0; u < 4; ++u) mac(o.x[u], o.b[u]);
      }
      put(3 + wv);
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < 6; ++m)
      if (m < L) update(m, red[m][er][ec]);
    __syncthreads();
    // the others, a step's poles dealt to the waves
#pragma unroll
    for (int m = 6; m < TLMAX; ++m) {
      if (m < L) {
        zero();
        for (int g = (1 << m) + 16 * wv; g < 2 << m; g += 16 * NW) {
          const Ops o = load(g);
#pragma unroll
          for (int u = 0; u < 4; ++u) mac(o.x[u], o.b[u]);
        }
        const int s0 = NW * (m & 1);  // two sets of slots: one barrier per step
        put(s0 + wv);
        __syncthreads();
        C64 T = mk(0.0, 0.0);
#pragma unroll
        for (int q = 0; q < NW; q += 4)
          if ((1 << m) > 16 * q)  // (waves past the step's poles leave zeros)
            T = T + ((red[s0 + q][er][ec] + red[s0 + q + 1][er][ec]) + (red[s0 + q + 2][er][ec] + red[s0 + q + 3][er][ec]));
        update(m, T);
      }
    }
    if (own) S_b[so] = s;
  }
#pragma unroll
  for (int m = 0; m < TLMAX; ++m) {
    if (m < L && wv < 4) {
      const double d = wave_sum(ds[m]), e = wave_sum(ns[m]);
      if (lane == 0) {
        sred[wv][2 * m] = d;
        sred[wv][2 * m + 1] = e;
      }
    }
  }
  __syncthreads();
  if (threadIdx.x < 2 * L)
    w.sums[((size_t)b * 2 * Lw + threadIdx.x) * w.nsum + blockIdx.x] =
        (sred[0][threadIdx.x] + sred[1][threadIdx.x]) + (sred[2][threadIdx.x] + sred[3][threadIdx.x]);
}

// the sums over the tiles, in a fixed order, into host memory: per matrix 2 L
// sums (one wave each), then 1.0 if the closed form does not cover the matrix
__global__ void __launch_bounds__(64) k_tri_sums(TriWs w, double* host) {
  const int b = blockIdx.y, m = blockIdx.x, n2 = gridDim.x;
  const double* p = w.sums + ((size_t)b * n2 + m) * w.nsum;
  double v = 0.0;
#pragma unroll 4
  for (int k = threadIdx.x; k < w.nsum; k += 64) v += p[k];
  v = wave_sum(v);
  if (threadIdx.x == 0) {
    host[(size_t)b * (n2 + 1) + m] = v;
    if (m == 0) host[(size_t)b * (n2 + 1) + n2] = w.sing[b] ? 1.0 : 0.0;
  }
}

DevBuf g_tri;
HostBuf g_tri_pin;

struct Layout {
  int np, nch, ntask;
  size_t bytes;
};

// workspace of a batch at L steps
Layout tri_layout(int batch, int ld, int maxn, int L) {
  Layout y;
  y.np = std::max(1 << L, 64);
  y.nch = (maxn + TB - 1) / TB;
  y.ntask = y.nch * TPARTS + y.nch * (y.nch - 1);
  const size_t el = (2 * (TB + 2) + 13 * TB) * (size_t)y.nch * batch * y.np + (size_t)batch * y.nch * (2 + y.nch) * y.np;
  y.bytes = el * sizeof(C64) +
            (2 * (size_t)batch * y.np + (size_t)batch * L + (size_t)batch * 2 * L * y.ntask) * sizeof(double) + 256;
  return y;
}

// the workspace of that layout, in g_tri
TriWs tri_ws(const Layout& y, int batch, int ld, int L, int* sing) {
  TriWs w{};
  w.ld = ld;
  w.np = y.np;
  w.nch = y.nch;
  w.nsum = y.ntask;
  C64* p = g_tri.as<C64>();
  auto take = [&](size_t n) {
    C64* r = p;
    p += n;
    return r;
  };
  for (C64** f : {&w.N, &w.M}) *f = take((size_t)batch * y.nch * (TB + 2) * y.np);
  for (C64** f : {&w.au, &w.ad, &w.bu, &w.bd, &w.gg, &w.fu[0], &w.fu[1], &w.fu[2], &w.fu[3], &w.fd[0], &w.fd[1],
                  &w.fd[2], &w.fd[3]})
    *f = take((size_t)batch * y.nch * TB * y.np);
  w.rt = take((size_t)batch * y.nch * 2 * y.np);
  w.rr = take((size_t)batch * y.nch * y.nch * y.np);
  w.rho = reinterpret_cast<double*>(p);
  w.kap = w.rho + (size_t)batch * y.np;
  w.mu = w.kap + (size_t)batch * y.np;
  w.sums = w.mu + (size_t)batch * L;
  w.sing = sing;
  return w;
}

// S_0 -> S_1 .. of every tile.  At most one workgroup per CU: sixteen waves for
// a tile, a step's poles in a quarter of the turns.  More workgroups fill the
// chip themselves, three of four waves to a CU.  Sixteen waves against four:
// n = 60 (48 workgroups) 27 and 38 us, n = 190 (240) 21 and 26, n = 230 (345)
// 34 and 28, n = 500 (1280) 94 and 54.
void tri_tiles(const TriWs& w, int batch, const int* nvec, int L, const int* steps, C64* S, hipStream_t st) {
  if (w.nsum * batch <= 256)
    hipLaunchKernelGGL(k_tri_tile<16>, dim3(w.nsum, 1, batch), dim3(1024), 0, st, w, nvec, L, steps, S);
  else
    hipLaunchKernelGGL(k_tri_tile<4>, dim3(w.nsum, 1, batch), dim3(256), 0, st, w, nvec, L, steps, S);
}

}  // namespace

// The steps to take in closed form: ten for orders up to 128 and nine above
// (a spectrum between 0.3 and 6.5 in modulus converges in eight or nine; each
// further step doubles the poles), nine when scaled (one workgroup's 512
// threads), never more than the cap; fewer when the workspace would pass
// 512 MB.  Fewer than five are not worth the detour: 0, and the caller
// iterates with explicit inverses from the start; so it does for a cap below
// one, under which no step is taken.
int tri_rh_steps(int batch, int ld, int maxn, int scaling, int maxit) {
  if (maxn < 1 || maxit < 1) return 0;
  int L = scaling == NK_RH_NONE && maxn <= 128 ? TLMAX : 9;
  L = std::min(L, maxit);
  while (L > 0 && tri_layout(batch, ld, maxn, L).bytes > (size_t)512 << 20) --L;
  return L >= std::min(5, maxit) ? L : 0;
}

int tri_rh_run(int batch, int ld, int maxn, const int* nvec, int* sing, const TriIn& h, C64* S, int scaling,
               const double* sched, int nsched, int L, const double** sums, hipStream_t st) {
  const Layout y = tri_layout(batch, ld, maxn, L);
  if (g_tri.ensure(y.bytes) || g_tri_pin.ensure((size_t)batch * (2 * L + 1) * sizeof(double))) return 1;
  const TriWs w = tri_ws(y, batch, ld, L, sing);
  const int pb = y.np / 64;
  if (scaling == NK_RH_NONE)
    hipLaunchKernelGGL(k_tri_chain, dim3(pb, 2, batch), dim3(64), 0, st, w, h, nvec, L);
  else
    hipLaunchKernelGGL(k_tri_chain_mu, dim3(1, 1, batch), dim3(512), 0, st, w, h, nvec, L, sched, nsched);
  hipLaunchKernelGGL(k_tri_mid, dim3(pb, 2 * y.nch, batch), dim3(64), 0, st, w, h, nvec);
  if (y.nch > 1) hipLaunchKernelGGL(k_tri_between, dim3(pb, 2 * y.nch, batch), dim3(64), 0, st, w, nvec);
  tri_tiles(w, batch, nvec, L, nullptr, S, st);
  hipLaunchKernelGGL(k_tri_sums, dim3(2 * L, batch), dim3(64), 0, st, w, g_tri_pin.dev<double>());
  NK_HIP(hipGetLastError());
  *sums = g_tri_pin.host<double>();
  return NK_OK;
}

__global__ void __launch_bounds__(256) k_tri_restart(int ld, const int* __restrict__ nvec,
                                                     const int* __restrict__ redo, TriIn h, C64* __restrict__ S_b) {
  const int b = blockIdx.y, n = nvec[b];
  if (!redo[b]) return;
  C64* S = S_b + (size_t)b * ld * ld;
  const size_t nn = (size_t)max(n, 0) * n;
  for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < nn; e += (size_t)gridDim.x * 256) {
    const int i = (int)(e / n), j = (int)(e % n);
    C64 v = mk(0.0, 0.0);
    if (i == j) v = h.a[b * h.stride + i];
    if (j == i + 1) v = h.b[b * h.stride + i];
    if (i == j + 1) v = h.d[b * h.stride + j];
    S[(size_t)i * ld + j] = v;
  }
}

int tri_rh_retake(int batch, int ld, int maxn, const int* nvec, const int* steps, const TriIn& h, C64* S, int L,
                  hipStream_t st) {
  hipLaunchKernelGGL(k_tri_restart, dim3(64, batch), dim3(256), 0, st, ld, nvec, steps, h, S);
  tri_tiles(tri_ws(tri_layout(batch, ld, maxn, L), batch, ld, L, nullptr), batch, nvec, L, steps, S, st);
  NK_HIP(hipGetLastError());
  return NK_OK;
}

}  // namespace nk
