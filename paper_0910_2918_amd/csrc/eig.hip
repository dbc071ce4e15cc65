// The critical eigenpairs that deflation treats exactly (Sec. 2), for the
// Hermitian case mu = 0: the m eigenvalues of H = gamma5 Dw(0) smallest in
// modulus, with orthonormal eigenvectors (left = right).  The paper takes them
// from earlier work; the method here is Chebyshev-filtered subspace iteration
// on H^2, which is positive semi-definite, so the wanted eigenvalues are its
// smallest and the filter damps the interval above them:
//   * a block of p >= m vectors is filtered by the degree-d Chebyshev
//     polynomial of H^2 mapped so that [a2, b2] goes to [-1, 1], where b2
//     bounds the spectrum of H^2 ((|4 + m_w| + 8)^2) and a2 is the largest
//     Ritz value of H^2 in the current block;
//   * the block is orthonormalised by Cholesky QR, twice;
//   * Rayleigh-Ritz with H^2 (no spurious interior Ritz values, unlike with
//     the indefinite H over the whole block) rotates it to Ritz vectors;
//     then Rayleigh-Ritz with H on the leading q >= m of them (q grows past
//     m while their H^2 values repeat) splits the pairs lambda, -lambda that
//     H^2 cannot tell apart (the free field's spectrum is exactly symmetric);
//     the eigenvalue of H of each vector is its Rayleigh quotient;
//   * it stops when the m leading residuals |H r - lambda r| are below
//     tol * sqrt(b2).
// Vector work runs in kernels on whole blocks: the stencil with the Chebyshev
// step in its epilogue (k_apply_block), Gram matrices (k_gram) and block
// rotations (k_rotate) on the FP64 matrix cores, residual norms (k_cols).
// The p x p Cholesky and Jacobi steps run on the host; their matrices pass
// through pinned memory.  The iteration works in the library's packed device
// layout: every step but the stencil is an inner product or a linear
// combination, which a fixed reordering of the entries leaves unchanged, so
// the start block is packed once and the result unpacked once.
#include <algorithm>
#include <cmath>
#include <utility>
#include <vector>

#include "nk_internal.h"
#include "small_dense.h"

namespace nk {

namespace {

typedef double nk_d4 __attribute__((ext_vector_type(4)));

using dense::cd;

// MFMA operand layout (16 x 16 x 4, FP64): lane l holds A[l % 16][l / 16] and
// B[l / 16][l % 16], and accumulator element i of lane l is
// D[4 i + l / 16][l % 16].

// Partial Gram matrices: for each pair (blockIdx.z) of blocks a, b of q
// vectors, part[((pair nch + c) q + j) q + i] = a_i^dag b_j over the entries of
// chunk c = blockIdx.y.  Four waves of one 16 x 16 tile each make a 32 x 32
// tile of the result (blockIdx.x); a lane reads runs of four entries (64 bytes)
// of its vector, dealt to the four products that they enter, so the loads need
// no LDS.  Bound by the loads of the two blocks and the products (on 8^4, 24
// vectors: 33 us for two or three pairs); column by column, as before, the
// block was read q / 2 times over, in 24 launches and 24 reductions of 4 us a
// matrix.
struct GramPairs {
  const C64* a[3];
  const C64* b[3];
};
__global__ void __launch_bounds__(256) k_gram(GramPairs ab, int q, size_t n, int ch, C64* __restrict__ part) {
  const int pair = blockIdx.z, c = blockIdx.y, nch = gridDim.y;
  const int tq = (q + 31) / 32;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int l16 = lane & 15, lq = lane >> 4;
  const int i0 = (blockIdx.x % tq) * 32 + (w & 1) * 16, j0 = (blockIdx.x / tq) * 32 + (w >> 1) * 16;
  if (i0 >= q || j0 >= q) return;
  const C64* a = pair == 0 ? ab.a[0] : pair == 1 ? ab.a[1] : ab.a[2];
  const C64* b = pair == 0 ? ab.b[0] : pair == 1 ? ab.b[1] : ab.b[2];
  a += (size_t)min(i0 + l16, q - 1) * n;  // vectors past the block repeat its last; their results are not stored
  b += (size_t)min(j0 + l16, q - 1) * n;
  const size_t e0 = (size_t)c * ch, e1 = min(n, e0 + ch);
  nk_d4 re = {0.0, 0.0, 0.0, 0.0}, im = {0.0, 0.0, 0.0, 0.0};
  for (size_t e = e0; e < e1; e += 16) {
    C64 av[4], bv[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const size_t x = e + 4 * lq + s;
      const bool in = x < e1;
      av[s] = a[in ? x : e0];
      bv[s] = b[in ? x : e0];
      if (!in) av[s] = bv[s] = mk(0.0, 0.0);
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s].re, bv[s].re, re, 0, 0, 0);
      re = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s].im, bv[s].im, re, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(av[s].re, bv[s].im, im, 0, 0, 0);
      im = __builtin_amdgcn_mfma_f64_16x16x4f64(-av[s].im, bv[s].re, im, 0, 0, 0);
    }
  }
  C64* out = part + (size_t)(pair * nch + c) * q * q;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = i0 + 4 * r + lq, j = j0 + l16;
    if (i < q && j < q) out[(size_t)j * q + i] = mk(re[r], im[r]);
  }
}

// out[pair qq + o] = sum over the chunks of part[(pair nch + c) qq + o], in a
// fixed order; 64 results per workgroup, four threads each; out is host memory
__global__ void __launch_bounds__(256) k_gram_sum(int nch, int qq, const C64* __restrict__ part, C64* out) {
  __shared__ C64 sh[4][64];
  const int t = threadIdx.x & 63, seg = threadIdx.x >> 6;
  const int o = blockIdx.x * 64 + t;
  const C64* p = part + (size_t)blockIdx.y * nch * qq + (o < qq ? o : 0);
  C64 acc = mk(0.0, 0.0);
#pragma unroll 8
  for (int c = seg; c < nch; c += 4) acc = acc + p[(size_t)c * qq];
  sh[seg][t] = acc;
  __syncthreads();
  if (seg == 0 && o < qq) out[(size_t)blockIdx.y * qq + o] = (sh[0][t] + sh[1][t]) + (sh[2][t] + sh[3][t]);
}

// In-place rotation of blocks of p vectors, y_j <- sum_i y_i m[i + j p] (block
// blockIdx.y with its own matrix): a wave loads its 16 NE entries of all p
// vectors (PT = ceil(p / 16) groups of 16), so that it may overwrite them, and
// forms 16 new vectors at a time on the matrix cores, the matrix read from L2.
// Each block is read and written once (two or four blocks of 24 vectors on
// 8^4: 33 us); as one combination per new vector, before, it was read p times,
// in 24 launches of 4 us a block.
struct RotBlocks {
  C64* y[4];
  const C64* m[4];
};
template <int PT, int NE>
__global__ void __launch_bounds__(256) k_rotate(RotBlocks rb, int p, size_t n) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int l16 = lane & 15, lq = lane >> 4;
  C64* y = blockIdx.y == 0 ? rb.y[0] : blockIdx.y == 1 ? rb.y[1] : blockIdx.y == 2 ? rb.y[2] : rb.y[3];
  const C64* m = blockIdx.y == 0 ? rb.m[0] : blockIdx.y == 1 ? rb.m[1] : blockIdx.y == 2 ? rb.m[2] : rb.m[3];
  const size_t e0 = ((size_t)blockIdx.x * 4 + w) * 16 * NE;
  if (e0 >= n) return;
  C64 yv[4 * PT][NE];
#pragma unroll
  for (int kk = 0; kk < 4 * PT; ++kk)
#pragma unroll
    for (int h = 0; h < NE; ++h) {
      const int k = 4 * kk + lq;
      const size_t e = e0 + 16 * h + l16;
      const bool in = k < p && e < n;
      yv[kk][h] = y[in ? (size_t)k * n + e : e0];
      if (!in) yv[kk][h] = mk(0.0, 0.0);
    }
#pragma unroll 1
  for (int jt = 0; jt < PT; ++jt) {
    const int j = 16 * jt + l16;
    nk_d4 re[NE], im[NE];
#pragma unroll
    for (int h = 0; h < NE; ++h) {
      re[h] = nk_d4{0.0, 0.0, 0.0, 0.0};
      im[h] = nk_d4{0.0, 0.0, 0.0, 0.0};
    }
#pragma unroll
    for (int kk = 0; kk < 4 * PT; ++kk) {
      const int k = 4 * kk + lq;
      const bool in = j < p && k < p;
      C64 c = m[in ? k + (size_t)j * p : 0];
      if (!in) c = mk(0.0, 0.0);
#pragma unroll
      for (int h = 0; h < NE; ++h) {
        re[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(c.re, yv[kk][h].re, re[h], 0, 0, 0);
        re[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(-c.im, yv[kk][h].im, re[h], 0, 0, 0);
        im[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(c.re, yv[kk][h].im, im[h], 0, 0, 0);
        im[h] = __builtin_amdgcn_mfma_f64_16x16x4f64(c.im, yv[kk][h].re, im[h], 0, 0, 0);
      }
    }
#pragma unroll
    for (int h = 0; h < NE; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int jo = 16 * jt + 4 * i + lq;
        const size_t e = e0 + 16 * h + l16;
        if (jo < p && e < n) y[(size_t)jo * n + e] = mk(re[h][i], im[h][i]);
      }
  }
}

// Per-column partial sums over chunks of RCH entries (blockIdx.x), column
// blockIdx.y, side blockIdx.z:
//   MODE 0: a_i^dag b_i
//   MODE 1: |b_i - th_i a_i|^2 (re) and |a_i|^2 (im), th conjugated on side 1
constexpr int RT = 256, RE = 8, RCH = RT * RE;
struct ColArgs {
  const C64* a[2];
  const C64* b[2];
  const C64* th;
};
template <int MODE>
__global__ void __launch_bounds__(RT) k_cols(ColArgs ca, size_t n, C64* __restrict__ part) {
  __shared__ C64 sh[RT / 64];
  const int side = blockIdx.z;
  const size_t col = (size_t)blockIdx.y * n;
  const C64* a = (side ? ca.a[1] : ca.a[0]) + col;
  const C64* b = (side ? ca.b[1] : ca.b[0]) + col;
  C64 th = mk(0.0, 0.0);
  if (MODE == 1) {
    th = ca.th[blockIdx.y];
    if (side) th = conj(th);
  }
  C64 acc = mk(0.0, 0.0);
#pragma unroll
  for (int u = 0; u < RE; ++u) {
    const size_t e = (size_t)blockIdx.x * RCH + u * RT + threadIdx.x;
    if (e < n) {
      const C64 x = a[e], z = b[e];
      if (MODE == 0)
        acc = acc + cmulc(x, z);
      else
        acc = acc + mk(norm2(z - cmul(th, x)), norm2(x));
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    acc.re += __shfl_xor(acc.re, o, 64);
    acc.im += __shfl_xor(acc.im, o, 64);
  }
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0)
    part[((size_t)side * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x] = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

// c[i] = sum_b part[i nb + b] in a fixed order, one wave per column; c2, if
// given, receives the real part alone (the quotient of a Hermitian operator)
__global__ void __launch_bounds__(64) k_cols_sum(const C64* __restrict__ part, int nb, C64* c, C64* c2) {
  const C64* p = part + (size_t)blockIdx.x * nb;
  C64 acc = mk(0.0, 0.0);
  for (int b = threadIdx.x; b < nb; b += 64) acc = acc + p[b];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    acc.re += __shfl_xor(acc.re, o, 64);
    acc.im += __shfl_xor(acc.im, o, 64);
  }
  if (threadIdx.x == 0) {
    c[blockIdx.x] = acc;
    if (c2) c2[blockIdx.x] = mk(acc.re, 0.0);
  }
}

// column i of y scaled by f[i] (real), in place
__global__ void __launch_bounds__(RT) k_scale_cols(C64* __restrict__ y, const C64* __restrict__ f, size_t n) {
  const size_t e = (size_t)blockIdx.x * RT + threadIdx.x;
  if (e >= n) return;
  C64* c = y + (size_t)blockIdx.y * n;
  c[e] = f[blockIdx.y].re * c[e];
}

// device and pinned workspace of one solve: p x p matrices and partial sums
struct EigWork {
  size_t n;
  int p, nch, ch, nbc;
  C64* part;   // partial sums
  C64* dm;     // two p x p coefficient matrices, then 2 p per-column scalars
  C64* up;     // their pinned staging (host address)
  C64 *hg, *hg_dev;  // pinned results: three p x p matrices, 2 p per-column sums
  hipStream_t st;
  size_t pp() const { return (size_t)p * p; }
};

// chunks of a Gram matrix: enough workgroups to fill the device, the partial
// matrices bounded by 16 MB a pair
int gram_chunks(size_t n, int p) {
  const size_t most = std::max<size_t>(8, std::min<size_t>(256, (size_t)(1 << 20) / ((size_t)p * p)));
  return (int)std::max<size_t>(1, std::min<size_t>(most, (n + 255) / 256));
}

// elements of workspace beside the blocks of vectors
size_t eig_small(size_t n, int p) {
  const size_t parts = std::max((size_t)3 * gram_chunks(n, p) * p * p, (size_t)2 * p * ((n + RCH - 1) / RCH));
  return parts + 2 * (size_t)p * p + 2 * (size_t)p;
}

int eig_work(nk_lattice* lat, int p, C64* small, hipStream_t st, EigWork* w) {
  w->n = (size_t)12 * lat->g.V;
  w->p = p;
  w->nch = gram_chunks(w->n, p);
  const size_t per = (w->n + w->nch - 1) / w->nch;
  w->ch = (int)((per + 15) & ~(size_t)15);
  w->nch = (int)((w->n + w->ch - 1) / w->ch);
  w->nbc = (int)((w->n + RCH - 1) / RCH);
  w->dm = small;
  w->part = small + 2 * (size_t)p * p + 2 * (size_t)p;
  w->st = st;
  const size_t nup = 2 * w->pp() + 2 * (size_t)p, ng = 3 * w->pp() + 2 * (size_t)p;
  if (lat->eig_pin.ensure((nup + ng) * sizeof(C64))) return NK_ENOMEM;
  w->up = lat->eig_pin.host<C64>();
  w->hg = w->up + nup;
  w->hg_dev = lat->eig_pin.dev<C64>() + nup;
  return NK_OK;
}

// h[s][i + j p] = a_i^dag b_j for np pairs of blocks; waits for the stream
int grams(const EigWork& w, const GramPairs& ab, int np, std::vector<cd>* h) {
  const int p = w.p, tq = (p + 31) / 32;
  hipLaunchKernelGGL(k_gram, dim3(tq * tq, w.nch, np), dim3(256), 0, w.st, ab, p, w.n, w.ch, w.part);
  hipLaunchKernelGGL(k_gram_sum, dim3((p * p + 63) / 64, np), dim3(256), 0, w.st, w.nch, p * p,
                     (const C64*)w.part, w.hg_dev);
  NK_HIP(hipGetLastError());
  NK_HIP(hipStreamSynchronize(w.st));
  for (int s = 0; s < np; ++s) {
    h[s].resize(w.pp());
    for (size_t i = 0; i < w.pp(); ++i) h[s][i] = cd(w.hg[s * w.pp() + i].re, w.hg[s * w.pp() + i].im);
  }
  return NK_OK;
}

// the upper triangle of a Gram matrix mirrored into an exactly Hermitian one
void mirror(std::vector<cd>& h, int p) {
  for (int j = 0; j < p; ++j)
    for (int i = 0; i <= j; ++i) {
      const cd v = h[i + (size_t)j * p];
      h[i + (size_t)j * p] = i == j ? cd(v.real(), 0.0) : v;
      h[j + (size_t)i * p] = i == j ? cd(v.real(), 0.0) : std::conj(v);
    }
}

// a matrix (or scalars) into slot `at` of the device's coefficient array.
// The staging area is rewritten only after a synchronisation that followed
// its last upload: every caller's uploads alternate with grams() or a wait.
int upload(const EigWork& w, size_t at, const cd* v, size_t count) {
  for (size_t i = 0; i < count; ++i) w.up[at + i] = mk(v[i].real(), v[i].imag());
  NK_HIP(hipMemcpyAsync(w.dm + at, w.up + at, count * sizeof(C64), hipMemcpyHostToDevice, w.st));
  return NK_OK;
}

// blocks y[0 .. nblk) rotated in place, block i by matrix which[i] (0 or 1) of m
int rotate_blocks(const EigWork& w, int nblk, C64* const* y, const int* which, const std::vector<cd>* m, int nm) {
  for (int k = 0; k < nm; ++k)
    if (int e = upload(w, k * w.pp(), m[k].data(), w.pp())) return e;
  RotBlocks rb{};
  for (int i = 0; i < nblk; ++i) {
    rb.y[i] = y[i];
    rb.m[i] = w.dm + which[i] * w.pp();
  }
#define NK_ROT(PT_, NE_)                                                                                       \
  hipLaunchKernelGGL((k_rotate<PT_, NE_>), dim3((unsigned)((w.n + 64 * NE_ - 1) / (64 * NE_)), nblk), dim3(256), 0, \
                     w.st, rb, w.p, w.n);                                                                      \
  break
  switch ((w.p + 15) / 16) {
    case 1: NK_ROT(1, 4);
    case 2: NK_ROT(2, 4);
    case 3: NK_ROT(3, 2);
    case 4: NK_ROT(4, 2);
    case 5: NK_ROT(5, 1);
    case 6: NK_ROT(6, 1);
    case 7: NK_ROT(7, 1);
    default: NK_ROT(8, 1);
  }
#undef NK_ROT
  NK_HIP(hipGetLastError());
  return NK_OK;
}

// y_s <- y_s C_s^{-1} with y_s^dag y_s = C_s^dag C_s, twice, for ns blocks
int orthonormalise(const EigWork& w, int ns, C64* const* y) {
  const int which[2] = {0, 1};
  for (int pass = 0; pass < 2; ++pass) {
    GramPairs ab{};
    for (int s = 0; s < ns; ++s) ab.a[s] = ab.b[s] = y[s];
    std::vector<cd> g[2];
    if (int e = grams(w, ab, ns, g)) return e;
    for (int s = 0; s < ns; ++s) {
      mirror(g[s], w.p);
      if (!dense::chol_inv_upper(g[s], w.p)) {
        set_error("eigensolver: the block lost rank (Gram matrix not positive definite)");
        return NK_EINVAL;
      }
    }
    if (int e = rotate_blocks(w, ns, y, which, g, ns)) return e;
  }
  return NK_OK;
}

// The degree-d Chebyshev filter in A(mu_s)^2, mapped so that [a2, b2] goes to
// [-1, 1], of ns blocks at once: x[s] ends up holding the result and y[s] the
// other buffer of its pair; t[s] is scratch.  Two launches per degree.
int cheb_filter(nk_lattice* lat, double m_w, int ns, const double* mu, C64** x, C64** y, C64* const* t, int p,
                int degree, double a2, double b2, hipStream_t st) {
  const double c = 0.5 * (a2 + b2), e = 0.5 * (b2 - a2);
  ApplyBlock ab{};
  ab.p = p;
  for (int s = 0; s < ns; ++s) {
    ab.ef[s] = std::exp(mu[s]);
    ab.eb[s] = std::exp(-mu[s]);
  }
  C64 *prev[2] = {nullptr, nullptr}, *cur[2] = {nullptr, nullptr};
  for (int j = 1; j <= degree; ++j) {
    for (int s = 0; s < ns; ++s) {
      if (j == 1) {
        prev[s] = x[s];
        cur[s] = y[s];
      }
      ab.x[s] = j == 1 ? x[s] : cur[s];
      ab.out[s] = t[s];
    }
    if (int er = apply_block_dev(lat, m_w, ab, ns, false, st)) return er;
    // Y_1 = (A^2 X - c X) / e, then Y_{j+1} = 2 (A^2 Y_j - c Y_j) / e - Y_{j-1} written over Y_{j-1}
    for (int s = 0; s < ns; ++s) {
      ab.y[s] = ab.x[s];
      ab.x[s] = t[s];
      ab.out[s] = j == 1 ? cur[s] : prev[s];
    }
    const double f = j == 1 ? 1.0 : 2.0;
    ab.ca = f / e;
    ab.cb = -f * c / e;
    ab.cc = j == 1 ? 0.0 : -1.0;
    if (int er = apply_block_dev(lat, m_w, ab, ns, true, st)) return er;
    if (j > 1)
      for (int s = 0; s < ns; ++s) std::swap(prev[s], cur[s]);
  }
  for (int s = 0; s < ns; ++s) {
    C64* other = cur[s] == x[s] ? y[s] : x[s];
    x[s] = cur[s];
    y[s] = other;
  }
  return NK_OK;
}

// out[s] = A(mu_s) x[s] for ns blocks
int apply_blocks_of(nk_lattice* lat, double m_w, int ns, const double* mu, C64* const* x, C64* const* out, int p,
                    hipStream_t st) {
  ApplyBlock ab{};
  ab.p = p;
  for (int s = 0; s < ns; ++s) {
    ab.x[s] = x[s];
    ab.out[s] = out[s];
    ab.ef[s] = std::exp(mu[s]);
    ab.eb[s] = std::exp(-mu[s]);
  }
  return apply_block_dev(lat, m_w, ab, ns, false, st);
}

// c = a b for column-major p x p matrices
std::vector<cd> matmul(const std::vector<cd>& a, const std::vector<cd>& b, int p) {
  std::vector<cd> c((size_t)p * p, cd(0.0, 0.0));
  for (int j = 0; j < p; ++j)
    for (int k = 0; k < p; ++k) {
      const cd v = b[k + (size_t)j * p];
      for (int i = 0; i < p; ++i) c[i + (size_t)j * p] += a[i + (size_t)k * p] * v;
    }
  return c;
}

// the leading q x q block of z^dag k y
std::vector<cd> projected(const std::vector<cd>& z, const std::vector<cd>& k, const std::vector<cd>& y, int p, int q) {
  const std::vector<cd> ky = matmul(k, y, p);
  std::vector<cd> c((size_t)q * q, cd(0.0, 0.0));
  for (int j = 0; j < q; ++j)
    for (int i = 0; i < q; ++i)
      for (int l = 0; l < p; ++l) c[i + (size_t)j * q] += std::conj(z[l + (size_t)i * p]) * ky[l + (size_t)j * p];
  return c;
}

}  // namespace

// The critical eigenpairs of A = gamma5 Dw(mu) for any mu (Sec. 2, the
// deflation paragraph): the m eigenvalues nearest the imaginary axis, with
// right vectors R (A R = R Lambda) and left vectors L (L^dag A = Lambda
// L^dag), L^dag R = I.  Two-sided filtered subspace iteration:
//   * a right block V and a left block W of p vectors are filtered by the
//     degree-d Chebyshev polynomial in A^2 (V) and in (A^dag)^2 = A(-mu)^2
//     (W), mapped so that [a2, b2] goes to [-1, 1]: b2 bounds |lambda|^2
//     ((|4 + m_w| + 6 + 2 cosh mu)^2: the mass term plus the six spatial and
//     two temporal hops), a2 is the largest Re sigma of the current Ritz
//     values of A^2 (below).  The eigenvalues of A near the imaginary axis have the
//     smallest Re lambda^2 (often below zero), outside that interval, so
//     the filter amplifies them, as long as the spectrum keeps small
//     imaginary parts where |Re lambda| is large (mu of order 0.1-1 on
//     these lattices: |Im lambda| < 0.14 against |Re lambda| up to 6);
//   * both blocks are orthonormalised (Cholesky QR, twice);
//   * two-sided Rayleigh-Ritz in two steps.  First with A^2: with
//     G = W^dag V and K2 = (A^dag W)^dag (A V) = W^dag A^2 V, the p x p
//     eigenproblem of G^{-1} K2 gives values sigma, right coefficients Y and
//     left ones U with U^dag Y = I, so the block rotated to V Y and
//     W G^{-dag} U is biorthonormal, sorted by Re sigma.  Then with A itself
//     on the leading q >= m of these vectors (q grows past m while sigma
//     repeats): the eigenvalues theta of their q x q W^dag A V, which split
//     pairs lambda, -lambda that A^2 cannot tell apart.  Rayleigh-Ritz with
//     A on the whole block would not do: A is indefinite, and a mixture of
//     eigenvectors of large positive and negative eigenvalue has a Rayleigh
//     quotient near zero, a spurious critical value with a large residual
//     (at mu = 0 the iteration then never converges);
//   * the leading q vectors are sorted by |Re theta|, and the iteration
//     stops when the m leading residuals |A r - theta r| / |r| and
//     |A^dag l - conj(theta) l| / |l| are below tol * sqrt(b2).
// Vector work runs in kernels; the p x p steps (LU inverse, Hessenberg QR
// eigen-decomposition) run on the host.
int eig_critical(nk_lattice* lat, double m_w, double mu, int m, int p, int degree, double tol, int maxit,
                 const C64* v0, double* lam, C64* r_out, C64* l_out, int* passes, double* resid, hipStream_t st) {
  const size_t n = (size_t)12 * lat->g.V;
  const size_t blk = (size_t)p * n;
  if (lat->eig.ensure((6 * blk + eig_small(n, p)) * sizeof(C64))) return NK_ENOMEM;
  C64* base = lat->eig.as<C64>();
  // right and left side: the block, the filter's second buffer and A times it
  C64* X[2] = {base, base + blk};
  C64* Y[2] = {base + 2 * blk, base + 3 * blk};
  C64* AX[2] = {base + 4 * blk, base + 5 * blk};
  EigWork w;
  if (int e = eig_work(lat, p, base + 6 * blk, st, &w)) return e;
  const double mus[2] = {mu, -mu};
  const double hb = std::fabs(4.0 + m_w) + 6.0 + 2.0 * std::cosh(mu), b2 = hb * hb;
  std::vector<cd> th(p), sg(p);
  std::vector<double> rv(p), rw(p), vn(p);
  // the q x q eigenproblem of Gi K (Gi = I when null): values, right and left
  // coefficient matrices (the left ones already mapped by Gi^dag)
  auto small_eig = [&](const std::vector<cd>& K, const std::vector<cd>* Gi, int q, std::vector<cd>& val,
                       std::vector<cd>& yr, std::vector<cd>& zl) -> int {
    std::vector<cd> ul;
    if (!dense::eig_general(Gi ? matmul(*Gi, K, q) : K, q, val, yr, ul)) {
      set_error("eigensolver: the projected %d x %d eigenproblem did not converge", q, q);
      return NK_EINVAL;
    }
    if (!Gi) {
      zl = ul;
      return NK_OK;
    }
    zl.assign((size_t)q * q, cd(0.0, 0.0));
    for (int j = 0; j < q; ++j)
      for (int k = 0; k < q; ++k) {
        const cd u = ul[k + (size_t)j * q];
        for (int i = 0; i < q; ++i) zl[i + (size_t)j * q] += std::conj((*Gi)[k + (size_t)i * q]) * u;
      }
    return NK_OK;
  };
  // the columns of yr and zl reordered as idx lists them, into p x p
  // coefficient matrices that leave the columns past q unchanged
  auto reorder = [&](const std::vector<cd>& yr, const std::vector<cd>& zl, int q, const std::vector<int>& idx,
                     std::vector<cd>& Ys, std::vector<cd>& Zs) {
    Ys.assign((size_t)p * p, cd(0.0, 0.0));
    Zs.assign((size_t)p * p, cd(0.0, 0.0));
    for (int j = 0; j < p; ++j) {
      if (j < q) {
        for (int i = 0; i < q; ++i) {
          Ys[i + (size_t)j * p] = yr[i + (size_t)idx[j] * q];
          Zs[i + (size_t)j * p] = zl[i + (size_t)idx[j] * q];
        }
      } else {
        Ys[j + (size_t)j * p] = 1.0;
        Zs[j + (size_t)j * p] = 1.0;
      }
    }
  };
  // the two Rayleigh-Ritz steps on orthonormal X[0] = V and X[1] = W; leaves
  // them rotated (W^dag V = I), sg the Ritz values of A^2, th those of A on
  // the leading q, rv and rw the relative residuals and vn the squared norms
  // of the right Ritz vectors.  The second step's matrix W^dag A V is formed
  // from the first step's products, so both rotations go to the vectors as one.
  auto rayleigh_ritz = [&]() -> int {
    if (int e = apply_blocks_of(lat, m_w, 2, mus, X, AX, p, st)) return e;
    const GramPairs ab{{X[1], AX[1], X[1]}, {X[0], AX[0], AX[0]}};
    std::vector<cd> g[3], Gi, val, yr, zl, Ys, Zs, Yq, Zq;
    if (int e = grams(w, ab, 3, g)) return e;  // W^dag V, (A^dag W)^dag (A V), W^dag A V
    if (!dense::lu_inverse(g[0], p, Gi)) {
      set_error("eigensolver: the left and right blocks became orthogonal (W^dag V singular)");
      return NK_EINVAL;
    }
    if (int e = small_eig(g[1], &Gi, p, val, yr, zl)) return e;
    std::vector<int> idx(p);
    for (int i = 0; i < p; ++i) idx[i] = i;
    std::stable_sort(idx.begin(), idx.end(), [&](int x, int y) { return val[x].real() < val[y].real(); });
    for (int j = 0; j < p; ++j) sg[j] = val[idx[j]];
    reorder(yr, zl, p, idx, Ys, Zs);
    int q = m;
    while (q < p && std::fabs(sg[q].real() - sg[q - 1].real()) <= 1e-8 * std::fabs(sg[q].real())) ++q;
    if (int e = small_eig(projected(Zs, g[2], Ys, p, q), nullptr, q, val, yr, zl)) return e;
    idx.resize(q);
    for (int i = 0; i < q; ++i) idx[i] = i;
    std::stable_sort(idx.begin(), idx.end(),
                     [&](int x, int y) { return std::fabs(val[x].real()) < std::fabs(val[y].real()); });
    for (int j = 0; j < q; ++j) th[j] = val[idx[j]];
    for (int j = q; j < p; ++j) th[j] = std::sqrt(sg[j]);  // only for completeness: past q, A^2 values
    reorder(yr, zl, q, idx, Yq, Zq);
    const std::vector<cd> rot[2] = {matmul(Ys, Yq, p), matmul(Zs, Zq, p)};
    C64* const blocks[4] = {X[0], AX[0], X[1], AX[1]};
    const int which[4] = {0, 0, 1, 1};
    if (int e = rotate_blocks(w, 4, blocks, which, rot, 2)) return e;
    // squared norms of the residuals A r - theta r and A^dag l - conj(theta) l and of the vectors, leading m
    if (int e = upload(w, 2 * w.pp(), th.data(), m)) return e;
    const ColArgs ca{{X[0], X[1]}, {AX[0], AX[1]}, w.dm + 2 * w.pp()};
    hipLaunchKernelGGL(k_cols<1>, dim3(w.nbc, m, 2), dim3(RT), 0, st, ca, n, w.part);
    hipLaunchKernelGGL(k_cols_sum, dim3(2 * m), dim3(64), 0, st, (const C64*)w.part, w.nbc, w.hg_dev, (C64*)nullptr);
    NK_HIP(hipGetLastError());
    NK_HIP(hipStreamSynchronize(st));
    for (int i = 0; i < m; ++i) {
      vn[i] = std::max(w.hg[i].im, 0.0);
      rv[i] = std::sqrt(w.hg[i].re / std::max(vn[i], 1e-300));
      rw[i] = std::sqrt(w.hg[m + i].re / std::max(w.hg[m + i].im, 1e-300));
    }
    return NK_OK;
  };

  if (int e = nk_spinor_pack_device(lat, v0, X[0], p, st)) return e;
  NK_HIP(hipMemcpyAsync(X[1], X[0], blk * sizeof(C64), hipMemcpyDeviceToDevice, st));
  if (int e = orthonormalise(w, 2, X)) return e;
  if (int e = rayleigh_ritz()) return e;
  auto worst_of = [&]() {
    double x = 0.0;
    for (int i = 0; i < m; ++i) x = std::max(x, std::max(rv[i], rw[i]));
    return x;
  };
  int it = 0;
  double worst = worst_of();
  while (it < maxit && worst > tol * hb) {
    ++it;
    double a2 = 0.0;
    for (int i = 0; i < p; ++i) a2 = std::max(a2, sg[i].real());
    if (!(a2 < b2)) a2 = 0.5 * b2;
    if (int er = cheb_filter(lat, m_w, 2, mus, X, Y, AX, p, degree, a2, b2, st)) return er;
    if (int er = orthonormalise(w, 2, X)) return er;
    if (int er = rayleigh_ritz()) return er;
    worst = worst_of();
  }
  // unit right vectors, the left ones scaled to keep l_i^dag r_i = 1
  std::vector<cd> sc(2 * (size_t)m);
  for (int i = 0; i < m; ++i) {
    const double c = std::sqrt(vn[i]);
    sc[i] = 1.0 / c;
    sc[m + i] = c;
  }
  if (int e = upload(w, 2 * w.pp(), sc.data(), sc.size())) return e;
  const dim3 gs((unsigned)((n + RT - 1) / RT), m);
  hipLaunchKernelGGL(k_scale_cols, gs, dim3(RT), 0, st, X[0], (const C64*)(w.dm + 2 * w.pp()), n);
  hipLaunchKernelGGL(k_scale_cols, gs, dim3(RT), 0, st, X[1], (const C64*)(w.dm + 2 * w.pp() + m), n);
  NK_HIP(hipGetLastError());
  if (int e = nk_spinor_unpack_device(lat, X[0], r_out, m, st)) return e;
  if (int e = nk_spinor_unpack_device(lat, X[1], l_out, m, st)) return e;
  NK_HIP(hipStreamSynchronize(st));
  for (int i = 0; i < m; ++i) {
    lam[2 * i] = th[i].real();
    lam[2 * i + 1] = th[i].imag();
  }
  *passes = it;
  *resid = worst;
  return worst <= tol * hb ? NK_OK : NK_WARN_NOTCONV;
}

int eig_hermitian(nk_lattice* lat, double m_w, int m, int p, int degree, double tol, int maxit, const C64* v0,
                  double* lam, C64* r_out, int* passes, double* resid, hipStream_t st) {
  const size_t n = (size_t)12 * lat->g.V;
  const size_t blk = (size_t)p * n;
  if (lat->eig.ensure((4 * blk + eig_small(n, p)) * sizeof(C64))) return NK_ENOMEM;
  C64* base = lat->eig.as<C64>();
  C64* V = base;            // current orthonormal block
  C64* Y = base + blk;      // the filter's second buffer
  C64* Wb = base + 2 * blk; // H V
  C64* T = base + 3 * blk;  // H times the iterate inside the filter
  EigWork w;
  if (int e = eig_work(lat, p, base + 4 * blk, st, &w)) return e;
  const double hb = std::fabs(4.0 + m_w) + 8.0, b2 = hb * hb;
  const double mu0 = 0.0;

  std::vector<double> t2, th(p), res(p);
  // Rayleigh-Ritz with H^2 on the orthonormal V, then with H on the leading
  // Ritz vectors; leaves V rotated, Wb = H V, th the Rayleigh quotients of H
  // and res the residual norms of the leading m.  The second step's matrix
  // V^dag H V is formed from the first step's products, so both rotations go
  // to the vectors as one.
  auto rayleigh_ritz = [&]() -> int {
    if (int e = apply_blocks_of(lat, m_w, 1, &mu0, &V, &Wb, p, st)) return e;
    const GramPairs ab{{Wb, V, nullptr}, {Wb, Wb, nullptr}};
    std::vector<cd> g[2], q1;
    if (int e = grams(w, ab, 2, g)) return e;  // V^dag H^2 V = (H V)^dag (H V), and V^dag H V
    mirror(g[0], p);
    dense::jacobi_herm(g[0], p, t2, q1);
    // with H itself on the leading nq >= m vectors (nq grows past m while the
    // H^2 values repeat), which splits pairs lambda, -lambda that H^2 cannot
    // tell apart; sorted by |theta|
    int nq = m;
    while (nq < p && std::fabs(t2[nq] - t2[nq - 1]) <= 1e-8 * std::fabs(t2[nq])) ++nq;
    std::vector<cd> kq = projected(q1, g[1], q1, p, nq), qq;
    for (int j = 0; j < nq; ++j)
      for (int i = 0; i <= j; ++i) {
        const cd h = 0.5 * (kq[i + (size_t)j * nq] + std::conj(kq[j + (size_t)i * nq]));
        kq[i + (size_t)j * nq] = i == j ? cd(h.real(), 0.0) : h;
        kq[j + (size_t)i * nq] = i == j ? cd(h.real(), 0.0) : std::conj(h);
      }
    std::vector<double> tq;
    dense::jacobi_herm(kq, nq, tq, qq);
    std::vector<int> idx(nq);
    for (int i = 0; i < nq; ++i) idx[i] = i;
    std::stable_sort(idx.begin(), idx.end(), [&](int x, int y) { return std::fabs(tq[x]) < std::fabs(tq[y]); });
    std::vector<cd> q2((size_t)p * p, cd(0.0, 0.0));
    for (int j = 0; j < p; ++j) {
      if (j < nq) {
        for (int i = 0; i < nq; ++i) q2[i + (size_t)j * p] = qq[i + (size_t)idx[j] * nq];
      } else {
        q2[j + (size_t)j * p] = 1.0;
      }
    }
    const std::vector<cd> rot[1] = {matmul(q1, q2, p)};
    C64* const blocks[2] = {V, Wb};
    const int which[2] = {0, 0};
    if (int e = rotate_blocks(w, 2, blocks, which, rot, 1)) return e;
    // Rayleigh quotients v_i^dag H v_i, then the residuals H v_i - th_i v_i and their norms, leading m
    const ColArgs ca{{V, V}, {Wb, Wb}, w.dm + 2 * w.pp()};
    hipLaunchKernelGGL(k_cols<0>, dim3(w.nbc, m, 1), dim3(RT), 0, st, ca, n, w.part);
    hipLaunchKernelGGL(k_cols_sum, dim3(m), dim3(64), 0, st, (const C64*)w.part, w.nbc, w.hg_dev, w.dm + 2 * w.pp());
    hipLaunchKernelGGL(k_cols<1>, dim3(w.nbc, m, 1), dim3(RT), 0, st, ca, n, w.part);
    hipLaunchKernelGGL(k_cols_sum, dim3(m), dim3(64), 0, st, (const C64*)w.part, w.nbc, w.hg_dev + p, (C64*)nullptr);
    NK_HIP(hipGetLastError());
    NK_HIP(hipStreamSynchronize(st));
    for (int i = 0; i < m; ++i) {
      th[i] = w.hg[i].re;
      res[i] = std::sqrt(std::max(w.hg[p + i].re, 0.0));
    }
    return NK_OK;
  };

  if (int e = nk_spinor_pack_device(lat, v0, V, p, st)) return e;
  if (int e = orthonormalise(w, 1, &V)) return e;
  if (int e = rayleigh_ritz()) return e;
  int it = 0;
  double worst = *std::max_element(res.begin(), res.begin() + m);
  while (it < maxit && worst > tol * hb) {
    ++it;
    double a2 = t2[p - 1];
    if (!(a2 < b2)) a2 = 0.5 * b2;
    if (int er = cheb_filter(lat, m_w, 1, &mu0, &V, &Y, &T, p, degree, a2, b2, st)) return er;
    if (int er = orthonormalise(w, 1, &V)) return er;
    if (int er = rayleigh_ritz()) return er;
    worst = *std::max_element(res.begin(), res.begin() + m);
  }
  if (int e = nk_spinor_unpack_device(lat, V, r_out, m, st)) return e;
  NK_HIP(hipStreamSynchronize(st));
  for (int i = 0; i < m; ++i) lam[i] = th[i];
  *passes = it;
  *resid = worst;
  return worst <= tol * hb ? NK_OK : NK_WARN_NOTCONV;
}

}  // namespace nk
