// Learned scaling of the Roberts-Higham iteration of Eq. (4) on gfx950.
//
// The scaled iteration S <- (mu S + (mu S)^{-1}) / 2 has the limit sgn(S)
// for every mu > 0 (the scalar argument of Eq. (7) holds for mu z as well),
// so the factors change only the iteration count.  For the first T steps the
// factor is determinant scaling times a learned correction,
//   mu_t = |det S_t|^{-1/n} exp(y_t),
// with y predicted by a 16-64-64-64-T network (tanh, FP32 weights) from cheap
// features f of S_0:
//   x = (f - mean) * inv_std,  a_l = tanh(W_l a_{l-1} + b_l) (l = 1, 2, 3),
//   y = W4 a3 + b4,
// so y = 0 is plain determinant scaling.  It is trained without labels: each
// eigenvalue of a diagonalisable S_0 follows the scalar map and
// log|det S_t| = sum_i log|z_{i,t}|, so the distance
// d_i = log |z_{i,T} - sgn Re lambda_i| after T steps follows from the
// spectrum; the loss is the smooth maximum (1/kappa) log mean exp(kappa d).
//
// Kernels: features of a batch of dense matrices, forward pass, the
// spectral loss with its gradient, backward pass (per-sample deltas, then the
// weight gradients summed over the batch in a fixed order -- deterministic),
// and Adam.  The forward pass and the weight gradients are contractions over
// the units and over the batch and run on the matrix cores, in FP64 and in
// FP32; the per-sample deltas are small matrix-vector products on the vector
// ALUs.
#include <cmath>
#include <mutex>

#include "nk_internal.h"
#include "wave.h"

namespace nk {

constexpr int MI = NK_MLP_IN, MH = NK_MLP_HIDDEN, MT = NK_MLP_STEPS;
// flat parameter offsets
constexpr int OW1 = 0, OB1 = OW1 + MH * MI, OW2 = OB1 + MH, OB2 = OW2 + MH * MH, OW3 = OB2 + MH,
              OB3 = OW3 + MH * MH, OW4 = OB3 + MH, OB4 = OW4 + MT * MH, OMEAN = OB4 + MT, OISTD = OMEAN + MI;
static_assert(OMEAN == NK_MLP_NTRAIN, "trainable block size");
static_assert(OISTD + MI == NK_MLP_NPARAMS, "parameter count");
// FLOOR: squared distance below which an eigenvalue counts as converged (one
// more quadratic step takes 1e-7 to 1e-14); it also keeps the loss free of
// the sharp valleys of log 0
constexpr double KAPPA = 4.0, TINYF = 1e-30, FLOOR = 1e-14;

__device__ __forceinline__ double clampf(double v) { return fmin(50.0, fmax(-50.0, v)); }

__device__ __forceinline__ C64 cdiv1(C64 z) {  // 1 / z
  const double r = 1.0 / norm2(z);
  return mk(z.re * r, -z.im * r);
}

template <class T>
__device__ __forceinline__ T wsum(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double wmax(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ double wmin(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
  return v;
}

// ---------------------------------------------------------------------------
// features of the dense n x n matrix b (row-major, leading dimension ld); one
// 256-thread workgroup per matrix, O(n^2) reads
__global__ void __launch_bounds__(256) k_rh_features(int ld, const int* __restrict__ nvec,
                                                     const C64* __restrict__ S_b, float* __restrict__ feat) {
  const int b = blockIdx.x;
  const int n = nvec[b];
  const C64* S = S_b + (size_t)b * ld * ld;
  // four consecutive lanes per row i = tid / 4 + 64 m, each adding the
  // columns j = tid % 4 + 4 q of it (row sums, Hermitian defect), met by
  // shuffles; the group's first lane keeps the row's statistics (diagonal
  // entries and the row-sum ones).  The column sums the same way, columns
  // j = tid / 4 + 64 m over rows i = tid % 4 + 4 q.
  const int gr = threadIdx.x >> 2, gl = threadIdx.x & 3;
  double fro = 0, rowmax = 0, colmax = 0, herm = 0, dsq = 0, dmax = 0, dmin = INFINITY, rmin = INFINITY;
  double npos = 0, lsum = 0, lsq = 0, radmax = 0, ncross = 0, tr_re = 0, tr_im = 0;
  for (int i0 = 0; i0 < n; i0 += 64) {
    const int i = i0 + gr;
    double rs = 0, rq = 0, hd = 0;
    if (i < n) {
#pragma unroll 4
      for (int j = gl; j < n; j += 4) {
        const C64 a = S[(size_t)i * ld + j];
        const double m = sqrt(norm2(a));
        rs += m;
        rq += m * m;
        const C64 t = a - conj(S[(size_t)j * ld + i]);
        hd += norm2(t);
      }
    }
#pragma unroll
    for (int o = 1; o < 4; o <<= 1) {
      rs += __shfl_xor(rs, o, 64);
      rq += __shfl_xor(rq, o, 64);
      hd += __shfl_xor(hd, o, 64);
    }
    if (i < n && gl == 0) {
      const C64 d = S[(size_t)i * ld + i];
      const double ad = sqrt(norm2(d));
      fro += rq;
      rowmax = fmax(rowmax, rs);
      herm += hd;
      dsq += ad * ad;
      dmax = fmax(dmax, ad);
      dmin = fmin(dmin, ad);
      rmin = fmin(rmin, fabs(d.re));
      npos += d.re > 0 ? 1.0 : 0.0;
      const double ld_ = log(ad + TINYF);
      lsum += ld_;
      lsq += ld_ * ld_;
      const double rad = rs - ad;
      radmax = fmax(radmax, rad);
      ncross += fabs(d.re) < rad ? 1.0 : 0.0;
      tr_re += d.re;
      tr_im += d.im;
    }
  }
  for (int j0 = 0; j0 < n; j0 += 64) {
    const int j = j0 + gr;
    double cs = 0;
    if (j < n) {
#pragma unroll 4
      for (int i = gl; i < n; i += 4) cs += sqrt(norm2(S[(size_t)i * ld + j]));
    }
#pragma unroll
    for (int o = 1; o < 4; o <<= 1) cs += __shfl_xor(cs, o, 64);
    if (j < n && gl == 0) colmax = fmax(colmax, cs);
  }
  __shared__ double sh[4][16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double sums[9] = {fro, herm, dsq, npos, lsum, lsq, ncross, tr_re, tr_im};
  double maxs[4] = {rowmax, colmax, dmax, radmax};
  double mins[2] = {dmin, rmin};
#pragma unroll
  for (int q = 0; q < 9; ++q) sums[q] = wsum(sums[q]);
#pragma unroll
  for (int q = 0; q < 4; ++q) maxs[q] = wmax(maxs[q]);
#pragma unroll
  for (int q = 0; q < 2; ++q) mins[q] = wmin(mins[q]);
  if (lane == 0) {
#pragma unroll
    for (int q = 0; q < 9; ++q) sh[w][q] = sums[q];
#pragma unroll
    for (int q = 0; q < 4; ++q) sh[w][9 + q] = maxs[q];
#pragma unroll
    for (int q = 0; q < 2; ++q) sh[w][13 + q] = mins[q];
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  double v[15];
  for (int q = 0; q < 9; ++q) v[q] = (sh[0][q] + sh[1][q]) + (sh[2][q] + sh[3][q]);
  for (int q = 9; q < 13; ++q) v[q] = fmax(fmax(sh[0][q], sh[1][q]), fmax(sh[2][q], sh[3][q]));
  for (int q = 13; q < 15; ++q) v[q] = fmin(fmin(sh[0][q], sh[1][q]), fmin(sh[2][q], sh[3][q]));
  const double nd = (double)n;
  const double frob = sqrt(v[0]);
  const double rms = frob / sqrt(nd);
  const double lr = log(rms + TINYF);
  const double lmean = v[4] / nd;
  const double lvar = fmax(v[5] / nd - lmean * lmean, 0.0);
  const double offd = sqrt(fmax(v[0] - v[2], 0.0));
  double f[16];
  f[0] = log(nd);
  f[1] = lr;
  f[2] = log(v[9] + TINYF) - lr;
  f[3] = log(v[10] + TINYF) - lr;
  f[4] = v[7] / (nd * (rms + TINYF));
  f[5] = v[8] / (nd * (rms + TINYF));
  f[6] = log(v[11] + TINYF) - lr;
  f[7] = log(v[13] + TINYF) - lr;
  f[8] = log(v[14] + TINYF) - lr;
  f[9] = v[3] / nd;
  f[10] = lmean - lr;
  f[11] = sqrt(lvar);
  f[12] = log(sqrt(v[1]) / (frob + TINYF) + TINYF);
  f[13] = log(offd / (sqrt(v[2]) + TINYF) + TINYF);
  f[14] = log(v[12] + TINYF) - lr;
  f[15] = v[6] / nd;
  for (int q = 0; q < 16; ++q) feat[(size_t)b * MI + q] = (float)clampf(f[q]);
}

// ---------------------------------------------------------------------------
// forward pass: 16 samples per 256-thread workgroup on the FP64 matrix cores
// (v_mfma_f64_16x16x4f64), rounded to FP32 only where y and the activations
// are stored: the spectral loss multiplies an error of y by up to a hundred,
// and with FP32 sums and activations (2.3e-7 of y) the gradient of a few
// samples was off by a few 1e-6; now 2.5e-8 of y and 1e-7.  Wave w finishes units 16 w ..
// 16 w + 15 of a hidden layer, wave 0 the output layer.  Operand layout: lane
// l holds A[l % 16][l / 16] and B[l / 16][l % 16], accumulator element i of
// lane l is D[4 i + l / 16][l % 16].  The products of a layer of NV inputs are
// dealt so that lane group q = l / 16 takes the inputs q NV/4 ..
// (q + 1) NV/4 - 1: a lane then reads contiguous runs of its weight row
// (16-byte loads) and of its sample's activations.
// Bound by latency (three layers, one weight read each): with one lane per
// unit, as this kernel was before, every lane walked its own weight row in
// 4-byte loads, 64 cache lines per load, and a layer took 64 of them; 12.7 us
// for 2048 samples, now 9.0 (11.4 with tanh(), 8.3 in FP32).
// act (optional) keeps a1, a2, a3 for the backward pass.
typedef float nk_f4 __attribute__((ext_vector_type(4)));
typedef double nk_d4 __attribute__((ext_vector_type(4)));
constexpr int FS = 16;       // samples per workgroup
constexpr int FLD = MH + 2;  // padded row of activations (16-byte aligned)

// tanh to a few 1e-16, absolute, and to as much relative to its value below
// 2^-10 (three terms of the series): half the instructions of tanh(), which
// were most of the kernel's time
__device__ __forceinline__ double tanh_of(double x) {
  const double x2 = x * x;
  const double s = x * fma(x2, fma(x2, 2.0 / 15.0, -1.0 / 3.0), 1.0);
  const double t = 1.0 - 2.0 / (exp(2.0 * x) + 1.0);
  return fabs(x) < 0x1p-10 ? s : t;
}

// this lane's weights of 16 units, whose rows of NV start at W; units past nu
// read row 0 and are ignored by the caller
template <int NV>
__device__ __forceinline__ void weights16(const float* __restrict__ W, int nu, int lane, float (&wv)[NV / 4]) {
  const int l16 = lane & 15;
  const float* wr = W + (size_t)(l16 < nu ? l16 : 0) * NV + (lane >> 4) * (NV / 4);
#pragma unroll
  for (int c = 0; c < NV / 4; ++c) wv[c] = wr[c];  // (the flat parameter array gives no more than 4-byte alignment)
}
// the pre-activations of the 16 samples (rows of in, leading dimension FLD) and those units
template <int NV>
__device__ __forceinline__ nk_d4 layer16(const float (&wv)[NV / 4], const double* in, int lane) {
  const double* ar = in + (lane & 15) * FLD + (lane >> 4) * (NV / 4);
  nk_d4 acc[4] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};
#pragma unroll
  for (int c = 0; c < NV / 4; ++c)
    acc[c & 3] = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[c], (double)wv[c], acc[c & 3], 0, 0, 0);
  return (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

__global__ void __launch_bounds__(256) k_mlp_fwd(int B, const float* __restrict__ P, const float* __restrict__ feat,
                                                 float* __restrict__ y, float* __restrict__ act) {
  __shared__ __align__(16) double sx[FS][FLD];
  __shared__ __align__(16) double sa[2][FS][FLD];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int b0 = blockIdx.x * FS;
  const int u = 16 * w + (lane & 15), r0 = lane >> 4;  // this lane's unit, and its samples r0 + 4 i
  // every layer's weights are known at launch: one memory round trip for all
  float w1[MI / 4], w2[MH / 4], w3[MH / 4], w4[MH / 4];
  weights16<MI>(P + OW1 + 16 * w * MI, 16, lane, w1);
  weights16<MH>(P + OW2 + 16 * w * MH, 16, lane, w2);
  weights16<MH>(P + OW3 + 16 * w * MH, 16, lane, w3);
  weights16<MH>(P + OW4, MT, lane, w4);
  const float h1 = P[OB1 + u], h2 = P[OB2 + u], h3 = P[OB3 + u], h4 = P[OB4 + min(lane & 15, MT - 1)];
  {
    const int sl = tid / MI, v = tid % MI;  // 16 samples x 16 features
    const int b = b0 + sl;
    sx[sl][v] = b < B ? ((double)feat[(size_t)b * MI + v] - (double)P[OMEAN + v]) * (double)P[OISTD + v] : 0.0;
  }
  __syncthreads();
  auto finish = [&](nk_d4 h, float bias, int layer, double (*out)[FLD]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const double a = tanh_of(h[i] + (double)bias);
      const int r = r0 + 4 * i, b = b0 + r;
      out[r][u] = a;
      if (act && b < B) act[((size_t)b * 3 + layer) * MH + u] = (float)a;
    }
  };
  finish(layer16<MI>(w1, &sx[0][0], lane), h1, 0, sa[0]);
  __syncthreads();
  finish(layer16<MH>(w2, &sa[0][0][0], lane), h2, 1, sa[1]);
  __syncthreads();
  finish(layer16<MH>(w3, &sa[1][0][0], lane), h3, 2, sa[0]);
  __syncthreads();
  if (w == 0) {
    const nk_d4 o = layer16<MH>(w4, &sa[0][0][0], lane);
    const int t = lane & 15;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int b = b0 + r0 + 4 * i;
      if (t < MT && b < B) y[(size_t)b * MT + t] = (float)(o[i] + (double)h4);
    }
  }
}

// ---------------------------------------------------------------------------
// spectral loss of sample b (eigenvalues lam[off[b] .. off[b+1])) and its
// gradient with respect to y, scaled by gscale; one workgroup per sample,
// FP64 arithmetic.  Step t uses mu_t = exp(y_t - mean_i log|z_{i,t}|): the
// determinant scale of the eigenvalues times the learned correction.
// SPT eigenvalues per thread: 1 for spectra of up to 256, 2 up to 512, in one
// launch, and 4 up to 1024 in a second one.  Each launch takes the samples of
// its own class and returns at once on the others (their sizes are on the
// device); slots and whole waves past a
// sample's spectrum are branched over.  Bound by FP64 issue: the logarithm,
// exponential and division of every step and eigenvalue.  So a step divides
// once, and the backward sweep reuses its 1/w: 1/w^2 = (1/w)^2 and
// z/|z|^2 = conj(1/z) = mu conj(1/w).  With four slots for every sample, each
// of them computed, and two more divisions and an exponential per step, as
// before, 2048 samples of 16 to 300 eigenvalues took 52.6 us; as two launches
// of one and of four slots 22 + 19 (the few large samples leave the chip half
// empty), and now 26 + 4, FP64 issue busy for 16 of them.  Registers: 106 for
// one and two slots together, 188 for four, which would hold every sample to two
// workgroups per compute unit.

// sum over the 256 threads of the workgroup, the same value in every thread;
// on: whether this wave has a value at all.  The calls of a kernel take turns
// of the two halves of sh, so one barrier a call is enough.
__device__ __forceinline__ double block_sum256(double v, bool on, double* sh) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (on) v = wave_xsum(v);
  if (lane == 0) sh[w] = v;
  __syncthreads();
  return (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

template <int SPT>
__device__ __forceinline__ void spec_loss_of(int b, int i0, int n, const C64* __restrict__ lam,
                                             const float* __restrict__ y, float gscale, float* __restrict__ loss,
                                             float* __restrict__ dy, double* sh) {
  if (n <= 0) {  // no eigenvalues: nothing to learn from this sample
    if (threadIdx.x < MT) dy[(size_t)b * MT + threadIdx.x] = 0.f;
    if (threadIdx.x == 0) loss[b] = 0.f;
    return;
  }
  const bool wave_on = __builtin_amdgcn_readfirstlane(threadIdx.x) < n;
  bool on[SPT];
  C64 z[SPT];                  // z_t of the current step
  C64 w[SPT][MT], iw[SPT][MT];  // w_t = mu_t z_t and 1 / w_t
  double sg[SPT], mu[MT];
#pragma unroll
  for (int r = 0; r < SPT; ++r) {
    const int i = threadIdx.x + r * 256;
    on[r] = i < n;
    z[r] = mk(1.0, 0.0);
    if (on[r]) z[r] = lam[i0 + i];
    sg[r] = z[r].re > 0 ? 1.0 : -1.0;
  }
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    double ls = 0.0;
#pragma unroll
    for (int r = 0; r < SPT; ++r)
      if (on[r]) ls += 0.5 * log(norm2(z[r]));
    const double lm = block_sum256(ls, wave_on, sh + 4 * (t & 1)) / n;
    mu[t] = wave_on ? exp((double)y[(size_t)b * MT + t] - lm) : 1.0;
#pragma unroll
    for (int r = 0; r < SPT; ++r)
      if (on[r]) {
        w[r][t] = mu[t] * z[r];
        iw[r][t] = cdiv1(w[r][t]);
        z[r] = 0.5 * (w[r][t] + iw[r][t]);
      }
  }
  double dl[SPT], e[SPT], dmax = -INFINITY;
#pragma unroll
  for (int r = 0; r < SPT; ++r)
    if (on[r]) {
      e[r] = norm2(z[r] - mk(sg[r], 0.0));
      dl[r] = 0.5 * log(e[r] + FLOOR);
      dmax = fmax(dmax, dl[r]);
    }
  if (wave_on) dmax = wmax(dmax);
  double* shm = sh + 4 * (MT & 1);
  if ((threadIdx.x & 63) == 0) shm[threadIdx.x >> 6] = dmax;
  __syncthreads();
  const double m = fmax(fmax(shm[0], shm[1]), fmax(shm[2], shm[3]));
  double ex[SPT], se = 0.0;
#pragma unroll
  for (int r = 0; r < SPT; ++r)
    if (on[r]) {
      ex[r] = exp(KAPPA * (dl[r] - m));
      se += ex[r];
    }
  const double S = block_sum256(se, wave_on, sh + 4 * ((MT + 1) & 1));
  // backward: gradients as complex numbers dRe + i dIm
  C64 gz[SPT];
#pragma unroll
  for (int r = 0; r < SPT; ++r)
    if (on[r]) gz[r] = (ex[r] / (S * (e[r] + FLOOR))) * (z[r] - mk(sg[r], 0.0));
  double g[MT];
#pragma unroll
  for (int t = MT - 1; t >= 0; --t) {
    double pg = 0.0;
#pragma unroll
    for (int r = 0; r < SPT; ++r)
      if (on[r]) {
        const C64 q = cmul(iw[r][t], iw[r][t]);
        gz[r] = cmulc(mk(0.5 * (1.0 - q.re), -0.5 * q.im), gz[r]);  // conj(f'(w)) gz, through z_{t+1} = (w + 1/w) / 2
        pg += gz[r].re * w[r][t].re + gz[r].im * w[r][t].im;
      }
    const double glm = block_sum256(pg, wave_on, sh + 4 * ((MT + 2 + MT - 1 - t) & 1));  // dL/dlog mu_t = dL/dy_t
    g[t] = glm;
    // through w = mu z_t, and through the determinant scale -mean log|z_t|
#pragma unroll
    for (int r = 0; r < SPT; ++r)
      if (on[r]) gz[r] = mu[t] * (gz[r] - (glm / n) * conj(iw[r][t]));
  }
  if (threadIdx.x == 0) {
    loss[b] = (float)(m + log(S / n) / KAPPA);
#pragma unroll
    for (int t = 0; t < MT; ++t) dy[(size_t)b * MT + t] = (float)(gscale * g[t]);
  }
}

template <bool LARGE>
__global__ void __launch_bounds__(256) k_spec_loss(const int* __restrict__ off, const C64* __restrict__ lam,
                                                   const float* __restrict__ y, float gscale,
                                                   float* __restrict__ loss, float* __restrict__ dy) {
  __shared__ double sh[8];
  const int b = blockIdx.x;
  const int i0 = off[b], n = off[b + 1] - off[b];
  if (LARGE != (n > 512)) return;  // the other launch's sample
  if constexpr (LARGE)
    spec_loss_of<4>(b, i0, n, lam, y, gscale, loss, dy, sh);
  else if (n <= 256)
    spec_loss_of<1>(b, i0, n, lam, y, gscale, loss, dy, sh);
  else
    spec_loss_of<2>(b, i0, n, lam, y, gscale, loss, dy, sh);
}

// ---------------------------------------------------------------------------
// backward, step 1: per-sample deltas of the three hidden layers
__global__ void __launch_bounds__(256) k_mlp_delta(int B, const float* __restrict__ P, const float* __restrict__ act,
                                                   const float* __restrict__ dy, float* __restrict__ delta) {
  __shared__ float sd[4][MH];
  const int sl = threadIdx.x >> 6, u = threadIdx.x & 63;
  const int b = blockIdx.x * 4 + sl;
  const bool live = b < B;
  const size_t ab = (size_t)(live ? b : 0) * 3 * MH;
  // layer 3: (W4^T dy) * (1 - a3^2)
  float s = 0.f;
  for (int t = 0; t < MT; ++t) s += P[OW4 + t * MH + u] * (live ? dy[(size_t)b * MT + t] : 0.f);
  float a = act[ab + 2 * MH + u];
  float d = s * (1.f - a * a);
  sd[sl][u] = d;
  if (live) delta[ab + 2 * MH + u] = d;
  __syncthreads();
  // layer 2: (W3^T d3) * (1 - a2^2)
  s = 0.f;
  for (int v = 0; v < MH; ++v) s += P[OW3 + v * MH + u] * sd[sl][v];
  a = act[ab + 1 * MH + u];
  d = s * (1.f - a * a);
  __syncthreads();
  sd[sl][u] = d;
  if (live) delta[ab + 1 * MH + u] = d;
  __syncthreads();
  // layer 1: (W2^T d2) * (1 - a1^2)
  s = 0.f;
  for (int v = 0; v < MH; ++v) s += P[OW2 + v * MH + u] * sd[sl][v];
  a = act[ab + 0 * MH + u];
  d = s * (1.f - a * a);
  if (live) delta[ab + 0 * MH + u] = d;
}

// backward, step 2: the weight gradients sum_b delta[b][u] in[b][v] as matrix
// products over the batch on the FP32 matrix cores (layout:
// A = delta^T, B = the layer's input).  One workgroup of 16 waves per 16 x 16
// tile of a weight matrix: 4 tiles of W1, 16 of W2, 16 of W3 and 4 of W4 (its
// 4 rows of 16).  Wave w takes samples 4 w .. 4 w + 3 of every 64, one product
// each, in order; the 16 accumulators then meet in LDS and are added in wave
// order, so the result does not depend on timing.  The bias gradient of 16
// units comes from the same delta entries, in the workgroups of the first
// column tile.  No scratch memory.
// Bound by the latency of the loads (the batch's deltas and activations stay
// in L2 between the 40 workgroups): one thread per parameter walking the
// whole batch, as before, is a chain of 2048 dependent additions, 519 us for
// 2048 samples; now 10.7.
constexpr int WGT = 1024, WGW = WGT / 64;
constexpr int NWT = 40;  // weight tiles

__global__ void __launch_bounds__(WGT) k_mlp_wgrad(int B, const float* __restrict__ P, const float* __restrict__ feat,
                                                   const float* __restrict__ act, const float* __restrict__ dy,
                                                   const float* __restrict__ delta, float* __restrict__ grad) {
  __shared__ float sacc[WGW][16][17];
  __shared__ float sb[WGW][16];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, q = lane >> 4;
  // the tile: layer 0..3, first unit u0 and first input v0
  const int tile = blockIdx.x;
  const int layer = tile < 4 ? 0 : tile < 20 ? 1 : tile < 36 ? 2 : 3;
  const int tl = tile - (layer == 0 ? 0 : layer == 1 ? 4 : layer == 2 ? 20 : 36);
  const int u0 = layer == 0 ? 16 * tl : layer == 3 ? 0 : 16 * (tl >> 2);
  const int v0 = layer == 0 ? 0 : layer == 3 ? 16 * tl : 16 * (tl & 3);
  const int u = u0 + l16, v = v0 + l16;
  // element (b, u) of the output-side gradients and (b, v) of the input side
  const float* ga = layer == 3 ? dy : delta + layer * MH;
  const int lda = layer == 3 ? MT : 3 * MH;
  const float* gb = layer == 0 ? feat : act + (layer - 1) * MH;
  const int ldb = layer == 0 ? MI : 3 * MH;
  const bool ua = layer != 3 || u < MT;
  const float mv = layer == 0 ? P[OMEAN + v] : 0.f, iv = layer == 0 ? P[OISTD + v] : 1.f;
  nk_f4 acc = {0.f, 0.f, 0.f, 0.f};
  float bsum = 0.f;
  constexpr int U = 4;  // loads of four products in flight
  for (int b0 = 4 * w; b0 < B; b0 += 64 * U) {  // wave-uniform: every lane takes part in the products
    float av[U], bv[U];
#pragma unroll
    for (int s = 0; s < U; ++s) {
      const int b = b0 + 64 * s + q;
      const bool in = b < B;
      const size_t bb = in ? b : 0;
      const float x = ga[bb * lda + (ua ? u : 0)], z = gb[bb * ldb + v];
      av[s] = in && ua ? x : 0.f;
      bv[s] = in ? (layer == 0 ? (z - mv) * iv : z) : 0.f;
    }
#pragma unroll
    for (int s = 0; s < U; ++s) {
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s], bv[s], acc, 0, 0, 0);
      bsum += av[s];
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) sacc[w][4 * q + i][l16] = acc[i];
  bsum += __shfl_xor(bsum, 16, 64);
  bsum += __shfl_xor(bsum, 32, 64);
  if (q == 0) sb[w][l16] = bsum;
  __syncthreads();
  if (tid < 256) {
    const int r = tid >> 4, c = tid & 15;
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < WGW; ++k) t += sacc[k][r][c];
    const int ow = layer == 0 ? OW1 : layer == 1 ? OW2 : layer == 2 ? OW3 : OW4;
    const int ld = layer == 0 ? MI : MH;
    if (layer != 3 || r < MT) grad[ow + (u0 + r) * ld + v0 + c] = t;
  }
  if (v0 == 0 && tid < 16 && (layer != 3 || tid < MT)) {
    float t = 0.f;
#pragma unroll
    for (int k = 0; k < WGW; ++k) t += sb[k][tid];
    const int ob = layer == 0 ? OB1 : layer == 1 ? OB2 : layer == 2 ? OB3 : OB4;
    grad[ob + u0 + tid] = t;
  }
}

__global__ void k_adam(int n, float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, float c1, float c2, float lr, float b1, float b2, float eps) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.f - b1) * gi;
  const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi * c1) / (sqrtf(vi * c2) + eps);
}

// y -> exp(y), the correction factor on top of determinant scaling, in FP64
// for the Roberts-Higham kernels; a non-finite or implausible prediction
// becomes -1 (the step then uses determinant scaling alone)
__global__ void k_mu_from_y(int n, const float* __restrict__ y, double* __restrict__ mu) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double v = (double)y[i];
  mu[i] = (v == v && fabs(v) < 30.0) ? exp(v) : -1.0;
}

// ---------------------------------------------------------------------------
// host side
namespace {
std::mutex g_model_mu;
DevBuf g_model, g_feat, g_y, g_n;
bool g_have_model = false;
}  // namespace

int mlp_features(int batch, int ld, const int* nvec_dev, const C64* S, float* feat, hipStream_t st) {
  hipLaunchKernelGGL(k_rh_features, dim3(batch), dim3(256), 0, st, ld, nvec_dev, S, feat);
  NK_HIP(hipGetLastError());
  return NK_OK;
}

int mlp_forward(int batch, const float* P, const float* feat, float* y, float* act, hipStream_t st) {
  if (batch <= 0) return NK_OK;
  hipLaunchKernelGGL(k_mlp_fwd, dim3((batch + FS - 1) / FS), dim3(256), 0, st, batch, P, feat, y, act);
  NK_HIP(hipGetLastError());
  return NK_OK;
}

int mlp_spectral_loss(int batch, const int* off, const C64* lam, const float* y, float gscale, float* loss,
                      float* dy, hipStream_t st) {
  if (batch <= 0) return NK_OK;
  hipLaunchKernelGGL(k_spec_loss<false>, dim3(batch), dim3(256), 0, st, off, lam, y, gscale, loss, dy);
  hipLaunchKernelGGL(k_spec_loss<true>, dim3(batch), dim3(256), 0, st, off, lam, y, gscale, loss, dy);
  NK_HIP(hipGetLastError());
  return NK_OK;
}

int mlp_backward(int batch, const float* P, const float* feat, const float* act, const float* dy, float* delta,
                 float* grad, hipStream_t st) {
  if (batch > 0) hipLaunchKernelGGL(k_mlp_delta, dim3((batch + 3) / 4), dim3(256), 0, st, batch, P, act, dy, delta);
  hipLaunchKernelGGL(k_mlp_wgrad, dim3(NWT), dim3(WGT), 0, st, batch, P, feat, act, dy, delta, grad);
  NK_HIP(hipGetLastError());
  return NK_OK;
}

int mlp_adam(int n, float* p, const float* g, float* m, float* v, int t, float lr, float b1, float b2, float eps,
             hipStream_t st) {
  const float c1 = (float)(1.0 / (1.0 - std::pow((double)b1, t)));
  const float c2 = (float)(1.0 / (1.0 - std::pow((double)b2, t)));
  hipLaunchKernelGGL(k_adam, dim3((n + 255) / 256), dim3(256), 0, st, n, p, g, m, v, c1, c2, lr, b1, b2, eps);
  NK_HIP(hipGetLastError());
  return NK_OK;
}

int mlp_model_set(const float* params_host) {
  std::lock_guard<std::mutex> lock(g_model_mu);
  if (!params_host) {
    g_have_model = false;
    return NK_OK;
  }
  if (g_model.ensure(NK_MLP_NPARAMS * sizeof(float))) return NK_ENOMEM;
  NK_HIP(hipMemcpy(g_model.p, params_host, NK_MLP_NPARAMS * sizeof(float), hipMemcpyHostToDevice));
  g_have_model = true;
  return NK_OK;
}

// correction factors [batch][NK_MLP_STEPS] (device, FP64) predicted by the
// installed model for the batch of dense matrices S; *have = 0 without a model
int mlp_schedule(int batch, int ld, const int* nvec_dev, const C64* S, double* mu_dev, int* have, hipStream_t st) {
  std::lock_guard<std::mutex> lock(g_model_mu);
  *have = g_have_model ? 1 : 0;
  if (!g_have_model || batch <= 0) return NK_OK;
  if (g_feat.ensure((size_t)batch * MI * sizeof(float)) || g_y.ensure((size_t)batch * MT * sizeof(float)))
    return NK_ENOMEM;
  if (int e = mlp_features(batch, ld, nvec_dev, S, g_feat.as<float>(), st)) return e;
  if (int e = mlp_forward(batch, g_model.as<float>(), g_feat.as<float>(), g_y.as<float>(), nullptr, st)) return e;
  hipLaunchKernelGGL(k_mu_from_y, dim3((batch * MT + 255) / 256), dim3(256), 0, st, batch * MT, g_y.as<float>(),
                     mu_dev);
  NK_HIP(hipGetLastError());
  return NK_OK;
}

}  // namespace nk
