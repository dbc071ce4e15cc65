// Stand-alone applications of gamma5 Dw(mu): the single operator and the
// fused pair (A v, A^dag w) of two-sided Lanczos (A^dag = A(-mu)).
#include <algorithm>

#include "stencil.h"

namespace nk {

// y_f = [gamma5] ((4 + m_w) x_f - 1/2 hop(x_f)) for NF fields, device layout.
// Directions split over the waves of the workgroup (hop_group); NF lanes per
// site, lane f on field f.  Bound by the caches: an XCD's 4 MB L2 holds about
// eight tiles' links and spinors, so the spinors that cross a tile in z and t
// are fetched again (529 to 573 MB read for 318 on 24^4).  PAST: results, a fifth of
// what would share that L2, are stored past it (see apply_pair_dev).
template <class R, int NF, class LK, int NG, bool PAST = false>
__global__ void __launch_bounds__(256) k_apply(Geom g, LK lk, R diag, int g5, FieldPtrs<R, NF> in,
                                                FieldPtrsW<R, NF> out, TFac<R, NF> tf) {
  constexpr int M = 12 / NG;
  constexpr int SPW = 64 / NF;         // sites per wave
  constexpr int NSB = (256 / 64) / NG;  // site blocks per workgroup
  __shared__ XBuf<R, NG> xb;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int gi = w % NG, sb = w / NG;
  const int f = NF == 1 ? 0 : lane & 1;
  const Cx<R>* x = NF == 1 ? in.p[0] : (f ? in.p[NF - 1] : in.p[0]);
  Cx<R>* y = NF == 1 ? out.p[0] : (f ? out.p[NF - 1] : out.p[0]);
  const R ef = NF == 1 ? tf.f[0] : (f ? tf.f[NF - 1] : tf.f[0]);
  const R eb = NF == 1 ? tf.b[0] : (f ? tf.b[NF - 1] : tf.b[0]);
  const int s = (xcd_block() * NSB + sb) * SPW + lane / NF;
  const bool live = s < g.V;
  Cx<R> mine[M];
  hop_group<NG>(g, live ? s : 0, lk, x, gi, ef, eb, xb, w, lane, mine);  // a lane past the end hops at site 0
  __builtin_amdgcn_sched_barrier(0);  // the stencil's registers are free before these loads
  // this site's input entries go out before the exchange's barrier, which
  // they then overlap
  int se = s;
  asm volatile("" : "+v"(se));  // keeps the epilogue addresses out of the stencil's registers
  Cx<R> ein[M];
#pragma unroll
  for (int cl = 0; cl < M; ++cl) ein[cl] = x[sidx<R>(g.V, gi * M + cl, live ? se : 0)];
  __syncthreads();
  if (!live) return;
#pragma unroll
  for (int cl = 0; cl < M; ++cl) {
    const int cc = gi * M + cl;
    const Cx<R> hs = xsum<NG>(xb, sb, gi, lane, cl, mine[cl]);
    const size_t i = sidx<R>(g.V, cc, se);
    Cx<R> o = diag * ein[cl] - R(0.5) * hs;
    if (g5 && cc >= 6) o = mk<R>(-o.re, -o.im);
    if (PAST)
      store_nt(&y[i], o);
    else
      y[i] = o;
  }
}

// The same operator on a block of vectors (grid y = vector, of one or two
// sides with their own chemical potential), optionally finishing a step of a
// three-term recurrence in its epilogue:
//   out = A x,  or (CHEB)  out = ca A x + cb y + cc old,
// with old the vector that out replaces (each entry is read before it is
// written; cc = 0 reads none).  One launch per application of the block: on
// 8^4 one vector is 64 workgroups, a quarter of the compute units, and its
// launches follow each other no faster than every 5 us; the block runs 48
// vectors in 28 us (with the recurrence step 34).  The hardware deals
// workgroup b to XCD b mod 8, so where a vector has a multiple of eight site
// blocks, each lands on the XCD that holds its links.  Folding the recurrence step in saves writing and
// reading A x (a third of the bytes of the step).
template <int NG, bool CHEB>
__global__ void __launch_bounds__(256) k_apply_block(Geom g, LinksPlain<double> lk, double diag, ApplyBlock a) {
  constexpr int M = 12 / NG;
  constexpr int NSB = (256 / 64) / NG;
  __shared__ XBuf<double, NG> xb;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int gi = w % NG, sb = w / NG;
  const int side = (int)blockIdx.y >= a.p ? 1 : 0;
  const size_t off = (size_t)((int)blockIdx.y - side * a.p) * 12 * g.V;
  const C64* x = (side ? a.x[1] : a.x[0]) + off;
  const double ef = side ? a.ef[1] : a.ef[0], eb = side ? a.eb[1] : a.eb[0];
  const int s = (xcd_block() * NSB + sb) * 64 + lane;
  const bool live = s < g.V;
  C64 mine[M];
  hop_group<NG>(g, live ? s : 0, lk, x, gi, ef, eb, xb, w, lane, mine);  // a lane past the end hops at site 0
  __builtin_amdgcn_sched_barrier(0);  // the stencil's registers are free before these loads
  const C64* y = CHEB ? (side ? a.y[1] : a.y[0]) + off : nullptr;
  C64* out = (side ? a.out[1] : a.out[0]) + off;
  int se = live ? s : 0;
  asm volatile("" : "+v"(se));  // keeps the epilogue addresses out of the stencil's registers
  C64 ein[M], ey[M], eo[M];
#pragma unroll
  for (int cl = 0; cl < M; ++cl) {
    const size_t i = sidx<double>(g.V, gi * M + cl, se);
    ein[cl] = x[i];
    if (CHEB) {
      ey[cl] = y[i];
      eo[cl] = a.cc != 0.0 ? out[i] : mk(0.0, 0.0);
    }
  }
  __syncthreads();
  if (!live) return;
#pragma unroll
  for (int cl = 0; cl < M; ++cl) {
    const int cc = gi * M + cl;
    const C64 hs = xsum<NG>(xb, sb, gi, lane, cl, mine[cl]);
    C64 o = diag * ein[cl] - 0.5 * hs;
    if (cc >= 6) o = mk(-o.re, -o.im);
    if (CHEB) {
      o = mk(a.ca * o.re + a.cb * ey[cl].re, a.ca * o.im + a.cb * ey[cl].im);
      if (a.cc != 0.0) o = mk(o.re + a.cc * eo[cl].re, o.im + a.cc * eo[cl].im);
    }
    out[sidx<double>(g.V, cc, se)] = o;
  }
}

// The operator on canonical vectors, out of the stencil's epilogue into the
// canonical layout: the 64 sites' results meet in LDS (over the exchange's
// buffer) and go out as they lie in memory, 12 components of a site together
// and whole x lines of sites behind each other.  CIN: the input is canonical
// too, each lane reading its neighbours' 192 bytes where they lie (twelve loads
// that share their lines; the L1 holds a wave's 12 KB of them); grid y =
// vector.  That spares the packing launch and its pass over memory.  The
// results are stored past the L2, which the neighbours and links need, on every
// lattice: with them kept in it and past it, 24^4 95 and 79 us, 16^4 18.6 and
// 17.6, 20736 sites 9.7 and 9.4, 8^4 5.45 and 5.47 (y read back by the next
// application: 98 and 90, 18.9 and 18.3, 10.5 and 10.4, 5.86 and 5.86; so on 4^4
// and 6^4, 5.5 and 5.5, 5.8 and 5.7: what one XCD stored, seven others read).
template <int NG, bool CIN>
__global__ void __launch_bounds__(256) k_apply_canon(Geom g, LinksPlain<double> lk, double diag, int g5, const C64* in,
                                                     C64* out, double ef, double eb) {
  constexpr int M = 12 / NG, NSB = (256 / 64) / NG, SITES = 64 * NSB, LD = 13;  // LD: padded sites in LDS
  __shared__ union {
    XBuf<double, NG> xb;
    C64 y[SITES][LD];
  } sh;
  __shared__ int s_can[SITES];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int gi = w % NG, sb = w / NG;
  const int s0 = xcd_block() * SITES, s = s0 + sb * 64 + lane;
  const size_t off = CIN ? (size_t)blockIdx.y * 12 * g.V : 0;
  const C64* x = in + off;
  C64* y = out + off;
  const bool live = s < g.V;
  const int sl = live ? s : 0;  // a lane past the end hops at site 0
  const int sc = canon_site(g, site_coords(g, sl));
  if (gi == 0) s_can[sb * 64 + lane] = sc;
  C64 mine[M];
  if constexpr (CIN)
    hop_group<NG>(g, sl, lk, CanonField{x, sc}, gi, ef, eb, sh.xb, w, lane, mine);
  else
    hop_group<NG>(g, sl, lk, x, gi, ef, eb, sh.xb, w, lane, mine);
  __builtin_amdgcn_sched_barrier(0);  // the stencil's registers are free before these loads
  int se = CIN ? sc : sl;
  asm volatile("" : "+v"(se));  // keeps the epilogue addresses out of the stencil's registers
  C64 ein[M];
#pragma unroll
  for (int cl = 0; cl < M; ++cl) ein[cl] = CIN ? x[(size_t)se * 12 + gi * M + cl] : x[sidx<double>(g.V, gi * M + cl, se)];
  __syncthreads();
  C64 o[M];
#pragma unroll
  for (int cl = 0; cl < M; ++cl) {
    const int cc = gi * M + cl;
    const C64 hs = xsum<NG>(sh.xb, sb, gi, lane, cl, mine[cl]);
    o[cl] = diag * ein[cl] - 0.5 * hs;
    if (g5 && cc >= 6) o[cl] = mk(-o[cl].re, -o[cl].im);
  }
  __syncthreads();
#pragma unroll
  for (int cl = 0; cl < M; ++cl) sh.y[sb * 64 + lane][gi * M + cl] = o[cl];
  __syncthreads();
#pragma unroll
  for (int m = 0; m < SITES * 12 / 256; ++m) {
    const int e = threadIdx.x + 256 * m, q = e / 12, c = e % 12;
    if (s0 + q < g.V) store_nt(&y[(size_t)s_can[q] * 12 + c], sh.y[q][c]);
  }
}

// workgroups of k_apply for NF fields
static int apply_blocks(const Geom& g, int nf) {
  const int spb = (64 / nf) * ((256 / 64) / NK_GROUPS);
  return (g.V + spb - 1) / spb;
}

static int check_gauge(nk_lattice* lat) {
  if (!lat->have_gauge) {
    set_error("no gauge field set on the lattice handle");
    return NK_ENOGAUGE;
  }
  return NK_OK;
}

int apply_dw_dev(nk_lattice* lat, double m_w, double mu, int g5, const C64* x, C64* y, hipStream_t st) {
  if (int e = check_gauge(lat)) return e;
  const Geom& g = lat->g;
  FieldPtrs<double, 1> in{{x}};
  FieldPtrsW<double, 1> out{{y}};
  TFac<double, 1> tf{{exp(mu)}, {exp(-mu)}};
  LinksPlain<double> lk{lat->U64.as<C64>(), g.V};
  hipLaunchKernelGGL((k_apply<double, 1, LinksPlain<double>, NK_GROUPS>), dim3(apply_blocks(g, 1)), dim3(256), 0,
                     st, g, lk, 4.0 + m_w, g5, in, out, tf);
  NK_HIP(hipGetLastError());
  return NK_OK;
}

// y = [gamma5] Dw x for nrhs canonical vectors.  The one launch needs x and y
// apart, since it writes y while it reads x; where they overlap, each x is
// packed into tmp(), one vector, before its y is written, one vector after the
// other.  Measured (one vector; through the packed layout with this epilogue;
// pack, stencil and unpack; the first two with results kept in the L2): 4096
// sites 7.4, 10.8, 12.6 us; 65536 18.8, 23.2, 31.0; 331776 96, 114, 157.
int apply_canon_dev(nk_lattice* lat, double m_w, double mu, int g5, const C64* x, C64* y, int nrhs,
                    int (*tmp)(nk_lattice*, C64**), hipStream_t st) {
  if (int e = check_gauge(lat)) return e;
  const Geom& g = lat->g;
  const size_t n = (size_t)12 * g.V;
  LinksPlain<double> lk{lat->U64.as<C64>(), g.V};
  const double ef = exp(mu), eb = exp(-mu);
  if (x + n * nrhs <= y || y + n * nrhs <= x) {
    for (int r = 0; r < nrhs; r += 65535)
      hipLaunchKernelGGL((k_apply_canon<NK_GROUPS, true>), dim3(apply_blocks(g, 1), std::min(nrhs - r, 65535)),
                         dim3(256), 0, st, g, lk, 4.0 + m_w, g5, x + r * n, y + r * n, ef, eb);
  } else {
    C64* p = nullptr;
    if (int e = tmp(lat, &p)) return e;
    for (int r = 0; r < nrhs; ++r) {
      if (int e = pack_spinor<double>(g, x + r * n, p, st)) return e;
      hipLaunchKernelGGL((k_apply_canon<NK_GROUPS, false>), dim3(apply_blocks(g, 1)), dim3(256), 0, st, g, lk,
                         4.0 + m_w, g5, p, y + r * n, ef, eb);
    }
  }
  NK_HIP(hipGetLastError());
  return NK_OK;
}

int apply_block_dev(nk_lattice* lat, double m_w, const ApplyBlock& a, int sides, bool cheb, hipStream_t st) {
  if (int e = check_gauge(lat)) return e;
  const Geom& g = lat->g;
  LinksPlain<double> lk{lat->U64.as<C64>(), g.V};
  const dim3 grid(apply_blocks(g, 1), sides * a.p);
  if (cheb)
    hipLaunchKernelGGL((k_apply_block<NK_GROUPS, true>), grid, dim3(256), 0, st, g, lk, 4.0 + m_w, a);
  else
    hipLaunchKernelGGL((k_apply_block<NK_GROUPS, false>), grid, dim3(256), 0, st, g, lk, 4.0 + m_w, a);
  NK_HIP(hipGetLastError());
  return NK_OK;
}

int apply_pair_dev(nk_lattice* lat, double m_w, double mu, const C64* v, const C64* w, C64* av, C64* adw,
                   hipStream_t st) {
  if (int e = check_gauge(lat)) return e;
  const Geom& g = lat->g;
  FieldPtrs<double, 2> in{{v, w}};
  FieldPtrsW<double, 2> out{{av, adw}};
  TFac<double, 2> tf{{exp(mu), exp(-mu)}, {exp(-mu), exp(mu)}};
  LinksPlain<double> lk{lat->U64.as<C64>(), g.V};
  // Links and fields beyond the 256 MB Infinity Cache: nobody finds the results
  // there anyway, and stored past the L2 they leave it to the neighbours.  With
  // the results in the caches and past the L2, read back by the next call:
  // 160000 sites 57.8, 68.8 us; 221184 86.2, 80.1; 331776 154.9, 150.0 (not read
  // back: 58.3, 57.4; 83.6, 66.9; 152.5, 143.0).
  const size_t bytes = ((size_t)4 * 9 + 4 * 12) * g.V * sizeof(C64);
  auto* const k = bytes > (size_t)256 << 20 ? k_apply<double, 2, LinksPlain<double>, NK_GROUPS, true>
                                            : k_apply<double, 2, LinksPlain<double>, NK_GROUPS>;
  hipLaunchKernelGGL(k, dim3(apply_blocks(g, 2)), dim3(256), 0, st, g, lk, 4.0 + m_w, 1, in, out, tf);
  NK_HIP(hipGetLastError());
  return NK_OK;
}

}  // namespace nk
