// The per-site steps of the even-odd solvers, used by the grouped kernels (one
// launch a step, solver_kernels.hip) and by the one-work-group solver of small
// lattices (solo.hip).  Each works on site s of system d, whose state st may lie
// in global memory or in LDS, and gives the site's share of the step's sums in v.
#pragma once
#include "solver_dev.h"

namespace qiral {

enum : int { A_ONE = 0, A_KAPPA = 1, A_MKAPPA2 = 2, A_MKAPPA = 3 };

__device__ __forceinline__ double coef(int amode, double k) {
  return amode == A_ONE ? 1.0 : amode == A_KAPPA ? k : amode == A_MKAPPA2 ? -k * k : -k;
}

template <int S> __device__ __forceinline__ const void *links_of(const SysDesc &d) {
  return S == S_F64 ? d.g64 : d.glo;
}

// A hop's epilogue on its sum acc = (H in)(s): out = C_o (a acc), or with `epi`
// C_o (C_x x + a acc), C_o and C_x the twisted-mass site factors chio and chix.
// red: 0 none; 1 ||out||^2; 2 (rt | out); 3 (out | x) and ||out||^2 (epi only);
// 4 (z | out).  ont: streaming store.
template <int S>
__device__ __forceinline__ void hop_site(const SysDesc &d, cpx<typename SpinorIO<S>::R> acc[12], int epi,
                                         typename SpinorIO<S>::R a, int fx, int fout, int s, int red, int chio,
                                         int chix, int ont, double v[NV]) {
  using R = typename SpinorIO<S>::R;
  if (!epi) {
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = cscale(a, acc[k]);
    apply_chi(acc, chio, d.tmu);
  } else {
    cpx<R> xv[12], ax[12];
    SpinorIO<S>::load(d.f[fx], s, d.npad, xv);
#pragma unroll
    for (int k = 0; k < 12; ++k) ax[k] = xv[k];
    apply_chi(ax, chix, d.tmu);
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = cadd(ax[k], cscale(a, acc[k]));
    apply_chi(acc, chio, d.tmu);
    if (red == 3) { dot12(acc, xv, v[0], v[1]); v[2] = norm12(acc); }
  }
  if (ont) SpinorIO<S>::template store_fast<true>(d.f[fout], s, d.npad, acc);
  else SpinorIO<S>::template store_fast<false>(d.f[fout], s, d.npad, acc);
  if (red == 1) v[0] = norm12(acc);
  if (red == 2 || red == 4) {
    cpx<R> rt[12];
    SpinorIO<S>::load(d.f[red == 2 ? F_RT : F_Z], s, d.npad, rt);
    dot12(rt, acc, v[0], v[1]);
  }
}

// Unit 0 of site s in a packed F64 half-field.
__device__ __forceinline__ size_t f64_at(int s) { return (size_t)(s >> 6) * (12 * WAVE) + (s & 63); }

// The reliable update at an odd site, acc = (H_oe T64)(s): y = XH + X; XH = y;
// X = 0; r_hat = BH - (A y - kappa^2 acc) in FP64; R = r_hat rounded to the
// iterate precision; ||r_hat||^2 (and (rt | r_hat) for BiCGStab).
template <int SO, bool HASLO, bool BICG>
__device__ __forceinline__ void upd_site(const SysDesc &d, const SysState *st, cpx<double> acc[12], int s,
                                         double v[NV]) {
  using RO = typename SpinorIO<SO>::R;
  const double k2 = d.kappa * d.kappa;
  double2 *xh = (double2 *)d.f[F_XH] + f64_at(s);
  const double2 *bh = (const double2 *)d.f[F_BH] + f64_at(s);
  float4 *xl = HASLO ? (float4 *)d.f[F_X] + (size_t)(s >> 6) * (6 * WAVE) + (s & 63) : nullptr;
#pragma unroll
  for (int c = 0; c < 3; ++c) {   // a colour at a time: three waves per SIMD keep their registers
    double2 y[4], b[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) { y[j] = xh[(4 * c + j) * WAVE]; b[j] = bh[(4 * c + j) * WAVE]; }
    if (HASLO) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const float4 l = xl[(2 * c + j) * WAVE];
        y[2 * j] = make_double2(y[2 * j].x + (double)l.x, y[2 * j].y + (double)l.y);
        y[2 * j + 1] = make_double2(y[2 * j + 1].x + (double)l.z, y[2 * j + 1].y + (double)l.w);
        xl[(2 * c + j) * WAVE] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) xh[(4 * c + j) * WAVE] = y[j];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const cpx<double> ay = chi1(cmake(y[j].x, y[j].y), j, CHI_A, d.tmu);
      acc[4 * c + j] = cadd(csub(cmake(b[j].x, b[j].y), ay), cscale(k2, acc[4 * c + j]));
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  v[0] = norm12(acc);
  cpx<RO> r[12];
  cvt12(acc, r);
  SpinorIO<SO>::store(d.f[F_R], s, d.npad, r);
  if (BICG && st->iter > 0) {
    cpx<RO> rt[12];
    SpinorIO<SO>::load(d.f[F_RT], s, d.npad, rt);
    cpx<double> rtd[12];
    cvt12(rt, rtd);
    dot12(rtd, acc, v[1], v[2]);
  }
}

// ||b - D x||^2 at a site of parity par, acc = (H x_{1-par})(s).
__device__ __forceinline__ void res_site(const SysDesc &d, cpx<double> acc[12], int par, int s, double v[NV]) {
  const double2 *xp = (const double2 *)d.f[par ? F_XH : F_XE] + f64_at(s);
  const double2 *bp = (const double2 *)d.f[par ? F_BO : F_BE] + f64_at(s);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    double2 x[4], b[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) { x[j] = xp[(4 * c + j) * WAVE]; b[j] = bp[(4 * c + j) * WAVE]; }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const cpx<double> ax = chi1(cmake(x[j].x, x[j].y), j, CHI_A, d.tmu);
      acc[4 * c + j] = cadd(csub(cmake(b[j].x, b[j].y), ax), cscale(d.kappa, acc[4 * c + j]));
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  v[0] = norm12(acc);
}

// ||b||^2 over both parities.
__device__ __forceinline__ void bnorm_site(const SysDesc &d, int s, double v[NV]) {
  cpx<double> a[12], b[12];
  SpinorIO<S_F64>::load(d.f[F_BE], s, d.npad, a);
  SpinorIO<S_F64>::load(d.f[F_BO], s, d.npad, b);
  v[0] = norm12(a);
  v[0] += norm12(b);
}

// CGNR: X += alpha P; R -= alpha AP; ||R||^2.  A plain (FP64) solve leaves X
// to cg2_site, which reads P anyway: X += alpha P there, before P changes, is
// the same arithmetic one pass over the vectors cheaper; xfin_site applies the
// last one when the solve stops here.  V: streaming level (vec_stream).  The
// loads come before the first store: one that might alias them would hold them
// back a memory round trip.
template <int S, int XS, int V>
__device__ __forceinline__ void cg1_site(const SysDesc &d, const SysState *st, int s, double v[NV]) {
  using R = typename SpinorIO<S>::R;
  using RX = typename SpinorIO<XS>::R;
  constexpr bool xhere = S != S_F64;
  const double al = st->alpha;
  cpx<R> r[12], ap[12];
  SpinorIO<S>::template load<(V > 1)>(d.f[F_R], s, d.npad, r);
  SpinorIO<S>::template load<(V > 0)>(d.f[F_AP], s, d.npad, ap);
  if (xhere) {
    cpx<R> p[12];
    cpx<RX> x[12];
    SpinorIO<S>::template load<(V > 1)>(d.f[F_P], s, d.npad, p);
    SpinorIO<XS>::template load<(V > 0)>(d.f[F_X], s, d.npad, x);
#pragma unroll
    for (int k = 0; k < 12; ++k) x[k] = cadd(x[k], cscale((RX)al, cmake((RX)p[k].re, (RX)p[k].im)));
    SpinorIO<XS>::template store<(V > 0)>(d.f[F_X], s, d.npad, x);
  }
#pragma unroll
  for (int k = 0; k < 12; ++k) r[k] = csub(r[k], cscale((R)al, ap[k]));
  SpinorIO<S>::template store<(V > 1)>(d.f[F_R], s, d.npad, r);
  v[0] = norm12(r);
}

// The x += alpha p that a plain CGNR solve stopped before (status done after
// cg1_site, flag set by the residual check).
__device__ __forceinline__ void xfin_site(const SysDesc &d, const SysState *st, int s) {
  const double al = st->alpha;
  cpx<double> p[12], x[12];
  SpinorIO<S_F64>::load(d.f[F_P], s, d.npad, p);
  SpinorIO<S_F64>::load(d.f[F_X], s, d.npad, x);
#pragma unroll
  for (int k = 0; k < 12; ++k) x[k] = cadd(x[k], cscale(al, cmake(p[k].re, p[k].im)));
  SpinorIO<S_F64>::store(d.f[F_X], s, d.npad, x);
}

// CGNR: P = Z + beta P; with XUPD (plain solves, in the iterations) first
// X += alpha P with the old P (the update cg1_site left).
template <int S, bool XUPD, int V>
__device__ __forceinline__ void cg2_site(const SysDesc &d, const SysState *st, int s) {
  using R = typename SpinorIO<S>::R;
  const R be = (R)st->beta;
  cpx<R> p[12], z[12];
  cpx<double> x[12];
  SpinorIO<S>::template load<(V > 1)>(d.f[F_P], s, d.npad, p);
  if (XUPD) SpinorIO<S_F64>::load<(V > 0)>(d.f[F_X], s, d.npad, x);
  SpinorIO<S>::template load<(V > 0)>(d.f[F_Z], s, d.npad, z);
  if (XUPD) {
    const double al = st->alpha;
#pragma unroll
    for (int k = 0; k < 12; ++k) x[k] = cadd(x[k], cscale(al, cmake((double)p[k].re, (double)p[k].im)));
    SpinorIO<S_F64>::store<(V > 0)>(d.f[F_X], s, d.npad, x);
  }
#pragma unroll
  for (int k = 0; k < 12; ++k) p[k] = cadd(z[k], cscale(be, p[k]));
  SpinorIO<S>::template store<(V > 1)>(d.f[F_P], s, d.npad, p);
}

// Conjugate residual on S^dagger S: X += alpha P; R -= alpha U (U = S P);
// Z -= alpha Q (Q = S^dagger S P); ||R||^2 (the Schur residual).
template <int S>
__device__ __forceinline__ void cr1_site(const SysDesc &d, const SysState *st, int s, double v[NV]) {
  using R = typename SpinorIO<S>::R;
  const R al = (R)st->alpha;
  const int dst[3] = {F_X, F_R, F_Z}, src[3] = {F_P, F_T, F_AP};
#pragma unroll
  for (int f = 0; f < 3; ++f) {   // one pair after the other: all six at once leave too few waves (2% slower)
    cpx<R> a[12], b[12];
    SpinorIO<S>::load(d.f[src[f]], s, d.npad, b);
    SpinorIO<S>::load(d.f[dst[f]], s, d.npad, a);
#pragma unroll
    for (int k = 0; k < 12; ++k) a[k] = f == 0 ? cadd(a[k], cscale(al, b[k])) : csub(a[k], cscale(al, b[k]));
    SpinorIO<S>::store(d.f[dst[f]], s, d.npad, a);
    if (f == 1) v[0] = norm12(a);
  }
}

// Conjugate residual: P = Z + beta P; Q = W + beta Q; U = V + beta U (INIT:
// beta = 0, old values not read); ||Q||^2.
template <int S, bool INIT>
__device__ __forceinline__ void cr2_site(const SysDesc &d, const SysState *st, int s, double v[NV]) {
  using R = typename SpinorIO<S>::R;
  const R be = (R)st->beta;
  const int src[3] = {F_Z, F_W, F_RT}, dst[3] = {F_P, F_AP, F_T};
#pragma unroll
  for (int f = 0; f < 3; ++f) {
    cpx<R> a[12];
    SpinorIO<S>::load(d.f[src[f]], s, d.npad, a);
    if (!INIT) {
      cpx<R> b[12];
      SpinorIO<S>::load(d.f[dst[f]], s, d.npad, b);
#pragma unroll
      for (int k = 0; k < 12; ++k) a[k] = cadd(a[k], cscale(be, b[k]));
    }
    SpinorIO<S>::store(d.f[dst[f]], s, d.npad, a);
    if (f == 1) v[0] = norm12(a);
  }
}

// BiCGStab: P = R + beta (P - omega V)    (V lives in F_AP)
template <int S, int V> __device__ __forceinline__ void bi_p_site(const SysDesc &d, const SysState *st, int s) {
  using R = typename SpinorIO<S>::R;
  const cpx<R> be = cmake((R)st->be_re, (R)st->be_im), om = cmake((R)st->om_re, (R)st->om_im);
  cpx<R> p[12], r[12], vv[12];
  SpinorIO<S>::template load<(V > 1)>(d.f[F_P], s, d.npad, p);
  SpinorIO<S>::template load<(V > 1)>(d.f[F_R], s, d.npad, r);
  SpinorIO<S>::template load<(V > 0)>(d.f[F_AP], s, d.npad, vv);
#pragma unroll
  for (int k = 0; k < 12; ++k) p[k] = cadd(r[k], cmul(be, csub(p[k], cmul(om, vv[k]))));
  SpinorIO<S>::template store<(V > 1)>(d.f[F_P], s, d.npad, p);
}

// BiCGStab: S = R - alpha V    (S lives in F_Z)
template <int S, int V> __device__ __forceinline__ void bi_s_site(const SysDesc &d, const SysState *st, int s) {
  using R = typename SpinorIO<S>::R;
  const cpx<R> al = cmake((R)st->al_re, (R)st->al_im);
  cpx<R> r[12], vv[12];
  SpinorIO<S>::template load<(V > 0)>(d.f[F_R], s, d.npad, r);
  SpinorIO<S>::template load<(V > 1)>(d.f[F_AP], s, d.npad, vv);
#pragma unroll
  for (int k = 0; k < 12; ++k) r[k] = csub(r[k], cmul(al, vv[k]));
  SpinorIO<S>::template store<(V > 1)>(d.f[F_Z], s, d.npad, r);
}

// BiCGStab: X += alpha P + omega S; R = S - omega T; (rt | R) and ||R||^2.
// LATE: T and rt are loaded once P and X are used up, for a kernel without registers
// for five FP64 vectors at once.
template <int S, int XS, int V, bool LATE = false>
__device__ __forceinline__ void bi_xr_site(const SysDesc &d, const SysState *st, int site, double v[NV]) {
  using R = typename SpinorIO<S>::R;
  using RX = typename SpinorIO<XS>::R;
  const cpx<RX> al = cmake((RX)st->al_re, (RX)st->al_im), om = cmake((RX)st->om_re, (RX)st->om_im);
  const cpx<R> omr = cmake((R)st->om_re, (R)st->om_im);
  cpx<R> p[12], s[12], t[12], rt[12];
  cpx<RX> x[12];
  SpinorIO<S>::template load<(V > 1)>(d.f[F_P], site, d.npad, p);
  SpinorIO<S>::template load<(V > 0)>(d.f[F_Z], site, d.npad, s);
  SpinorIO<XS>::template load<(V > 0)>(d.f[F_X], site, d.npad, x);
  auto second = [&]() {
    SpinorIO<S>::template load<(V > 0)>(d.f[F_T], site, d.npad, t);
    SpinorIO<S>::template load<(V > 1)>(d.f[F_RT], site, d.npad, rt);
  };
  if (!LATE) second();
#pragma unroll
  for (int k = 0; k < 12; ++k)
    x[k] = cadd(x[k], cadd(cmul(al, cmake((RX)p[k].re, (RX)p[k].im)), cmul(om, cmake((RX)s[k].re, (RX)s[k].im))));
  SpinorIO<XS>::template store<(V > 0)>(d.f[F_X], site, d.npad, x);
  if (LATE) {
    __builtin_amdgcn_sched_barrier(0);
    second();
  }
#pragma unroll
  for (int k = 0; k < 12; ++k) s[k] = csub(s[k], cmul(omr, t[k]));
  SpinorIO<S>::template store<(V > 1)>(d.f[F_R], site, d.npad, s);
  dot12(rt, s, v[0], v[1]);
  v[2] = norm12(s);
}

// dst = C src for a half-field, C the twisted-mass site factor chi.
template <int S> __device__ __forceinline__ void copy_site(const SysDesc &d, int fsrc, int fdst, int chi, int s) {
  cpx<typename SpinorIO<S>::R> a[12];
  SpinorIO<S>::load(d.f[fsrc], s, d.npad, a);
  apply_chi(a, chi, d.tmu);
  SpinorIO<S>::store(d.f[fdst], s, d.npad, a);
}

// BiCGStab start: rho = (r~ | r) = ||r||^2 with r~ = r, alpha = omega = 1, beta = 0.
__device__ __forceinline__ void bi_start(SysState *st) {
  st->rho_re = st->nr; st->rho_im = 0.0;
  st->rho0_re = st->nr; st->rho0_im = 0.0;
  st->al_re = 1.0; st->al_im = 0.0;
  st->om_re = 1.0; st->om_im = 0.0;
  st->be_re = 0.0; st->be_im = 0.0;
}

}  // namespace qiral
