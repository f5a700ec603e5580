// Grouped kernels of the even-odd solvers (CGNR of Fig. "CG" on the Schur
// system of the "schur" template, and BiCGStab), plus the FP64 reliable update
// and true-residual kernels.  Every kernel takes the system table and the work
// table; see solver_dev.h.
#include "qiral_int.h"
#include "solver_steps.h"
#include "solver_kernels.h"

namespace qiral {

// out = C_o (a H in) (EPI 0) or out = C_o (C_x x + a H in) (EPI 1), parity
// `par` out, for the (up to NR) systems of a grouped work item (they share the
// lattice, so each link is loaded once for all of them); see hop_site.
// T waves per item (see hop_wave); padded lanes compute on site 0 and store
// nothing.  Every wave reaches wave_combine's barrier.
template <int S, int L, bool DAG, int EPI, int T, int NR, bool NT>
__global__ __launch_bounds__(WG, HOP_MIN_WAVES(S, T, NR)) void k_hop_sys(const SysDesc *__restrict__ sdesc,
                                                                 const uint32_t *__restrict__ work, int nwork,
                                                                 int fin_id, int fout, int fx, int par, int amode,
                                                                 int mask, int red, int slot, int chio, int chix,
                                                                 int ont) {
  using R = typename SpinorIO<S>::R;
  using LDS = HopLds<T, NR, R>;
  __shared__ typename LDS::V lds[LDS::VECS];
  const Item it = fetch_item<T>(work, nwork);
  bool act[NR];
  bool any = false;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    act[r] = it.active && r < it.cnt && (sdesc[it.sys + r].st->status & mask);
    any = any || act[r];
  }
  const SysDesc &d0 = sdesc[it.sys];
  const bool site_ok = it.active && it.s < d0.g.vh;
  const size_t npad = d0.npad;
  FieldLd<S, NR> ld;
  ld.npad = npad;
#pragma unroll
  for (int r = 0; r < NR; ++r) ld.base[r] = sdesc[it.sys + min(r, it.cnt - 1)].f[fin_id];
  cpx<R> acc[NR][12];
  if (any) hop_wave<L, DAG, T, NT>(d0.g, links_of<S>(d0), ld, site_ok ? it.s : 0, par, it.grp, acc);
  else zero_acc<NR>(acc);
  wave_combine<T, NR>(acc, it.slot, it.grp, lds);
  if (!any) return;
  const R a = (R)coef(amode, d0.kappa);
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    if (!act[r]) continue;
    const SysDesc &d = sdesc[it.sys + r];
    double v[NV] = {0.0, 0.0, 0.0};
    if (site_ok && it.grp == 0) hop_site<S>(d, acc[r], EPI, a, fx, fout, it.s, red, chio, chix, ont, v);
    if (red) sys_partial(d, slot, it, v);
  }
}

// The FP64 hops of the reliable update and the true residual: 4 waves per
// item, directions summed in LDS.
constexpr int T64 = 4;
using Lds64 = HopLds<T64, 1, double>;

// The `chunk` consecutive items of a work-group of k_hop_upd: calls
// each(item) for those whose system has an update pending.  Most iterations have
// none, and a work-group then only has to find that out: for 12 systems at
// 24^3x48, 62208 work-groups of one item of k_hop_upd took 42 us to come and go,
// 15552 of four take 15 (a system's items follow one another, so one look at its
// state serves the chunk).
template <class Each>
__device__ __forceinline__ void update_items(const SysDesc *sdesc, const uint32_t *work, int nwork, int chunk,
                                             Each each) {
  static_assert(WG / WAVE == T64, "one work item at a time");
  const int i0 = xcd_remap(blockIdx.x, gridDim.x) * chunk;
  int sys = -1;
  bool on = false;
#pragma unroll 1
  for (int i = i0; i < i0 + chunk && i < nwork; ++i) {
    const Item it = fetch_item_at<T64>(work, nwork, i);
    if (it.sys != sys) {
      sys = it.sys;
      on = sdesc[sys].st->status & ST_UPDATE;   // uniform
    }
    if (!on) continue;
    each(it);
    if (chunk > 1) __syncthreads();   // the next item overwrites the combine buffer
  }
}

// T64 = A^-1 H_eo (XH + X): the hop of the current solution for the FP64 residual.
// Two waves per SIMD: held to three its sums come a colour at a time and it runs
// 1006 instead of 870 us (12 systems at 24^3x48).  One item a work-group: those of a
// chunk wait for each other (870 -> 1000 us), as much as the idle launches save.
template <bool HASLO>
__global__ __launch_bounds__(WG, 2) void k_hop_sum(const SysDesc *__restrict__ sdesc,
                                                   const uint32_t *__restrict__ work, int nwork) {
  static_assert(WG / WAVE == T64, "one work item a work-group");
  __shared__ Lds64::V lds[Lds64::VECS];
  const Item it = fetch_item<T64>(work, nwork);
  const SysDesc &d = sdesc[it.sys];
  if (!it.active || !(d.st->status & ST_UPDATE)) return;   // uniform
  const bool site_ok = it.s < d.g.vh;
  cpx<double> acc[1][12];
  SumLd ld{d.f[F_XH], HASLO ? d.f[F_X] : nullptr, d.npad};
  hop_wave<L_F64R18, false, T64, false>(d.g, d.g64, ld, site_ok ? it.s : 0, 0, it.grp, acc);
  wave_combine<T64, 1>(acc, it.slot, it.grp, lds);
  if (site_ok && it.grp == 0) {
    apply_chi(acc[0], CHI_AINV, d.tmu);
    SpinorIO<S_F64>::store(d.f[F_T64], it.s, d.npad, acc[0]);
  }
}

// Reliable update on the odd sites (upd_site), with its sums.  Three waves per
// SIMD, which the epilogue allows by going a colour at a time: 1200 -> 1110 us for
// 12 systems at 24^3x48, k_hop_res 800 -> 715.  Items of two systems (links read
// once for both) were tried for the three and gained nothing: 890 to 1370 us.
template <int SO, bool HASLO, bool BICG>
__global__ __launch_bounds__(WG, 3) void k_hop_upd(const SysDesc *__restrict__ sdesc,
                                                   const uint32_t *__restrict__ work, int nwork, int chunk) {
  __shared__ Lds64::V lds[Lds64::VECS];
  update_items(sdesc, work, nwork, chunk, [&](const Item &it) {
    const SysDesc &d = sdesc[it.sys];
    const bool site_ok = it.s < d.g.vh;
    double v[NV] = {0.0, 0.0, 0.0};
    cpx<double> acc1[1][12];
    FieldLd<S_F64, 1> ld{{d.f[F_T64]}, d.npad};
    hop_wave<L_F64R18, false, T64, false>(d.g, d.g64, ld, site_ok ? it.s : 0, 1, it.grp, acc1);
    wave_combine<T64, 1>(acc1, it.slot, it.grp, lds);
    if (site_ok && it.grp == 0) upd_site<SO, HASLO, BICG>(d, d.st, acc1[0], it.s, v);
    sys_partial(d, SL_UPD, it, v);
  });
}

// ||b - D x||^2 on the sites of parity p: B_p - A X_p + kappa H X_{1-p}.
__global__ __launch_bounds__(WG, 3) void k_hop_res(const SysDesc *__restrict__ sdesc, const uint32_t *__restrict__ work,
                                                int nwork, int par) {
  __shared__ Lds64::V lds[Lds64::VECS];
  const Item it = fetch_item<T64>(work, nwork);
  const SysDesc &d = sdesc[it.sys];
  const int fin_id = par ? F_XE : F_XH;
  const bool site_ok = it.active && it.s < d.g.vh;
  double v[NV] = {0.0, 0.0, 0.0};
  cpx<double> acc1[1][12];
  FieldLd<S_F64, 1> ld{{d.f[fin_id]}, d.npad};
  if (it.active) hop_wave<L_F64R18, false, T64, false>(d.g, d.g64, ld, site_ok ? it.s : 0, par, it.grp, acc1);
  else zero_acc<1>(acc1);
  wave_combine<T64, 1>(acc1, it.slot, it.grp, lds);
  if (!it.active) return;
  if (site_ok && it.grp == 0) res_site(d, acc1[0], par, it.s, v);
  sys_partial(d, par ? SL_RES_O : SL_RES_E, it, v);
}

// Sum a system's partials of one reduction slot and run the solver's scalar
// step (one work-group of RED_WG threads per system), in the fixed order of
// red_part: the result does not depend on scheduling.
__global__ __launch_bounds__(RED_WG) void k_reduce(const SysDesc *__restrict__ sdesc, int slot, int fin,
                                                   int mask) {
  static_assert(sizeof(SysState) % 8 == 0 && sizeof(SysState) / 8 <= RED_WG, "state copy");
  constexpr int NW8 = (int)(sizeof(SysState) / 8);
  const SysDesc &d = sdesc[blockIdx.x];
  // The reliable-update reduction has nothing to do in most iterations: look at
  // the state first there (the other reductions almost always run).
  if (fin == FIN_UPDATE && !(d.st->status & mask)) return;   // uniform over the work-group
  // The system's state is copied to LDS while the partials load, so the scalar
  // step below does not wait for another round trip to memory; the whole state
  // is written back afterwards (no other kernel runs meanwhile).
  __shared__ SysState sst;
  const int tid = threadIdx.x, w = tid >> 6;
  if (tid < NW8) ((unsigned long long *)&sst)[tid] = ((const unsigned long long *)d.st)[tid];
  __shared__ double red[NV][RED_WG / WAVE];
  double sp[NV];
  red_part<NV>(part_row(d, slot, 0), (size_t)d.g.nb * 4, d.g.nb, tid, sp);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const double v = wave_sum(sp[i]);
    if (lane_id() == 0) red[i][w] = v;
  }
  __syncthreads();
  if (!(sst.status & mask)) return;   // uniform over the work-group
  if (tid == 0) {
    double t[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      double v = 0.0;
      for (int j = 0; j < RED_WG / WAVE; ++j) v += red[i][j];
      t[i] = v;
    }
    finalize(&sst, fin, slot, t);
  }
  __syncthreads();
  if (tid < NW8) ((unsigned long long *)d.st)[tid] = ((const unsigned long long *)&sst)[tid];
}

// The vector steps (solver_steps.h), one wave per 64-site block of a system
// whose status matches: SUM names the reduction slot of the step's sums, -1 for
// none.
#define QVECTOR_KERNEL(NAME, TEMPLATE, MASK, SUM, CALL)                                                              \
  TEMPLATE __global__ __launch_bounds__(WG) void NAME(const SysDesc *__restrict__ sdesc,                             \
                                                      const uint32_t *__restrict__ work, int nwork) {                \
    const Item it = fetch_item<1>(work, nwork);                                                                      \
    if (!it.active) return;                                                                                          \
    const SysDesc &d = sdesc[it.sys];                                                                                \
    if ((MASK) != ST_ANY && !(d.st->status & (MASK))) return;                                                        \
    double v[NV] = {0.0, 0.0, 0.0};                                                                                  \
    const int s = it.s;                                                                                              \
    if (s < d.g.vh) CALL;                                                                                            \
    if ((SUM) >= 0) sys_partial(d, SUM, it, v);                                                                      \
  }
#define QT(...) template <__VA_ARGS__>
QVECTOR_KERNEL(k_bnorm, , ST_ANY, SL_B, bnorm_site(d, s, v))
QVECTOR_KERNEL(k_cg1, QT(int S, int XS, int V), ST_RUN, SL_R, (cg1_site<S, XS, V>(d, d.st, s, v)))
QVECTOR_KERNEL(k_cg2, QT(int S, bool XUPD, int V), ST_RUN, -1, (cg2_site<S, XUPD, V>(d, d.st, s)))
QVECTOR_KERNEL(k_cg_xfin, , ST_DONE, -1, if (d.st->xpend) xfin_site(d, d.st, s))
QVECTOR_KERNEL(k_cr1, QT(int S), ST_RUN, SL_R, cr1_site<S>(d, d.st, s, v))
QVECTOR_KERNEL(k_cr2, QT(int S, bool INIT), ST_RUN, SL_AP, (cr2_site<S, INIT>(d, d.st, s, v)))
QVECTOR_KERNEL(k_bi_p, QT(int S, int V), ST_RUN, -1, (bi_p_site<S, V>(d, d.st, s)))
QVECTOR_KERNEL(k_bi_s, QT(int S, int V), ST_RUN, -1, (bi_s_site<S, V>(d, d.st, s)))
QVECTOR_KERNEL(k_bi_xr, QT(int S, int XS, int V), ST_RUN, SL_BI3, (bi_xr_site<S, XS, V>(d, d.st, s, v)))
#undef QT
#undef QVECTOR_KERNEL

// copy a half-field of the iterate precision: dst = src
template <int S>
__global__ __launch_bounds__(WG) void k_copy(const SysDesc *__restrict__ sdesc, const uint32_t *__restrict__ work,
                                             int nwork, int fsrc, int fdst, int mask, int chi) {
  const Item it = fetch_item<1>(work, nwork);
  if (!it.active) return;
  const SysDesc &d = sdesc[it.sys];
  if (!(d.st->status & mask) || it.s >= d.g.vh) return;
  copy_site<S>(d, fsrc, fdst, chi, it.s);
}

__global__ void k_bi_init(const SysDesc *__restrict__ sdesc, int nsys) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nsys && (sdesc[i].st->status & ST_RUN)) bi_start(sdesc[i].st);
}

// ---------------------------------------------------------------------------
// launchers
static inline dim3 grid_of(int nwork, int T = 1) { return dim3(grid_for(nwork, T)); }

template <int S, int L, int T, int NR, bool NT>
static void hop_sys_tt(const Launch &l, bool dag, int epi, int fi, int fo, int fx, int par, int amode, int mask,
                       int red, int slot) {
  const dim3 g = grid_of(l.nwork, T), b(WG);
#define QARGS l.desc, l.work, l.nwork, fi, fo, fx, par, amode, mask, red, slot, l.chio, l.chix, l.ont
  if (!dag) {
    if (epi == 0) hipLaunchKernelGGL((k_hop_sys<S, L, false, 0, T, NR, NT>), g, b, 0, l.stream, QARGS);
    else hipLaunchKernelGGL((k_hop_sys<S, L, false, 1, T, NR, NT>), g, b, 0, l.stream, QARGS);
  } else {
    if (epi == 0) hipLaunchKernelGGL((k_hop_sys<S, L, true, 0, T, NR, NT>), g, b, 0, l.stream, QARGS);
    else hipLaunchKernelGGL((k_hop_sys<S, L, true, 1, T, NR, NT>), g, b, 0, l.stream, QARGS);
  }
#undef QARGS
}

template <int S, int L, int T, int NR>
static void hop_sys_t(const Launch &l, bool dag, int epi, int fi, int fo, int fx, int par, int amode, int mask, int red,
                      int slot) {
  if (l.NT) hop_sys_tt<S, L, T, NR, true>(l, dag, epi, fi, fo, fx, par, amode, mask, red, slot);
  else hop_sys_tt<S, L, T, NR, false>(l, dag, epi, fi, fo, fx, par, amode, mask, red, slot);
}

template <int S, int L, int T>
static void hop_sys_n(const Launch &l, bool dag, int epi, int fi, int fo, int fx, int par, int amode, int mask, int red,
                      int slot) {
  // l.NR never exceeds hop_nr_max(S, T): the solver takes (T, NR) from hop_config.
  constexpr int NM = hop_nr_max(S, T);
  if constexpr (NM > 0) {
    if constexpr (NM >= 4) if (l.NR == 4) return hop_sys_t<S, L, T, 4>(l, dag, epi, fi, fo, fx, par, amode, mask, red, slot);
    if constexpr (NM >= 3) if (l.NR == 3) return hop_sys_t<S, L, T, 3>(l, dag, epi, fi, fo, fx, par, amode, mask, red, slot);
    if constexpr (NM >= 2) if (l.NR == 2) return hop_sys_t<S, L, T, 2>(l, dag, epi, fi, fo, fx, par, amode, mask, red, slot);
    hop_sys_t<S, L, T, 1>(l, dag, epi, fi, fo, fx, par, amode, mask, red, slot);
  }
}

template <int S, int L>
static void hop_sys_p(const Launch &l, bool dag, int epi, int fi, int fo, int fx, int par, int amode, int mask, int red,
                      int slot) {
  if constexpr (S == S_F64) hop_sys_n<S, L, 4>(l, dag, epi, fi, fo, fx, par, amode, mask, red, slot);
  else if (l.T == 4) hop_sys_n<S, L, 4>(l, dag, epi, fi, fo, fx, par, amode, mask, red, slot);
  else hop_sys_n<S, L, 2>(l, dag, epi, fi, fo, fx, par, amode, mask, red, slot);
}

void reduce(const Launch &l, int slot, int fin, int mask) {
  hipLaunchKernelGGL(k_reduce, dim3(l.nsys), dim3(RED_WG), 0, l.stream, l.desc, slot, fin, mask);
}

void hop_sys(const Launch &l, int prec, bool dag, int epi, int fi, int fo, int fx, int par, int amode, int mask,
             int red, int slot, int fin, int chio, int chix) {
  // the iterate-precision hop walks the grouped table; an FP64 hop of a mixed
  // solve (source, reconstruction) walks the plain one
  const bool grouped = (prec == S_F64) == (l.prec == S_F64);
  Launch lp = l;
  lp.chio = chio;
  lp.chix = chix;
  if (grouped) { lp.work = l.work_hop; lp.nwork = l.nwork_hop; lp.T = l.T; lp.NR = l.NR; lp.NT = l.NT; }
  else { lp.T = 4; lp.NR = 1; lp.NT = l.NT64; lp.ont = l.ont64; }
  if (prec == S_F64) hop_sys_p<S_F64, L_F64R18>(lp, dag, epi, fi, fo, fx, par, amode, mask, red, slot);
  else if (prec == S_F32) hop_sys_p<S_F32, L_F32R12>(lp, dag, epi, fi, fo, fx, par, amode, mask, red, slot);
  else hop_sys_p<S_F16S, L_F16R12>(lp, dag, epi, fi, fo, fx, par, amode, mask, red, slot);
  if (red) reduce(l, slot, fin, mask);
}

// Items per work-group of k_hop_upd: four while there are many times more than
// the card holds, one where each should have its own (8^4 in FP32 with four: 3%
// slower).
static int upd_chunk(const Launch &l) { return l.nwork >= 8192 ? 4 : 1; }

void hop_sum(const Launch &l, bool haslo) {
  const dim3 g = grid_of(l.nwork, T64), b(WG);
  if (haslo) hipLaunchKernelGGL((k_hop_sum<true>), g, b, 0, l.stream, l.desc, l.work, l.nwork);
  else hipLaunchKernelGGL((k_hop_sum<false>), g, b, 0, l.stream, l.desc, l.work, l.nwork);
}

void hop_upd(const Launch &l, int prec, bool bicg) {
  const int c = upd_chunk(l);
  const dim3 g((l.nwork + c - 1) / c), b(WG);
#define QU(SO, LO, BI) \
  hipLaunchKernelGGL((k_hop_upd<SO, LO, BI>), g, b, 0, l.stream, l.desc, l.work, l.nwork, c)
  if (prec == S_F64) { if (bicg) QU(S_F64, false, true); else QU(S_F64, false, false); }
  else if (prec == S_F32) { if (bicg) QU(S_F32, true, true); else QU(S_F32, true, false); }
  else { if (bicg) QU(S_F16S, true, true); else QU(S_F16S, true, false); }
#undef QU
  reduce(l, SL_UPD, FIN_UPDATE, ST_UPDATE);
}

void hop_res(const Launch &l, int par) {
  const dim3 g = grid_of(l.nwork, T64), b(WG);
  hipLaunchKernelGGL(k_hop_res, g, b, 0, l.stream, l.desc, l.work, l.nwork, par);
  reduce(l, par ? SL_RES_O : SL_RES_E, FIN_NONE, ST_ANY);
}

void bnorm(const Launch &l) {
  hipLaunchKernelGGL(k_bnorm, grid_of(l.nwork), dim3(WG), 0, l.stream, l.desc, l.work, l.nwork);
  reduce(l, SL_B, FIN_BNORM, ST_ANY);
}

// A vector kernel in the form of the launch's streaming level (vec_stream).
#define QVEC(KERNEL0, KERNEL1, KERNEL2)                                                                \
  hipLaunchKernelGGL(l.vec == 0 ? (KERNEL0) : l.vec == 1 ? (KERNEL1) : (KERNEL2), grid_of(l.nwork), dim3(WG), 0, \
                     l.stream, l.desc, l.work, l.nwork)

void cg1(const Launch &l, int prec) {
  if (prec == S_F64) QVEC((k_cg1<S_F64, S_F64, 0>), (k_cg1<S_F64, S_F64, 1>), (k_cg1<S_F64, S_F64, 2>));
  else if (prec == S_F32) QVEC((k_cg1<S_F32, S_F32, 0>), (k_cg1<S_F32, S_F32, 1>), (k_cg1<S_F32, S_F32, 2>));
  else QVEC((k_cg1<S_F16S, S_F32, 0>), (k_cg1<S_F16S, S_F32, 1>), (k_cg1<S_F16S, S_F32, 2>));
  reduce(l, SL_R, FIN_NR, ST_RUN);
}

void cg2(const Launch &l, int prec, bool xupd) {
  if (prec == S_F64) {
    if (xupd) QVEC((k_cg2<S_F64, true, 0>), (k_cg2<S_F64, true, 1>), (k_cg2<S_F64, true, 2>));
    else QVEC((k_cg2<S_F64, false, 0>), (k_cg2<S_F64, false, 1>), (k_cg2<S_F64, false, 2>));
  } else if (prec == S_F32) QVEC((k_cg2<S_F32, false, 0>), (k_cg2<S_F32, false, 1>), (k_cg2<S_F32, false, 2>));
  else QVEC((k_cg2<S_F16S, false, 0>), (k_cg2<S_F16S, false, 1>), (k_cg2<S_F16S, false, 2>));
}

void cg_xfin(const Launch &l) {
  hipLaunchKernelGGL(k_cg_xfin, grid_of(l.nwork), dim3(WG), 0, l.stream, l.desc, l.work, l.nwork);
}

void cr1(const Launch &l) {
  hipLaunchKernelGGL(k_cr1<S_F64>, grid_of(l.nwork), dim3(WG), 0, l.stream, l.desc, l.work, l.nwork);
  reduce(l, SL_R, FIN_NR, ST_RUN);
}

void cr2(const Launch &l, bool init) {
  if (init) hipLaunchKernelGGL((k_cr2<S_F64, true>), grid_of(l.nwork), dim3(WG), 0, l.stream, l.desc, l.work, l.nwork);
  else hipLaunchKernelGGL((k_cr2<S_F64, false>), grid_of(l.nwork), dim3(WG), 0, l.stream, l.desc, l.work, l.nwork);
  reduce(l, SL_AP, FIN_CR_ALPHA, ST_RUN);
}

void bi_p(const Launch &l, int prec) {
  if (prec == S_F64) QVEC((k_bi_p<S_F64, 0>), (k_bi_p<S_F64, 1>), (k_bi_p<S_F64, 2>));
  else if (prec == S_F32) QVEC((k_bi_p<S_F32, 0>), (k_bi_p<S_F32, 1>), (k_bi_p<S_F32, 2>));
  else QVEC((k_bi_p<S_F16S, 0>), (k_bi_p<S_F16S, 1>), (k_bi_p<S_F16S, 2>));
}

void bi_s(const Launch &l, int prec) {
  if (prec == S_F64) QVEC((k_bi_s<S_F64, 0>), (k_bi_s<S_F64, 1>), (k_bi_s<S_F64, 2>));
  else if (prec == S_F32) QVEC((k_bi_s<S_F32, 0>), (k_bi_s<S_F32, 1>), (k_bi_s<S_F32, 2>));
  else QVEC((k_bi_s<S_F16S, 0>), (k_bi_s<S_F16S, 1>), (k_bi_s<S_F16S, 2>));
}

void bi_xr(const Launch &l, int prec) {
  if (prec == S_F64) QVEC((k_bi_xr<S_F64, S_F64, 0>), (k_bi_xr<S_F64, S_F64, 1>), (k_bi_xr<S_F64, S_F64, 2>));
  else if (prec == S_F32) QVEC((k_bi_xr<S_F32, S_F32, 0>), (k_bi_xr<S_F32, S_F32, 1>), (k_bi_xr<S_F32, S_F32, 2>));
  else QVEC((k_bi_xr<S_F16S, S_F32, 0>), (k_bi_xr<S_F16S, S_F32, 1>), (k_bi_xr<S_F16S, S_F32, 2>));
  reduce(l, SL_BI3, FIN_BI_RHO, ST_RUN);
}
#undef QVEC

void copy_field(const Launch &l, int prec, int fsrc, int fdst, int mask, int chi) {
  const dim3 g = grid_of(l.nwork), b(WG);
  if (prec == S_F64) hipLaunchKernelGGL(k_copy<S_F64>, g, b, 0, l.stream, l.desc, l.work, l.nwork, fsrc, fdst, mask, chi);
  else if (prec == S_F32) hipLaunchKernelGGL(k_copy<S_F32>, g, b, 0, l.stream, l.desc, l.work, l.nwork, fsrc, fdst, mask, chi);
  else hipLaunchKernelGGL(k_copy<S_F16S>, g, b, 0, l.stream, l.desc, l.work, l.nwork, fsrc, fdst, mask, chi);
}

void bi_init(const Launch &l, int nsys) {
  hipLaunchKernelGGL(k_bi_init, dim3((nsys + 63) / 64), dim3(64), 0, l.stream, l.desc, nsys);
}

}  // namespace qiral
