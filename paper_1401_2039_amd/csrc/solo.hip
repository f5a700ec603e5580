// The even-odd solvers on small lattices: one work-group solves one system from
// the canonical source to the canonical solution in one launch.
//
// On a lattice of a few 64-site blocks every launch of the grouped solver is
// latency: nine kernels of 4 to 6 us an iteration, each starting with the chain
// work table, system table, state, data. Here the steps of the same sequence
// (solver_steps.h) follow one another inside a work-group of eight waves, with a
// barrier where the grouped solver has a kernel boundary; the state and the
// system's description lie in LDS, the fields stay in the compute unit's cache.
// The sums are taken in the grouped solver's order, so the iterates are the same
// bit for bit in FP64 (in the reduced precisions up to the hop's wave split).
// What bounds it is the chain of one compute unit: loads, about 500 FP64
// instructions a wave, the combine in LDS and a store's acknowledgement in each
// of the four hops of an iteration.  See solo_line for the times of both and where
// it pays.
#include "qiral_int.h"
#include "solver_steps.h"
#include "solo.h"

namespace qiral {

namespace {

constexpr int SW = 8;          // waves of the work-group: two hop items at a time, four waves each
constexpr int MAX_RUN = 256;   // iterations per launch

struct Solo {
  SysDesc d;
  SysState st;
  double part[NV][SOLO_BLOCKS];   // a step's sums, one per 64-site block
};

// Four waves' partial sums of a hop item, two items (wave_combine).
constexpr int LDS_VECS = 2 * HopLds<4, 1, double>::VECS;

__device__ __forceinline__ void put_part(Solo &so, int sb, double v[NV]) {
#pragma unroll
  for (int i = 0; i < NV; ++i) v[i] = wave_sum(v[i]);
  if (lane_id() == 0)
#pragma unroll
    for (int i = 0; i < NV; ++i) so.part[i][sb] = v[i];
}

// The scalar step on the sums of `part`, in k_reduce's order (its first wave).
__device__ __forceinline__ void solo_reduce(Solo &so, int slot, int fin, int w) {
  static_assert(SOLO_BLOCKS <= 128 && SOLO_BLOCKS % 2 == 0, "one wave's pairs");
  __syncthreads();
  if (w == 0) {
    double sp[NV], t[NV];
    red_part<NV>(so.part[0], SOLO_BLOCKS, so.d.g.nb, lane_id(), sp);
#pragma unroll
    for (int i = 0; i < NV; ++i) t[i] = 0.0 + wave_sum(sp[i]);
    if (lane_id() == 0) finalize(&so.st, fin, slot, t);
  }
}

// One hop over every block: EACH(acc, s, v) is the epilogue at a site.
template <int L, bool BOTH, class Ld, class Each>
__device__ __forceinline__ void solo_hop(Solo &so, const void *links, const Ld &ld, int par, bool dag, bool sum, int w,
                                         typename Vec16<typename Ld::R>::T *lds, Each each) {
  using R = typename Ld::R;
  const int slot = w >> 2, grp = w & 3;
#pragma unroll 1
  for (int b0 = 0; b0 < so.d.g.nb; b0 += 2) {
    const int sb = b0 + slot, s = sb * WAVE + lane_id();
    const bool act = sb < so.d.g.nb, site_ok = act && s < so.d.g.vh;
    cpx<R> acc[1][12];
    if (!act) zero_acc<1>(acc);
    else if (BOTH && dag) hop_wave<L, true, 4, false>(so.d.g, links, ld, site_ok ? s : 0, par, grp, acc);
    else hop_wave<L, false, 4, false>(so.d.g, links, ld, site_ok ? s : 0, par, grp, acc);
    wave_combine<4, 1>(acc, slot, grp, lds);
    if (act && grp == 0) {
      double v[NV] = {0.0, 0.0, 0.0};
      if (site_ok) each(acc[0], s, v);
      if (sum) put_part(so, sb, v);
    }
    __syncthreads();   // the next two items overwrite the combine buffer
  }
}

// A vector step over every block of the half-field.
template <class Each> __device__ __forceinline__ void solo_vec(Solo &so, bool sum, int w, Each each) {
#pragma unroll 1
  for (int sb = w; sb < so.d.g.nb; sb += SW) {
    const int s = sb * WAVE + lane_id();
    double v[NV] = {0.0, 0.0, 0.0};
    if (s < so.d.g.vh) each(s, v);
    if (sum) put_part(so, sb, v);
  }
}

// Canonical site index of checkerboard site s of parity p.
__device__ __forceinline__ size_t canon_site(const Geo &g, int s, int p) {
  const SiteC c = site_c(g, s, p);
  return (((size_t)c.t * g.lz + c.z) * g.ly + c.y) * g.lx + c.x;
}

// The steps of a solve, from the template chain's own sequence (solver.hip's
// run_solve enqueues the same as launches).
constexpr SoloProg solo_program(int solver, int prec, bool twisted, bool guess) {
  SoloProg p{};
  int n = 0;
  auto add = [&](int kind, int mask) -> SoloStep & {
    SoloStep &q = p.step[n++];
    q.kind = (int8_t)kind;
    q.mask = (int8_t)mask;
    q.fin_red = -1;
    return q;
  };
  auto sums = [&](SoloStep &q, int slot, int fin) {
    q.slot = (int8_t)slot;
    q.fin_red = (int8_t)fin;
  };
  auto hop = [&](int f64, bool dag, int epi, int fi, int fo, int fx, int par, int amode, int mask, int red, int slot,
                 int fin, int chio = CHI_ONE, int chix = CHI_ONE) {
    SoloStep &q = add(SK_HOP, mask);
    q.f64 = (int8_t)f64; q.dag = dag; q.epi = (int8_t)epi; q.fin = (int8_t)fi; q.fout = (int8_t)fo; q.fx = (int8_t)fx;
    q.par = (int8_t)par; q.amode = (int8_t)amode; q.red = (int8_t)red; q.chio = (int8_t)chio; q.chix = (int8_t)chix;
    if (red) sums(q, slot, fin);
  };
  auto zero = [&](int field, int prec_) {
    SoloStep &q = add(SK_ZERO, ST_ANY);
    q.fout = (int8_t)field;
    q.f64 = (int8_t)prec_;
  };
  auto import = [&](bool x) {
    SoloStep &q = add(SK_IMPORT, ST_ANY);
    q.par = x;
    q.fin = x ? F_XE : F_BE;
    q.fout = x ? F_XH : F_BO;
  };
  const bool mixed = prec != QIRAL_F64, bicg = solver == QIRAL_BICGSTAB_EO, cr = solver == QIRAL_CRNR_EO;
  auto schur = [&](bool dag, int fi, int fo, int red, int slot, int fin) {   // fo = S fi or S^dagger fi, through TMP
    hop(!mixed, dag, 0, fi, F_TMP, 0, 0, A_ONE, ST_RUN, 0, 0, FIN_NONE, dag ? CHI_AINVDAG : CHI_AINV);
    hop(!mixed, dag, 1, F_TMP, fo, fi, 1, A_MKAPPA2, ST_RUN, red, slot, fin, CHI_ONE, dag ? CHI_ADAG : CHI_A);
  };
  auto update = [&]() {
    SoloStep &q = add(SK_SUM, ST_UPDATE);
    q.fin = F_XH;
    SoloStep &u = add(SK_UPD, ST_UPDATE);
    u.fin = F_T64;
    u.par = 1;
    sums(u, SL_UPD, FIN_UPDATE);
  };
  auto cr_apply = [&](int fin) {
    schur(false, F_Z, F_RT, 0, 0, FIN_NONE);
    schur(true, F_RT, F_W, 4, SL_Z, fin);
  };
  auto cr2 = [&](bool init) {
    SoloStep &q = add(SK_CR2, ST_RUN);
    q.par = init;
    sums(q, SL_AP, FIN_CR_ALPHA);
  };
  // the source
  import(false);
  if (guess) import(true);
  else zero(F_XH, S_F64);
  if (mixed) zero(F_X, S_F32);
  zero(F_P, prec);
  zero(F_AP, prec);
  sums(add(SK_BNORM, ST_ANY), SL_B, FIN_BNORM);
  if (twisted) {
    SoloStep &q = add(SK_COPY, ST_ANY);
    q.f64 = 1; q.fin = F_BE; q.fout = F_T64; q.chio = CHI_AINV;
  }
  hop(1, false, 1, twisted ? F_T64 : F_BE, F_BH, F_BO, 1, A_KAPPA, ST_ANY, 0, 0, FIN_NONE);
  // the start of the iterations
  p.start = n;
  update();
  if (cr) {
    schur(true, F_R, F_Z, 0, 0, FIN_NONE);
    cr_apply(FIN_CR_ZW);
    cr2(true);
  } else if (bicg) {
    SoloStep &q = add(SK_COPY, ST_RUN);
    q.fin = F_R; q.fout = F_RT; q.f64 = !mixed;
    add(SK_BIINIT, ST_RUN);
  } else {
    schur(true, F_R, F_Z, 1, SL_Z, FIN_NZ_INIT);
    add(SK_CG2, ST_RUN);
  }
  // an iteration
  p.iter = n;
  if (cr) {
    sums(add(SK_CR1, ST_RUN), SL_R, FIN_NR);
    cr_apply(FIN_CR_BETA);
    cr2(false);
  } else if (bicg) {
    add(SK_BIP, ST_RUN);
    schur(false, F_P, F_AP, 2, SL_BI1, FIN_BI_ALPHA);
    add(SK_BIS, ST_RUN);
    schur(false, F_Z, F_T, 3, SL_BI2, FIN_BI_OMEGA);
    sums(add(SK_BIXR, ST_RUN), SL_BI3, FIN_BI_RHO);
    if (mixed) update();
  } else {
    schur(false, F_P, F_AP, 1, SL_AP, FIN_ALPHA);
    sums(add(SK_CG1, ST_RUN), SL_R, FIN_NR);
    if (mixed) update();
    schur(true, F_R, F_Z, 1, SL_Z, FIN_BETA);
    add(SK_CG2, ST_RUN).par = !mixed;
  }
  // x_e, the true residual, the solution
  p.post = n;
  if (!mixed && !bicg && !cr) add(SK_XFIN, ST_DONE);
  hop(1, false, 1, F_XH, F_XE, F_BE, 0, A_KAPPA, ST_ANY, 0, 0, FIN_NONE, CHI_AINV);
  for (int par = 0; par < 2; ++par) {
    SoloStep &q = add(SK_RES, ST_ANY);
    q.fin = par ? F_XE : F_XH;
    q.par = (int8_t)par;
    sums(q, par ? SL_RES_O : SL_RES_E, FIN_NONE);
  }
  SoloStep &q = add(SK_EXPORT, ST_ANY);
  q.fin = F_XE;
  q.fout = F_XH;
  p.end = n;
  return p;
}

// Every program: [solver][precision][twisted][guess], solvers in the order of SOLO_SOLVER.
constexpr int SOLO_SOLVER[3] = {QIRAL_CGNR_EO, QIRAL_BICGSTAB_EO, QIRAL_CRNR_EO};
struct SoloProgs { SoloProg p[3 * 3 * 2 * 2]; };
constexpr SoloProgs solo_programs() {
  SoloProgs t{};
  for (int i = 0; i < 36; ++i) t.p[i] = solo_program(SOLO_SOLVER[i / 12], i / 4 % 3, i & 2, i & 1);
  return t;
}
__constant__ SoloProgs solo_table = solo_programs();

template <int S> __global__ __launch_bounds__(SW *WAVE, 2) void k_solo(const SysDesc *__restrict__ sdesc, int id,
                                                                       int mode) {
  const SoloProg &prog = solo_table.p[id];
  using R = typename SpinorIO<S>::R;
  constexpr bool MIXED = S != S_F64;
  constexpr int XS = MIXED ? S_F32 : S_F64;
  constexpr int L = S == S_F64 ? L_F64R18 : S == S_F32 ? L_F32R12 : L_F16R12;
  __shared__ Solo so;
  __shared__ double2 lds[LDS_VECS];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const SysDesc *dg = sdesc + blockIdx.x;
  static_assert(sizeof(SysDesc) % 8 == 0 && sizeof(SysState) % 8 == 0, "copies");
  for (int i = threadIdx.x; i < (int)(sizeof(SysDesc) / 8); i += SW * WAVE)
    ((unsigned long long *)&so.d)[i] = ((const unsigned long long *)dg)[i];
  for (int i = threadIdx.x; i < (int)(sizeof(SysState) / 8); i += SW * WAVE)
    ((unsigned long long *)&so.st)[i] = ((const unsigned long long *)dg->st)[i];
  __syncthreads();
  // done in an earlier launch, its end steps with it: they must not run again (the
  // last x += alpha p would be added twice)
  if (mode != SOLO_NEW && (so.st.status & ST_DONE)) return;

  auto run = [&](const SoloStep &q) {
    if (!(so.st.status & q.mask)) return;   // uniform: the state changes between barriers only
    switch (q.kind) {
      case SK_HOP: {
        const double a = coef(q.amode, so.d.kappa);
        if (MIXED && !q.f64) {
          if constexpr (MIXED) {
            FieldLd<S, 1, true> ld{{so.d.f[q.fin]}, so.d.npad};
            solo_hop<L, true>(so, so.d.glo, ld, q.par, q.dag, q.red, w, (typename Vec16<R>::T *)lds,
                              [&](cpx<R> *acc, int s, double v[NV]) {
                                hop_site<S>(so.d, acc, q.epi, (R)a, q.fx, q.fout, s, q.red, q.chio, q.chix, 0, v);
                              });
          }
        } else {
          FieldLd<S_F64, 1, true> ld{{so.d.f[q.fin]}, so.d.npad};
          solo_hop<L_F64R18, !MIXED>(so, so.d.g64, ld, q.par, q.dag, q.red, w, lds,
                                     [&](cpx<double> *acc, int s, double v[NV]) {
                                       hop_site<S_F64>(so.d, acc, q.epi, a, q.fx, q.fout, s, q.red, q.chio, q.chix, 0, v);
                                     });
        }
        break;
      }
      case SK_SUM:   // T64 = A^-1 H_eo (XH + X)
      case SK_UPD:   // the reliable update
      case SK_RES: { // ||b - D x||^2 on one parity
        SumLd ld{so.d.f[q.fin], MIXED && q.kind == SK_SUM ? so.d.f[F_X] : nullptr, so.d.npad};
        solo_hop<L_F64R18, false>(so, so.d.g64, ld, q.par, false, q.kind != SK_SUM, w, lds,
                                  [&](cpx<double> *acc, int s, double v[NV]) {
                                    if (q.kind == SK_SUM) {
                                      apply_chi(acc, CHI_AINV, so.d.tmu);
                                      SpinorIO<S_F64>::store(so.d.f[F_T64], s, so.d.npad, acc);
                                    } else if (q.kind == SK_RES) {
                                      res_site(so.d, acc, q.par, s, v);
                                    } else if (so.st.solver == SOLVER_BICG) {
                                      upd_site<S, MIXED, true>(so.d, &so.st, acc, s, v);
                                    } else {
                                      upd_site<S, MIXED, false>(so.d, &so.st, acc, s, v);
                                    }
                                  });
        break;
      }
      case SK_BNORM: solo_vec(so, true, w, [&](int s, double v[NV]) { bnorm_site(so.d, s, v); }); break;
      case SK_CG1: solo_vec(so, true, w, [&](int s, double v[NV]) { cg1_site<S, XS, 0>(so.d, &so.st, s, v); }); break;
      case SK_CG2:
        if (!MIXED && q.par) solo_vec(so, false, w, [&](int s, double *) { cg2_site<S, true, 0>(so.d, &so.st, s); });
        else solo_vec(so, false, w, [&](int s, double *) { cg2_site<S, false, 0>(so.d, &so.st, s); });
        break;
      case SK_XFIN:
        if (so.st.xpend) solo_vec(so, false, w, [&](int s, double *) { xfin_site(so.d, &so.st, s); });
        break;
      case SK_CR1:
        if constexpr (!MIXED) solo_vec(so, true, w, [&](int s, double v[NV]) { cr1_site<S>(so.d, &so.st, s, v); });
        break;
      case SK_CR2:
        if constexpr (!MIXED) {
          if (q.par) solo_vec(so, true, w, [&](int s, double v[NV]) { cr2_site<S, true>(so.d, &so.st, s, v); });
          else solo_vec(so, true, w, [&](int s, double v[NV]) { cr2_site<S, false>(so.d, &so.st, s, v); });
        }
        break;
      case SK_BIP: solo_vec(so, false, w, [&](int s, double *) { bi_p_site<S, 0>(so.d, &so.st, s); }); break;
      case SK_BIS: solo_vec(so, false, w, [&](int s, double *) { bi_s_site<S, 0>(so.d, &so.st, s); }); break;
      case SK_BIXR:
        solo_vec(so, true, w, [&](int s, double v[NV]) { bi_xr_site<S, XS, 0, !MIXED>(so.d, &so.st, s, v); });
        break;
      case SK_COPY:
        if (q.f64) solo_vec(so, false, w, [&](int s, double *) { copy_site<S_F64>(so.d, q.fin, q.fout, q.chio, s); });
        else solo_vec(so, false, w, [&](int s, double *) { copy_site<S>(so.d, q.fin, q.fout, q.chio, s); });
        break;
      case SK_BIINIT:
        if (threadIdx.x == 0) bi_start(&so.st);
        break;
      case SK_IMPORT:   // both parities of b or x, FP64; padding sites are zero
      case SK_EXPORT:
#pragma unroll 1
        for (int i = w; i < 2 * so.d.g.nb; i += SW) {
          const int p = i & 1, s = (i >> 1) * WAVE + lane_id();
          void *f = so.d.f[p ? q.fout : q.fin];
          const bool ok = s < so.d.g.vh;
          const size_t at = ok ? canon_site(so.d.g, s, p) * 12 : 0;
          cpx<double> v[12];
          if (q.kind == SK_IMPORT) {
            const double2 *src = (const double2 *)(q.par ? so.d.x : so.d.b) + at;
#pragma unroll
            for (int k = 0; k < 12; ++k) v[k] = ok ? cmake(src[k].x, src[k].y) : cmake(0.0, 0.0);
            SpinorIO<S_F64>::store(f, s, so.d.npad, v);
          } else if (ok) {
            SpinorIO<S_F64>::load(f, s, so.d.npad, v);
#pragma unroll
            for (int k = 0; k < 12; ++k) ((double2 *)so.d.x)[at + k] = make_double2(v[k].re, v[k].im);
          }
        }
        break;
      case SK_ZERO: {
        const size_t n = so.d.npad * (q.f64 == S_F64 ? SpinorIO<S_F64>::SITE_BYTES
                                      : q.f64 == S_F32 ? SpinorIO<S_F32>::SITE_BYTES : SpinorIO<S_F16S>::SITE_BYTES);
        for (size_t i = threadIdx.x; i < n / 16; i += SW * WAVE) ((uint4 *)so.d.f[q.fout])[i] = make_uint4(0, 0, 0, 0);
        break;
      }
      default: break;
    }
    if (q.fin_red >= 0) solo_reduce(so, q.slot, q.fin_red, w);
    __syncthreads();
  };

  // One place that runs a step: with several the body becomes a function, and its
  // call a stack, for which the runtime would allocate device memory.
#pragma unroll 1
  for (int i = mode == SOLO_NEW ? 0 : mode == SOLO_RESTART ? prog.start : prog.iter, k = 0; i < prog.end;) {
    if (i >= prog.iter && i < prog.post) {   // in the iterations: to the end once done
      if (so.st.status & ST_DONE) i = prog.post;
      else if (k == MAX_RUN) break;
    }
    run(prog.step[i]);
    if (++i == prog.post) { i = prog.iter; ++k; }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < (int)(sizeof(SysState) / 8); i += SW * WAVE)
    ((unsigned long long *)so.d.st)[i] = ((const unsigned long long *)&so.st)[i];
}

}  // namespace

hipError_t solo_launch(const SysDesc *desc, int nsys, int solver, int prec, bool twisted, bool guess, int mode,
                       hipStream_t s) {
  const int so = solver == QIRAL_BICGSTAB_EO ? 1 : solver == QIRAL_CRNR_EO ? 2 : 0;
  const int id = ((so * 3 + prec) * 2 + twisted) * 2 + guess;
  const dim3 g(nsys), b(SW * WAVE);
  if (prec == QIRAL_F64) hipLaunchKernelGGL(k_solo<S_F64>, g, b, 0, s, desc, id, mode);
  else if (prec == QIRAL_F32) hipLaunchKernelGGL(k_solo<S_F32>, g, b, 0, s, desc, id, mode);
  else hipLaunchKernelGGL(k_solo<S_F16S>, g, b, 0, s, desc, id, mode);
  return hipGetLastError();
}

}  // namespace qiral
