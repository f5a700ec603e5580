// C ABI of the library: argument validation, lattice handles, packing of links
// and fields, the hopping-term and operator entry points.
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdio>
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <string>

#include "qiral_int.h"

using namespace qiral;

// ---------------------------------------------------------------------------
// errors
namespace qiral {
static thread_local std::string g_last_error;
void set_error(const std::string &msg) { g_last_error = msg; }
qiral_status hip_fail(hipError_t e, const char *what) {
  set_error(std::string(what) + ": " + hipGetErrorString(e));
  return QIRAL_ERR_HIP;
}
}  // namespace qiral

extern "C" const char *qiral_last_error(void) { return g_last_error.c_str(); }

extern "C" const char *qiral_status_string(qiral_status s) {
  switch (s) {
    case QIRAL_OK: return "ok";
    case QIRAL_ERR_INVALID_ARG: return "invalid argument";
    case QIRAL_ERR_BAD_DIMS: return "bad lattice dimensions";
    case QIRAL_ERR_UNSUPPORTED: return "unsupported";
    case QIRAL_ERR_HIP: return "HIP runtime error";
    case QIRAL_ERR_NOT_CONVERGED: return "not converged";
    case QIRAL_ERR_NONFINITE: return "non-finite value";
    case QIRAL_ERR_WORKSPACE: return "workspace allocation failed";
  }
  return "unknown status";
}

static qiral_status fail(qiral_status s, const char *msg) {
  set_error(msg);
  return s;
}

static qiral_status check_dims(const int32_t *d) {
  if (!d) return fail(QIRAL_ERR_INVALID_ARG, "dims is NULL");
  int64_t v = 1;
  for (int i = 0; i < 4; ++i) {
    if (d[i] < 2 || (d[i] & 1)) return fail(QIRAL_ERR_BAD_DIMS, "every lattice extent must be even and >= 2");
    v *= d[i];
  }
  if (v / 2 > (1ll << 30)) return fail(QIRAL_ERR_BAD_DIMS, "lattice too large (more than 2^30 sites per parity)");
  return QIRAL_OK;
}

static bool valid_prec(int p) { return p == QIRAL_F64 || p == QIRAL_F32 || p == QIRAL_F16S; }

namespace qiral {
static size_t site_bytes(int prec) {
  return prec == QIRAL_F64 ? SpinorIO<S_F64>::SITE_BYTES
       : prec == QIRAL_F32 ? SpinorIO<S_F32>::SITE_BYTES : SpinorIO<S_F16S>::SITE_BYTES;
}
size_t half_bytes(const Geo &g, int prec) { return npad_of(g) * site_bytes(prec); }
const void *links_for(const qiral_lattice *lat, int prec) {
  return prec == QIRAL_F64 ? lat->g64 : prec == QIRAL_F32 ? lat->g32 : lat->g16;
}
size_t link_store_bytes(const Geo &g, int prec) {
  const size_t link = prec == QIRAL_F64 ? LinkIO<L_F64R18>::LINK_BYTES
                    : prec == QIRAL_F32 ? LinkIO<L_F32R12>::LINK_BYTES
                    : prec == QIRAL_F16S ? LinkIO<L_F16R12>::LINK_BYTES : 0;
  return 8 * npad_of(g) * link;   // 4 forward links per site of each parity
}
}  // namespace qiral

extern "C" size_t qiral_gauge_bytes(const int32_t dims[4], qiral_prec prec, qiral_recon recon) {
  if (check_dims(dims) != QIRAL_OK || !valid_prec(prec)) return 0;
  if ((prec == QIRAL_F64) != (recon == QIRAL_RECON18)) return 0;   // F64: 18 reals; F32, F16: 12
  if (recon != QIRAL_RECON18 && recon != QIRAL_RECON12) return 0;
  return link_store_bytes(make_geo(dims), prec);
}

extern "C" size_t qiral_field_bytes(const int32_t dims[4], qiral_subset subset, qiral_prec prec, int32_t nrhs) {
  if (check_dims(dims) != QIRAL_OK || !valid_prec(prec) || nrhs < 1) return 0;
  if (subset != QIRAL_EVEN && subset != QIRAL_ODD && subset != QIRAL_FULL) return 0;
  Geo g = make_geo(dims);
  size_t h = half_bytes(g, prec);
  return (subset == QIRAL_FULL ? 2 * h : h) * (size_t)nrhs;
}

// ---------------------------------------------------------------------------
// kernels: packing
__device__ __forceinline__ void site_coords(const Geo &g, int s, int p, int &x, int &y, int &z, int &t) {
  int xh = s % g.lxh;
  int r = s / g.lxh;
  y = r % g.ly; r /= g.ly;
  z = r % g.lz;
  t = r / g.lz;
  x = 2 * xh + ((p + y + z + t) & 1);
}

__device__ __forceinline__ size_t lex_of(const Geo &g, int x, int y, int z, int t) {
  return (((size_t)t * g.lz + z) * g.ly + y) * g.lx + x;
}

template <int L>
__global__ __launch_bounds__(WG) void k_pack_gauge(Geo g, const double *__restrict__ canon, void *__restrict__ dst) {
  const size_t npad = (size_t)g.nb * WAVE;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= 8 * npad) return;
  const int s = (int)(i % npad);
  const int pm = (int)(i / npad);   // parity * 4 + mu
  const int p = pm >> 2, mu = pm & 3;
  if (s >= g.vh) return;
  int x, y, z, t;
  site_coords(g, s, p, x, y, z, t);
  const double *src = canon + (lex_of(g, x, y, z, t) * 4 + mu) * 18;
  const size_t blk = (size_t)pm * g.nb + (s >> 6);
  if (L == L_F64R18) {
    double2 *d = (double2 *)dst + blk * 9 * WAVE + (s & 63);
    for (int j = 0; j < 9; ++j) d[j * WAVE] = make_double2(src[2 * j], src[2 * j + 1]);
  } else if (L == L_F32R12) {
    float4 *d = (float4 *)dst + blk * 3 * WAVE + (s & 63);
    for (int j = 0; j < 3; ++j)
      d[j * WAVE] = make_float4((float)src[4 * j], (float)src[4 * j + 1], (float)src[4 * j + 2], (float)src[4 * j + 3]);
  } else {
    uint2 *d = (uint2 *)dst + blk * 3 * WAVE + (s & 63);
    for (int j = 0; j < 3; ++j) {
      unsigned a = d2h(src[4 * j]) | ((unsigned)d2h(src[4 * j + 1]) << 16);
      unsigned b = d2h(src[4 * j + 2]) | ((unsigned)d2h(src[4 * j + 3]) << 16);
      d[j * WAVE] = make_uint2(a, b);
    }
  }
}

// FP16 links: each real is rounded FP64 -> FP16 once, to nearest even (d2h);
// FP32 links: FP64 -> FP32, to nearest even.

// Import and export.  The 64-site blocks b of both parities are the 128
// consecutive canonical sites 128 b .. 128 b + 127 (the checkerboard index is lex
// / 2), so a work-group of two waves takes one such run: it moves the canonical
// side as one contiguous 24 KB piece and passes it through LDS to one lane per
// site, whose packed accesses are contiguous over a wave as everywhere.  A lane
// that reads its 192 bytes of the canonical field itself has its wave touch every
// line twelve times.  Bound by memory; see canon_stream for the rates.  The LDS rows
// are 13 units long: a wave's reads of one component (every second row, 104 words
// apart) then fall on different banks.
constexpr int PK_ROW = 13;

// Parity of canonical site `lex` (x fastest, Lx even).
__device__ __forceinline__ int lex_parity(const Geo &g, int lex) {
  const int q1 = qdiv(lex >> 1, g.rlxh);   // (t Lz + z) Ly + y
  const int q2 = qdiv(q1, g.rly), t = qdiv(q2, g.rlz);
  return (lex + (q1 - q2 * g.ly) + (q2 - t * g.lz) + t) & 1;
}

// Both parities; parity p's packed half-field starts at dst + p * hoff.
template <int S, int NT>
__global__ __launch_bounds__(2 * WAVE) void k_import(Geo g, const double *__restrict__ canon, size_t canon_stride,
                                                     void *__restrict__ dst, size_t dst_stride, size_t hoff) {
  using R = typename SpinorIO<S>::R;
  __shared__ double2 lds[2 * WAVE * PK_ROW];
  const int r = blockIdx.x / g.nb, b = blockIdx.x - r * g.nb;
  const int l0 = 2 * WAVE * b, n = min(2 * WAVE, 2 * g.vh - l0);   // sites of the run
  const double2 *src = (const double2 *)(canon + r * canon_stride) + (size_t)l0 * 12;
  auto put = [&](int m, double2 q) {
    const int i = m * 2 * WAVE + threadIdx.x, j = i / 12;
    lds[j * PK_ROW + (i - 12 * j)] = q;
  };
  auto get = [&](int m) {
    const double2 *at = src + m * 2 * WAVE + threadIdx.x;
    return NT ? ld_nt(at) : *at;
  };
  // A whole run has all twelve loads in flight; under a test each they go one after
  // the other: one F16S field of 24^3x48 27 / 42 us, 3 FP64 of 16^3x32 26 / 35.
  if (n == 2 * WAVE) {
    double2 q[12];
#pragma unroll
    for (int m = 0; m < 12; ++m) q[m] = get(m);
#pragma unroll
    for (int m = 0; m < 12; ++m) put(m, q[m]);
  } else {
#pragma unroll
    for (int m = 0; m < 12; ++m)
      if (m * 2 * WAVE + (int)threadIdx.x < 12 * n) put(m, get(m));
  }
  __syncthreads();
  const int p = threadIdx.x >> 6, lane = threadIdx.x & (WAVE - 1), s = b * WAVE + lane;
  cpx<R> v[12];
  if (s < g.vh) {
    const double2 *row = lds + (2 * lane + (lex_parity(g, 2 * s) ^ p)) * PK_ROW;
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = cmake((R)row[k].x, (R)row[k].y);
  } else {
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = cmake((R)0, (R)0);
  }
  SpinorIO<S>::template store<(NT > 1)>((char *)dst + r * dst_stride + p * hoff, s, (size_t)g.nb * WAVE, v);
}

// Parity p alone: every second site of a run is skipped, so it is no contiguous
// piece, and a lane reads its own 192 bytes, all twelve loads at once.  Through LDS,
// each load under the test of its site's parity, this half took 42 us for one FP64
// field of 24^3x48 and this takes 25; 12 F16S fields 390 and 235.
template <int S>
__global__ __launch_bounds__(WG) void k_import_half(Geo g, const double *__restrict__ canon, size_t canon_stride,
                                                    void *__restrict__ dst, size_t dst_stride, int p, int nrhs) {
  using R = typename SpinorIO<S>::R;
  const size_t npad = (size_t)g.nb * WAVE;
  const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= npad * nrhs) return;
  const int s = (int)(i % npad), r = (int)(i / npad);
  cpx<R> v[12];
  if (s < g.vh) {
    const double2 *src = (const double2 *)(canon + r * canon_stride) + (size_t)(2 * s + (lex_parity(g, 2 * s) ^ p)) * 12;
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = cmake((R)src[k].x, (R)src[k].y);
  } else {
#pragma unroll
    for (int k = 0; k < 12; ++k) v[k] = cmake((R)0, (R)0);
  }
  SpinorIO<S>::store((char *)dst + r * dst_stride, s, npad, v);
}

// half: 0 or 1 for that parity alone, 2 for both; parity p's packed half-field
// starts at src + p * hoff.
template <int S, int NT>
__global__ __launch_bounds__(2 * WAVE) void k_export(Geo g, double *__restrict__ canon, size_t canon_stride,
                                                     const void *__restrict__ src, size_t src_stride, size_t hoff,
                                                     int half) {
  using R = typename SpinorIO<S>::R;
  __shared__ double2 lds[2 * WAVE * PK_ROW];
  const int r = blockIdx.x / g.nb, b = blockIdx.x - r * g.nb;
  const int l0 = 2 * WAVE * b, n = min(2 * WAVE, 2 * g.vh - l0);
  const int p = threadIdx.x >> 6, lane = threadIdx.x & (WAVE - 1), s = b * WAVE + lane;
  if (s < g.vh && (half == 2 || p == half)) {
    cpx<R> v[12];
    SpinorIO<S>::template load<(NT > 1)>((const char *)src + r * src_stride + p * hoff, s, (size_t)g.nb * WAVE, v);
    double2 *row = lds + (2 * lane + (lex_parity(g, 2 * s) ^ p)) * PK_ROW;
#pragma unroll
    for (int k = 0; k < 12; ++k) row[k] = make_double2((double)v[k].re, (double)v[k].im);
  }
  __syncthreads();
  double2 *d = (double2 *)(canon + r * canon_stride) + (size_t)l0 * 12;
#pragma unroll
  for (int m = 0; m < 12; ++m) {
    const int i = m * 2 * WAVE + threadIdx.x, j = i / 12;
    if (j < n && (half == 2 || lex_parity(g, l0 + j) == half)) {
      const double2 q = lds[j * PK_ROW + (i - 12 * j)];
      if (NT) st_nt(d + i, q);
      else d[i] = q;
    }
  }
}

// ---------------------------------------------------------------------------
// kernel: hopping term on one lattice, nrhs consecutive fields.  A work item
// is one 64-site block of a group of NR right-hand sides (each lane applies
// every link it loads to all NR of them).  Items run tile by tile: within a
// tile of at least two t-slices, every group sweeps the tile's blocks in turn,
// so a group's neighbour spinors are re-read while still cached and the tile's
// links are re-read from cache by the next group.  T waves cover an item, each
// taking 4/T directions for all 64 sites (hop_wave), and their sums are added
// in LDS (wave_combine).
// p >= 0: the fields are half-fields, out of parity p.  p < 0: they are full
// fields whose odd half starts hoff bytes on, and blockIdx.y is the output
// parity: D on every right-hand side in one launch.
template <int S, int L, bool DAG, int EPI, int T, int NR, bool NT>
__global__ __launch_bounds__(WG, HOP_MIN_WAVES(S, T, NR)) void k_hop(Geo g, const void *__restrict__ gauge,
                                                             const void *__restrict__ in, void *__restrict__ out,
                                                             const void *__restrict__ xin, size_t fstride, int nrhs,
                                                             int p, size_t hoff, double a, int tile, int zb, int chio,
                                                             int chix, double tmu, int ont) {
  using R = typename SpinorIO<S>::R;
  using LDS = HopLds<T, NR, R>;
  if (p < 0) {
    p = (int)blockIdx.y;
    in = (const char *)in + (1 - p) * hoff;
    out = (char *)out + p * hoff;
    xin = (const char *)xin + p * hoff;
  }
  __shared__ typename LDS::V lds[LDS::VECS];
  const int wg = xcd_remap(blockIdx.x, gridDim.x);
  const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // wave-uniform
  const int slot = w / T, grp = w % T;
  const int item = wg * (4 / T) + slot;
  // item order: (tile of `tile` blocks, right-hand-side group, block in tile)
  const int ngr = (nrhs + NR - 1) / NR;
  const int per_tile = ngr * tile;
  const int ti = item / per_tile, rem = item - ti * per_tile;
  const int rg = rem / tile;
  const int sbl = ti * tile + (rem - rg * tile);
  const bool item_ok = sbl < g.nb;   // uniform over the item's waves
  const int sb = item_ok ? block_order(g, sbl, zb) : 0;
  const int r0 = rg * NR;
  const int cnt = item_ok ? min(NR, nrhs - r0) : 1;
  const int s = sb * WAVE + (int)(threadIdx.x & (WAVE - 1));
  const bool site_ok = item_ok && s < g.vh;
  const size_t npad = (size_t)g.nb * WAVE;
  FieldLd<S, NR> ld;
  ld.npad = npad;
#pragma unroll
  for (int r = 0; r < NR; ++r) ld.base[r] = (const char *)in + (size_t)(r0 + min(r, cnt - 1)) * fstride;
  cpx<R> acc[NR][12];
  if (item_ok) hop_wave<L, DAG, T, NT>(g, gauge, ld, site_ok ? s : 0, p, grp, acc);
  else zero_acc<NR>(acc);
  wave_combine<T, NR>(acc, slot, grp, lds);
  if (!site_ok || grp != 0) return;
  const R ar = (R)a;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    if (r >= cnt) continue;
    if (EPI == 0) {
#pragma unroll
      for (int k = 0; k < 12; ++k) acc[r][k] = cscale(ar, acc[r][k]);
    } else {
      cpx<R> xv[12];
      SpinorIO<S>::load((const char *)xin + (size_t)(r0 + r) * fstride, s, npad, xv);
      apply_chi(xv, chix, tmu);
#pragma unroll
      for (int k = 0; k < 12; ++k) acc[r][k] = cadd(xv[k], cscale(ar, acc[r][k]));
    }
    apply_chi(acc[r], chio, tmu);
    if (ont) SpinorIO<S>::template store_fast<true>((char *)out + (size_t)(r0 + r) * fstride, s, npad, acc[r]);
    else SpinorIO<S>::template store_fast<false>((char *)out + (size_t)(r0 + r) * fstride, s, npad, acc[r]);
  }
}

namespace qiral {
// Right-hand sides per lane of a hop that was not tuned.  Two read each link once
// for both, but keep two thirds of the waves: while the items are few, or in a
// solver's hops (whose links the last-level cache serves and whose epilogues read
// more), one is faster.  The F16S hop is bound by its vector work and gains from two
// much earlier, where the right-hand sides come in pairs (with an odd number half of
// the last group's work is for nothing).  One / two per lane, us:
//   S, FP64: 12 fields of 12^3x24 78 / 83, 2 of 20^3x40 118 / 123, 12 of 16^3x32
//     248 / 249, 2 of 24^3x48 261 / 231, 12 of 20^3x40 721 / 690
//   S, FP32: 12 of 12^3x24 40 / 42, 2 of 24^3x48 96 / 123, 4 of 24^3x48 228 / 224
//   S, F16S: 2 of 16^3x32 18.6 / 20.3, 5 35.1 / 37.8, 7 47.0 / 48.8, 2 of 24^3x48
//     69 / 75; in pairs 6 of 14^3x28 28.4 / 29.3, 12 of 12^3x24 29.2 / 29.2, 8 of
//     14^3x28 34.4 / 33.2, 6 of 16^3x32 41.1 / 39.6, 10 66.3 / 62.4, 4 of 20^3x40
//     67 / 62; H on 4 of 20^3x40 31.9 / 29.8, D on 4 of 16^3x32 27.5 / 25.9, on 8 of
//     12^3x24 19.0 / 19.4
//   CGNR in ms, FP64: 12 of 12^3x24 9.7 / 11.4, 4 of 16^3x32 10.3 / 11.9, 2 of 24^3x48
//     28.9 / 28.3, 4 52.3 / 55.9, 12 147 / 158; FP32: 3 of 20^3x40 12.3 / 13.8, 12 of
//     24^3x48 93.5 / 97.3; F16S: 12 of 12^3x24 6.73 / 6.78, 6 of 16^3x32 8.85 / 8.98, 12
//     of 14^3x28 10.32 / 10.30, 8 of 16^3x32 11.07 / 10.99, 10 13.37 / 13.14, 2 of
//     24^3x48 12.9 / 13.7, 4 22.8 / 22.0
static int default_nr(int prec, long items, long nrhs, bool solver) {
  if (solver && prec != QIRAL_F16S) return 1;
  if (prec == QIRAL_F16S && nrhs >= 4 && nrhs % 2 == 0) return items < (solver ? 7000 : 3800) ? 1 : 2;
  return items < (prec == QIRAL_F64 ? 8000 : 11000) ? 1 : 2;
}

HopCfg hop_config(const qiral_lattice *lat, int prec, long nrhs, bool solver) {
  HopCfg c;
  const long nb = lat->geo.nb;
  // The tuner times the plain hop.  Its shape with several right-hand sides per lane
  // and more than one group of them is none for a solver whose hops take one: CGNR on
  // 12 FP64 sources of 24^3x48 took 182 ms with it and takes 170 (2 sources, one group:
  // 32.5 ms with it, 33.3 without).
  const int tnr = tuned_nr(lat, prec, (int)nrhs);
  const bool tuned = !(solver && prec != QIRAL_F16S && tnr > 1 && nrhs > tnr);
  if (const char *e = getenv("QIRAL_HOP_NR")) c.nr = atoi(e);
  else if (!(c.nr = tuned ? tnr : 0)) c.nr = default_nr(prec, nb * nrhs, nrhs, solver);
  c.nr = std::max(1, std::min(c.nr, 4));
  if (c.nr > nrhs) c.nr = (int)nrhs;
  const long nitems = nb * ((nrhs + c.nr - 1) / c.nr);
  c.t = hop_split(prec, nitems);
  const int tt = tuned ? lat->tuned_t[prec][nrhs < 4 ? nrhs : 4] : 0;
  if (tt && !getenv("QIRAL_HOP_SPLIT") && hop_nr_max(prec, tt) >= 1) c.t = tt;
  c.tile = tuned ? lat->tuned_tile[prec][nrhs < 4 ? nrhs : 4] : 0;
  if (c.nr > hop_nr_max(prec, c.t)) c.t = (c.t == 1 && c.nr <= hop_nr_max(prec, 2)) ? 2 : 4;
  c.nr = std::min(c.nr, hop_nr_max(prec, c.t));   // FP64 takes at most 2
  return c;
}

bool hop_stream(const Geo &g, int prec, long nrhs, long ngroups) {
  if (const char *e = getenv("QIRAL_HOP_NT")) return atoi(e) != 0;
  if (ngroups > 1) return false;   // the groups re-read the tile's links
  const double link = prec == QIRAL_F64 ? 96 : prec == QIRAL_F32 ? 48 : 24;   // bytes a hop reads per link
  const double sp = prec == QIRAL_F64 ? 192 : prec == QIRAL_F32 ? 96 : 52;
  const double bytes = (double)g.vh * (8 * link + 2 * sp * nrhs);
  return bytes > 128e6;   // half the 256 MB last-level cache
}

// Both sides of the solvers' rules, in ms per FP64 CGNR solve unless said otherwise
// (streaming stores of the hops' outputs off / on, then the vector kernels'
// level 0 / 1 / 2 with the better of them):
//   one system, 20^3x40 (31 MB a vector): 8.72 / 9.14, 8.72 / 8.81 / 8.86
//   one system, 24^3x48 (64 MB): 16.7 / 17.2, 16.7 / 16.0 / 16.2
//   one system, 32^3x64 (201 MB): 52.9 / 49.3, 49.3 / 47.4 / 49.0
//   one system, 32^3x64 in FP32 (100 MB): 31.3 / 31.0, 31.0 / 30.1 / 30.0
//   2 of 16^3x32 (25 MB): 6.86 / -, - / 6.82 / 6.83; 3 (38 MB): 10.4, 9.92 / 10.0
//   2 of 24^3x48 (127 MB): level 1 28.6, level 2 29.2
//   12 of 24^3x48 (764 MB): 163.9 / 162.5 / 159.5; FP32 102.8 / 101.6 / 99.3;
//   F16S 69.9 / 68.6 / 66.7
//   8 lattices of 4 sizes, FP32 (48 MB): 14.35 (off, 0), 13.6 (on, 1), 13.2 (on, 2)
// Systems on lattices of their own do not meet in the cache as those of one lattice do
// (whose links they share).  Stores off / on, then level 0 / 1 / 2, stores off:
//   12^3x24 with 16^3x32, FP64 (17 MB): 5.86 / 5.98, 5.72 / 5.76 / 5.83, BiCGStab 2.99 /
//     3.04 / 3.15; 5 of 12^3x24 (20 MB) 6.58 / 6.71, 6.62 / 6.50 / 6.56
//   4 of 16^3x32, FP32 (25 MB): 9.05 / 9.09, 9.09 / 8.90 / 9.02
//   4 of two sizes, FP64 (33 MB): 9.53 / 9.50, 10.04 / 9.45 / 9.51, BiCGStab 5.33 / 5.10 /
//     4.99; 3 of three sizes, FP32 (33 MB), all stores / none: level 2 12.51 / - , level 1
//     - / 12.75
//   6 of 16^3x32, FP32 (38 MB): 12.97 / 12.80, 13.89 / 13.37 / 12.92
//   20^3x40 with 16^3x32, FP64 (43 MB): 13.55 / 13.06, 13.78 / 13.06 / 13.04
// Vectors of several right-hand sides of one lattice, level 0 / 1: 3 FP32 of 16^3x32 (19
// MB) 6.40 / 6.28, 2 FP64 (25 MB) 6.96 / 6.86, 2 FP32 of 20^3x40 (31 MB) 10.06 / 9.97
bool out_stream(size_t bytes, int nsys, bool same_lattice) {
  return bytes >= (nsys == 1 ? 80e6 : same_lattice ? 16e6 : 30e6);
}

// Several groups of right-hand sides stream from 16 MB on, one group with its links;
// neither while the next launch finds the output in the last-level cache (one field's
// line, 80 MB).  Cached / streamed, us:
//   the next launch reads it, S: 5 F32 of 16^3x32 (31 MB) 47.0 / 47.7, 12 FP64 of
//     12^3x24 (48 MB) 71.8 / 75.3, 2 FP64 of 20^3x40 (61 MB) 112.9 / 115.5, 12 F32 of
//     16^3x32 (75 MB) 111.4 / 113.6, 5 F32 of 20^3x40 (77 MB) 124.7 / 128.7; 3 FP64 of
//     20^3x40 (92 MB) 174.1 / 171.3, 3 F32 of 24^3x48 (95 MB) 202 / 171, 8 F32 of
//     20^3x40 (123 MB) 211 / 205
//   it does not: S on 4 FP64 of 12^3x24 (16 MB) 31.4 / 31.3, D on 2 FP64 of 16^3x32
//     (25 MB a parity) 46.0 / 45.5, H on 3 (38 MB) 30.8 / 30.1, on 4 F32 of 24^3x48
//     (127 MB) 109 / 78.5, D on 5 F32 of 20^3x40 (77 MB a parity) 140 / 126
// D's both parities count as one here: doubling its bytes changed none of 13 cases.
bool op_out_stream(size_t bytes, int ngroups, bool nt, bool reread) {
  if (reread && !out_stream(bytes, 1, true)) return false;
  return ngroups > 1 ? bytes >= 16e6 : nt;
}

int vec_stream(size_t bytes, int nsys, bool same_lattice) {
  if (nsys == 1) return bytes >= 48e6;
  if (bytes < 17e6) return 0;
  return bytes >= (same_lattice ? 200e6 : 30e6) ? 2 : 1;
}

bool zb_valid(const Geo &g, int zb) {
  return zb > 0 && zb < g.lz && g.lz % zb == 0 && (long)zb * g.sz % WAVE == 0 && g.st % WAVE == 0;
}

int hop_zb(const Geo &g) {
  if (g.st % WAVE != 0 || (long)g.nb * WAVE != g.vh) return 0;
  if (const char *e = getenv("QIRAL_HOP_ORDER")) {   // 0: plain order; n > 0: tiles of n planes
    const int n = atoi(e);
    return zb_valid(g, n) ? n : 0;
  }
  // A lattice whose FP64 hop (1152 B per site) fits the 256 MB last-level
  // cache keeps the plain order: its hops run from that cache, and tiling them
  // cost up to 10% (FP32 at 16^3x32).
  if ((double)g.vh * 1152.0 <= 256e6) return 0;
  // As many z-tiles as XCDs (else half or a quarter as many), so that the
  // contiguous range of blocks each XCD takes (xcd_remap) is one whole tile or
  // a whole part of one: a tile's z-neighbour planes are then read twice only
  // where two XCDs meet, and a block's t-neighbours were read one chunk earlier
  // on the same XCD.  Measured on the 1-RHS hops at 64^3x128, tiles of Lz/8
  // planes ran 21% (FP64), 15% (FP32) and 8% (F16S) faster than tiles of about
  // 0.5 MB of input spinors (1, 2 and 4 planes); at 32^3x64 and 24^3x48 the
  // best tiles were Lz/8 and Lz/4 planes as well.
  for (int ntz : {NXCD, NXCD / 2, NXCD / 4})
    if (g.lz % ntz == 0 && zb_valid(g, g.lz / ntz)) return g.lz / ntz;
  return 0;   // the plain order
}

int hop_tile(const Geo &g, int ngroups, int tuned) {
  if (ngroups <= 1) return g.nb;   // one group: plain block order
  if (const char *e = getenv("QIRAL_HOP_TILE")) {
    const int n = atoi(e);
    if (n > 0) return std::min(g.nb, n);
  }
  // Each group sweeps a tile before the next group does, so the tile's links are
  // re-read from the L2 while they are still there: 16 blocks (1.2 MB of FP64
  // links) measured within a few percent of the best tile at 24^3x48 for every
  // storage class, where tiles of two t-slices (216 blocks) were 5-25% slower.
  if (tuned > 0) return std::min(g.nb, tuned);
  return std::min(g.nb, 16);
}

int hop_split(int prec, long nwork) {
  if (const char *e = getenv("QIRAL_HOP_SPLIT")) {
    const int t = atoi(e);
    if (t == 4 || (t == 2 && prec != QIRAL_F64) || (t == 1 && prec == QIRAL_F16S)) return t;
  }
  // FP64 needs 4 waves per site block (fewer spill); otherwise 4 while the
  // blocks do not fill the SIMDs (more waves hide more latency), else 2 (less
  // LDS traffic and fewer redundant coordinate computations per site).  One
  // wave per block (F16S only) is left to the tuner.
  const long simds = 1024;   // 256 compute units x 4 SIMDs
  if (prec == QIRAL_F64 || nwork <= simds) return 4;
  return 2;
}

template <int S, int L, int T, int NR, bool NT>
static hipError_t launch_hop_ttt(const HopCfg &c, const qiral_lattice *lat, const HopCall &h) {
  const Geo &g = lat->geo;
  const double tmu = 2.0 * lat->kappa * lat->mu;
  const size_t hb = half_bytes(g, S), fstride = h.p < 0 ? 2 * hb : hb;
  const void *gauge = links_for(lat, S);
  const int tile = hop_tile(g, (h.nrhs + NR - 1) / NR, c.tile);
  const int zb = hop_zb(g);
  const long ntile = (g.nb + tile - 1) / tile;
  const long nitems = ntile * tile * ((h.nrhs + NR - 1) / NR);
  const int nwg = (int)((nitems * T + 3) / 4);
  const dim3 grid(nwg, h.p < 0 ? 2 : 1), block(WG);
  const int ont = op_out_stream(hb * (size_t)h.nrhs, (h.nrhs + NR - 1) / NR, NT, h.reread);
#define QARGS g, gauge, h.in, h.out, h.x, fstride, h.nrhs, h.p, hb, h.a, tile, zb, h.chio, h.chix, tmu, ont
  if (!h.dagger) {
    if (h.epi == 0) hipLaunchKernelGGL((k_hop<S, L, false, 0, T, NR, NT>), grid, block, 0, h.st, QARGS);
    else hipLaunchKernelGGL((k_hop<S, L, false, 1, T, NR, NT>), grid, block, 0, h.st, QARGS);
  } else {
    if (h.epi == 0) hipLaunchKernelGGL((k_hop<S, L, true, 0, T, NR, NT>), grid, block, 0, h.st, QARGS);
    else hipLaunchKernelGGL((k_hop<S, L, true, 1, T, NR, NT>), grid, block, 0, h.st, QARGS);
  }
#undef QARGS
  return hipGetLastError();
}

template <int S, int L, int T, int NR>
static hipError_t launch_hop_tt(const HopCfg &c, const qiral_lattice *lat, const HopCall &h) {
  if (hop_stream(lat->geo, S, h.nrhs, (h.nrhs + NR - 1) / NR)) return launch_hop_ttt<S, L, T, NR, true>(c, lat, h);
  return launch_hop_ttt<S, L, T, NR, false>(c, lat, h);
}

template <int S, int L, int T>
static hipError_t launch_hop_n(const HopCfg &c, const qiral_lattice *lat, const HopCall &h) {
  constexpr int NM = hop_nr_max(S, T);   // shapes beyond it are excluded by hop_config and the tuner
  if constexpr (NM == 0) {
    return hipErrorInvalidValue;
  } else {
    if (c.nr > NM) return hipErrorInvalidValue;
    if constexpr (NM >= 4) if (c.nr == 4) return launch_hop_tt<S, L, T, 4>(c, lat, h);
    if constexpr (NM >= 3) if (c.nr == 3) return launch_hop_tt<S, L, T, 3>(c, lat, h);
    if constexpr (NM >= 2) if (c.nr == 2) return launch_hop_tt<S, L, T, 2>(c, lat, h);
    return launch_hop_tt<S, L, T, 1>(c, lat, h);
  }
}

template <int S, int L>
static hipError_t launch_hop_t(const HopCfg &c, const qiral_lattice *lat, const HopCall &h) {
  if constexpr (S == S_F64) return launch_hop_n<S, L, 4>(c, lat, h);
  else {
    if (c.t == 4) return launch_hop_n<S, L, 4>(c, lat, h);
    if (c.t == 1) return launch_hop_n<S, L, 1>(c, lat, h);
    return launch_hop_n<S, L, 2>(c, lat, h);
  }
}

hipError_t launch_hop_cfg(const HopCfg &c, const qiral_lattice *lat, int prec, const HopCall &h) {
  if (prec == QIRAL_F64) return launch_hop_t<S_F64, L_F64R18>(c, lat, h);
  if (prec == QIRAL_F32) return launch_hop_t<S_F32, L_F32R12>(c, lat, h);
  return launch_hop_t<S_F16S, L_F16R12>(c, lat, h);
}

hipError_t launch_hop(const qiral_lattice *lat, int prec, int dagger, int p, int epi, double a, const void *in,
                      void *out, const void *x, int nrhs, hipStream_t st, int chio, int chix, bool reread) {
  return launch_hop_cfg(hop_config(lat, prec, nrhs), lat, prec,
                        HopCall{dagger, p, epi, a, in, out, x, nrhs, st, chio, chix, reread});
}

hipError_t launch_D(const qiral_lattice *lat, int prec, int dagger, void *out, const void *in, int nrhs,
                    hipStream_t st) {
  // D = A - kappa H (D^dagger = A^dagger - kappa H^dagger), A = 1 + 2 i kappa mu gamma_5.
  // One launch for both output parities of every right-hand side: a launch per
  // parity and right-hand side took 10 x 5.0 us for 5 F16S fields of 14x10x18x22
  // (433 blocks each, fewer than the SIMDs).
  return launch_hop(lat, prec, dagger, -1, 1, -lat->kappa, in, out, in, nrhs, st, CHI_ONE, dagger ? CHI_ADAG : CHI_A);
}
}  // namespace qiral

// ---------------------------------------------------------------------------
// lattice handle
static void release_handle(qiral_lattice *lat) {
  for (hipEvent_t e : lat->poll_ev) if (e) (void)hipEventDestroy(e);
  for (hipEvent_t e : lat->time_ev) if (e) (void)hipEventDestroy(e);
  if (lat->pinned) (void)hipHostFree(lat->pinned);
  delete lat;
}

extern "C" qiral_status qiral_lattice_create(qiral_lattice **out, const int32_t dims[4], double kappa, double mu,
                                             const double *gauge_canon, void *gauge_f64, void *gauge_f32,
                                             void *gauge_f16, qiral_stream_t stream) {
  if (!out) return fail(QIRAL_ERR_INVALID_ARG, "lat is NULL");
  *out = nullptr;
  qiral_status st = check_dims(dims);
  if (st != QIRAL_OK) return st;
  if (!gauge_canon) return fail(QIRAL_ERR_INVALID_ARG, "gauge_canon is NULL");
  if (!gauge_f64) return fail(QIRAL_ERR_INVALID_ARG, "gauge_f64 is NULL (the FP64 store is required)");
  if (!std::isfinite(kappa) || !std::isfinite(mu)) return fail(QIRAL_ERR_INVALID_ARG, "kappa and mu must be finite");
  for (const void *p : {gauge_f64, gauge_f32, gauge_f16})
    if (((uintptr_t)p & 15) != 0) return fail(QIRAL_ERR_INVALID_ARG, "link stores must be 16-byte aligned");
  if ((gauge_f32 && (gauge_f32 == gauge_f64 || gauge_f32 == gauge_f16)) || (gauge_f16 && gauge_f16 == gauge_f64))
    return fail(QIRAL_ERR_INVALID_ARG, "the link stores must be distinct buffers");

  qiral_lattice *lat = new qiral_lattice();
  for (int i = 0; i < 4; ++i) lat->dims[i] = dims[i];
  lat->geo = make_geo(dims);
  lat->kappa = kappa;
  lat->mu = mu;
  lat->g64 = gauge_f64;
  lat->g32 = gauge_f32;
  lat->g16 = gauge_f16;
  hipStream_t s = (hipStream_t)stream;
  const Geo &g = lat->geo;
  auto cleanup = [&](qiral_status r) {
    release_handle(lat);
    return r;
  };
  hipError_t e = hipGetDevice(&lat->device);
  if (e != hipSuccess) return cleanup(hip_fail(e, "hipGetDevice"));
  // host-side resources of later solves and tuning, made once here
  e = hipHostMalloc(&lat->pinned, poll_bytes(), hipHostMallocDefault);
  if (e != hipSuccess) { lat->pinned = nullptr; return cleanup(hip_fail(e, "hipHostMalloc(state polls)")); }
  lat->pinned_bytes = poll_bytes();
  for (hipEvent_t &ev : lat->poll_ev) {
    e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
    if (e != hipSuccess) { ev = nullptr; return cleanup(hip_fail(e, "hipEventCreate")); }
  }
  for (hipEvent_t &ev : lat->time_ev) {
    e = hipEventCreate(&ev);
    if (e != hipSuccess) { ev = nullptr; return cleanup(hip_fail(e, "hipEventCreate")); }
  }
  const size_t nlinks = 8 * npad_of(g);
  const int nblk = (int)((nlinks + WG - 1) / WG);
  hipLaunchKernelGGL(k_pack_gauge<L_F64R18>, dim3(nblk), dim3(WG), 0, s, g, gauge_canon, lat->g64);
  lat->gauge_bytes = link_store_bytes(g, QIRAL_F64);
  if (gauge_f32) {
    hipLaunchKernelGGL(k_pack_gauge<L_F32R12>, dim3(nblk), dim3(WG), 0, s, g, gauge_canon, lat->g32);
    lat->gauge_bytes += link_store_bytes(g, QIRAL_F32);
  }
  if (gauge_f16) {
    hipLaunchKernelGGL(k_pack_gauge<L_F16R12>, dim3(nblk), dim3(WG), 0, s, g, gauge_canon, lat->g16);
    lat->gauge_bytes += link_store_bytes(g, QIRAL_F16S);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return cleanup(hip_fail(e, "pack links"));
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) return cleanup(hip_fail(e, "hipStreamSynchronize(lattice_create)"));
  *out = lat;
  return QIRAL_OK;
}

extern "C" qiral_status qiral_lattice_destroy(qiral_lattice *lat) {
  if (!lat) return fail(QIRAL_ERR_INVALID_ARG, "lat is NULL");
  release_handle(lat);
  return QIRAL_OK;
}

extern "C" qiral_status qiral_lattice_query(const qiral_lattice *lat, int64_t *vh, int64_t *bytes) {
  if (!lat) return fail(QIRAL_ERR_INVALID_ARG, "lat is NULL");
  if (vh) *vh = lat->geo.vh;
  if (bytes) *bytes = (int64_t)lat->gauge_bytes;
  return QIRAL_OK;
}

// ---------------------------------------------------------------------------
// field import / export
static qiral_status check_field_args(const qiral_lattice *lat, const void *a, const void *b, int subset, int prec,
                                     int nrhs) {
  if (!lat) return fail(QIRAL_ERR_INVALID_ARG, "lat is NULL");
  if (!a || !b) return fail(QIRAL_ERR_INVALID_ARG, "field pointer is NULL");
  if (subset != QIRAL_EVEN && subset != QIRAL_ODD && subset != QIRAL_FULL)
    return fail(QIRAL_ERR_INVALID_ARG, "bad subset");
  if (!valid_prec(prec)) return fail(QIRAL_ERR_INVALID_ARG, "bad precision");
  if (nrhs < 1) return fail(QIRAL_ERR_INVALID_ARG, "nrhs must be >= 1");
  return QIRAL_OK;
}

// The canonical field is read or written once: streaming where it is far larger
// than an L2 keeps, and the packed field too where the last-level cache does not
// hold them.  12 FP64 fields of 24^3x48 (3.06 GB), both parities: import 684 us with
// one lane per site reading its own 192 bytes, 540 now (5.7 TB/s, as a device
// copy); export 806, 611 with the canonical side streaming, 534 with both.
static int canon_stream(const Geo &g, int nrhs) {
  const double bytes = (double)g.vh * 384 * nrhs;
  return bytes >= 256e6 ? 2 : bytes >= 64e6;
}

template <int S>
static void launch_import(const Geo &g, const double *src, void *dst, int subset, int nrhs, hipStream_t s) {
  const size_t canon_stride = (size_t)g.vh * 2 * 24;   // doubles per canonical field
  const size_t hb = half_bytes(g, S);
  if (subset != QIRAL_FULL) {
    const dim3 grid((unsigned)((npad_of(g) * nrhs + WG - 1) / WG)), block(WG);
    hipLaunchKernelGGL(k_import_half<S>, grid, block, 0, s, g, src, canon_stride, dst, hb, subset, nrhs);
    return;
  }
  const dim3 grid((unsigned)((long)g.nb * nrhs)), block(2 * WAVE);
  const int nt = canon_stream(g, nrhs);
  const auto kernel = nt == 0 ? k_import<S, 0> : nt == 1 ? k_import<S, 1> : k_import<S, 2>;
  hipLaunchKernelGGL(kernel, grid, block, 0, s, g, src, canon_stride, dst, 2 * hb, hb);
}

template <int S>
static void launch_export(const Geo &g, double *dst, const void *src, int subset, int nrhs, hipStream_t s) {
  const size_t canon_stride = (size_t)g.vh * 2 * 24;
  const size_t hb = half_bytes(g, S), hoff = subset == QIRAL_FULL ? hb : 0, stride = hb + hoff;
  const dim3 grid((unsigned)((long)g.nb * nrhs)), block(2 * WAVE);
  const int nt = canon_stream(g, nrhs);
  const auto kernel = nt == 0 ? k_export<S, 0> : nt == 1 ? k_export<S, 1> : k_export<S, 2>;
  hipLaunchKernelGGL(kernel, grid, block, 0, s, g, dst, canon_stride, src, stride, hoff, subset);
}

namespace qiral {
void import_field(const Geo &g, const double *src, void *dst, int subset, int prec, int nrhs, hipStream_t s) {
  if (prec == QIRAL_F64) launch_import<S_F64>(g, src, dst, subset, nrhs, s);
  else if (prec == QIRAL_F32) launch_import<S_F32>(g, src, dst, subset, nrhs, s);
  else launch_import<S_F16S>(g, src, dst, subset, nrhs, s);
}
void export_field(const Geo &g, double *dst, const void *src, int subset, int prec, int nrhs, hipStream_t s) {
  if (prec == QIRAL_F64) launch_export<S_F64>(g, dst, src, subset, nrhs, s);
  else if (prec == QIRAL_F32) launch_export<S_F32>(g, dst, src, subset, nrhs, s);
  else launch_export<S_F16S>(g, dst, src, subset, nrhs, s);
}
}  // namespace qiral

extern "C" qiral_status qiral_field_import(const qiral_lattice *lat, void *dst, const double *src_canon,
                                           qiral_subset subset, qiral_prec prec, int32_t nrhs, qiral_stream_t stream) {
  qiral_status st = check_field_args(lat, dst, src_canon, subset, prec, nrhs);
  if (st != QIRAL_OK) return st;
  import_field(lat->geo, src_canon, dst, subset, prec, nrhs, (hipStream_t)stream);
  QIRAL_HIP(hipGetLastError());
  return QIRAL_OK;
}

extern "C" qiral_status qiral_field_export(const qiral_lattice *lat, double *dst_canon, const void *src,
                                           qiral_subset subset, qiral_prec prec, int32_t nrhs, qiral_stream_t stream) {
  qiral_status st = check_field_args(lat, dst_canon, src, subset, prec, nrhs);
  if (st != QIRAL_OK) return st;
  export_field(lat->geo, dst_canon, src, subset, prec, nrhs, (hipStream_t)stream);
  QIRAL_HIP(hipGetLastError());
  return QIRAL_OK;
}

// ---------------------------------------------------------------------------
// operators
static qiral_status check_op_prec(const qiral_lattice *lat, int prec) {
  if (!valid_prec(prec)) return fail(QIRAL_ERR_INVALID_ARG, "bad precision");
  if (!links_for(lat, prec))
    return fail(QIRAL_ERR_INVALID_ARG, "the lattice holds no links of this precision (see lo_precs)");
  return QIRAL_OK;
}

extern "C" qiral_status qiral_dslash_eo(const qiral_lattice *lat, void *out, const void *in, int32_t out_parity,
                                        int32_t dagger, qiral_prec prec, int32_t nrhs, qiral_stream_t stream) {
  if (!lat) return fail(QIRAL_ERR_INVALID_ARG, "lat is NULL");
  if (!out || !in) return fail(QIRAL_ERR_INVALID_ARG, "field pointer is NULL");
  if (out == in) return fail(QIRAL_ERR_INVALID_ARG, "in and out must not alias");
  if (out_parity != 0 && out_parity != 1) return fail(QIRAL_ERR_INVALID_ARG, "out_parity must be 0 or 1");
  if (nrhs < 1) return fail(QIRAL_ERR_INVALID_ARG, "nrhs must be >= 1");
  qiral_status st = check_op_prec(lat, prec);
  if (st != QIRAL_OK) return st;
  QIRAL_HIP(launch_hop(lat, prec, dagger != 0, out_parity, 0, 1.0, in, out, nullptr, nrhs, (hipStream_t)stream));
  return QIRAL_OK;
}

extern "C" qiral_status qiral_apply_M(const qiral_lattice *lat, void *out, const void *in, void *tmp, qiral_op op,
                                      qiral_prec prec, int32_t nrhs, qiral_stream_t stream) {
  if (!lat) return fail(QIRAL_ERR_INVALID_ARG, "lat is NULL");
  if (!out || !in) return fail(QIRAL_ERR_INVALID_ARG, "field pointer is NULL");
  if (out == in) return fail(QIRAL_ERR_INVALID_ARG, "in and out must not alias");
  if (nrhs < 1) return fail(QIRAL_ERR_INVALID_ARG, "nrhs must be >= 1");
  if (op != QIRAL_OP_D && op != QIRAL_OP_DDAG && op != QIRAL_OP_SCHUR && op != QIRAL_OP_SCHUR_DAG)
    return fail(QIRAL_ERR_INVALID_ARG, "bad operator");
  if ((op == QIRAL_OP_SCHUR || op == QIRAL_OP_SCHUR_DAG) && (!tmp || tmp == in || tmp == out))
    return fail(QIRAL_ERR_INVALID_ARG, "the Schur operators need a separate tmp half-field");
  qiral_status st = check_op_prec(lat, prec);
  if (st != QIRAL_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  const double k = lat->kappa;
  const int dag = (op == QIRAL_OP_DDAG || op == QIRAL_OP_SCHUR_DAG);
  if (op == QIRAL_OP_D || op == QIRAL_OP_DDAG) {
    // full fields, [rhs][even | odd]; one after the other where a result lies in an
    // earlier right-hand side's place (out n fields below in), whose input is then used up
    const size_t fb = 2 * half_bytes(lat->geo, prec);
    const uintptr_t i = (uintptr_t)in, o = (uintptr_t)out, all = fb * (size_t)nrhs;
    const int step = i < o + all && o < i + all ? 1 : nrhs;
    for (int r = 0; r < nrhs; r += step)
      QIRAL_HIP(launch_D(lat, prec, dag, (char *)out + r * fb, (const char *)in + r * fb, step, s));
  } else {
    // S = A - kappa^2 H_oe A^-1 H_eo (S^dagger: daggered hops and site factors)
    QIRAL_HIP(launch_hop(lat, prec, dag, 0, 0, 1.0, in, tmp, nullptr, nrhs, s, dag ? CHI_AINVDAG : CHI_AINV, CHI_ONE,
                         true));
    QIRAL_HIP(launch_hop(lat, prec, dag, 1, 1, -k * k, tmp, out, in, nrhs, s, CHI_ONE, dag ? CHI_ADAG : CHI_A));
  }
  return QIRAL_OK;
}
