// The one-work-group solver of small lattices (solo.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "solver_dev.h"

namespace qiral {

// Most 64-site blocks per parity of a lattice that one work-group solves.
constexpr int SOLO_BLOCKS = 4;
// The line of a solve: the work-group does two blocks at a time, so its
// iteration grows by the hops of two blocks (about 20 us for CGNR in FP64) where
// the grouped solver's stays at its launches' latency, and grows with the number
// of systems instead.  Grouped / one work-group, us a solve from a Gaussian source on
// links near 1, kappa 0.12, in FP64 for one source unless said otherwise:
//   4^4 (2 blocks): CGNR 1950 / 1160, BiCGStab 1010 / 564, CRNR 2000 / 1273
//   4^3x6 (3): CGNR 2057 / 1908, CRNR 2117 / 2069
//   4^3x8 (4): BiCGStab 1076 / 998, CGNR in F32 2117 / 1719, F16S 2220 / 1936, 4 sources
//     2244 / 2235, 5 sources 2307 / 2238, CRNR 4 sources 2386 / 2452
// and on other links, before the work-group's steps were inlined (which took 2 to 9%
// off its times):
//   4^3x8 (4): CGNR 1820 / 1953, CRNR 1942 / 2141
//   4^2x6x8 (6): CGNR 1919 / 2905, 12 sources 2678 / 2926
inline int solo_line(int nsys, bool fp64, bool bicgstab) { return fp64 && !bicgstab && nsys < 4 ? 3 : SOLO_BLOCKS; }

// A solve as steps: the source [0, start), the start of the iterations [start,
// iter), one iteration [iter, post) and the end [post, end).  A step runs if
// the system's status matches its mask; fin_red >= 0: its sums (slot) go
// through the scalar step fin_red (FIN_*).
enum : int {
  SK_HOP = 0, SK_SUM, SK_UPD, SK_RES, SK_BNORM, SK_CG1, SK_CG2, SK_XFIN, SK_CR1, SK_CR2, SK_BIP, SK_BIS, SK_BIXR,
  SK_COPY, SK_BIINIT, SK_IMPORT, SK_EXPORT, SK_ZERO
};
struct SoloStep {
  int8_t kind, mask, fin, fout, fx, par, amode, red, slot, fin_red, chio, chix, epi, f64;
  bool dag;
  int8_t pad;
};
constexpr int SOLO_STEPS = 48;
struct SoloProg {
  SoloStep step[SOLO_STEPS];
  int start, iter, post, end;
};

// From the source; from the start of the iterations (a restart); more iterations.
enum : int { SOLO_NEW = 0, SOLO_RESTART = 1, SOLO_MORE = 2 };

// Solves nsys systems of at most SOLO_BLOCKS blocks, one work-group each, or
// goes on with those that the states do not say are done.  At most 256
// iterations a launch.
hipError_t solo_launch(const SysDesc *desc, int nsys, int solver, int prec, bool twisted, bool guess, int mode,
                       hipStream_t s);

}  // namespace qiral
