"""The rules that choose a hop's launch shape are host code: a small program links the
library and asks them, without a GPU."""
import os
import shutil
import subprocess

import pytest

from paper_1401_2039_amd import _lib as L
from paper_1401_2039_amd import build

pytestmark = pytest.mark.skipif(not os.path.exists(L.LIB_PATH) or
                                (not os.path.exists(build.HIPCC) and shutil.which("hipcc") is None),
                                reason="library not built or hipcc not available")

SOURCE = r"""
#include <cstdio>
#include "qiral_int.h"
using namespace qiral;
int main() {
  int nb, prec, nrhs, solver, nr, t, tile;
  while (scanf("%d %d %d %d %d %d %d", &nb, &prec, &nrhs, &solver, &nr, &t, &tile) == 7) {
    qiral_lattice lat{};
    lat.geo.nb = nb;
    lat.geo.vh = nb * WAVE;
    const int i = nrhs < 4 ? nrhs : 4;
    lat.tuned_nr[prec][i] = nr;
    lat.tuned_t[prec][i] = t;
    lat.tuned_tile[prec][i] = tile;
    const HopCfg c = hop_config(&lat, prec, nrhs, solver);
    printf("%d %d %d\n", c.nr, c.t, c.tile);
  }
}
"""


def _program(d, source):
    """Builds `source` against the library; a function from cases to rows of numbers."""
    src, exe = d / "rules.hip", d / "rules"
    src.write_text(source)
    flags = [f for f in build.CFLAGS if f != "-fPIC"] + ["-I", build.CSRC]
    lib = os.path.dirname(L.LIB_PATH)
    r = subprocess.run([build.HIPCC, *flags, str(src), "-o", str(exe), "-L", lib, "-lqiral_hip", f"-Wl,-rpath,{lib}"],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]

    def ask(*cases):
        text = "\n".join(" ".join(str(int(v)) for v in c) for c in cases)
        env = {k: v for k, v in os.environ.items() if not k.startswith("QIRAL_HOP_")}
        out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, env=env, timeout=60)
        assert out.returncode == 0, out.stderr[-2000:]
        return [tuple(int(v) for v in line.split()) for line in out.stdout.split("\n") if line]
    return ask


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    return _program(tmp_path_factory.mktemp("rules"), SOURCE)


@pytest.mark.parametrize("prec,t", [(L.F64, 4), (L.F32, 4), (L.F32, 2)])
def test_solver_hops_keep_one_right_hand_side_per_lane_on_a_tuned_handle(shapes, prec, t):
    """A plain hop tuned to two right-hand sides per lane does not set the grouped
    solver's shape, unless they are all there are; one tuned to one does."""
    nb = 5184   # 24^3x48
    plain, solver, untuned, all_in_one, one = shapes((nb, prec, 12, 0, 2, t, 8), (nb, prec, 12, 1, 2, t, 8),
                                                     (nb, prec, 12, 1, 0, 0, 0), (nb, prec, 2, 1, 2, t, 0),
                                                     (nb, prec, 12, 1, 1, t, 8))
    assert plain == (2, t, 8)
    assert solver == untuned and solver[0] == 1
    assert all_in_one[0] == 2
    assert one == (1, t, 8)


def test_f16s_solver_hops_take_the_tuned_shape(shapes):
    assert shapes((5184, L.F16S, 12, 1, 2, 4, 32)) == [(2, 4, 32)]


def test_f16s_right_hand_sides_go_in_pairs(shapes):
    """An even number of F16S fields of 16^3x32 or more takes two right-hand sides per
    lane, an odd number or two of them one (per-lane numbers, untuned)."""
    nb = 1024   # 16^3x32
    got = shapes(*((nb, L.F16S, n, 0, 0, 0, 0) for n in (1, 2, 3, 4, 5, 6, 8, 10, 12)))
    assert [c[0] for c in got] == [1, 1, 1, 2, 1, 2, 2, 2, 2]
    got = shapes(*((nb, L.F16S, n, 1, 0, 0, 0) for n in (4, 6, 8, 10, 12)))
    assert [c[0] for c in got] == [1, 1, 2, 2, 2]
    assert shapes((324, L.F16S, 8, 0, 0, 0, 0))[0][0] == 1   # 12^3x24: too few items


STREAMING = r"""
#include <cstdio>
#include "qiral_int.h"
using namespace qiral;
int main() {
  double mb;
  int groups, nt, reread;
  while (scanf("%lf %d %d %d", &mb, &groups, &nt, &reread) == 4)
    printf("%d\n", (int)op_out_stream((size_t)(mb * 1e6), groups, nt, reread));
}
"""


def test_an_intermediate_that_fits_the_cache_is_kept_there(tmp_path):
    """Schur's intermediate over several groups of right-hand sides is streamed only
    where the last-level cache would not keep it; one group as its links."""
    ask = _program(tmp_path, STREAMING)
    several = ask((31, 6, 0, 1), (75, 6, 0, 1), (95, 2, 0, 1), (15, 6, 0, 0), (38, 2, 0, 0))
    assert [v for (v,) in several] == [0, 0, 1, 0, 1]
    one = ask((64, 1, 1, 1), (64, 1, 1, 0), (201, 1, 1, 1), (25, 1, 0, 0))
    assert [v for (v,) in one] == [0, 1, 1, 0]


SOLVE_STREAMING = r"""
#include <cstdio>
#include "qiral_int.h"
using namespace qiral;
int main() {
  double mb;
  int nsys, same;
  while (scanf("%lf %d %d", &mb, &nsys, &same) == 3)
    printf("%d %d\n", (int)out_stream((size_t)(mb * 1e6), nsys, same), vec_stream((size_t)(mb * 1e6), nsys, same));
}
"""


def test_small_batches_of_lattices_stay_cached(tmp_path):
    """(streamed hop outputs, level of the vector kernels) of a solve, by the bytes of a
    vector over its systems: lattices of their own stream everything from 30 MB only."""
    ask = _program(tmp_path, SOLVE_STREAMING)
    assert ask((16, 2, 0), (25, 4, 0), (33, 4, 0), (38, 6, 0), (48, 8, 0)) == [(0, 0), (0, 1), (1, 2), (1, 2), (1, 2)]
    assert ask((12, 3, 1), (19, 3, 1), (48, 12, 1), (382, 12, 1)) == [(0, 0), (1, 1), (1, 1), (1, 2)]
    assert ask((31, 1, 1), (64, 1, 1), (100, 1, 1)) == [(0, 0), (0, 1), (1, 1)]
