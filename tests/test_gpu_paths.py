"""Launch paths chosen by a rule on sizes, at the sizes where they can go wrong,
against the complex128 oracle.  Tolerances: FP64 1e-12 and FP32 2e-6 relative
(5e-6 of the largest element), F16S half an FP16 ulp of each site's scale plus
FP32 rounding, as for the operators in general."""
import numpy as np
import pytest
import torch

import latgen
from oracle import ptc, solvers as S, storage, wilson as W
import paper_1401_2039_amd as q
from gpu_util import say, dev, host

pytestmark = pytest.mark.gpu


def _rounded(cfg, prec):
    U, b = cfg["U"], cfg["b"]
    if prec == q.F64:
        return U, b
    if prec == q.F32:
        return storage.round_links_r12(U, np.complex64), storage.round_f32(b)
    return storage.round_links_r12(U, "f16"), storage.round_f16s(b)


def _check(got, want, prec):
    d = np.abs(got - want)
    if prec == q.F64:
        assert d.max() < 1e-12 * np.abs(want).max()
    elif prec == q.F32:
        assert np.sqrt(W.norm2(got - want) / W.norm2(want)) < 2e-6 and d.max() < 5e-6 * np.abs(want).max()
    else:
        scale = np.abs(np.stack([want.real, want.imag])).reshape(2, -1, 12).max(axis=(0, 2))
        assert np.all(d.reshape(-1, 12).max(axis=1) <= 2.0 ** -11 * 1.01 * scale + 1e-6 * scale.max())


# one launch of D takes both output parities of every right-hand side: an odd
# number of fields (a short last group), a ragged last block, one block, two
@pytest.mark.parametrize("prec", [q.F64, q.F32, q.F16S], ids=["f64", "f32", "f16s"])
@pytest.mark.parametrize("dims,nrhs", [((6, 4, 2, 4), 5), ((2, 2, 2, 2), 3), ((4, 4, 4, 4), 2), ((6, 10, 2, 8), 1)])
def test_full_operator_of_several_fields(dims, nrhs, prec):
    say("D of several fields", dims, nrhs, prec)
    cfg = latgen.small_config(dims, seed=81, kind="expih", eps=0.4, nrhs=nrhs)
    lat = q.Lattice(dims, 0.12, cfg["U"], mu=0.35)
    Ur, br = _rounded(cfg, prec)
    inp, out = lat.import_field(dev(cfg["b"]), q.FULL, prec), lat.field(q.FULL, prec, nrhs)
    for op, ref in ((q.OP_D, W.apply_D), (q.OP_DDAG, W.apply_Ddag)):
        lat.apply_M(out, inp, None, op, prec, nrhs)
        got = host(lat.export_field(out, q.FULL, prec, nrhs=nrhs))
        for r in range(nrhs):
            _check(got[r], ref(Ur, 0.12, 0.35, br[r]), prec)


# The network's pass over all paths and the gradient of its folded weights work
# on tiles of 16 and 32 sites in a bounded number of work-groups: one partly
# filled block, a ragged last tile, whole tiles, and 12x12x16x24 with more blocks
# (864 of both parities) than work-groups.  FP32 sums of 72 products in each of
# two passes: 2e-6 relative.  A gradient entry sums a product per site and colour
# in FP32 pieces: 1e-5 of the largest.
@pytest.mark.parametrize("dims,H", [((2, 2, 2, 2), 8), ((6, 4, 2, 4), 2), ((4, 4, 4, 4), 4), ((6, 10, 2, 8), 8),
                                    ((12, 12, 16, 24), 2)])
def test_network_and_gradient_tiles(dims, H):
    say("network tiles", dims, H)
    cfg = latgen.small_config(dims, seed=83, kind="expih", eps=0.4, nrhs=2)
    lat = q.Lattice(dims, 0.125, cfg["U"])
    net = q.Network(lat, H)
    rng = np.random.default_rng(H)
    w1, w2 = (0.3 * (rng.standard_normal(n) + 1j * rng.standard_normal(n)) for n in ((9, H, 1, 4, 4), (9, 1, H, 4, 4)))
    net.set_weights(w1, w2)
    ws = [w.astype(np.complex64).astype(np.complex128) for w in (w1, w2)]
    Ur, br = _rounded(cfg, q.F32)
    src, tgt = (lat.import_field(dev(cfg["b"][i:i + 1]), q.FULL, q.F32) for i in (0, 1))
    out = lat.field(q.FULL, q.F32)
    for adj, ref in ((False, ptc.network), (True, ptc.network_adjoint)):
        net.apply(out, src, adjoint=adj)
        got, want = host(lat.export_field(out, q.FULL, q.F32))[0], ref(Ur, ws, br[0])
        assert np.sqrt(W.norm2(got - want) / W.norm2(want)) < 2e-6
    loss, g = net.grad(src, tgt)
    L, G = ptc.loss_and_grad(Ur, ws, br[0], br[1])
    want = np.concatenate([(2 * G[0]).ravel(), (2 * G[1]).ravel()])
    assert abs(loss - L) < 1e-6 * L
    assert np.abs(g[0::2] + 1j * g[1::2] - want).max() < 1e-5 * np.abs(want).max()


def test_network_streamed_for_several_systems():
    """The path fields of four systems of 12^3x16 (48 MB) are streamed, of one (12 MB)
    cached: the iterates in lockstep are those alone bit for bit."""
    dims = (12, 12, 12, 16)
    say("network streamed", dims)
    cfg = latgen.small_config(dims, seed=88, kind="expih", eps=0.4, nrhs=4)
    lat = q.Lattice(dims, 0.12, cfg["U"])
    net = q.Network(lat, 2)
    kw = dict(tol=1e-10, solver=q.BICGSTAB_EO, system=q.SYSTEM_SCHUR, precond=net.handle, fallback_cg=0)
    b = dev(cfg["b"])
    x, st, info = lat.solve(b, **kw)
    x = x.clone()
    assert st == 0
    for r in (0, 3):
        x1, st1, i1 = lat.solve(b[r:r + 1], **kw)
        assert st1 == 0 and i1[0]["iterations"] == info[r]["iterations"] and torch.equal(x[r:r + 1], x1)
    assert S.true_rel_residual(cfg["U"], 0.12, 0.0, host(x)[3], cfg["b"][3]) <= 1e-10


# One work-group solves a lattice of up to four 64-site blocks; a captured graph
# always takes the grouped kernels.  Both take the same steps with the same sums:
# equal bit for bit in FP64, and to the tolerance of the solves in the reduced
# precisions (their hops may split the directions over other waves).  One, two,
# three and four blocks, a partly filled last one, one and five systems (the line
# lies one block higher for several), with and without a twisted mass.
@pytest.mark.parametrize("dims,mu,nrhs", [((2, 2, 2, 2), 0.0, 1), ((4, 4, 4, 4), 0.35, 1), ((4, 4, 4, 6), 0.0, 1),
                                          ((4, 4, 4, 8), 0.0, 5), ((6, 2, 4, 10), 0.35, 2)])
@pytest.mark.parametrize("solver", [q.CGNR_EO, q.BICGSTAB_EO, q.CRNR_EO], ids=["cgnr", "bicgstab", "crnr"])
def test_one_work_group_solves(dims, mu, nrhs, solver):
    say("one work-group", dims, mu, nrhs, solver)
    cfg = latgen.small_config(dims, seed=85, kind="expih", eps=0.4, nrhs=nrhs)
    lat = q.Lattice(dims, 0.12, cfg["U"], mu=mu)
    b, side = dev(cfg["b"]), torch.cuda.Stream()
    for prec in (q.F64, q.F32, q.F16S)[:1 if solver == q.CRNR_EO else 3]:
        kw = dict(solver=solver, inner_prec=prec, tol=1e-10)
        x, st, info = lat.solve(b, **kw)
        with torch.cuda.stream(side):
            xg, sg, ig = lat.solve(b, use_graph=1, **kw)
        side.synchronize()
        x, xg = host(x), host(xg)
        assert st == 0 and sg == 0
        for r in range(nrhs):
            assert S.true_rel_residual(cfg["U"], 0.12, mu, x[r], cfg["b"][r]) <= 1e-10
        if prec == q.F64:
            assert np.array_equal(x, xg)
            assert [i["iterations"] for i in info] == [i["iterations"] for i in ig]
            assert [i["hop_applications"] for i in info] == [i["hop_applications"] for i in ig]
            assert [i["true_rel_resid"] for i in info] == [i["true_rel_resid"] for i in ig]


def test_one_work_group_goes_on():
    """More iterations than one launch takes (256), from a guess, and a stop at
    maxiter: the grouped solver's iterate bit for bit."""
    say("one work-group, 300 iterations")
    cfg = latgen.small_config((4, 4, 4, 4), seed=86, kind="haar", nrhs=1)
    lat = q.Lattice((4, 4, 4, 4), 0.12, cfg["U"])
    b, side = dev(cfg["b"]), torch.cuda.Stream()
    x0 = dev(0.1 * cfg["b"])
    for n in (3, 300):
        kw = dict(tol=1e-200, maxiter=n, x0_is_guess=1)
        x, st, info = lat.solve(b, x_canon=x0.clone(), **kw)
        with torch.cuda.stream(side):
            xg, sg, ig = lat.solve(b, x_canon=x0.clone(), use_graph=1, **kw)
        side.synchronize()
        assert st == sg and info[0]["iterations"] == ig[0]["iterations"] == n
        assert torch.equal(x, xg)


# Packing moves runs of 128 canonical sites: a run shorter than a wave's share, a
# ragged last one, whole ones; and, with 2 x 21 MB and 12 x 21 MB of FP64 fields of
# 12x12x12x32, both streaming forms.  Half subsets leave the other parity alone.
@pytest.mark.parametrize("dims,nrhs", [((2, 2, 2, 2), 2), ((6, 4, 2, 4), 3), ((4, 4, 4, 4), 1), ((6, 10, 2, 8), 2),
                                       ((12, 12, 12, 32), 4), ((12, 12, 12, 32), 13)])
def test_packing_runs(dims, nrhs):
    say("packing", dims, nrhs)
    lat = q.Lattice(dims, 0.12, latgen.gauge_field(1090, 0, dims, "unit"), lo_precs=0)
    psi = dev(latgen.complex_gaussian(np.random.default_rng(9), (nrhs,) + W.site_shape(dims) + (3, 4)))
    par = torch.from_numpy(W.parity_field(dims)).cuda().reshape(-1)
    for prec, rnd in ((q.F64, lambda a: a), (q.F32, storage.round_f32), (q.F16S, storage.round_f16s)):
        want = dev(rnd(host(psi)))
        assert torch.equal(lat.export_field(lat.import_field(psi, q.FULL, prec), q.FULL, prec, nrhs), want)
        for p in (0, 1):
            out = torch.full_like(psi, 7.0)
            lat.export_field(lat.import_field(psi, p, prec), p, prec, nrhs, out=out)
            o, w = out.reshape(nrhs, -1, 12), want.reshape(nrhs, -1, 12)
            assert torch.equal(o[:, par == p], w[:, par == p]) and bool((o[:, par != p] == 7.0).all())


def _batch(cfgs, kappas, dims, prec, xs=None, **kw):
    """qiral_solve_batch of one source per lattice: solutions, status, infos."""
    lats = [q.Lattice(dims, k, c["U"]) for k, c in zip(kappas, cfgs)]
    bs = [dev(c["b"]) for c in cfgs]
    xs = xs(bs) if xs else [lat.canon() for lat in lats]
    st, info = q.qiral_solve_batch([lat.handle for lat in lats], [dims] * len(lats), xs, bs,
                                   q.solve_params(inner_prec=prec, **kw))
    return xs, st, info


# Systems of one call that end in different launches of the one-work-group solver
# (256 iterations each): what is done stays as it is, and the others go on.  The
# grouped solver's results, bit for bit in FP64.
@pytest.mark.parametrize("dims,kappas", [((4, 4, 4, 4), (0.12, 0.24)), ((4, 4, 4, 8), (0.24, 0.12, 0.21, 0.1))])
def test_one_work_group_systems_end_apart(dims, kappas):
    say("one work-group, several launches", dims, kappas)
    cfgs = [latgen.small_config(dims, seed=89 + i, kind="haar", nrhs=1) for i in range(len(kappas))]
    kw = dict(tol=1e-10, maxiter=5000)
    xs, st, info = _batch(cfgs, kappas, dims, q.F64, **kw)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        xg, sg, ig = _batch(cfgs, kappas, dims, q.F64, use_graph=1, **kw)
    side.synchronize()
    its = [i["iterations"] for i in ig]
    assert st == sg == 0 and min(its) < 256 < max(its)
    for key in ("iterations", "hop_applications", "true_rel_resid"):
        assert [i[key] for i in info] == [i[key] for i in ig], key
    for x, y in zip(xs, xg):
        assert torch.equal(x, y)


# A solution may lie where another system's source was: every source is read
# before any solution is written.
@pytest.mark.parametrize("prec", [q.F64, q.F32], ids=["f64", "f32"])
def test_small_systems_sharing_memory(prec):
    say("one work-group, a solution in another's source", prec)
    dims, n = (4, 4, 4, 4), 3
    cfg = latgen.small_config(dims, seed=93, kind="expih", eps=0.4, nrhs=n)
    lat = q.Lattice(dims, 0.12, cfg["U"])
    kw = dict(inner_prec=prec, tol=1e-10)
    want, st, info = lat.solve(dev(cfg["b"]), use_graph=0, **kw)
    assert st == 0
    # the solutions one field before the sources
    buf = lat.canon(n + 1)
    buf[1:] = dev(cfg["b"])
    x, st, info = lat.solve(buf[1:], x_canon=buf[:n], **kw)
    assert st == 0
    # a batch: the first solution in the last source, each source read as it was given
    bs = [dev(cfg["b"][i:i + 1]) for i in range(n)]
    xs = [bs[n - 1], lat.canon(), lat.canon()]
    st, _ = q.qiral_solve_batch([lat.handle] * n, [dims] * n, xs, bs, q.solve_params(**kw))
    assert st == 0
    for i in range(n):
        for got in (x[i:i + 1], xs[i]):
            assert S.true_rel_residual(cfg["U"], 0.12, 0.0, host(got)[0], cfg["b"][i]) <= 1e-10
            assert prec != q.F64 or torch.equal(got, want[i:i + 1])


# The gradient's FP32 sums go on in FP64 after 32 products.  Integer fields on unit
# links, with the identity for a network and a target of norm^2 2^k, make every
# product (just under 2^19, one sign) and every sum of 32 an FP32 integer: nothing is
# rounded, where runs of 96 would leave the integers.  One item of 32 sites per
# work-group, and two.
@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (16, 16, 16, 8)])
def test_gradient_sums_leave_fp32_early(dims):
    say("gradient sums", dims)
    H, shape = 2, W.site_shape(dims) + (3, 4)
    U = latgen.gauge_field(1091, 0, dims, "unit")
    lat = q.Lattice(dims, 0.12, U, lo_precs=q.LINKS_F32)
    net = q.Network(lat, H)
    w1, w2 = np.zeros((9, H, 1, 4, 4), complex), np.zeros((9, 1, H, 4, 4), complex)
    w1[0, 0, 0] = w2[0, 0, 0] = np.eye(4)
    net.set_weights(w1, w2)
    rng = np.random.default_rng(11)
    src = rng.integers(719, 724, shape) + 1j * rng.integers(719, 724, shape)
    tgt = np.zeros(shape, complex)
    tgt[..., 0, :] = 1 + 1j   # 8 per site
    loss, g = net.grad(*(lat.import_field(dev(f[None]), q.FULL, q.F32) for f in (src, tgt)))
    L, G = ptc.loss_and_grad(U, [w1, w2], src, tgt)
    assert loss == L
    assert np.array_equal(g[0::2] + 1j * g[1::2], np.concatenate([(2 * G[0]).ravel(), (2 * G[1]).ravel()]))


# Training keeps what the folded weights lose in FP32: with identity matrices a and b
# on path 0 and a b half an FP32 ulp (2^-24) off, the loss without it is 6e-8 off, the
# same at every site.  With it the roundings of the sites are independent: about
# 2 * 5e-8 / sqrt(24 V) relative, 2e-10 here; ten times that.
@pytest.mark.parametrize("dims", [(8, 8, 8, 8), (6, 10, 4, 18)])
def test_training_keeps_the_folded_weights_remainder(dims):
    say("folded weights' remainder", dims)
    H = 2
    cfg = latgen.small_config(dims, seed=94, kind="expih", eps=0.4, nrhs=2)
    lat = q.Lattice(dims, 0.12, cfg["U"], lo_precs=q.LINKS_F32)
    net = q.Network(lat, H)
    w1, w2 = np.zeros((9, H, 1, 4, 4), complex), np.zeros((9, 1, H, 4, 4), complex)
    w1[0, 0, 0] = w2[0, 0, 0] = (1 + 3 * 2.0 ** -12) * np.eye(4)
    net.set_weights(w1, w2)
    Ur, br = _rounded(cfg, q.F32)
    loss, _ = net.grad(*(lat.import_field(dev(cfg["b"][i:i + 1]), q.FULL, q.F32) for i in (0, 1)))
    L, _ = ptc.loss_and_grad(Ur, [w1, w2], br[0], br[1])
    assert abs(loss - L) < 2e-9 * L


def _least_us(f, reps=40, batches=5):
    e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    best = float("inf")
    for _ in range(batches + 1):   # the first one warms up
        e[0].record()
        for _ in range(reps):
            f()
        e[1].record()
        torch.cuda.synchronize()
        best = min(best, 1e3 * e[0].elapsed_time(e[1]) / reps)
    return best


def test_import_keeps_its_loads_in_flight():
    """An import whose loads wait for one another took 1.8 times the export of the same
    field, and half a field as long as a whole one.  Now 1.2 times and 0.65; the lines
    lie between."""
    dims = (24, 24, 24, 48)
    say("import times", dims)
    unit = torch.eye(3, dtype=torch.complex128, device="cuda").expand(W.site_shape(dims) + (4, 3, 3))
    lat = q.Lattice(dims, 0.12, unit, lo_precs=0)
    psi, buf = lat.canon(), lat.field(q.FULL, q.F16S)
    imp, half = (_least_us(lambda: q.qiral_field_import(lat.handle, dims, buf, psi, sub, q.F16S))
                 for sub in (q.FULL, q.ODD))
    exp = _least_us(lambda: lat.export_field(buf, q.FULL, q.F16S, out=psi))
    assert imp < 1.5 * exp and half < 0.8 * imp, (imp, half, exp)


# The streaming forms on a ragged lattice (a last block of 8 sites): 7 fields of
# 14x10x18x22 (75 MB, the canonical side streamed) and 25 (266 MB, both sides), whole
# and one parity at a time.  The largest of the test above is 138 MB.
@pytest.mark.parametrize("nrhs", [7, 25])
def test_packing_streams_ragged_fields(nrhs):
    dims = (14, 10, 18, 22)
    say("packing, streamed, ragged", dims, nrhs)
    unit = torch.eye(3, dtype=torch.complex128, device="cuda").expand(W.site_shape(dims) + (4, 3, 3))
    lat = q.Lattice(dims, 0.12, unit, lo_precs=0)
    psi = dev(latgen.complex_gaussian(np.random.default_rng(10), (nrhs,) + W.site_shape(dims) + (3, 4)))
    par = torch.from_numpy(W.parity_field(dims)).cuda().reshape(-1)
    for prec, rnd in ((q.F64, lambda a: a), (q.F32, storage.round_f32), (q.F16S, storage.round_f16s)):
        want = dev(rnd(host(psi)))
        full = lat.import_field(psi, q.FULL, prec)
        assert torch.equal(lat.export_field(full, q.FULL, prec, nrhs), want)
        for p in (0, 1):
            half = lat.import_field(psi, p, prec)
            assert torch.equal(half.reshape(nrhs, -1), full.reshape(nrhs, 2, -1)[:, p])
            out = torch.full_like(psi, 7.0)
            lat.export_field(half, p, prec, nrhs, out=out)
            o, w = out.reshape(nrhs, -1, 12), want.reshape(nrhs, -1, 12)
            assert torch.equal(o[:, par == p], w[:, par == p]) and bool((o[:, par != p] == 7.0).all())


@pytest.mark.parametrize("prec", [q.F64, q.F32, q.F16S], ids=["f64", "f32", "f16s"])
def test_full_operator_into_used_up_fields(prec):
    """D writes each field into the place of the one before it, field by field."""
    dims, n = (4, 4, 6, 8), 3
    say("D in place, one field on", dims, prec)
    cfg = latgen.small_config(dims, seed=95, kind="expih", eps=0.4, nrhs=n)
    lat = q.Lattice(dims, 0.12, cfg["U"], mu=0.35)
    Ur, br = _rounded(cfg, prec)
    one = q.qiral_field_bytes(dims, q.FULL, prec)
    buf = lat.field(q.FULL, prec, n + 1)
    buf[one:] = lat.import_field(dev(cfg["b"]), q.FULL, prec)
    for op, ref in ((q.OP_D, W.apply_D), (q.OP_DDAG, W.apply_Ddag)):
        work = buf.clone()
        lat.apply_M(work[:n * one], work[one:], None, op, prec, n)
        got = host(lat.export_field(work[:n * one].clone(), q.FULL, prec, nrhs=n))
        for r in range(n):
            _check(got[r], ref(Ur, 0.12, 0.35, br[r]), prec)
