"""The work this library is used for, as measurable cases.

A case is a dict of plain values.  `prepare` makes what a user's program holds
before the call (links, sources, packed fields, handles, workspaces, a
network), `run` makes one pass through the public entry points and returns its
outputs, `work` says what a pass cannot do without, and `exact` gives the same
outputs from plain torch in 64 bits, without the library.

Kinds of cases:
  field    canonical fields packed and unpacked again (import, then export)
  op       one application of the hop (even or odd output), of D or of the Schur
           operator, or of an adjoint, on packed fields
  solve    D x = b from a canonical source to a canonical solution
  batch    the same for several lattices of different sizes in one call
  network  one application of the learned preconditioner, or of its adjoint
  train    a few steps of its training

Lattices are given as "LxLyLzLt" texts such as "24x24x24x48".
"""
import math

import torch

import paper_1401_2039_amd as q

PREC = {"f64": q.F64, "f32": q.F32, "f16s": q.F16S}
SITE_BYTES = {"f64": 192, "f32": 96, "f16s": 52}      # one spinor
LINK_BYTES = {"f64": 96, "f32": 48, "f16s": 24}       # rows 0 and 1 of one link, which determine it
OPS = {"D": q.OP_D, "Ddag": q.OP_DDAG, "S": q.OP_SCHUR, "Sdag": q.OP_SCHUR_DAG}
SOLVERS = {"cgnr": q.CGNR_EO, "bicgstab": q.BICGSTAB_EO, "crnr": q.CRNR_EO, "fgmres": q.FGMRES_NN, "fcg": q.FCG_NN}
HOP_FLOPS = 1320                                      # one hop, per output site
LR, STEPS = 1e-3, 4                                   # of a training case


def listed():
    return [
        # A source packed for the operator calls and a result unpacked: what a program that
        # composes its own solver from the operators does around it; 12 spin-colour sources.
        dict(name="field_f64_12", kind="field", dims="24x24x24x48", prec="f64", nrhs=12),
        # The smallest operator calls, where the launch and the latency of a chain of loads count.
        dict(name="schur_f64_8^4", kind="op", op="S", dims="8x8x8x8", prec="f64", nrhs=1, eps=0.3, kappa=0.12, mu=0.0),
        # The library's dominant kernel, on the lattice of the benchmark.
        dict(name="hop_f64_24^3x48", kind="op", op="Heo", dims="24x24x24x48", prec="f64", nrhs=1, eps=0.4, kappa=0.12,
             mu=0.0),
        # The operator of a batched reduced-precision solve of 12 spin-colour sources.
        dict(name="schurdag_f32_24^3x48_12", kind="op", op="Sdag", dims="24x24x24x48", prec="f32", nrhs=12, eps=0.4,
             kappa=0.12, mu=0.0),
        # An odd lattice (a last site block partly filled), an odd number of fields, twisted mass,
        # FP16 storage: the full operator.
        dict(name="D_f16s_twisted_odd", kind="op", op="D", dims="14x10x18x22", prec="f16s", nrhs=5, eps=0.3, kappa=0.11,
             mu=0.35),
        # The smallest solve (the plain method's own workload): an iteration is nothing but latency.
        dict(name="cgnr_f64_4^4", kind="solve", solver="cgnr", dims="4x4x4x4", prec="f64", nrhs=1, eps=-1.0, kappa=0.12,
             mu=0.0, source="gauss", net=False),
        # The benchmark's solve, one source.
        dict(name="cgnr_f64_24^3x48", kind="solve", solver="cgnr", dims="24x24x24x48", prec="f64", nrhs=1, eps=0.4,
             kappa=0.12, mu=0.0, source="point", net=False),
        # A propagator: the 12 point sources together in mixed precision, the fastest form there is.
        dict(name="cgnr_f16s_24^3x48_12", kind="solve", solver="cgnr", dims="24x24x24x48", prec="f16s", nrhs=12,
             eps=0.4, kappa=0.12, mu=0.0, source="point", net=False),
        # Independent lattices of uneven sizes in one call.
        dict(name="batch_f32_uneven", kind="batch", dims="8x8x8x8,8x8x8x8,12x12x12x24,12x12x12x24,16x16x16x32,"
             "16x16x16x32,20x20x20x40,20x20x20x40", prec="f32", eps=0.35, kappa=0.11, mu=0.0),
        # The preconditioned solve of 12 sources.
        dict(name="learned_24^3x48_12", kind="solve", solver="bicgstab", dims="24x24x24x48", prec="f64", nrhs=12,
             eps=0.5, kappa=0.125, mu=0.0, source="gauss", net=True),
        # The network on its own, as a smoother or a preconditioner of a program's own solver.
        dict(name="network_24^3x48", kind="network", dims="24x24x24x48", hidden=8, adjoint=False, eps=0.5, kappa=0.125),
        # Its training: forward, backward, Adam.
        dict(name="train_24^3x48", kind="train", dims="24x24x24x48", hidden=8, eps=0.5, kappa=0.125),
    ]


def _draw_dims(rng, lo, hi):
    """Even extents with a volume between lo and hi sites, spread over its logarithm."""
    while True:
        v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        r = [rng.uniform(0.75, 1.3) for _ in range(3)] + [rng.uniform(0.8, 2.2)]
        f = (v / math.prod(r)) ** 0.25
        d = [max(2, 2 * round(f * x / 2)) for x in r]
        if lo <= math.prod(d) <= hi:
            return "x".join(map(str, d))


def draw(rng):
    most = max(work(c)["bytes"] for c in listed())
    while True:
        case = _draw(rng)
        if work(case)["bytes"] <= most:
            return case


def _draw(rng):
    kind = rng.choice(["field", "op", "op", "op", "solve", "solve", "solve", "batch", "network", "train"])
    full = 24 * 24 * 24 * 48
    eps, kappa = round(rng.uniform(0.2, 0.5), 3), round(rng.uniform(0.10, 0.125), 4)
    mu = rng.choice([0.0, 0.0, 0.0, 0.2, 0.35])
    nrhs = rng.choice([1, 1, 2, 3, 4, 5, 7, 8, 12])
    if kind == "field":
        return dict(kind=kind, dims=_draw_dims(rng, 256, full), prec=rng.choice(list(PREC)), nrhs=nrhs)
    if kind == "op":
        return dict(kind=kind, op=rng.choice(["Heo", "Hoe", "D", "Ddag", "S", "S", "Sdag"]),
                    dims=_draw_dims(rng, 256, full), prec=rng.choice(list(PREC)), nrhs=nrhs, eps=eps, kappa=kappa, mu=mu)
    if kind == "solve":
        solver, net = rng.choice([("cgnr", False)] * 4 + [("bicgstab", False)] * 2 +
                                 [("crnr", False), ("bicgstab", True), ("fgmres", True), ("fcg", True)])
        prec = rng.choice(list(PREC)) if solver in ("cgnr", "bicgstab") and not net else "f64"
        if solver in ("fgmres", "fcg"):   # these solve their sources one after the other
            nrhs = min(nrhs, 2)
        return dict(kind=kind, solver=solver, dims=_draw_dims(rng, 256, full // (2 if net else 1)), prec=prec, nrhs=nrhs,
                    eps=eps, kappa=kappa, mu=mu, source=rng.choice(["gauss", "gauss", "point"]), net=net)
    if kind == "batch":
        n = rng.randint(2, 6)
        return dict(kind=kind, dims=",".join(_draw_dims(rng, 256, full // 4) for _ in range(n)),
                    prec=rng.choice(["f64", "f32", "f32", "f16s"]), eps=eps, kappa=round(min(kappa, 0.12), 4), mu=mu)
    hidden = rng.choice([2, 4, 8, 8])
    if kind == "network":
        return dict(kind=kind, dims=_draw_dims(rng, 4096, full), hidden=hidden, adjoint=rng.random() < 0.5, eps=eps,
                    kappa=kappa)
    return dict(kind=kind, dims=_draw_dims(rng, 4096, full), hidden=hidden, eps=eps, kappa=kappa)


# ---------------------------------------------------------------------------
# inputs


def _dims(case):
    return tuple(int(v) for v in case["dims"].split("x"))


def _sites(d):
    return (d[3], d[2], d[1], d[0])


def _mul3(a, b):
    return sum(a[..., :, k, None] * b[..., None, k, :] for k in range(3))


def _row2(r0, r1):
    """conj(r0 x r1): the last row of an SU(3) matrix."""
    return torch.linalg.cross(r0, r1).conj()


def _gauss(gen, shape):
    return torch.view_as_complex(torch.randn(tuple(shape) + (2,), generator=gen, device="cuda", dtype=torch.float64))


def _links(gen, d, eps):
    """Haar random links (eps < 0), or exp(i eps H) with H traceless Hermitian Gaussian."""
    a = _gauss(gen, _sites(d) + (4, 3, 3))
    if eps < 0:
        u = a
    else:
        h = 0.5 * (a + a.conj().transpose(-1, -2))
        h = h - torch.eye(3, device="cuda") * (torch.diagonal(h, dim1=-2, dim2=-1).real.sum(-1) / 3.0)[..., None, None]
        h = h * (1j * eps)
        u = torch.eye(3, device="cuda", dtype=torch.complex128).expand_as(h)
        for k in range(24, 0, -1):   # Horner's form of the exponential's series
            u = torch.eye(3, device="cuda") + _mul3(h, u) / k
    r0 = u[..., 0, :] / torch.linalg.vector_norm(u[..., 0, :], dim=-1, keepdim=True)
    r1 = u[..., 1, :] - (r0.conj() * u[..., 1, :]).sum(-1, keepdim=True) * r0
    r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
    return torch.stack([r0, r1, _row2(r0, r1)], dim=-2).contiguous()


def _source(gen, d, nrhs, kind):
    if kind == "gauss":
        return _gauss(gen, (nrhs,) + _sites(d) + (3, 4))
    b = torch.zeros((nrhs,) + _sites(d) + (3, 4), dtype=torch.complex128, device="cuda")
    at = [int(torch.randint(0, n, (1,), generator=gen, device="cuda")) for n in _sites(d)]
    for k in range(nrhs):
        b[(k, *at, (k // 4) % 3, k % 4)] = 1.0
    return b


def _weights(gen, hidden, kappa):
    """Weights near 1 + kappa H + kappa^2 H^2 with every channel in use, as in training."""
    n = (9, hidden, 4, 4)
    w1, w2 = (0.05 * _gauss(gen, n) for _ in range(2))
    w1[0, 0] += torch.eye(4, device="cuda")
    w2[0, 0] += torch.eye(4, device="cuda")
    for mu in range(4):
        g = _gamma(mu)
        one = torch.eye(4, device="cuda")
        w1[1 + mu, 1] += one - g
        w1[5 + mu, 1] += one + g
        w2[1 + mu, 1] += kappa * kappa * (one - g)
        w2[5 + mu, 1] += kappa * kappa * (one + g)
    w2[0, 1] += kappa * torch.eye(4, device="cuda")
    return w1.to(torch.complex64), w2.to(torch.complex64)


def _inputs(case, seed):
    """The inputs of a case in canonical form, from the seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    kind = case["kind"]
    if kind == "field":
        return dict(psi=_gauss(gen, (case["nrhs"],) + _sites(_dims(case)) + (3, 4)))
    if kind == "batch":
        out = []
        for t in case["dims"].split(","):
            d = _dims(dict(dims=t))
            out.append((d, _links(gen, d, case["eps"]), _gauss(gen, (1,) + _sites(d) + (3, 4))))
        return dict(systems=out)
    d = _dims(case)
    v = dict(U=_links(gen, d, case["eps"]))
    if kind == "op":
        v["psi"] = _gauss(gen, (case["nrhs"],) + _sites(d) + (3, 4))
    elif kind == "solve":
        v["b"] = _source(gen, d, case["nrhs"], case["source"])
    else:
        v["w1"], v["w2"] = _weights(gen, case["hidden"], case["kappa"])
        if kind == "network":
            v["psi"] = _gauss(gen, (1,) + _sites(d) + (3, 4))
        else:
            v["seed"] = int(seed) & 0x7FFFFFFF
    return v


# ---------------------------------------------------------------------------
# the cases


def _views(buf, nfields, prec):
    """A packed buffer as the numbers that it holds."""
    if prec == "f64":
        return [buf.view(torch.float64)]
    if prec == "f32":
        return [buf.view(torch.float32)]
    f = buf.view(nfields, -1)   # per half-field: 48 bytes of FP16 a site, then one FP32 scale a site
    at = f.shape[1] // 52 * 48
    return [f[:, :at].view(torch.float16), f[:, at:].view(torch.float32)]


def prepare(case, seed):
    v, kind = _inputs(case, seed), case["kind"]
    s = dict(case=case, kind=kind)
    if kind == "batch":
        lats, xs, bs, dims = [], [], [], []
        for d, U, b in v["systems"]:
            lats.append(q.Lattice(d, case["kappa"], U, lo_precs=_stores(case["prec"]), mu=case["mu"]))
            dims.append(d)
            bs.append(b)
            xs.append(lats[-1].canon())
        prm = q.solve_params(solver=q.CGNR_EO, inner_prec=PREC[case["prec"]])
        n = q.qiral_solve_batch_workspace_bytes([t.handle for t in lats], prm)
        return dict(s, lats=lats, handles=[t.handle for t in lats], dims=dims, xs=xs, bs=bs, prm=prm,
                    ws=torch.empty(n, dtype=torch.uint8, device="cuda"))
    d = _dims(case)
    if kind == "field":   # packing needs a lattice handle, not its links
        lat = q.Lattice(d, 0.12, torch.eye(3, dtype=torch.complex128, device="cuda").expand(_sites(d) + (4, 3, 3)),
                        lo_precs=0)
        p = PREC[case["prec"]]
        s.update(lat=lat, psi=v["psi"], back=torch.zeros_like(v["psi"]), buf=lat.field(q.FULL, p, case["nrhs"]))
        s["out"] = _views(s["buf"], 2 * case["nrhs"], case["prec"])
        return s
    prec = case.get("prec", "f32")
    lat = q.Lattice(d, case["kappa"], v["U"], lo_precs=_stores(prec) | (q.LINKS_F32 if case.get("net") else 0),
                    mu=case.get("mu", 0.0))
    s.update(lat=lat)
    if kind == "op":
        op, n, p = case["op"], case["nrhs"], PREC[case["prec"]]
        full = op in ("D", "Ddag")
        sub = q.FULL if full else {"Heo": q.ODD, "Hoe": q.EVEN}.get(op, q.ODD)
        s.update(op=op, n=n, p=p, inp=lat.import_field(v["psi"], sub, p), buf=lat.field(q.FULL if full else q.EVEN, p, n),
                 tmp=None if full else lat.field(q.EVEN, p, n))
        s["out"] = _views(s["buf"], n * (2 if full else 1), case["prec"])
    elif kind == "solve":
        s.update(b=v["b"], x=torch.zeros_like(v["b"]),
                 kw=dict(solver=SOLVERS[case["solver"]], tol=1e-10, inner_prec=PREC[case["prec"]]))
        if case["net"]:   # a network's weights as it is created; its handle stays with the program
            s["net"] = q.Network(lat, 8)
            s["kw"].update(precond=s["net"].handle, system=q.SYSTEM_SCHUR)
    else:
        s["net"] = q.Network(lat, case["hidden"])
        s["net"].set_weights(v["w1"].cpu().numpy(), v["w2"].cpu().numpy())
        if kind == "network":
            s.update(inp=lat.import_field(v["psi"], q.FULL, q.F32), buf=lat.field(q.FULL, q.F32))
            s["out"] = _views(s["buf"], 2, "f32")
        else:
            s["seed"] = v["seed"]
    return s


def _stores(prec):
    return {"f64": 0, "f32": q.LINKS_F32, "f16s": q.LINKS_F16}[prec]


def run(s):
    kind, case = s["kind"], s["case"]
    if kind == "op":
        if s["op"] in ("Heo", "Hoe"):
            s["lat"].dslash_eo(s["buf"], s["inp"], 0 if s["op"] == "Heo" else 1, 0, s["p"], s["n"])
        else:
            s["lat"].apply_M(s["buf"], s["inp"], s["tmp"], OPS[s["op"]], s["p"], s["n"])
        return s["out"]
    if kind == "field":
        lat, p, n = s["lat"], PREC[case["prec"]], case["nrhs"]
        q.qiral_field_import(lat.handle, lat.dims, s["buf"], s["psi"], q.FULL, p, n)
        lat.export_field(s["buf"], q.FULL, p, n, out=s["back"])
        return s["out"] + [s["back"]]
    if kind == "solve":
        x, status, info = s["lat"].solve(s["b"], x_canon=s["x"], **s["kw"])
        return [x, status]
    if kind == "batch":
        status, info = q.qiral_solve_batch(s["handles"], s["dims"], s["xs"], s["bs"], s["prm"], ws=s["ws"])
        return [s["xs"], status]
    if kind == "network":
        s["net"].apply(s["buf"], s["inp"], adjoint=case["adjoint"])
        return s["out"]
    loss = s["net"].train(STEPS, lr=LR, seed=s["seed"])
    w1, w2 = s["net"].get_weights()
    return [[float(v) for v in loss], w1, w2]


def work(case):
    """What a pass cannot do without.  A solve's count of iterations is not known beforehand: the
    one of its workload to 1e-10 (about 40 for CGNR's methods, 14 for BiCGStab, 8 with the network)
    is taken, each with its operator applications (links, input and output once each)."""
    kind = case["kind"]
    dims = [_dims(dict(dims=t)) for t in case["dims"].split(",")]
    vh = sum(math.prod(d) // 2 for d in dims)
    if kind == "field":
        both = 2 * vh * case["nrhs"] * (192 + SITE_BYTES[case["prec"]])
        return dict(bytes=2 * both, flops=0)
    if kind == "op":
        sp, n = SITE_BYTES[case["prec"]], case["nrhs"]
        links = 8 * LINK_BYTES[case["prec"]] * vh   # each link of the lattice once
        halves = 2 if case["op"] in ("D", "Ddag") else 1
        hops = 1 if case["op"] in ("Heo", "Hoe") else 2
        return dict(bytes=links + 2 * halves * sp * n * vh, flops=hops * HOP_FLOPS * n * vh)
    if kind in ("solve", "batch"):
        n, prec = case.get("nrhs", 1), case["prec"]
        solver = case.get("solver", "cgnr")
        its = 8 if case.get("net") else 14 if solver == "bicgstab" else 40
        apply = 8 * LINK_BYTES[prec] * vh + 2 * SITE_BYTES[prec] * n * vh
        return dict(bytes=its * 2 * apply + 4 * 192 * n * vh, flops=its * 4 * HOP_FLOPS * n * vh)
    links = 8 * LINK_BYTES["f32"] * vh
    h = case["hidden"]
    if kind == "network":   # nine transports (264 flop a spin component pair) and one 4x4 product a path, twice
        return dict(bytes=links + 4 * 96 * vh, flops=2 * vh * 2 * 9 * (4 * 66 + 3 * 16 * 8))
    # per step: the pair, forward, backward in the data and the weights; activations kept between
    fields = 2 * vh * 96
    return dict(bytes=STEPS * (6 * links + (4 + 4 * h) * fields), flops=STEPS * 2 * vh * 9 * 5 * (264 + h * 3 * 16 * 8))


# ---------------------------------------------------------------------------
# 64-bit values in plain torch


def _gamma(mu):
    """The chiral basis: gamma_mu = [[0, B], [B^+, 0]], B_k = -i sigma_k, B_t = 1."""
    B = {0: [[0, -1j], [-1j, 0]], 1: [[0, -1], [1, 0]], 2: [[-1j, 0], [0, 1j]], 3: [[1, 0], [0, 1]]}[mu]
    B = torch.tensor(B, dtype=torch.complex128, device="cuda")
    g = torch.zeros(4, 4, dtype=torch.complex128, device="cuda")
    g[:2, 2:], g[2:, :2] = B, B.conj().T
    return g


def _colour(u, psi):
    return sum(u[..., :, b, None] * psi[..., b, None, :] for b in range(3))


def _transport(U, psi, p):
    """Path p of psi[n][t][z][y][x][colour][spin]: 0 itself, 1..4 from x + mu, 5..8 from x - mu."""
    if p == 0:
        return psi
    mu = (p - 1) % 4
    u, ax = U[..., mu, :, :], 3 - mu
    if p <= 4:
        return _colour(u, torch.roll(psi, -1, ax + 1))
    return torch.roll(_colour(u.conj().transpose(-1, -2), psi), 1, ax + 1)


def _spin(psi, m):
    """m on the spin index."""
    return (psi.reshape(-1, 4) @ m.T.contiguous()).reshape(psi.shape)


def _hop(U, psi, dag=False):
    out, one = torch.zeros_like(psi), torch.eye(4, dtype=torch.complex128, device="cuda")
    for mu in range(4):
        g = _gamma(mu) * (-1 if dag else 1)
        out += _spin(_transport(U, psi, 1 + mu), one - g)
        out += _spin(_transport(U, psi, 5 + mu), one + g)
    return out


def _mass(psi, kappa, mu, dag=False, inverse=False):
    """A = 1 + 2 i kappa mu gamma_5 and its relatives."""
    t = 2 * kappa * mu * (-1 if dag != inverse else 1)
    c = torch.tensor([1 + 1j * t, 1 + 1j * t, 1 - 1j * t, 1 - 1j * t], dtype=torch.complex128, device="cuda")
    return psi * c / (1 + t * t if inverse else 1.0)


def _dirac(U, psi, kappa, mu, dag=False):
    return _mass(psi, kappa, mu, dag) - kappa * _hop(U, psi, dag)


def _parity(d):
    t, z, y, x = (torch.arange(n, device="cuda") for n in _sites(d))
    return (t[:, None, None, None] + z[:, None, None] + y[:, None] + x) % 2


def _pack(psi, d, prec, subset):
    """The packed layout's numbers of a canonical field: 64-site blocks, units of 16 bytes."""
    par = _parity(d).reshape(-1)
    halves = []
    for p in ((0, 1) if subset == "full" else (subset,)):
        h = psi.reshape(psi.shape[0], -1, 12)[:, par == p]
        halves.append(torch.nn.functional.pad(torch.view_as_real(h), (0, 0, 0, 0, 0, -h.shape[1] % 64)))
    f = torch.stack(halves, 1)   # [rhs][half][site][12][2]
    if prec == "f16s":
        sc = f.abs().amax((-1, -2))
        f = f / torch.where(sc > 0, sc, torch.ones_like(sc))[..., None, None]
    per = {"f64": 2, "f32": 4, "f16s": 8}[prec]
    f = f.reshape(f.shape[0] * f.shape[1], -1, 64, 24 // per, per).transpose(2, 3)
    if prec == "f16s":
        return [f.reshape(f.shape[0], -1), sc.reshape(f.shape[0], -1)]
    return [f.reshape(-1)]


def _held(psi, prec):
    """A field as its storage class holds it."""
    if prec == "f64":
        return psi
    r = torch.view_as_real(psi.to(torch.complex64))
    if prec == "f16s":
        sc = r.abs().amax((-1, -2, -3), keepdim=True)
        sc = torch.where(sc > 0, sc, torch.ones_like(sc))
        r = (r / sc).to(torch.float16).to(torch.float64) * sc.to(torch.float64)
    return torch.view_as_complex(r.to(torch.float64).contiguous())


def _links_held(U, prec):
    if prec == "f64":
        return U
    r = torch.view_as_real(U[..., :2, :].contiguous())
    r = r.to(torch.float32 if prec == "f32" else torch.float16).to(torch.float64)
    r = torch.view_as_complex(r.contiguous())
    return torch.cat([r, _row2(r[..., 0, :], r[..., 1, :])[..., None, :]], dim=-2)


def _solve(U, b, kappa, mu):
    """BiCGStab on D x = b, all right-hand sides as one system, as far as 64 bits go."""
    x, r = torch.zeros_like(b), b.clone()
    rt, p, best = r.clone(), r.clone(), None
    rho, nb = torch.vdot(rt.view(-1), r.view(-1)), torch.linalg.vector_norm(b)
    for _ in range(300):
        v = _dirac(U, p, kappa, mu)
        al = rho / torch.vdot(rt.view(-1), v.view(-1))
        s = r - al * v
        t = _dirac(U, s, kappa, mu)
        om = torch.vdot(t.view(-1), s.view(-1)) / torch.vdot(t.view(-1), t.view(-1))
        x = x + al * p + om * s
        r = s - om * t
        if float(torch.linalg.vector_norm(r) / nb) < 1e-14:
            break
        new = torch.vdot(rt.view(-1), r.view(-1))
        p = r + (new / rho) * (al / om) * (p - om * v)
        rho = new
    return x


def _layers(U, w1, w2, psi):
    """The network on psi[1][...]: 1 -> hidden -> 1 channels."""
    hidden = w1.shape[1]
    t = [_transport(U, psi, p)[0] for p in range(9)]
    act = [sum(_spin(t[p], w1[p, i]) for p in range(9)) for i in range(hidden)]
    out = 0
    for p in range(9):
        out = out + _transport(U, sum(_spin(act[j], w2[p, j]) for j in range(hidden))[None], p)
    return out


def _philox(seed, step, n):
    """Six Philox4x32-10 blocks for each of n counters: [n][24] words."""
    M = 0xFFFFFFFF
    c = [torch.arange(n, device="cuda")[:, None].expand(n, 6).clone(),
         torch.arange(6, device="cuda")[None].expand(n, 6).clone(),
         torch.full((n, 6), step & M, device="cuda"), torch.full((n, 6), step >> 32, device="cuda")]
    k = [seed & M, seed >> 32]
    for _ in range(10):
        a, b = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57   # modulo 2^64: the low and high words are right
        c = [((b >> 32) & M) ^ c[1] ^ k[0], b & M, ((a >> 32) & M) ^ c[3] ^ k[1], a & M]
        k = [(k[0] + 0x9E3779B9) & M, (k[1] + 0xBB67AE85) & M]
    return torch.stack(c, -1).reshape(n, 24)


def _train(U, d, kappa, w1, w2, seed):
    w = [w1.to(torch.complex128), w2.to(torch.complex128)]
    m = [torch.zeros_like(torch.view_as_real(t)) for t in w]
    v = [torch.zeros_like(t) for t in m]
    losses = []
    for k in range(STEPS):
        u = (_philox(seed, k, math.prod(d)).to(torch.float64) + 0.5) / 2.0**32
        rad, ang = torch.sqrt(-2 * torch.log(u[:, 0::2])), 2 * math.pi * u[:, 1::2]
        y = torch.complex(rad * torch.cos(ang), rad * torch.sin(ang)).reshape((1,) + _sites(d) + (3, 4))
        src = _dirac(U, y, kappa, 0.0)
        w = [t.detach().requires_grad_(True) for t in w]
        e = _layers(U, w[0], w[1], src) - y
        loss = (e.real.square() + e.imag.square()).sum() / (y.real.square() + y.imag.square()).sum()
        grad = [torch.view_as_real(g.resolve_conj()) for g in torch.autograd.grad(loss, w)]
        losses.append(float(loss))
        new = []
        for i in range(2):
            m[i] = 0.9 * m[i] + 0.1 * grad[i]
            v[i] = 0.999 * v[i] + 0.001 * grad[i] ** 2
            mh, vh = m[i] / (1 - 0.9 ** (k + 1)), v[i] / (1 - 0.999 ** (k + 1))
            new.append(torch.view_as_complex(torch.view_as_real(w[i].detach()) - LR * mh / (vh.sqrt() + 1e-8)))
        w = new
    h = w1.shape[1]
    return [losses, w[0].reshape(9, h, 1, 4, 4), w[1].reshape(9, 1, h, 4, 4)]


def exact(case, seed):
    v, kind = _inputs(case, seed), case["kind"]
    if kind == "field":
        psi, d, prec = v["psi"], _dims(case), case["prec"]
        return _pack(psi, d, prec, "full") + [_held(psi, prec)]
    if kind == "batch":
        return [[_solve(U, b, case["kappa"], case["mu"]) for d, U, b in v["systems"]], None]
    d, U = _dims(case), v["U"]
    if kind == "solve":
        return [_solve(U, v["b"], case["kappa"], case["mu"]), None]
    if kind == "op":
        op, prec, kappa, mu = case["op"], case["prec"], case["kappa"], case["mu"]
        U, psi = _links_held(U, prec), _held(v["psi"], prec)
        if op in ("D", "Ddag"):
            return _pack(_dirac(U, psi, kappa, mu, op == "Ddag"), d, prec, "full")
        keep = (_parity(d) == (1 if op != "Hoe" else 0))[..., None, None]
        psi = psi * keep
        if op in ("Heo", "Hoe"):
            return _pack(_hop(U, psi), d, prec, 0 if op == "Heo" else 1)
        dag = op == "Sdag"
        e = _mass(_hop(U, psi, dag), kappa, mu, dag, inverse=True)
        return _pack(_mass(psi, kappa, mu, dag) - kappa**2 * _hop(U, e, dag), d, prec, 1)
    U = _links_held(U, "f32")
    if kind == "train":
        return _train(U, d, case["kappa"], v["w1"], v["w2"], v["seed"])
    w1, w2 = (t.to(torch.complex128) for t in (v["w1"], v["w2"]))
    psi = _held(v["psi"], "f32")
    if case["adjoint"]:   # N^+ has the layers' weights swapped, conjugated and on the mirrored paths
        mir = [0, 5, 6, 7, 8, 1, 2, 3, 4]
        w1, w2 = (t[mir].conj().transpose(-1, -2).contiguous() for t in (w2, w1))
    return _pack(_layers(U, w1, w2, psi), d, "f32", "full")
