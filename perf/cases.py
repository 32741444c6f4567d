"""Timed cases of the library's main path: operator calls on canonical spinors,
operator chains on encoded fields, per-configuration setup, whole solves and
a burst of served solves, from 8^4 (a launch-latency problem) to 48^3 x 96 (an
HBM problem), in every storage format.

Every input is drawn on the device from a seed: links U = exp(i eps H) with H
traceless Hermitian and Gaussian, spinors complex Gaussian or spin-colour point
sources, t antiperiodic.  `exact` evaluates the same maths in complex128 with
plain torch.  Kinds of case:

  op      one call on canonical FP64 parity spinors (wilson_dslash,
          wilson_mat_pc or mdagm), conversions included
  fields  an iterative user of the fast path: encode once, apply the operator
          `chain` times on encoded fields, decode once
  setup   a new gauge configuration: fix it to temporal gauge, build the
          resident handle, rotate the source, apply the hopping term once
  solve   bicgstab_solve / cg_solve of (1 - kappa D) x = b
  serve   single-RHS solves of mixed lattice sizes through the scheduler
"""
import torch

import paper_0911_3191_amd as wd
from paper_0911_3191_amd.serve import Server

DEV = "cuda"
REAL_BYTES = {"fp64": 8, "fp32": 4, "i16": 2, "f16": 2}
SPINOR_BYTES = {"fp64": 192, "fp32": 96, "i16": 52, "f16": 52}
UK, DR = wd.WD_BASIS_UKQCD, wd.WD_BASIS_DEGRAND_ROSSI


def listed():
    return [
        # the smallest operator call: launches and host overhead decide it
        dict(name="mdagm-8x8x8x8-fp64", kind="op", op="mdagm", dims="8,8,8,8", prec="fp64", nrhs=1,
             dagger=0, recon=12, temporal=False, eps=0.3, kappa=0.12),
        # a lattice with Lz not a multiple of 8 and a last block that is not full; int16, adjoint, 5 RHS
        dict(name="mat_pc-20x14x10x18-i16-5rhs", kind="op", op="mat_pc", dims="20,14,10,18", prec="i16", nrhs=5,
             dagger=1, recon=12, temporal=False, eps=0.3, kappa=0.122),
        # the hopping term of a single-RHS half-precision solver on a medium lattice
        dict(name="chain-24x24x24x32-f16", kind="fields", dims="24,24,24,32", prec="f16", nrhs=1, basis="uk",
             chain=8, recon=12, temporal=False, eps=0.3, kappa=0.124),
        # M_hat with the most compressed links: 8 reals, temporal gauge, FP32
        dict(name="chain-32x32x32x64-fp32-recon8", kind="fields", dims="32,32,32,64", prec="fp32", nrhs=1,
             basis="dr", chain=4, recon=8, temporal=True, eps=0.3, kappa=0.124),
        # plain double precision on the large lattice
        dict(name="chain-48x48x48x96-fp64", kind="fields", dims="48,48,48,96", prec="fp64", nrhs=1, basis="uk",
             chain=4, recon=12, temporal=False, eps=0.3, kappa=0.124),
        # twelve spin-colour right-hand sides in binary16 on the large lattice
        dict(name="chain-48x48x48x96-f16-12rhs", kind="fields", dims="48,48,48,96", prec="f16", nrhs=12,
             basis="uk", chain=4, recon=12, temporal=False, eps=0.3, kappa=0.124),
        # what every new gauge configuration costs before the first solve
        dict(name="setup-24x24x24x32", kind="setup", dims="24,24,24,32", prec="f16", nrhs=1, recon=12, eps=0.3),
        # the smallest solve: plain FP64 BiCGstab to 1e-10
        dict(name="bicgstab-8x8x8x8-fp64", kind="solve", solver="bicgstab", dims="8,8,8,8", inner="fp64", nrhs=1,
             tol=1e-10, delta=0.0, graph=True, check_every=4, restart=False, source="gauss", eps=0.3, kappa=0.12),
        # mixed-precision solve of one source on a medium lattice
        dict(name="bicgstab-24x24x24x32-f16", kind="solve", solver="bicgstab", dims="24,24,24,32", inner="f16",
             nrhs=1, tol=1e-12, delta=0.1, graph=True, check_every=4, restart=False, source="gauss", eps=0.3,
             kappa=0.124),
        # CG on the normal equations, 12 point sources, rougher links
        dict(name="cg-24x24x24x32-f16-12rhs", kind="solve", solver="cg", dims="24,24,24,32", inner="f16", nrhs=12,
             tol=1e-12, delta=0.1, graph=True, check_every=4, restart=False, source="point", eps=0.5,
             kappa=0.1245),
        # a propagator: 12 point sources by mixed-precision BiCGstab on a production-size lattice
        dict(name="bicgstab-32x32x32x64-f16-12rhs", kind="solve", solver="bicgstab", dims="32,32,32,64",
             inner="f16", nrhs=12, tol=1e-12, delta=0.1, graph=True, check_every=0, restart=False, source="point",
             eps=0.3, kappa=0.124),
        # concurrent requests on the serving lattices: solves share the device
        dict(name="serve-burst-8", kind="serve", lattices="16,16,16,32;24,24,24,32;32,32,32,64", requests=8,
             inner="f16", tol=1e-12, delta=0.1, check_every=2, slots=8, eps=0.3),
    ]


def draw(rng):
    def dims(lo, hi, most):
        while True:
            base = lo * (hi / lo) ** rng.random()
            ext = [max(4, 2 * round(base * rng.uniform(0.75, 1.25) / 2)) for _ in range(3)]
            ext.append(max(4, 2 * round(base * rng.uniform(0.9, 2.0) / 2)))
            if _volume(ext) <= most:
                return ext

    def text(d):
        return ",".join(str(k) for k in d)

    def rhs(d, most):
        return max(1, min(rng.choice([1, 1, 1, 2, 3, 4, 5, 8, 12]), most // _volume(d)))

    eps, kappa = 0.3, round(rng.uniform(0.120, 0.1245), 5)
    prec = rng.choice(["fp64", "fp32", "i16", "f16", "f16"])
    links = dict(recon=rng.choice([12, 12, 12, 8]), temporal=rng.random() < 0.25)
    kind = rng.choice(["op", "op", "fields", "fields", "fields", "setup", "solve", "solve", "solve", "serve"])
    if kind == "op":
        d = dims(8, 48, 48 ** 3 * 96)
        return dict(kind=kind, op=rng.choice(["dslash", "mat_pc", "mdagm"]), dims=text(d), prec=prec,
                    nrhs=rhs(d, 6000000), dagger=rng.randrange(2), eps=eps, kappa=kappa, **links)
    if kind == "fields":
        d = dims(8, 48, 48 ** 3 * 96)
        return dict(kind=kind, dims=text(d), prec=prec, nrhs=rhs(d, 24000000), basis=rng.choice(["uk", "uk", "dr"]),
                    chain=rng.choice([2, 4, 6]), eps=eps, kappa=kappa, **links)
    if kind == "setup":
        d = dims(8, 32, 32 ** 3 * 64)
        return dict(kind=kind, dims=text(d), prec=prec, nrhs=rhs(d, 6000000), recon=links["recon"], eps=eps)
    if kind == "solve":
        solver = rng.choice(["bicgstab", "bicgstab", "cg"])
        inner = rng.choice(["fp64", "fp32", "i16", "f16", "f16"])
        d = dims(8, 32, 32 ** 3 * 64)
        return dict(kind=kind, solver=solver, dims=text(d), inner=inner, nrhs=rhs(d, 5000000), tol=1e-12,
                    delta=0.0 if inner == "fp64" else 0.1, graph=rng.random() < 0.75,
                    check_every=rng.choice([0, 2, 4]), restart=inner != "fp64" and rng.random() < 0.2,
                    source=rng.choice(["gauss", "point"]), eps=eps, kappa=kappa)
    lats = [text(dims(8, 24, 24 ** 3 * 48)) for _ in range(3)]
    return dict(kind=kind, lattices=";".join(lats), requests=rng.randrange(4, 13), inner=rng.choice(["i16", "f16"]),
                tol=1e-12, delta=0.1, check_every=rng.choice([0, 2, 4]), slots=rng.choice([4, 8, 16]), eps=eps)


# ---- what a program has in hand before the call -------------------------------------


def prepare(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    kind = case["kind"]
    if kind == "serve":
        return _prepare_serve(case, gen)
    dims = _dims(case["dims"])
    lat = wd.lattice(dims)
    V = _volume(dims)
    n = case["nrhs"]
    U = _links(dims, case["eps"], gen)
    s = dict(case=case, lat=lat)
    if kind == "setup":
        s["U"] = U
        s["b"] = _gauss((n, V, 4, 3, 2), gen)
        s["rb"] = torch.empty_like(s["b"])
        s["psi"] = _gauss((n, V // 2, 4, 3, 2), gen)
        s["out"] = torch.empty_like(s["psi"])
        s["ws"] = wd.new_operator_workspace(lat, case["prec"], n)
        return s
    if kind == "solve":
        s["gauge"] = wd.Gauge(lat, U, sorted({"fp64", case["inner"]}))
        s["b"] = _source(case["source"], dims, n, gen)
        s["x"] = torch.zeros_like(s["b"])
        s["params"] = wd.solve_params(tol=case["tol"], maxiter=20000, inner=case["inner"], delta=case["delta"],
                                      nrhs=n, use_graph=case["graph"], restart=case["restart"],
                                      check_every=case["check_every"])
        s["ws"] = wd.new_workspace(lat, s["params"], case["solver"])
        s["stream"] = torch.cuda.Stream()
        return s
    if case["temporal"]:
        U = _temporal_gauge(dims, U)[0]
    prec = case["prec"]
    s["gauge"] = wd.Gauge(lat, U, (prec,), recon=case["recon"], temporal=case["temporal"])
    s["in"] = _gauss((n, V // 2, 4, 3, 2), gen)
    s["out"] = torch.empty_like(s["in"])
    if kind == "op":
        s["ws"] = wd.new_operator_workspace(lat, prec, n)
    else:
        s["f"] = [wd.new_field(lat, prec, n) for _ in range(3)]
    return s


def run(state):
    return {"op": _run_op, "fields": _run_fields, "setup": _run_setup, "solve": _run_solve,
            "serve": _run_serve}[state["case"]["kind"]](state)


def _run_op(s):
    c = s["case"]
    g, out, inp, n = s["gauge"], s["out"], s["in"], c["nrhs"]
    if c["op"] == "dslash":
        wd.wilson_dslash(g, out, inp, 0, c["dagger"], c["prec"], n, s["ws"])
    elif c["op"] == "mat_pc":
        wd.wilson_mat_pc(g, c["kappa"], out, inp, c["dagger"], c["prec"], n, s["ws"])
    else:
        wd.mdagm(g, c["kappa"], out, inp, c["prec"], n, s["ws"])
    return out


def _run_fields(s):
    c = s["case"]
    g, prec, n = s["gauge"], c["prec"], c["nrhs"]
    a, b, odd = s["f"]
    basis = UK if c["basis"] == "uk" else DR
    wd.wd_spinor_encode_basis(s["lat"], prec, n, basis, a, s["in"])
    if basis == UK:  # hopping terms, even -> odd -> even
        for _ in range(c["chain"] // 2):
            wd.wd_dslash_field_basis(g, odd, a, 1, 0, prec, n, UK)
            wd.wd_dslash_field_basis(g, b, odd, 0, 0, prec, n, UK)
            a, b = b, a
    else:
        for _ in range(c["chain"] // 2):
            wd.wd_mat_pc_field(g, c["kappa"], b, a, odd, 0, prec, n)
            a, b = b, a
    wd.wd_spinor_decode_basis(s["lat"], prec, n, basis, s["out"], a)
    return s["out"]


def _run_setup(s):
    c = s["case"]
    lat, n, prec = s["lat"], c["nrhs"], c["prec"]
    Ut, g = wd.gauge_fix_temporal(lat, s["U"])
    gauge = wd.Gauge(lat, Ut, sorted({"fp64", prec}), recon=c["recon"], temporal=True)
    wd.wd_gauge_rotate_spinor(lat, g, s["rb"], s["b"], n)
    wd.wilson_dslash(gauge, s["out"], s["psi"], 0, 0, prec, n, s["ws"])
    return {"links": Ut, "g": g, "b": s["rb"], "out": s["out"]}


def _run_solve(s):
    c = s["case"]
    fn = wd.bicgstab_solve if c["solver"] == "bicgstab" else wd.cg_solve
    st, infos = fn(s["gauge"], c["kappa"], s["x"], s["b"], s["params"], s["ws"], s["stream"])
    if st != 0:
        raise RuntimeError(f"solve ended with status {st}: {wd.last_error()}")
    return s["x"]


def _run_serve(s):
    srv = s["server"]
    waiting = [srv.submit("bicgstab", g, kappa, x, b, s["params"]) for g, kappa, x, b in s["requests"]]
    while waiting:
        srv.pump()
        left = []
        for rid in waiting:
            done = srv.poll(rid)
            if done is None:
                left.append(rid)
            elif done[0] != 0:
                raise RuntimeError(f"request ended with status {done[0]}")
        waiting = left
    return [x for _, _, x, _ in s["requests"]]


def _prepare_serve(case, gen):
    lats = [_dims(t) for t in case["lattices"].split(";")]
    params = wd.solve_params(tol=case["tol"], maxiter=20000, inner=case["inner"], delta=case["delta"], nrhs=1,
                             use_graph=True, check_every=case["check_every"])
    gauges = []
    for d in lats:
        gauges.append(wd.Gauge(wd.lattice(d), _links(d, case["eps"], gen), sorted({"fp64", case["inner"]})))
    requests = []
    for k in range(case["requests"]):
        j = k % len(lats)
        b = _source("gauss", lats[j], 1, gen)
        requests.append((gauges[j], _serve_kappa(k), torch.zeros_like(b), b))
    need = max(wd.wd_solve_workspace_bytes(g.lat, params, "bicgstab") for g in gauges)
    torch.cuda.current_stream().synchronize()  # the server's streams do not wait on this one
    return dict(case=case, params=params, requests=requests,
                server=Server(int(case["slots"] * need * 1.05), max_slots=case["slots"]))


def _serve_kappa(k):
    return 0.120 + 0.0045 * ((k * 5) % 8) / 7


# ---- what a pass cannot do without ---------------------------------------------------


def work(case):
    if case["kind"] == "serve":
        lats = [_dims(t) for t in case["lattices"].split(";")]
        per = [_solve_work(lats[k % len(lats)], "bicgstab", case["inner"], 1, 30) for k in range(case["requests"])]
        return {"bytes": sum(p[0] for p in per), "flops": sum(p[1] for p in per)}
    d = _dims(case["dims"])
    V, n = _volume(d), case["nrhs"]
    canon = 192 * (V // 2) * n
    if case["kind"] == "setup":
        # U read, U' and g written, links encoded in one or two formats, b rotated, one hopping term
        formats = sum(REAL_BYTES[p] for p in {"fp64", case["prec"]})
        nbytes = V * (2 * 576 + 144) + V * 4 * case["recon"] * formats + 4 * canon + 2 * canon
        return {"bytes": nbytes + _link_bytes(d, case["prec"], case["recon"], True), "flops": n * 1320 * V // 2}
    if case["kind"] == "solve":
        its = 50 if case["solver"] == "cg" else 31
        nbytes, flops = _solve_work(d, case["solver"], case["inner"], n, its)
        return {"bytes": nbytes, "flops": flops}
    links = _link_bytes(d, case["prec"], case["recon"], case["temporal"])
    if case["kind"] == "op":  # the links, the spinor in and the spinor out
        hops = {"dslash": 1, "mat_pc": 2, "mdagm": 4}[case["op"]]
        return {"bytes": links + 2 * canon, "flops": hops * n * 1320 * V // 2}
    field = SPINOR_BYTES[case["prec"]] * (V // 2) * n
    hops = case["chain"]
    nbytes = 2 * (canon + field) + hops * (links + 2 * field)
    if case["basis"] == "dr":  # x + a D y reads x as well
        nbytes += hops // 2 * field
    return {"bytes": nbytes, "flops": hops * n * 1320 * V // 2}


def _link_bytes(d, prec, recon, temporal):
    kept = 3 + 1 / d[3] if temporal else 4
    return int(_volume(d) * kept * recon * REAL_BYTES[prec])


def _solve_work(d, solver, inner, n, its):
    """Bytes and flops of a solve of `its` inner iterations: the hopping terms and
    the vector updates of each iteration, each field once, and the FP64
    source and solution."""
    Vh = _volume(d) // 2
    links, field = _link_bytes(d, inner, 12, False), SPINOR_BYTES[inner] * Vh * n
    hops, fields = (4, 4 * 2 + 2 + 7) if solver == "cg" else (4, 4 * 2 + 3 + 4 + 3 + 7)
    nbytes = its * (hops * links + fields * field) + 2 * 384 * Vh * n
    return nbytes, its * n * Vh * (hops * 1320 + 24 * 15)


# ---- inputs --------------------------------------------------------------------------


def _dims(text):
    return tuple(int(t) for t in text.split(","))


def _volume(d):
    return d[0] * d[1] * d[2] * d[3]


def _grid(d):
    return (d[3], d[2], d[1], d[0])  # tensors run over [t, z, y, x]


def _gauss(shape, gen):
    return torch.randn(shape, generator=gen, dtype=torch.float64, device=DEV)


def _source(kind, d, n, gen):
    V = _volume(d)
    if kind == "gauss":
        return _gauss((n, V, 4, 3, 2), gen)
    # spin-colour unit vectors at one site that the seed picks
    b = torch.zeros((n, V, 4, 3, 2), dtype=torch.float64, device=DEV)
    site = int(torch.randint(V, (1,), generator=gen, device=DEV))
    for k in range(n):
        b[k, site, (k % 12) // 3, k % 3, 0] = 1.0
    return b


def _mm(A, B):
    """3x3 products of matrices kept as lists of component tensors."""
    out = []
    for i in range(3):
        row = []
        for j in range(3):
            c = A[i][0] * B[0][j]
            c = c.addcmul_(A[i][1], B[1][j])
            row.append(c.addcmul_(A[i][2], B[2][j]))
        out.append(row)
    return out


def _dagger(A):
    return [[A[j][i].conj().resolve_conj() for j in range(3)] for i in range(3)]


def _links(d, eps, gen):
    """exp(i eps H), H = (A + A^dagger) / 2 less its trace, A complex Gaussian."""
    V = _volume(d)
    U = torch.empty((V, 4, 3, 3, 2), dtype=torch.float64, device=DEV)
    for mu in range(4):
        diag = [eps * _gauss((V,), gen) for _ in range(3)]
        mean = (diag[0] + diag[1] + diag[2]) / 3
        Q = [[None] * 3 for _ in range(3)]
        for i in range(3):
            Q[i][i] = torch.complex(torch.zeros_like(mean), diag[i] - mean)
            for j in range(i):
                h = torch.view_as_complex(_gauss((V, 2), gen)) * (eps * 0.5 ** 0.5)
                Q[i][j], Q[j][i] = 1j * h, 1j * h.conj()
        # Horner: 1 + Q (1 + Q/2 (1 + Q/3 (...)))
        E = [[(1.0 + q / 12 if i == j else q / 12) for j, q in enumerate(row)] for i, row in enumerate(Q)]
        for k in range(11, 0, -1):
            E = _mm(Q, E)
            E = [[(1.0 + q / k if i == j else q / k) for j, q in enumerate(row)] for i, row in enumerate(E)]
        a, b = E[0], E[1]
        norm = torch.sqrt(sum(z.real ** 2 + z.imag ** 2 for z in a))
        a = [z / norm for z in a]
        ab = sum(x.conj() * y for x, y in zip(a, b))
        b = [y - ab * x for x, y in zip(a, b)]
        norm = torch.sqrt(sum(z.real ** 2 + z.imag ** 2 for z in b))
        b = [z / norm for z in b]
        c = [(a[(j + 1) % 3] * b[(j + 2) % 3] - a[(j + 2) % 3] * b[(j + 1) % 3]).conj() for j in range(3)]
        for i, row in enumerate((a, b, c)):
            for j, z in enumerate(row):
                U[:, mu, i, j] = torch.view_as_real(z.resolve_conj())
    return U


# ---- the same maths in 64 bits -----------------------------------------------------------


def _parts(d, U):
    """W[mu][i][j][t, z, y, x] of canonical links."""
    W = torch.view_as_complex(U).view(_grid(d) + (4, 3, 3))
    return [[[W[..., mu, i, j].contiguous() for j in range(3)] for i in range(3)] for mu in range(4)]


def _canonical(d, W):
    U = torch.empty((_volume(d), 4, 3, 3, 2), dtype=torch.float64, device=DEV)
    for mu in range(4):
        for i in range(3):
            for j in range(3):
                U[:, mu, i, j] = torch.view_as_real(W[mu][i][j].contiguous()).view(-1, 2)
    return U


def _temporal_gauge(d, U):
    """(U', g): g(t = 0) = 1, g(t + 1) = g(t) U_t(t), U'_mu(x) = g(x) U_mu(x) g(x + mu)^dagger."""
    W = _parts(d, U)
    g = [[torch.zeros_like(W[0][0][0]) for _ in range(3)] for _ in range(3)]
    for i in range(3):
        g[i][i][0] = 1.0
    for t in range(d[3] - 1):
        nxt = _mm([[z[t] for z in row] for row in g], [[z[t] for z in row] for row in W[3]])
        for i in range(3):
            for j in range(3):
                g[i][j][t + 1] = nxt[i][j]
    gd = _dagger(g)
    for mu in range(4):
        W[mu] = _mm(_mm(g, W[mu]), [[torch.roll(z, -1, 3 - mu) for z in row] for row in gd])
    flat = torch.empty((_volume(d), 3, 3, 2), dtype=torch.float64, device=DEV)
    for i in range(3):
        for j in range(3):
            flat[:, i, j] = torch.view_as_real(g[i][j]).view(-1, 2)
    return _canonical(d, W), flat


# gamma_mu = [[0, A], [A^dagger, 0]]: row k of A has its entry in column P[k] with value PH[k]
_P = [(1, 0), (1, 0), (0, 1), (0, 1)]
_PH = [(1j, 1j), (-1.0, 1.0), (1j, -1j), (1.0, 1.0)]


class _Exact:
    """D, M_hat and their inverses on [n, t, z, y, x] component tensors psi[spin][colour]."""

    def __init__(self, d, U):
        self.d, self.W = d, _parts(d, U)
        self.Wd = [_dagger(w) for w in self.W]
        x, y, z, t = (torch.arange(k, device=DEV) for k in d)
        par = (t[:, None, None, None] + z[:, None, None] + y[:, None] + x) & 1
        self.even = (par == 0).to(torch.float64)
        self.odd = 1.0 - self.even
        lex = torch.arange(_volume(d), device=DEV)
        self.index = [lex[par.reshape(-1) == p] for p in (0, 1)]  # cb order is lex order within a parity

    def load(self, a, parity=None):
        """Canonical spinors (one parity, or the full lattice) to component tensors."""
        n = a.shape[0]
        out = []
        for s in range(4):
            row = []
            for c in range(3):
                z = torch.view_as_complex(a[:, :, s, c].contiguous())
                if parity is not None:
                    full = torch.zeros((n, _volume(self.d)), dtype=torch.complex128, device=DEV)
                    full[:, self.index[parity]] = z
                    z = full
                row.append(z.view((n,) + _grid(self.d)))
            out.append(row)
        return out

    def store(self, psi, parity=None):
        n = psi[0][0].shape[0]
        V = _volume(self.d)
        out = torch.empty((n, V if parity is None else V // 2, 4, 3, 2), dtype=torch.float64, device=DEV)
        for s in range(4):
            for c in range(3):
                z = psi[s][c].reshape(n, V)
                if parity is not None:
                    z = z[:, self.index[parity]]
                out[:, :, s, c] = torch.view_as_real(z.contiguous())
        return out

    def shift(self, z, mu, back):
        out = torch.roll(z, 1 if back else -1, 4 - mu)
        if mu == 3:  # antiperiodic in t
            out[:, 0 if back else -1] *= -1.0
        return out

    def hop(self, psi, dagger=0):
        """D psi: sum over mu of (1 - gamma) U(x) psi(x + mu) + (1 + gamma) U(x - mu)^dagger psi(x - mu)."""
        out = [[torch.zeros_like(psi[0][0]) for _ in range(3)] for _ in range(4)]
        for mu in range(4):
            for back in (False, True):
                sign = (1.0 if back else -1.0) * (-1.0 if dagger else 1.0)
                for k in range(2):
                    lo, ph = 2 + _P[mu][k], sign * _PH[mu][k]
                    h = [psi[k][c] + ph * psi[lo][c] for c in range(3)]
                    if back:
                        w = [self.shift(sum(self.Wd[mu][i][j] * h[j] for j in range(3)), mu, True) for i in range(3)]
                    else:
                        h = [self.shift(z, mu, False) for z in h]
                        w = [sum(self.W[mu][i][j] * h[j] for j in range(3)) for i in range(3)]
                    back_ph = sign * complex(_PH[mu][k]).conjugate()
                    for c in range(3):
                        out[k][c] += w[c]
                        out[lo][c] += back_ph * w[c]
        return out

    def mhat(self, psi, kappa, dagger=0):
        """psi - kappa^2 D D psi for an even psi."""
        t = self.hop(self.hop(psi, dagger), dagger)
        return [[a - kappa * kappa * b for a, b in zip(x, y)] for x, y in zip(psi, t)]

    def solve(self, b, kappa):
        """(1 - kappa D) x = b: even-odd BiCGstab until the residual stops at rounding."""
        Db = self.hop([[self.odd * z for z in row] for row in b])
        rhs = [[self.even * (z + kappa * y) for z, y in zip(r, q)] for r, q in zip(b, Db)]
        x = self._bicgstab(rhs, kappa)
        Dx = self.hop(x)
        return [[z + self.odd * (y + kappa * w) for z, y, w in zip(r, q, s)] for r, q, s in zip(x, b, Dx)]

    def _bicgstab(self, b, kappa):
        def flat(psi):
            return torch.stack([z for row in psi for z in row], 1)  # [n, 12, t, z, y, x]

        def split(v):
            return [[v[:, 3 * s + c] for c in range(3)] for s in range(4)]

        def dot(u, v):
            return (u.conj() * v).sum(dim=(1, 2, 3, 4, 5))

        def each(a):
            return a.view(-1, 1, 1, 1, 1, 1)

        B = flat(b)
        norm = torch.sqrt(dot(B, B).real)
        x, r = torch.zeros_like(B), B.clone()
        for _ in range(3):  # restarted from the true residual
            rt, p = r.clone(), r.clone()
            rho = dot(rt, r)
            for _ in range(200):
                v = flat(self.mhat(split(p), kappa))
                alpha = rho / dot(rt, v)
                s = r - each(alpha) * v
                t = flat(self.mhat(split(s), kappa))
                omega = dot(t, s) / dot(t, t)
                x += each(alpha) * p + each(omega) * s
                r = s - each(omega) * t
                if float((torch.sqrt(dot(r, r).real) / norm).max()) < 2e-15:
                    break
                new = dot(rt, r)
                p = r + each(new / rho * alpha / omega) * (p - each(omega) * v)
                rho = new
            r = B - flat(self.mhat(split(x), kappa))
            if float((torch.sqrt(dot(r, r).real) / norm).max()) < 3e-15:
                break
        return split(x)


def exact(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    kind = case["kind"]
    if kind == "serve":
        lats = [_dims(t) for t in case["lattices"].split(";")]
        fields = [_links(d, case["eps"], gen) for d in lats]
        out = []
        for k in range(case["requests"]):
            d = lats[k % len(lats)]
            b = _source("gauss", d, 1, gen)
            if _volume(d) > 600000:  # left out: the 64-bit solve takes too long
                out.append(None)
                continue
            e = _Exact(d, fields[k % len(lats)])
            out.append(e.store(e.solve(e.load(b), _serve_kappa(k))))
        return out
    d = _dims(case["dims"])
    V, n = _volume(d), case["nrhs"]
    U = _links(d, case["eps"], gen)
    if kind == "solve":
        if V * n > 6000000:  # the 64-bit solve takes too long
            return None
        b = _source(case["source"], d, n, gen)
        e = _Exact(d, U)
        return e.store(e.solve(e.load(b), case["kappa"]))
    if kind == "setup":
        b = _gauss((n, V, 4, 3, 2), gen)
        psi = _gauss((n, V // 2, 4, 3, 2), gen)
        Ut, g = _temporal_gauge(d, U)
        G = torch.view_as_complex(g)
        rb = torch.view_as_complex(b)
        rb = torch.stack([sum(G[:, i, j, None] * rb[..., j] for j in range(3)) for i in range(3)], -1)
        e = _Exact(d, Ut)
        return {"links": Ut, "g": g, "b": torch.view_as_real(rb), "out": e.store(e.hop(e.load(psi, 1)), 0)}
    psi = _gauss((n, V // 2, 4, 3, 2), gen)
    if case["temporal"]:
        U = _temporal_gauge(d, U)[0]
    e = _Exact(d, U)
    out = torch.empty_like(psi)
    for k in range(n):  # one right-hand side at a time bounds the memory
        if kind == "op" and case["op"] == "dslash":
            out[k:k + 1] = e.store(e.hop(e.load(psi[k:k + 1], 1), case["dagger"]), 0)
            continue
        v = e.load(psi[k:k + 1], 0)
        if kind == "op" and case["op"] == "mat_pc":
            v = e.mhat(v, case["kappa"], case["dagger"])
        elif kind == "op":
            v = e.mhat(e.mhat(v, case["kappa"]), case["kappa"], 1)
        else:
            for _ in range(case["chain"] // 2):
                v = e.hop(e.hop(v)) if case["basis"] == "uk" else e.mhat(v, case["kappa"])
        out[k:k + 1] = e.store(v, 0)
    return out
