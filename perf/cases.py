"""Workloads that the library's speed is measured on.

Each case is one pass of the work that a program built on this library does
again and again, through the public Python entry points: fitting steps and
operator applications of a few hundred microseconds, single designs from 24^3
to 256^3 in either precision and with each solver, a differentiable design
step, and the continuous-batching engine under a mixed and under a uniform
load.  Sizes and material data are those of ``workloads.py``, the tests and
``bench.py``; odd sizes stand for the grids that a user brings along.

``prepare`` makes what such a program holds before the call (charges, moduli,
a workspace, an engine), ``run`` is the pass, ``work`` what it cannot do
without, and ``exact`` the same results from plain torch in FP64.
"""
import numpy as np
import torch

from paper_2511_04025_amd import api, autograd, serving
from paper_2511_04025_amd.workloads import Design

DEV = "cuda"
# grids that the multigrid hierarchy coarsens (n = m 2^k, m <= 8)
MG_SIZES = (16, 20, 24, 28, 32, 40, 48, 56, 64, 80, 96, 112, 128)
# CG tolerances: that of the adjoint tests in mixed precision (C^H, whose error goes with the square, then has
# its last digits too and can be differenced between designs), the default in FP64
RTOL = {"mixed": 1e-7, "fp64": 1e-10}


def listed():
    return [
        # one step of the surface fit (2,048 points on the surface, 2,048 off it): the field there and its adjoint
        {"name": "fit_4096", "kind": "fit", "points": 4096, "charges": 24},
        # the stiffness operator inside a caller's own iteration, six load cases, an odd grid, single precision
        {"name": "operator_101_f32", "kind": "operator", "n": 101, "rhs": 6, "precision": "mixed"},
        # the occupancy of a design, for inspection and export
        {"name": "field_128", "kind": "field", "n": 128, "charges": 48, "vf": 0.1, "kappa": 0.0},
        # the smallest design, solved to the last digits: the reference calls of a test suite
        {"name": "shell_24_f64", "kind": "design", "n": 24, "charges": 16, "vf": 0.12, "void": 1e-3,
         "solver": "mg", "precision": "fp64"},
        # an ordinary design at preview resolution
        {"name": "shell_48", "kind": "design", "n": 48, "charges": 48, "vf": 0.1, "void": 1e-6,
         "solver": "mg", "precision": "mixed"},
        # a caller's own solid/void byte grid of a size that does not coarsen (the Jacobi path)
        {"name": "grid_45_auto", "kind": "grid", "n": 45, "charges": 32, "vf": 0.12, "void": 1e-3,
         "dtype": "uint8", "solver": "auto", "precision": "mixed"},
        # the headline resolution, one design at a time: what an interactive user waits for
        {"name": "shell_128", "kind": "design", "n": 128, "charges": 48, "vf": 0.1, "void": 1e-6,
         "solver": "mg", "precision": "mixed"},
        # the same with the culled solve on the active nodes
        {"name": "culled_128", "kind": "design", "n": 128, "charges": 48, "vf": 0.1, "void": 1e-6,
         "solver": "selective", "precision": "mixed"},
        # the largest grid of the workloads
        {"name": "shell_256", "kind": "design", "n": 256, "charges": 64, "vf": 0.1, "void": 1e-6,
         "solver": "mg", "precision": "mixed"},
        # one step of gradient-based design, eight logistic shells: forward, loss, adjoint to single-precision parameters
        {"name": "design_step_8x96", "kind": "step", "n": 96, "batch": 8, "charges": 32, "vf": 0.1, "solver": "mg",
         "precision": "mixed"},
        # the engine under a mixed load: three resolutions, more requests than slots
        {"name": "serve_mixed_12", "kind": "serve", "count": 12, "n": 0, "slots": 8, "solver": "mg"},
        # the engine under the headline load: eight designs at 128^3
        {"name": "serve_8x128", "kind": "serve", "count": 8, "n": 128, "slots": 8, "solver": "mg"},
    ]


def _log_int(rng, lo, hi):
    """A whole number spread evenly over the logarithm of [lo, hi]."""
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(("fit", "operator", "field", "design", "design", "design", "grid", "step", "serve"))
    vf = round(rng.uniform(0.08, 0.18), 4)
    charges = rng.randint(16, 64)
    if kind == "fit":
        return {"kind": kind, "points": _log_int(rng, 256, 32768), "charges": charges}
    if kind == "operator":
        return {"kind": kind, "n": _log_int(rng, 12, 160), "rhs": rng.randint(1, 6),
                "precision": rng.choice(("mixed", "fp64"))}
    if kind == "field":
        return {"kind": kind, "n": _log_int(rng, 16, 160), "charges": charges, "vf": vf,
                "kappa": rng.choice((0.0, 4.0))}
    if kind == "design":
        solver = rng.choice(("mg", "mg", "selective"))
        n = rng.choice(MG_SIZES) if solver == "mg" else _log_int(rng, 20, 128)
        return {"kind": kind, "n": n, "charges": charges, "vf": vf, "void": rng.choice((1e-3, 1e-6)),
                "solver": solver, "precision": rng.choice(("mixed", "mixed", "fp64"))}
    if kind == "grid":
        return {"kind": kind, "n": _log_int(rng, 20, 72), "charges": charges, "vf": vf, "void": 1e-3,
                "dtype": rng.choice(("uint8", "float32", "float64")), "solver": "auto",
                "precision": rng.choice(("mixed", "fp64"))}
    if kind == "step":
        solver, precision = rng.choice((("mg", "mixed"), ("mg", "mixed"), ("selective", "fp64")))
        return {"kind": kind, "n": rng.choice((24, 32, 40, 48, 64, 80, 96)), "batch": rng.randint(1, 6),
                "charges": charges, "vf": vf, "solver": solver, "precision": precision}
    return {"kind": kind, "count": rng.randint(2, 8), "n": rng.choice((0, 64, 96)), "slots": rng.randint(2, 8),
            "solver": rng.choice(("mg", "selective"))}


# ---- inputs ------------------------------------------------------------------
def _design(rng, n, charges, vf, void, kappa=0.0):
    """Uniform positions, magnitudes U[-1, 1] shifted to zero net charge."""
    q = rng.uniform(-1.0, 1.0, charges)
    return Design(pos=rng.random((charges, 3)), q=q - q.mean(), n=n, target_vf=vf, kappa=kappa, E_void=void)


def _designs(case, seed):
    """The designs of a case, from the seed alone."""
    rng = np.random.default_rng([seed, 4000])
    kind = case["kind"]
    if kind == "serve":  # resolutions and volume fractions as in the serving trace
        out = []
        for i in range(case["count"]):
            n = case["n"] or (64, 96, 128)[i % 3]
            out.append(_design(rng, n, int(rng.integers(16, 65)), float(rng.uniform(0.05, 0.2)), 1e-6))
        return out
    if kind == "step":
        n, m = case["n"], case["charges"]
        out = []
        for _ in range(case["batch"]):
            q = np.where(np.arange(m) < m // 2, 1.0, -1.0)
            out.append(Design(pos=rng.random((m, 3)).astype(np.float32).astype(np.float64), q=q, n=n,
                              target_vf=case["vf"], kappa=4.0 * n, E_void=1e-6))
        return out
    kappa = case.get("kappa", 0.0) * case["n"]
    return [_design(rng, case["n"], case["charges"], case["vf"], case.get("void", 1e-3), kappa)]


def _fit_inputs(case, seed):
    rng = np.random.default_rng([seed, 4001])
    m = case["charges"]
    q = np.where(np.arange(m) < m // 2, 1.0, -1.0)
    d = Design(pos=rng.random((m, 3)), q=q, n=2, alpha=rng.uniform(0.5, 1.5, (4, 4, 4)), thickness=0.1)
    return d, rng.random((case["points"], 3)), rng.standard_normal(case["points"])


def _operator_inputs(case, seed):
    """A solid/void grid (12 % solid) and random displacements."""
    n = case["n"]
    g = torch.Generator(device=DEV).manual_seed(seed)
    solid = torch.rand((n, n, n), generator=g, device=DEV) < 0.12
    E = solid.to(torch.float64).clamp(min=1e-6)
    p = torch.randn((case["rhs"], 3, n, n, n), generator=g, device=DEV, dtype=torch.float64)
    return E, p if case["precision"] == "fp64" else p.float()


def _grid_inputs(case, seed):
    d = _designs(case, seed)[0]
    solid = (_occupancy(d)[0] > 0.5).contiguous()
    if case["dtype"] == "uint8":
        return solid.to(torch.uint8)
    E = solid.to(torch.float64).clamp(min=case["void"])
    return E.float() if case["dtype"] == "float32" else E


def prepare(case, seed):
    kind, s = case["kind"], {"case": case}
    if kind == "fit":
        s["design"], pts, g = _fit_inputs(case, seed)
        s["pts"] = torch.tensor(pts, device=DEV)
        s["g"] = torch.tensor(g, device=DEV)
    elif kind == "operator":
        s["E"], s["p"] = _operator_inputs(case, seed)
    elif kind == "field":
        s["design"] = _designs(case, seed)[0]
    elif kind == "design":
        s["design"] = _designs(case, seed)[0]
        opts = api.B.make_opts(case["precision"], solver=case["solver"])
        s["ws"] = api.Workspace(api.workspace_bytes(s["design"], opts))
    elif kind == "grid":
        s["E"] = _grid_inputs(case, seed)
    elif kind == "step":
        ds = _designs(case, seed)
        s["spec"] = autograd.Spec(n=case["n"], thickness=autograd.initial_thickness(ds), kappa=ds[0].kappa,
                                  E_void=1e-6, precision=case["precision"], solver=case["solver"],
                                  rtol=RTOL[case["precision"]])
        s["pos"] = torch.tensor(np.stack([d.pos for d in ds]), dtype=torch.float32, requires_grad=True)
        s["q"] = torch.tensor(np.stack([d.q for d in ds]), dtype=torch.float32, requires_grad=True)
    else:
        s["designs"] = _designs(case, seed)
        opts = api.B.make_opts("mixed", solver=case["solver"])
        need = sorted((api.workspace_bytes(d, opts) for d in s["designs"]), reverse=True)
        s["engine"] = serving.Engine(sum(need[:case["slots"]]) + (64 << 20), max_slots=case["slots"],
                                     precision="mixed", rtol=RTOL["mixed"], solver=case["solver"])
    return s


# ---- one pass ----------------------------------------------------------------
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "fit":
        F = api.field_points(s["design"], s["pts"])
        return (F,) + tuple(api.field_points_grad(s["design"], s["pts"], s["g"]))
    if kind == "operator":
        return api.apply_stiffness(s["E"], s["p"], 0.3, precision=case["precision"])
    if kind == "field":
        return api.field(s["design"])
    if kind == "design":
        r = api.homogenize(s["design"], precision=case["precision"], rtol=RTOL[case["precision"]],
                           solver=case["solver"], workspace=s["ws"])
        return {"C": r["C"], "V": r["V"], "t": r["t"], "status": r["status"]}
    if kind == "grid":
        r = api.homogenize_field(s["E"], 0.3, E_solid=1.0, E_void=case["void"], precision=case["precision"],
                                 rtol=RTOL[case["precision"]], solver=case["solver"])
        return {"C": r["C"], "V": r["V"], "status": r["status"]}
    if kind == "step":
        s["pos"].grad = s["q"].grad = None
        C, V = autograd.Homogenize.apply(s["pos"], s["q"], s["spec"])
        (-autograd.voigt_bulk(C).sum()).backward()
        return {"C": C.detach(), "V": V, "pos": s["pos"].grad, "q": s["q"].grad}
    eng = s["engine"]
    for i, d in enumerate(s["designs"]):
        eng.submit(d, i)
    got = {}
    while len(got) < len(s["designs"]):
        eng.step(4)
        got.update(eng.poll())
    res = [got[i] for i in range(len(got))]
    return {"C": np.stack([r["C"] for r in res]), "V": np.array([r["V"] for r in res]),
            "status": np.array([r["status"] for r in res])}


def work(case):
    """Grids and vectors that the pass takes in or has to produce, once each.

    A solve cannot do without its moduli and the six displacement fields; the
    operations are one application of the element operator to those."""
    kind = case["kind"]
    if kind == "fit":
        m = case["points"]
        return {"bytes": 8 * (3 * m + m + 3 * m + m), "flops": 2 * m * (2 * 7 ** 3 + 2 * 7 ** 2)}
    if kind == "serve":
        ns = [case["n"] or (64, 96, 128)[i % 3] for i in range(case["count"])]
    else:
        ns = [case["n"]] * case.get("batch", 1)
    nn = float(sum(n ** 3 for n in ns))
    if kind == "field":
        return {"bytes": 48 * nn, "flops": 2 * nn * (4 * 7 + 3 * 7)}
    element = 2.0 * (45 * 3 + 24 * 4)  # multiply-adds of the factored element, the transforms and the corner sums
    if kind == "operator":
        size = 8 if case["precision"] == "fp64" else 4
        return {"bytes": nn * (8 + 2 * 3 * size * case["rhs"]), "flops": nn * case["rhs"] * element}
    size = 8 if case.get("precision") == "fp64" else 4
    active = 0.2 if case.get("solver") == "selective" else 1.0
    return {"bytes": nn * (8 + 2 * 18 * size * active), "flops": nn * 6 * element * active}


# ---- the same in FP64, with torch alone ---------------------------------------
K = 3  # truncation order of the series


def _basis(x):
    """1, cos 2 pi h x, sin 2 pi h x for h = 1 .. K, and derivatives: (M, 2K + 1) each."""
    val, der = [torch.ones_like(x)], [torch.zeros_like(x)]
    for h in range(1, K + 1):
        w = 2.0 * np.pi * h
        c, s = torch.cos(w * x), torch.sin(w * x)
        val += [c, s]
        der += [-w * s, w * c]
    return torch.stack(val, 1), torch.stack(der, 1)


def _coefficients(pos, q, alpha=None):
    """The charge sum of Eq. (6) as a tensor over the products of the 1D functions."""
    bx, by, bz = (_basis(pos[:, a])[0] for a in range(3))
    h = torch.tensor([(u + 1) // 2 for u in range(2 * K + 1)], device=pos.device)
    hh, kk, ll = h[:, None, None], h[None, :, None], h[None, None, :]
    zeros = (hh == 0).int() + (kk == 0).int() + (ll == 0).int()
    r2 = (hh * hh + kk * kk + ll * ll).double()
    w = torch.where(r2 > 0, 0.5 ** zeros.double() / r2.clamp(min=1.0), torch.zeros_like(r2))
    if alpha is not None:
        w = w * alpha[hh.expand_as(w), kk.expand_as(w), ll.expand_as(w)]
    return w * torch.einsum("j,ju,jv,jw->uvw", q, bx, by, bz)


def _grid_field(coef, n):
    """F and its gradient at the voxel centres, indexed [k, j, i]."""
    x = (torch.arange(n, device=coef.device, dtype=torch.float64) + 0.5) / n
    v, d = _basis(x)
    f = lambda a, b, c: torch.einsum("uvw,iu,jv,kw->kji", coef, a, b, c)
    return f(v, v, v), torch.stack([f(d, v, v), f(v, d, v), f(v, v, d)])


def _shell(F, G):
    gn = (G * G).sum(0).sqrt()
    return F.abs() / torch.maximum(gn, 1e-12 * gn.max().detach())


def _thickness(d, vf, kappa):
    """The midpoint of the two order statistics, or a bisection on the mean occupancy."""
    if kappa == 0.0:
        k = int(np.floor(vf * d.numel() + 0.5))
        s = d.reshape(-1).sort().values
        return float(0.5 * (s[k - 1] + s[k]))
    lo, hi = float(d.min()) - 40.0 / kappa, float(d.max()) + 40.0 / kappa
    for _ in range(200):
        t = 0.5 * (lo + hi)
        V = float(torch.sigmoid(kappa * (t - d)).mean())
        if abs(V - vf) <= 1e-12:
            break
        lo, hi = (t, hi) if V < vf else (lo, t)
    return t


def _occupancy(design):
    """(beta, d, F, G, t) of a design on its voxel grid."""
    pos = torch.tensor(design.pos, device=DEV)
    F, G = _grid_field(_coefficients(pos, torch.tensor(design.q, device=DEV)), design.n)
    d = _shell(F, G)
    t = _thickness(d, design.target_vf, design.kappa)
    beta = (d < t).double() if design.kappa == 0.0 else torch.sigmoid(design.kappa * (t - d))
    return beta, d, F, G, t


def _element(nu):
    """The 24 x 24 stiffness of the unit voxel (E = 1) and the six unit-strain
    corner displacements, by 2 x 2 x 2 Gauss points; dof 3 a + c, corner
    a = ax + 2 ay + 4 az."""
    lam, mu = nu / ((1 + nu) * (1 - 2 * nu)), 1 / (2 * (1 + nu))
    D = np.zeros((6, 6))
    D[:3, :3] = lam
    D[np.arange(6), np.arange(6)] += [2 * mu] * 3 + [mu] * 3
    corners = np.array([[a & 1, (a >> 1) & 1, a >> 2] for a in range(8)], float)
    K0 = np.zeros((24, 24))
    for g in np.ndindex(2, 2, 2):
        p = 0.5 + (np.array(g) - 0.5) / np.sqrt(3.0)
        f = np.where(corners > 0, p, 1 - p)
        sg = np.where(corners > 0, 1.0, -1.0)
        dN = np.stack([sg[:, 0] * f[:, 1] * f[:, 2], f[:, 0] * sg[:, 1] * f[:, 2], f[:, 0] * f[:, 1] * sg[:, 2]], 1)
        Bm = np.zeros((6, 24))
        for a in range(8):
            x, y, z = dN[a]
            Bm[:, 3 * a:3 * a + 3] = [[x, 0, 0], [0, y, 0], [0, 0, z], [0, z, y], [z, 0, x], [y, x, 0]]
        K0 += Bm.T @ D @ Bm / 8.0
    eps = np.zeros((6, 3, 3))
    for k, (i, j) in enumerate(((0, 0), (1, 1), (2, 2), (1, 2), (0, 2), (0, 1))):
        eps[k, i, j] = eps[k, j, i] = 1.0 if i == j else 0.5
    chi = np.einsum("kcd,ad->kac", eps, corners).reshape(6, 24)
    return torch.tensor(K0, device=DEV), torch.tensor(chi, device=DEV)


def _gather(u):
    """Nodal fields (m, 3, n, n, n) to element values (24, m, n^3)."""
    cols = []
    for a in range(8):
        r = torch.roll(u, (-(a >> 2), -((a >> 1) & 1), -(a & 1)), (2, 3, 4))
        cols += [r[:, c].reshape(u.shape[0], -1) for c in range(3)]
    return torch.stack(cols)


def _scatter(ue, n):
    """The transpose of _gather."""
    m = ue.shape[1]
    out = torch.zeros((m, 3, n, n, n), dtype=ue.dtype, device=ue.device)
    for a in range(8):
        v = ue[3 * a:3 * a + 3].transpose(0, 1).reshape(m, 3, n, n, n)
        out += torch.roll(v, (a >> 2, (a >> 1) & 1, a & 1), (2, 3, 4))
    return out


def _apply(E, p, K0):
    n = E.shape[0]
    ue = _gather(p)
    return _scatter((K0 @ ue.reshape(24, -1)).reshape(ue.shape) * E.reshape(1, 1, -1), n)


def _solve(E, nu):
    """(C, total element displacements chi + u (24, 6, n^3)) of a modulus grid,
    by Jacobi-preconditioned CG to the FP64 floor."""
    n = E.shape[0]
    K0, chi = _element(nu)
    fe = -(K0 @ chi.T)[:, :, None] * E.reshape(1, 1, -1)
    f = _scatter(fe, n)
    diag = _scatter((torch.diag(K0)[:, None, None] * E.reshape(1, 1, -1)), n)
    Dinv = torch.where(diag > 0, 1.0 / diag.clamp(min=1e-300), torch.zeros_like(diag))
    dot = lambda a, b: (a * b).sum((1, 2, 3, 4), keepdim=True)
    x, r = torch.zeros_like(f), f.clone()
    z = Dinv * r
    p, rho, ff = z.clone(), dot(r, z), dot(f, f).clamp(min=1e-300)
    for it in range(20000):
        q = _apply(E, p, K0)
        a = rho / dot(p, q).clamp(min=1e-300)
        x += a * p
        r -= a * q
        if it % 25 == 0 and float((dot(r, r) / ff).max()) <= 1e-24:
            break
        z = Dinv * r
        new = dot(r, z)
        p = z + (new / rho.clamp(min=1e-300)) * p
        rho = new
    ue = _gather(x) + chi.T[:, :, None]
    ke = (K0 @ ue.reshape(24, -1)).reshape(ue.shape)
    C = torch.einsum("aie,aje,e->ij", ue, ke, E.reshape(-1)) / n ** 3
    return C, ue, ke


def _moduli(design, solver):
    beta, _, _, _, t = _occupancy(design)
    if solver == "selective":  # voxels with beta <= 1e-3 are culled, the others carry E beta
        return torch.where(beta > 1e-3, beta, torch.zeros_like(beta)), beta.mean(), t
    return design.E_void + (1.0 - design.E_void) * beta, beta.mean(), t


def _exact_step(design, solver):
    """C, V and the gradient of -K_Voigt with respect to the positions and values."""
    E, V, t = _moduli(design, solver)
    C, ue, ke = _solve(E, 0.3)
    # dC_ij/dE_e = (chi + u)_i . K_0 (chi + u)_j / n^3; K_Voigt = sum of the 3 x 3 normal block / 9
    gE = -(ue[:, :3].sum(1) * ke[:, :3].sum(1)).sum(0) / (9.0 * design.n ** 3)
    pos = torch.tensor(design.pos, device=DEV, requires_grad=True)
    q = torch.tensor(design.q, device=DEV, requires_grad=True)
    d = _shell(*_grid_field(_coefficients(pos, q), design.n))
    beta = torch.sigmoid(design.kappa * (t - d))
    if solver == "selective":
        Et = torch.where(beta > 1e-3, beta, torch.zeros_like(beta))
    else:
        Et = design.E_void + (1.0 - design.E_void) * beta
    (gE.reshape(Et.shape) * Et).sum().backward()
    return C, V, pos.grad, q.grad


def exact(case, seed):
    kind = case["kind"]
    if kind == "fit":
        d, pts, g = _fit_inputs(case, seed)
        pos, q, al = (torch.tensor(v, device=DEV, requires_grad=True) for v in (d.pos, d.q, d.alpha))
        pts = torch.tensor(pts, device=DEV)
        bx, by, bz = (_basis(pts[:, a])[0] for a in range(3))
        F = torch.einsum("uvw,iu,iv,iw->i", _coefficients(pos, q, al), bx, by, bz)
        F.backward(torch.tensor(g, device=DEV))
        return (F.detach(), pos.grad, q.grad, al.grad)
    if kind == "operator":
        E, p = _operator_inputs(case, seed)
        K0, _ = _element(0.3)
        return torch.cat([_apply(E, p[k:k + 1].double(), K0) for k in range(p.shape[0])])
    if kind == "field":
        beta, d, F, G, t = _occupancy(_designs(case, seed)[0])
        return {"F": F, "G": G, "d": d, "beta": beta, "V": float(beta.mean()), "t": t}
    # thousands of iterations in plain torch: only where they end within seconds
    if kind == "serve" or case["n"] ** 3 * case.get("batch", 1) > 600000:
        return None
    if kind == "grid":
        E = _grid_inputs(case, seed)
        m = E.to(torch.float64).clamp(min=case["void"])
        V = float((E > 0).double().mean()) if case["dtype"] == "uint8" else float(m.mean() / m.max())
        return {"C": _solve(m, 0.3)[0], "V": V, "status": None}
    if kind == "design":
        d = _designs(case, seed)[0]
        E, V, t = _moduli(d, case["solver"])
        return {"C": _solve(E, 0.3)[0], "V": float(V), "t": t, "status": None}
    out = [_exact_step(d, case["solver"]) for d in _designs(case, seed)]
    C, V, gp, gq = (torch.stack(v) for v in zip(*out))
    return {"C": C, "V": V, "pos": gp, "q": gq}
