"""Timed cases of the coupled block solver's public entry points.

Every input is synthetic and seeded: hexahedral boxes with jittered nodes, the
density-based 5x5 matrix from cell states and face areas, the pressure-based
4x4 matrix from face coefficients, cells in mesh order or renumbered at random.
A case is a dict of plain values:

  path              what a pass runs (the functions _run_* below)
  n                 block size: 4 pressure-based, 5 density-based
  nx ny nz          cells of the box (a batch: count, and cells from lo to hi)
  precision solver precond smoother cycle   options of the solver
  renumbered stretch walls                  cell order, wall-normal growth,
                                            boundary faces

Solves start from a right side b = A x* with a known x*, so the exact solution
needs no second solver.  Their tolerance is that of verification solves and of
gradients checked by differences (1e-12).
"""
import math

import torch

import paper_2403_07882_amd as P

F64 = torch.float64


# ------------------------------------------------------------------ geometry
def _gen(seed, salt=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + salt)
    return g


def _rand(g, *shape, lo=0.0, hi=1.0):
    return lo + (hi - lo) * torch.rand(*shape, generator=g, dtype=F64, device="cuda")


def _dot(a, b):
    return (a * b).sum(-1)


def _mesh(nx, ny, nz, g, stretch=1.0):
    """A jittered hexahedral box, node spacing h = 1/nz (z spacing growing by
    `stretch` per layer towards h).  Per axis: area vectors and centres of all
    node planes, oriented towards the higher cell; cell centres and volumes."""
    h = 1.0 / nz
    dz = torch.full((nz,), h, dtype=F64, device="cuda")
    if stretch > 1.0:
        dz = torch.minimum(dz, h * 1e-3 * stretch ** torch.arange(nz, dtype=F64, device="cuda"))
    z = torch.cat([torch.zeros(1, dtype=F64, device="cuda"), torch.cumsum(dz, 0)])
    ax = torch.arange(nx + 1, dtype=F64, device="cuda") * h
    ay = torch.arange(ny + 1, dtype=F64, device="cuda") * h
    X = torch.stack(torch.meshgrid(z, ay, ax, indexing="ij")[::-1], dim=-1).contiguous()     # [k, j, i, xyz]
    jit = _rand(g, nz + 1, ny + 1, nx + 1, 3, lo=-0.2, hi=0.2)
    jit[..., :2] *= h
    step = torch.cat([dz[:1], torch.minimum(dz[1:], dz[:-1]), dz[-1:]])
    jit[..., 2] *= step[:, None, None]
    X[1:-1, 1:-1, 1:-1] += jit[1:-1, 1:-1, 1:-1]
    C = (X[:-1, :-1, :-1] + X[:-1, :-1, 1:] + X[:-1, 1:, :-1] + X[:-1, 1:, 1:]
         + X[1:, :-1, :-1] + X[1:, :-1, 1:] + X[1:, 1:, :-1] + X[1:, 1:, 1:]) * 0.125
    quads = [(X[:-1, :-1], X[:-1, 1:], X[1:, 1:], X[1:, :-1]),
             (X[:-1, :, :-1], X[1:, :, :-1], X[1:, :, 1:], X[:-1, :, 1:]),
             (X[:, :-1, :-1], X[:, :-1, 1:], X[:, 1:, 1:], X[:, 1:, :-1])]
    S, c = [], []
    for p0, p1, p2, p3 in quads:
        S.append(0.5 * torch.linalg.cross(p2 - p0, p3 - p1, dim=-1))
        c.append(0.25 * (p0 + p1 + p2 + p3))
    vol = torch.zeros(nz, ny, nx, dtype=F64, device="cuda")
    for a in range(3):
        q = _dot(S[a], c[a]) / 3.0
        vol += _hi(q, a) - _lo(q, a)
    return {"h": h, "S": S, "c": c, "C": C, "vol": vol, "shape": (nz, ny, nx)}


# slices along mesh axis a (x, y, z = tensor dims 2, 1, 0) of plane and cell arrays
def _lo(q, a):
    return q.narrow(2 - a, 0, q.shape[2 - a] - 1)


def _hi(q, a):
    return q.narrow(2 - a, 1, q.shape[2 - a] - 1)


def _inner(q, a):
    return q.narrow(2 - a, 1, q.shape[2 - a] - 2)


def _end(q, a, last):
    return q.narrow(2 - a, q.shape[2 - a] - 1 if last else 0, 1)


def _faces(nx, ny, nz):
    ids = torch.arange(nx * ny * nz, dtype=torch.int32, device="cuda").reshape(nz, ny, nx)
    return (torch.cat([_lo(ids, a).reshape(-1) for a in range(3)]),
            torch.cat([_hi(ids, a).reshape(-1) for a in range(3)]))


# ------------------------------------------------------------------ matrices
# A matrix is kept on the grid while it is formed: diag[nz, ny, nx, n, n] and
# per axis up[a], lo[a] over the inner planes (row of the lower cell, column of
# the higher one, and the reverse), so every sum runs in a fixed order.
def _apply(M, x):
    """A x on the grid (x[nz, ny, nx, n])."""
    mv = lambda B, v: (B * v.unsqueeze(-2)).sum(-1)
    y = mv(M["diag"], x)
    for a in range(3):
        if M["up"][a].numel():
            _lo(y, a).add_(mv(M["up"][a], _hi(x, a)))
            _hi(y, a).add_(mv(M["lo"][a], _lo(x, a)))
    return y


def _apply_t(M, x):
    mv = lambda B, v: (B * v.unsqueeze(-1)).sum(-2)
    y = mv(M["diag"], x)
    for a in range(3):
        if M["up"][a].numel():
            _lo(y, a).add_(mv(M["lo"][a], _hi(x, a)))
            _hi(y, a).add_(mv(M["up"][a], _lo(x, a)))
    return y


def _luo_fields(m, g):
    """States and geometry of the density-based assembly (Mach 0.5 free stream
    with perturbations, CFL about 10)."""
    N, gamma = m["vol"].numel(), 1.4
    rho = _rand(g, N, lo=0.8, hi=1.2)
    p = _rand(g, N, lo=0.8, hi=1.2) / gamma
    vel = torch.tensor([0.5, 0.1, 0.05], dtype=F64, device="cuda") + 0.05 * torch.randn(
        N, 3, generator=g, dtype=F64, device="cuda")
    Sf = torch.cat([_inner(m["S"][a], a).reshape(-1, 3) for a in range(3)])
    area = torch.stack([m["S"][a].norm(dim=-1).mean() for a in range(3)]).max()
    lam = _rand(g, Sf.shape[0], hi=0.05)
    cfl = 10.0 * _rand(g, N, lo=0.5, hi=2.0)
    Q = torch.cat([rho[:, None], rho[:, None] * vel, (p / (gamma - 1) + 0.5 * rho * _dot(vel, vel))[:, None]], 1)
    v_dt = area * (vel.norm(dim=1) + torch.sqrt(gamma * p / rho)) / cfl
    return {"Q": Q.contiguous(), "Sf": Sf.contiguous(), "lam_visc": lam, "v_dt": v_dt, "gamma": gamma}


def _euler_jac(Q, s, gamma):
    """d(F(Q).s)/dQ of an ideal gas, [..., 5, 5]."""
    u = Q[..., 1:4] / Q[..., :1]
    q2 = _dot(u, u)
    g1 = gamma - 1.0
    p = g1 * (Q[..., 4] - 0.5 * Q[..., 0] * q2)
    H = (Q[..., 4] + p) / Q[..., 0]
    V, phi = _dot(u, s), 0.5 * g1 * q2
    J = torch.zeros(*Q.shape[:-1], 5, 5, dtype=F64, device=Q.device)
    J[..., 0, 1:4] = s
    for k in range(3):
        J[..., 1 + k, 0] = phi * s[..., k] - u[..., k] * V
        for c in range(3):
            J[..., 1 + k, 1 + c] = u[..., k] * s[..., c] - g1 * u[..., c] * s[..., k]
        J[..., 1 + k, 1 + k] += V
        J[..., 1 + k, 4] = g1 * s[..., k]
    J[..., 4, 0] = V * (phi - H)
    for c in range(3):
        J[..., 4, 1 + c] = H * s[..., c] - g1 * u[..., c] * V
    J[..., 4, 4] = gamma * V
    return J, u, H


def _luo_matrix(m, f):
    """The matrix that the density-based assembly forms from `f`."""
    nz, ny, nx = m["shape"]
    gamma, Q = f["gamma"], f["Q"].reshape(nz, ny, nx, 5)
    eye = torch.eye(5, dtype=F64, device="cuda")
    diag = f["v_dt"].reshape(nz, ny, nx, 1, 1) * eye
    up, lo, at = [], [], 0
    for a in range(3):
        s = _inner(m["S"][a], a)
        count = s.shape[0] * s.shape[1] * s.shape[2]
        lv = f["lam_visc"][at:at + count].reshape(s.shape[:3])
        at += count
        Jl, ul, Hl = _euler_jac(_lo(Q, a), s, gamma)
        Jr, ur, Hr = _euler_jac(_hi(Q, a), s, gamma)
        wl, wr = torch.sqrt(_lo(Q, a)[..., 0]), torch.sqrt(_hi(Q, a)[..., 0])
        ua = (wl[..., None] * ul + wr[..., None] * ur) / (wl + wr)[..., None]
        Ha = (wl * Hl + wr * Hr) / (wl + wr)
        c = torch.sqrt((gamma - 1.0) * (Ha - 0.5 * _dot(ua, ua)))
        Sm = torch.sqrt(_dot(s, s))
        L = (_dot(ua, s).abs() + c * Sm + lv * Sm)[..., None, None] * eye
        up.append(0.5 * (Jr - L))
        lo.append(0.5 * (-Jl - L))
        _lo(diag, a).add_(0.5 * (Jl + L))
        _hi(diag, a).add_(0.5 * (-Jr + L))
    return {"diag": diag, "up": up, "lo": lo}


def _pu_fields(m, g):
    """Face geometry and fields of the pressure-based assembly, per axis: area
    vector, owner weight, centroid distance, flux of a smooth flow, viscosity;
    and the cell sums that boundary faces and relaxation add to the diagonals."""
    nz, ny, nx = m["shape"]
    u0 = _rand(g, 3, lo=0.2, hi=1.0)
    fc = []
    for a in range(3):
        S, x = _inner(m["S"][a], a), _inner(m["c"][a], a)
        d = _hi(m["C"], a) - _lo(m["C"], a)
        u = u0 * (1.0 + 0.3 * torch.sin(2.0 * math.pi * x[..., [1, 2, 0]]))
        fx = _dot(S, _hi(m["C"], a) - x) / _dot(S, d)
        fc.append({"S": S, "fx": fx, "d": d, "flux": _dot(S, u), "nu": _rand(g, *S.shape[:3], lo=0.005, hi=0.02)})
    uu = m["vol"] * (u0.norm() / m["h"]) * _rand(g, nz, ny, nx, lo=0.5, hi=1.5)
    pp = 1e-3 * m["h"] * _rand(g, nz, ny, nx, lo=0.5, hi=1.5)
    return fc, uu, pp, u0


def _pu_matrix(m, fields, walls):
    """The pressure-based 4x4 blocks: upwind convection and diffusion,
    interpolated face areas, Rhie-Chow pressure Laplacian.  walls: boundary
    faces on the diagonal (fixed velocity in a uniform flow, p = 0 at outflow)
    in place of the fields' diagonal sums."""
    fc, uu_add, pp_add, u0 = fields
    nz, ny, nx = m["shape"]
    eye = torch.eye(3, dtype=F64, device="cuda")
    C = m["C"]
    auu = torch.zeros(nz, ny, nx, dtype=F64, device="cuda") if walls else uu_add.clone()
    parts = []
    for a in range(3):
        f = fc[a]
        Sm = torch.sqrt(_dot(f["S"], f["S"]))
        nd = _dot(f["S"], f["d"]) / Sm
        Fl, k = f["flux"], f["nu"] * Sm / nd
        _lo(auu, a).add_(Fl.clamp(min=0) + k)
        _hi(auu, a).add_((-Fl).clamp(min=0) + k)
        bnd = []
        for last in (False, True) if walls else ():
            Sb = _end(m["S"][a], a, last) * (1.0 if last else -1.0)
            Sbm = torch.sqrt(_dot(Sb, Sb))
            ndb = _dot(Sb, _end(m["c"][a], a, last) - _end(C, a, last)) / Sbm
            Fb = _dot(Sb, u0)
            uu = Fb.clamp(min=0) + 0.01 * Sbm / ndb
            _end(auu, a, last).add_(uu)
            bnd.append((last, Sb, Sbm / ndb, (Fb > 0).to(F64), uu))
        parts.append((Sm / nd, Fl, k, bnd))
    D = m["vol"] / auu

    def block(pp, cpl, uu):
        B = torch.zeros(*pp.shape, 4, 4, dtype=F64, device="cuda")
        B[..., 0, 0] = pp
        B[..., 0, 1:] = cpl
        B[..., 1:, 0] = cpl
        B[..., 1:, 1:] = uu[..., None, None] * eye
        return B

    zero = torch.zeros(nz, ny, nx, 3, dtype=F64, device="cuda")
    diag = block(zero[..., 0], zero, zero[..., 0]) if walls else block(pp_add, zero, uu_add)
    up, lo = [], []
    for a in range(3):
        f, (geo, Fl, k, bnd) = fc[a], parts[a]
        pp = (f["fx"] * _lo(D, a) + (1.0 - f["fx"]) * _hi(D, a)) * geo
        own, oth = f["fx"][..., None] * f["S"], (1.0 - f["fx"])[..., None] * f["S"]
        out, back = Fl.clamp(min=0) + k, (-Fl).clamp(min=0) + k
        up.append(block(-pp, oth, -back))
        lo.append(block(-pp, -own, -out))
        _lo(diag, a).add_(block(pp, own, out))
        _hi(diag, a).add_(block(pp, -oth, back))
        for last, Sb, geo_b, outflow, uu in bnd:
            B = block(outflow * _end(D, a, last) * geo_b, Sb, uu)
            B[..., 0, 1:] *= outflow[..., None]
            _end(diag, a, last).add_(B)
    return {"diag": diag, "up": up, "lo": lo}


def _ldu(M, perm=None):
    """LDU arrays of a grid matrix, cells renumbered by perm (new id of each)."""
    nz, ny, nx, n, _ = M["diag"].shape
    la, ua = _faces(nx, ny, nz)
    cat = lambda parts: torch.cat([q.reshape(-1, n, n) for q in parts]).contiguous()
    diag = M["diag"].reshape(-1, n, n)
    if perm is not None:
        la, ua = perm[la.long()].int(), perm[ua.long()].int()
        d = torch.empty_like(diag)
        d[perm] = diag
        diag = d
    return {"N": nx * ny * nz, "n": n, "la": la, "ua": ua, "diag": diag.contiguous(), "up": cat(M["up"]),
            "lo": cat(M["lo"])}


def _cells(x, perm):
    x = x.reshape(-1, x.shape[-1])
    if perm is None:
        return x.contiguous()
    y = torch.empty_like(x)
    y[perm] = x
    return y


def _box(case, seed):
    """One box: its LDU arrays, the right side of a known solution x, and of
    the transposed system for a known lam."""
    g = _gen(seed)
    nx, ny, nz, n = case["nx"], case["ny"], case["nz"], case["n"]
    m = _mesh(nx, ny, nz, g, case.get("stretch", 1.0))
    fields = _luo_fields(m, g) if n == 5 else _pu_fields(m, g)
    M = _luo_matrix(m, fields) if n == 5 else _pu_matrix(m, fields, case.get("walls", True))
    perm = torch.randperm(nx * ny * nz, generator=g, device="cuda") if case.get("renumbered") else None
    x, lam = _rand(g, nz, ny, nx, n, lo=-1.0), _rand(g, nz, ny, nx, n, lo=-1.0)
    L = _ldu(M, perm)
    L.update(b=_cells(_apply(M, x), perm), x=_cells(x, perm), fields=fields, mesh=m)
    if case["path"] == "adjoint":
        L.update(g=_cells(_apply_t(M, lam), perm), lam=_cells(lam, perm))
    if case["path"] == "spmv_t":
        L.update(b=_cells(_apply_t(M, x), perm))
    return L


def _handle(L):
    return P.System(L["N"], L["n"], L["la"], L["ua"], L["diag"], L["up"], L["lo"])


def _options(case, **kw):
    mixed = case.get("precision", "mixed") == "mixed"
    o = {"precision": P.PRECISION_MIXED if mixed else P.PRECISION_FP64, "tol": 1e-12}
    o["solver"] = {"bicgstab": P.SOLVER_BICGSTAB, "fgmres": P.SOLVER_FGMRES,
                   "gmres": P.SOLVER_GMRES}[case.get("solver", "bicgstab")]
    if case.get("precond") == "sgs":
        o["precond"] = P.PREC_SGS
    if case.get("cycle") == "w":            # the benchmark's cycle
        o.update(w_levels=1, pre_sweeps=1, post_sweeps=2, coarse_omega=1.4)
    if case.get("smoother") == "dilu":
        o.update(smoother=P.SMOOTH_DILU, dilu_levels=1)
    return P.default_options(**o, **kw)


# ------------------------------------------------------------------ paths
# Each path: what the program holds before the call, and one pass.
def _prep_step(case, seed):
    """A linear step: new LDU coefficients, fresh preconditioner, solve from
    fields kept per variable (packed before and unpacked after)."""
    L = _box(case, seed)
    return {"s": _handle(L), "o": _options(case), "diag": L["diag"], "up": L["up"], "lo": L["lo"],
            "b": L["b"].t().contiguous()}


def _run_step(st):
    s = st["s"]
    b = P.pack_fields(st["b"])
    s.update_values(st["diag"], st["up"], st["lo"])
    s.setup(st["o"])
    x, _ = s.solve(b)
    return P.unpack_fields(x)


def _exact_step(case, seed):
    return _box(case, seed)["x"].t().contiguous()


def _prep_newton(case, seed):
    """The next nonlinear iteration on one mesh: assembly from the fields,
    preconditioner on the kept aggregates, solve from the last iterate."""
    L = _box(case, seed)
    s = _handle(L).setup(_options(case))
    x0 = L["x"] * (1.0 + 1e-2 * _rand(_gen(seed, 7), *L["x"].shape, lo=-1.0))
    return {"s": s, "o": _options(case, reuse_aggregates=1), "f": _assembly_arrays(L), "n": L["n"], "b": L["b"],
            "x0": x0}


def _assembly_arrays(L):
    f = L["fields"]
    if L["n"] == 5:
        return f
    fc, uu, pp, _ = f
    cat = lambda key: torch.cat([q[key].reshape(-1, 3) if q[key].dim() == 4 else q[key].reshape(-1)
                                 for q in fc]).contiguous()
    return {"Sf": cat("S"), "fx": cat("fx"), "d": cat("d"), "flux": cat("flux"), "nu_eff": cat("nu"),
            "vol": L["mesh"]["vol"].reshape(-1).contiguous(), "uu_add": uu.reshape(-1), "pp_add": pp.reshape(-1)}


def _run_newton(st):
    s = st["s"]
    (s.assemble_luo if st["n"] == 5 else s.assemble_pu)(**st["f"])
    s.setup(st["o"])
    return s.solve(st["b"], st["x0"])[0]


def _exact_x(case, seed):
    return _box(case, seed)["x"]


def _prep_defect(case, seed):
    """Assembly and the product with the current iterate, for the defect."""
    L = _box(case, seed)
    return {"s": _handle(L), "f": _assembly_arrays(L), "n": L["n"], "x": L["x"]}


def _run_defect(st):
    s = st["s"]
    (s.assemble_luo if st["n"] == 5 else s.assemble_pu)(**st["f"])
    return s.spmv(st["x"])


def _exact_b(case, seed):
    return _box(case, seed)["b"]


def _prep_adjoint(case, seed):
    """A differentiable solve: forward, then the gradients of all inputs."""
    L = _box(case, seed)
    s = _handle(L).setup(_options(case))
    return {"s": s, "in": [L[k].requires_grad_() for k in ("diag", "up", "lo", "b")], "g": L["g"]}


def _run_adjoint(st):
    x = P.coupled_solve(st["s"], *st["in"])
    return [x.detach()] + list(torch.autograd.grad(x, st["in"], st["g"]))


def _exact_adjoint(case, seed):
    L = _box(case, seed)
    l, u = L["la"].long(), L["ua"].long()
    outer = lambda a, b: -a.unsqueeze(-1) * b.unsqueeze(-2)
    return [L["x"], outer(L["lam"], L["x"]), outer(L["lam"][l], L["x"][u]), outer(L["lam"][u], L["x"][l]), L["lam"]]


def _batch(case, seed):
    """`count` density-based boxes, sizes spread evenly in their logarithm."""
    out = []
    for i in range(case["count"]):
        side = (case["lo"] * (case["hi"] / case["lo"]) ** (i / max(1, case["count"] - 1))) ** (1.0 / 3.0)
        a = max(2, round(side))
        c = dict(path="step", n=5, nx=a, ny=max(2, a - i % 3), nz=max(2, a + i % 2))
        out.append(_box(c, 1000 * seed + i))
    off = lambda sizes: [sum(sizes[:k]) for k in range(len(sizes) + 1)]
    L = {k: torch.cat([q[k] for q in out]) for k in ("la", "ua", "diag", "up", "lo", "b", "x")}
    L.update(cell_off=off([q["N"] for q in out]), face_off=off([q["la"].numel() for q in out]))
    return L


def _prep_batch(case, seed):
    L = _batch(case, seed)
    s = P.System(L["cell_off"][-1], 5, L["la"], L["ua"], L["diag"], L["up"], L["lo"], cell_off=L["cell_off"],
                 face_off=L["face_off"])
    return {"s": s, "o": _options(case), "diag": L["diag"], "up": L["up"], "lo": L["lo"], "b": L["b"]}


def _run_batch(st):
    s = st["s"]
    s.update_values(st["diag"], st["up"], st["lo"])
    s.setup(st["o"])
    return s.solve_batch(st["b"])[0]


def _exact_batch(case, seed):
    return _batch(case, seed)["x"]


def _prep_spmv(case, seed):
    L = _box(case, seed)
    return {"s": _handle(L), "x": L["x"]}


def _run_spmv(st):
    return st["s"].spmv(st["x"])


def _run_spmv_t(st):
    return st["s"].spmv(st["x"], transpose=True)


def _prep_precond(case, seed):
    """The preconditioner inside a caller's own outer iteration."""
    L = _box(case, seed)
    return {"s": _handle(L).setup(_options(case)), "r": L["b"]}


def _run_precond(st):
    return st["s"].apply_precond(st["r"])


_PATHS = {
    "step": (_prep_step, _run_step, _exact_step),
    "newton": (_prep_newton, _run_newton, _exact_x),
    "defect": (_prep_defect, _run_defect, _exact_b),
    "adjoint": (_prep_adjoint, _run_adjoint, _exact_adjoint),
    "batch": (_prep_batch, _run_batch, _exact_batch),
    "spmv": (_prep_spmv, _run_spmv, _exact_b),
    "spmv_t": (_prep_spmv, _run_spmv_t, _exact_b),
    "precond": (_prep_precond, _run_precond, None),
}


def listed():
    box = lambda name, path, n, nx, ny, nz, **kw: dict(name=name, path=path, n=n, nx=nx, ny=ny, nz=nz, **kw)
    return [
        # the smallest steps: a regression or design-loop case, where launches and read-backs count
        box("pu_step_960", "step", 4, 12, 10, 8, renumbered=True, precision="fp64"),
        # a correctness-sized density-based iteration
        box("density_newton_8k", "newton", 5, 20, 20, 20),
        # an ordinary pressure-based step, odd sizes, the library's default cycle
        box("pu_step_55k", "step", 4, 41, 39, 35, renumbered=True),
        # a differentiable solve in a training or optimisation loop
        box("pu_adjoint_35k", "adjoint", 4, 33, 31, 35, renumbered=True, precision="fp64"),
        # density-based nonlinear iteration on a mid-size mesh
        box("density_newton_219k", "newton", 5, 63, 57, 61),
        # boundary-layer mesh, flexible GMRES
        box("density_fgmres_164k", "step", 5, 64, 64, 40, solver="fgmres", stretch=1.2),
        # GMRES with symmetric Gauss-Seidel, the light-weight configuration
        box("density_sgs_59k", "step", 5, 39, 39, 39, solver="gmres", precond="sgs", precision="fp64"),
        # the benchmark: one million cells, W-cycle
        box("pu_step_1m", "step", 4, 100, 100, 100, renumbered=True, cycle="w"),
        # many small and mid-size systems at once
        dict(name="density_batch_24", path="batch", n=5, count=24, lo=1000, hi=60000),
        # assembly and one product: the defect of a nonlinear iteration
        box("pu_defect_1m", "defect", 4, 100, 100, 100, walls=False),
        # products with the matrix and its transpose in a caller's own iteration
        box("density_spmv_t_387k", "spmv_t", 5, 73, 71, 75, renumbered=True),
        # one preconditioner application in FP64, coloured smoother
        box("pu_precond_dilu_262k", "precond", 4, 64, 64, 64, renumbered=True, precision="fp64", smoother="dilu"),
    ]


def draw(rng):
    """One more case: a listed path and its options at another size."""
    c = dict(rng.choice(listed()))
    del c["name"]
    if c["path"] == "batch":
        c.update(count=rng.randint(4, 32), lo=rng.randint(400, 2000), hi=rng.randint(8000, 60000))
        return c
    top = {"step": 3e5, "newton": 2.2e5, "adjoint": 1e5, "defect": 1e6, "spmv": 1e6, "spmv_t": 6e5,
           "precond": 3e5}[c["path"]]
    if c.get("cycle") == "w":
        top = 9e5
    elif c["n"] == 5 and c["path"] == "step":
        top = 1.6e5
    low = 500 if c["path"] in ("step", "newton", "adjoint") else 8000
    N = math.exp(rng.uniform(math.log(low), math.log(top)))
    side = N ** (1.0 / 3.0)
    nx, ny = max(3, round(side * rng.uniform(0.8, 1.2))), max(3, round(side * rng.uniform(0.8, 1.2)))
    c.update(nx=nx, ny=ny, nz=max(3, int(N / (nx * ny))))
    if c["path"] in ("spmv", "spmv_t"):
        c.update(path=rng.choice(["spmv", "spmv_t"]), n=rng.choice([4, 5]), renumbered=rng.random() < 0.5)
    elif c["path"] == "step" and "precond" not in c:
        c["precision"] = rng.choice(["mixed", "fp64"])
    elif c["path"] == "precond" and rng.random() < 0.5:
        c.pop("smoother")
    return c


def prepare(case, seed):
    st = _PATHS[case["path"]][0](case, seed)
    st["path"] = case["path"]
    return st


def run(state):
    return _PATHS[state["path"]][1](state)


def exact(case, seed):
    fn = _PATHS[case["path"]][2]
    return fn(case, seed) if fn else None


def _counts(case):
    if case["path"] == "batch":
        N = F = 0
        for i in range(case["count"]):
            side = (case["lo"] * (case["hi"] / case["lo"]) ** (i / max(1, case["count"] - 1))) ** (1.0 / 3.0)
            a = max(2, round(side))
            x, y, z = a, max(2, a - i % 3), max(2, a + i % 2)
            N, F = N + x * y * z, F + 3 * x * y * z - x * y - y * z - z * x
        return N, F
    x, y, z = case["nx"], case["ny"], case["nz"]
    return x * y * z, 3 * x * y * z - x * y - y * z - z * x


def work(case):
    """One pass, each input read once and each output written once: a solve
    reads the coefficients, the right side and writes the solution (the passes
    over the matrix that its iterations need are the method's, not counted)."""
    N, F = _counts(case)
    n = case["n"]
    vec, mat = 8.0 * N * n, 8.0 * (N + 2 * F) * n * n
    product = 2.0 * (N + 2 * F) * n * n
    faces = 8.0 * F * (9 if n == 4 else 4) + 8.0 * N * (3 if n == 4 else 6)
    return {"step": {"bytes": mat + 2 * vec, "flops": product},
            "batch": {"bytes": mat + 2 * vec, "flops": product},
            "newton": {"bytes": faces + 3 * vec, "flops": product},
            "adjoint": {"bytes": 2 * mat + 4 * vec, "flops": 2 * product},
            "defect": {"bytes": faces + 2 * vec, "flops": product},
            "spmv": {"bytes": mat + 2 * vec, "flops": product},
            "spmv_t": {"bytes": mat + 2 * vec, "flops": product},
            "precond": {"bytes": mat + 2 * vec, "flops": product}}[case["path"]]
