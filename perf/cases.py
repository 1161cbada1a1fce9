"""The work a program gives this library, as measurable cases.

Node sets of closed surfaces at spacing h = 1/m with delta = 3h (the ratio
every configuration of this repository uses), on which programs

* apply one layer sum on a staged surface ("layer"): the matvec of a solver
  of their own, a field at the nodes, an accuracy study;
* apply one to a surface given directly, without a plan ("noalloc");
* stage a surface that was not seen before and apply one layer sum ("stage");
* solve the Darcy, the Stokes or the coupled problem ("darcy", "stokes",
  "ddm"), in double or with float pairs;
* take the drag and its gradient with respect to nodes, log K and alpha, as a
  step of a shape or parameter optimisation does ("gradient").

The outputs of a layer sum with float pairs are good to about 1e-7; a program
that asks for them keeps them in single precision, and so do the cases here.
Solves with float pairs end on double residuals: their outputs are double,
at the tolerances that the repository's smoke check uses (local 1e-12,
interface 1e-11).  Double solves run at the default tolerances.

Quadrature as in the paper: the points of the surface on the grid lines of
spacing h parallel to each axis, kept where the unit normal is within 70
degrees of that axis, weighted by a partition of unity on the normals.
"""
import math

import numpy as np
import torch

import paper_2110_10749_amd as sd

# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
MU = 1.0


def _layer(name, family, layer, surface, m, prec):
    return dict(name=name, op="layer", family=family, layer=layer, surface=surface, m=m, prec=prec)


def _solve(name, op, surface, m, prec, K=1e-2, alpha=1.0):
    return dict(name=name, op=op, surface=surface, m=m, prec=prec, K=K, alpha=alpha)


def listed():
    return [
        # the smallest call: a coarse sphere (N = 1062, the size of the smoke check), one Darcy matvec;
        # launches and latency are all there is
        _layer("laplace dl fp64 h/8", "laplace", "dl_sub", "sphere", 8, "fp64"),
        # the paper's coarsest grid on its ellipsoid (N = 2650, ten tiles and a ragged one): a Stokes matvec
        _layer("stokes dl fp64 h/16", "stokes", "dl_sub", "ellipsoid", 16, "fp64"),
        # the middle grid of the convergence studies (N = 17070): one Stokes single layer with float pairs,
        # as for the right-hand side of a loose solve
        _layer("stokes sl mixed h/32", "stokes", "sl", "perturbed", 32, "mixed"),
        # the benchmark's grid on the ellipsoid (N = 42342): the Stokes matvec that double solves consist of
        _layer("stokes dl fp64 h/64", "stokes", "dl_sub", "ellipsoid", 64, "fp64"),
        # the large surface (N = 272718): the matvec of the matrix-free mixed solve
        _layer("stokes dl mixed h/128", "stokes", "dl_sub", "sphere", 128, "mixed"),
        # a caller that cannot allocate and hands the surface over on every call (N = 9582)
        dict(name="noalloc sl fp64 h/24", op="noalloc", family="stokes", layer="sl", surface="sphere", m=24,
             prec="fp64"),
        # a new surface at the benchmark's grid (N = 68166): staging and one Laplace single layer on it
        dict(name="stage + laplace sl h/64", op="stage", family="laplace", layer="sl", surface="perturbed", m=64,
             prec="mixed"),
        # the Darcy problem alone at the middle grid, double
        _solve("darcy solve fp64 h/32", "darcy", "sphere", 32, "fp64"),
        # the Stokes problem with slip alone on an odd grid, float pairs
        _solve("stokes solve mixed h/41", "stokes", "perturbed", 41, "mixed"),
        # the coupled problem on the paper's coarsest ellipsoid grid, double: many small passes and Krylov steps
        _solve("ddm solve fp64 h/16", "ddm", "ellipsoid", 16, "fp64"),
        # the benchmark: the coupled problem on the sphere at h = 1/64 with float pairs
        _solve("ddm solve mixed h/64", "ddm", "sphere", 64, "mixed"),
        # one step of a shape optimisation: drag, its gradient, a new plan each time
        _solve("drag gradient fp64 h/16", "gradient", "perturbed", 16, "fp64"),
    ]


# grid ranges per kind of work, fp64 and mixed: up to what a program waits for interactively
_RANGE = {"layer": (8, 80, 120), "noalloc": (8, 40, 40), "stage": (8, 80, 80), "darcy": (8, 64, 64),
          "stokes": (8, 40, 48), "ddm": (8, 28, 40), "gradient": (8, 18, 18)}


def draw(rng):
    op = rng.choice(["layer", "layer", "layer", "noalloc", "stage", "darcy", "stokes", "ddm", "gradient"])
    prec = rng.choice(["fp64", "mixed"])
    lo, hi64, hi32 = _RANGE[op]
    hi = hi64 if prec == "fp64" else hi32
    c = dict(op=op, prec=prec, surface=rng.choice(["sphere", "ellipsoid", "perturbed"]),
             m=round(math.exp(rng.uniform(math.log(lo), math.log(hi))), 2))
    if op in ("layer", "noalloc", "stage"):
        c["family"] = "stokes" if op == "noalloc" else rng.choice(["laplace", "stokes"])
        c["layer"] = rng.choice(["sl", "dl_sub", "dl_sub", "dl_raw"])
    else:
        # slip beta = alpha / sqrt(K) up to 10: the range the default restart length serves
        c["K"], c["alpha"] = rng.choice([(1.0, 0.1), (1.0, 1.0), (1e-2, 0.1), (1e-2, 1.0), (1e-3, 0.3)])
    return c


# ---------------------------------------------------------------------------
# surfaces
# ---------------------------------------------------------------------------
_COS70 = math.cos(math.radians(70.0))


def _partition(n):
    r = np.arccos(np.clip(np.abs(n), 0.0, 1.0)) / math.radians(70.0)
    b = np.zeros_like(r)
    inside = r < 1.0
    b[inside] = np.exp(r[inside] ** 2 / (r[inside] ** 2 - 1.0))
    return b / b.sum(axis=0, keepdims=True)


def _ellipsoid(m, axes):
    """Nodes, normals and weights of the ellipsoid with semi-axes `axes` at spacing 1/m."""
    h = 1.0 / m
    X, NRM, W = [], [], []
    for i in range(3):
        a, b = [k for k in range(3) if k != i]
        ga = np.arange(-int(axes[a] * m) - 1, int(axes[a] * m) + 2) * h
        gb = np.arange(-int(axes[b] * m) - 1, int(axes[b] * m) + 2) * h
        A, B = [v.ravel() for v in np.meshgrid(ga, gb, indexing="ij")]
        s = 1.0 - (A / axes[a]) ** 2 - (B / axes[b]) ** 2
        A, B, s = A[s > 0], B[s > 0], s[s > 0]
        for sign in (-1.0, 1.0):
            x = np.empty((3, A.size))
            x[a], x[b], x[i] = A, B, sign * axes[i] * np.sqrt(s)
            n = x / np.asarray(axes)[:, None] ** 2
            n /= np.linalg.norm(n, axis=0)
            keep = np.abs(n[i]) >= _COS70
            x, n = x[:, keep], n[:, keep]
            X.append(x)
            NRM.append(n)
            W.append(_partition(n)[i] * h * h / np.abs(n[i]))
    return np.concatenate(X, axis=1), np.concatenate(NRM, axis=1), np.concatenate(W)


def _perturbed(m, seed):
    """The unit sphere's nodes moved radially by a cubic polynomial of the direction, coefficients of
    size 0.03 from the seed; normals and weights of the moved surface."""
    o, _, w = _ellipsoid(m, (1.0, 1.0, 1.0))
    rng = np.random.default_rng(seed)
    q, t = 0.03 * rng.normal(size=(3, 3)), 0.03 * rng.normal(size=(3, 3, 3))
    r = 1.0 + np.einsum("ij,in,jn->n", q, o, o) + np.einsum("ijk,in,jn,kn->n", t, o, o, o)
    g = np.einsum("ij,jn->in", q + q.T, o) + np.einsum(
        "ijk,jn,kn->in", t + t.transpose(1, 0, 2) + t.transpose(2, 0, 1), o, o)
    g -= o * (o * g).sum(axis=0)  # tangential part
    n = r * o - g
    length = np.linalg.norm(n, axis=0)
    return r * o, n / length, w * r * length


def _surface(case, seed):
    if case["surface"] == "perturbed":
        return _perturbed(case["m"], seed)
    return _ellipsoid(case["m"], (1.0, 1.0, 1.0) if case["surface"] == "sphere" else (1.0, 0.8, 0.6))


def _size(case):
    return _surface(case, 0)[2].size


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _fields(x, rng, comps):
    """Densities as they occur in a solve: a smooth field, some roughness on top."""
    f = np.empty((comps, x.shape[1]))
    for c in range(comps):
        a = rng.normal(size=7)
        f[c] = (a[0] + a[1] * x[0] + a[2] * x[1] + a[3] * x[2] + a[4] * x[0] * x[1] + a[5] * x[1] * x[2]
                + a[6] * x[2] ** 2 + 0.05 * rng.normal(size=x.shape[1]))
    return f


def _inputs(case, seed):
    """Everything a pass reads, as numpy arrays (shared by prepare and exact)."""
    x, n, w = _surface(case, seed)
    rng = np.random.default_rng([seed, 7])
    s = dict(x=x, n=n, w=w, delta=3.0 / case["m"])
    if case["op"] in ("layer", "noalloc", "stage"):
        s["dens"] = _fields(x, rng, 1)[0] if case["family"] == "laplace" else _fields(x, rng, 3)
    elif case["op"] == "darcy":
        v = _fields(x, rng, 1)[0]
        s["vn"] = v - (w * v).sum() / w.sum()  # no net flux through the closed surface
    else:
        # every component of the flow is present, so is every component of the drag
        s["U"] = [float(v) for v in rng.choice([-1.0, 1.0], size=3) * rng.uniform(0.4, 1.0, size=3)]
        s["e"] = [float(v) for v in rng.normal(size=3)]
        if case["op"] == "stokes":
            s["p"] = _fields(x, rng, 1)[0]
    return s


def _opts(case):
    if case["prec"] == "mixed":
        return dict(prec="mixed", tol_gmres=1e-12, tol_ddm=1e-11)
    return dict(prec="fp64")


def prepare(case, seed):
    s = _inputs(case, seed)
    for k in ("x", "n", "w", "dens", "vn", "p"):
        if k in s:
            s[k] = torch.from_numpy(np.ascontiguousarray(s[k])).to("cuda")
    s["case"] = case
    if case["op"] in ("layer", "darcy", "stokes", "ddm"):
        s["plan"] = sd.Plan(s["x"], s["n"], s["w"], s["delta"])
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def _kept(case, out):
    return out.float() if case["prec"] == "mixed" else out


def run(s):
    case = s["case"]
    op, prec = case["op"], case["prec"]
    if op == "noalloc":
        return _kept(case, sd.stokes_layer_apply_noalloc(s["x"], s["n"], s["w"], s["delta"], MU, case["layer"],
                                                         s["dens"], prec=prec))
    if op in ("layer", "stage"):
        plan = s["plan"] if op == "layer" else sd.Plan(s["x"], s["n"], s["w"], s["delta"])
        if case["family"] == "laplace":
            return _kept(case, sd.laplace_layer_apply(plan, case["layer"], s["dens"], prec=prec))
        return _kept(case, sd.stokes_layer_apply(plan, MU, case["layer"], s["dens"], prec=prec))
    K, alpha = case["K"], case["alpha"]
    if op == "darcy":
        return sd.darcy_solve(s["plan"], MU, K, alpha, s["vn"], opts=_opts(case))[0]
    if op == "stokes":
        return sd.stokes_solve(s["plan"], MU, K, alpha, s["U"], s["p"], opts=_opts(case))[0]
    if op == "ddm":
        p, u, drag, _ = sd.ddm_solve(s["plan"], MU, K, alpha, s["U"], opts=_opts(case))
        return {"p": p, "u": u, "drag": np.array(drag)}
    x = s["x"].detach().requires_grad_(True)
    log_K = torch.tensor(math.log(K), dtype=torch.float64, device="cuda", requires_grad=True)
    al = torch.tensor(alpha, dtype=torch.float64, device="cuda", requires_grad=True)
    drag = sd.drag(x, log_K, al, s["n"], s["w"], s["delta"], MU, s["U"], opts=_opts(case))
    (drag * torch.tensor(s["e"], dtype=torch.float64, device="cuda")).sum().backward()
    return {"drag": drag.detach(), "x": x.grad, "log_K": log_K.grad, "alpha": al.grad}


# flops per ordered pair of each kernel (FMA = 2): Laplace single and double layer, Stokeslet, stresslet
_FLOPS = {("laplace", "sl"): 10, ("laplace", "dl"): 20, ("stokes", "sl"): 28, ("stokes", "dl"): 33}


def work(case):
    n = float(_size(case))
    op = case["op"]
    if op in ("layer", "noalloc", "stage"):
        comps = 1 if case["family"] == "laplace" else 3
        return {"bytes": 8 * n * (7 + 2 * comps), "flops": n * n * _FLOPS[case["family"], case["layer"][:2]]}
    # the fewest products any Krylov solve of these problems has shown here: a right-hand side and
    # 6 matvecs (Darcy), 8 with slip (Stokes), 3 interface products (coupled), twice that and the
    # position derivatives (gradient)
    lap = n * n * (_FLOPS["laplace", "sl"] + 6 * _FLOPS["laplace", "dl"])
    sto = n * n * (_FLOPS["stokes", "sl"] + 8 * (_FLOPS["stokes", "dl"] + _FLOPS["stokes", "sl"]))
    flops = {"darcy": lap, "stokes": sto, "ddm": 3 * (lap + sto), "gradient": 6 * (lap + sto)}[op]
    return {"bytes": 8 * n * {"darcy": 9, "stokes": 11, "ddm": 11, "gradient": 14}[op], "flops": flops}


# ---------------------------------------------------------------------------
# the same in plain 64-bit torch: dense sums and dense solves
# ---------------------------------------------------------------------------
def _smoothed(x2, rho):
    """s1/rho, s2/rho^3, s3/rho^3, s4/rho^5 as functions of x2 = rho^2 (rho: its root).  Below rho^2 = 1 the
    erf series: erf(rho) = 2/sqrt(pi) rho exp(-rho^2) sum_k (2 rho^2)^k / (2k+1)!!, whose first terms cancel
    against the polynomials of the closed forms."""
    c = 2.0 / math.sqrt(math.pi)
    small = x2 < 1.0
    r = torch.where(small, torch.ones_like(rho), rho)
    y = r * r
    e = torch.exp(-y)
    ef, ce = torch.erf(r), c * r * e
    k1 = (ef - ce * (2 * y - 5) / 3) / r
    k2 = (ef + ce * (2 * y - 3) / 3) / r**3
    k3 = (ef - ce * ((4 * y - 14) * y + 3) / 3) / r**3
    k4 = (ef - ce * (((8 * y - 36) * y + 6) * y + 9) / 9) / r**5
    if bool(small.any()):
        z = x2[small]
        terms, dfact = [], 1.0
        for k in range(26):  # a_k = 2^k / (2k+1)!!
            dfact *= 2 * k + 1
            terms.append(2.0**k / dfact)

        def series(extra, first):  # sum_k (a_k + extra_k) z^(k - first)
            s = torch.zeros_like(z)
            for k in range(len(terms) - 1, first - 1, -1):
                s = s * z + terms[k] + extra.get(k, 0.0)
            return c * torch.exp(-z) * s

        k1[small] = series({0: 5 / 3, 1: -2 / 3}, 0)
        k2[small] = series({0: -1.0, 1: 2 / 3}, 1)
        k3[small] = series({0: -1.0, 1: 14 / 3, 2: -4 / 3}, 1)
        k4[small] = series({0: -1.0, 1: -2 / 3, 2: 4.0, 3: -8 / 9}, 2)
    return k1, k2, k3, k4


class _Dense:
    """Rows of the smoothed kernels over target chunks."""

    def __init__(self, s):
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")  # noqa: E731
        self.x, self.n, self.w, self.delta = t(s["x"]), t(s["n"]), t(s["w"]), s["delta"]
        self.N = self.w.numel()

    def chunks(self):
        step = max(1, min(self.N, 60_000_000 // self.N))
        for i in range(0, self.N, step):
            yield slice(i, min(i + step, self.N))

    def pairs(self, sl):
        D = [self.x[c, sl, None] - self.x[c, None, :] for c in range(3)]
        r2 = D[0] ** 2 + D[1] ** 2 + D[2] ** 2
        x2 = r2 / self.delta**2
        k1, k2, k3, k4 = _smoothed(x2, x2.sqrt())
        d = self.delta
        dn = D[0] * self.n[0] + D[1] * self.n[1] + D[2] * self.n[2]
        return D, dn, k1 / d, k2 / d**3, k3 / d**3, k4 / d**5

    def layer(self, family, layer, dens):
        q = torch.from_numpy(np.ascontiguousarray(dens)).to("cuda")
        out = torch.empty_like(q)
        for sl in self.chunks():
            D, dn, k1, k2, k3, k4 = self.pairs(sl)
            if family == "laplace":
                if layer == "sl":
                    out[sl] = -(k1 @ (self.w * q)) / (4 * math.pi)
                else:
                    m = dn * k2 * self.w
                    out[sl] = -(m @ q) if layer == "dl_raw" else m @ q - q[sl] * m.sum(dim=1)
                    out[sl] /= 4 * math.pi
                continue
            qd = sum(D[c] * q[c] for c in range(3))
            if layer == "sl":
                for c in range(3):
                    out[c, sl] = ((q[c] * k1 + D[c] * qd * k3) @ self.w) / (8 * math.pi * MU)
            else:
                if layer == "dl_sub":
                    qd = qd - sum(D[c] * q[c, sl, None] for c in range(3))
                m = qd * dn * k4
                for c in range(3):
                    out[c, sl] = -3.0 / (4 * math.pi) * ((m * D[c]) @ self.w) + (q[c, sl] if layer == "dl_sub" else 0.0)
        return out

    def darcy(self):
        """Matrices of S_L and of the completed subtracted double layer."""
        S, A = (torch.empty(self.N, self.N, dtype=torch.float64, device="cuda") for _ in range(2))
        for sl in self.chunks():
            _, dn, k1, k2, _, _ = self.pairs(sl)
            S[sl] = -k1 * self.w / (4 * math.pi)
            m = dn * k2 * self.w / (4 * math.pi)
            A[sl] = m + self.w / self.w.sum()
            i = torch.arange(sl.start, sl.stop, device="cuda")
            A[i, i] -= m.sum(dim=1)
        return S, A

    def stokes(self, beta):
        """Matrices [3N, 3N] of V and of the completed subtracted stresslet with implicit slip."""
        N = self.N
        V, A = (torch.empty(3, N, 3, N, dtype=torch.float64, device="cuda") for _ in range(2))
        i = torch.arange(N, device="cuda")
        for sl in self.chunks():
            D, dn, k1, _, k3, k4 = self.pairs(sl)
            for a in range(3):
                for b in range(3):
                    V[a, sl, b] = ((k1 if a == b else 0.0) + D[a] * D[b] * k3) * self.w / (8 * math.pi * MU)
                    m = -3.0 / (4 * math.pi) * dn * k4 * D[a] * D[b] * self.w
                    A[a, sl, b] = m + self.n[a, sl, None] * (self.w * self.n[b]) / self.w.sum()
                    A[a, i[sl], b, i[sl]] -= m.sum(dim=1)
        for a in range(3):
            A[a, i, a, i] += 1.0
        for b in range(3):  # + beta V (I - n n^T)
            Vn = sum(V[:, :, c] * self.n[c] for c in range(3))
            A[:, :, b] += beta * (V[:, :, b] - Vn * self.n[b])
        return V.view(3 * N, 3 * N), A.view(3 * N, 3 * N)


def exact(case, seed):
    op = case["op"]
    n = _size(case)
    # about 20 seconds of dense work: larger sums and systems have no value here
    if op == "gradient" or n > {"darcy": 18000, "stokes": 4500, "ddm": 4500}.get(op, 90000):
        return None
    s = _inputs(case, seed)
    d = _Dense(s)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda")  # noqa: E731
    if op in ("layer", "noalloc", "stage"):
        return _kept(case, d.layer(case["family"], case["layer"], s["dens"]))
    mean = lambda p: p - (d.w * p).sum() / d.w.sum()  # noqa: E731
    if op == "darcy":
        S, A = d.darcy()
        return mean(torch.linalg.solve(A, MU / case["K"] * (S @ t(s["vn"]))))
    beta = case["alpha"] * MU / math.sqrt(case["K"])
    V, A = d.stokes(beta)
    N = d.N
    U = torch.tensor(s["U"], dtype=torch.float64, device="cuda").repeat_interleave(N)
    if op == "stokes":
        return torch.linalg.solve(A, U + V @ (d.n * t(s["p"])).reshape(-1)).view(3, N)
    # coupled: A_D p - (mu/K) S_L[u.n] = 0,  A_S u - V[(p - mean) n] = U
    S, AD = d.darcy()
    M = torch.empty(4 * N, 4 * N, dtype=torch.float64, device="cuda")
    M[:N, :N], M[N:, N:] = AD, A
    for c in range(3):
        M[:N, (1 + c) * N:(2 + c) * N] = -MU / case["K"] * S * d.n[c]
    P = sum(V[:, c * N:(c + 1) * N] * d.n[c] for c in range(3))
    M[N:, :N] = -(P - P.sum(dim=1, keepdim=True) * (d.w / d.w.sum()))
    z = torch.linalg.solve(M, torch.cat([torch.zeros(N, dtype=torch.float64, device="cuda"), U]))
    p, u = mean(z[:N]), z[N:].view(3, N)
    f = -p * d.n + beta * (u - (u * d.n).sum(dim=0) * d.n)
    return {"p": p, "u": u, "drag": (f * d.w).sum(dim=1).cpu().numpy()}
