"""Timed cases of the library: each one call of a public entry point, over the sizes it is used at.

Kinds of a case (its "kind"):
  assemble  the dense EFIE matrix of a closed surface;
  product   Z X for one or many right-hand sides;
  sweep     plane-wave excitation and far field of a monostatic sweep;
  solve     a Krylov solve, plain or Calderon-preconditioned;
  calderon  the preconditioner P = T_BC(k~) G_mix^-1;
  gradient  the vertex gradient of a far-field objective;
  contour   the three boundary operators of a closed curve in 2-D.

Surfaces are geodesic spheres of frequency f (T = 20 f^2 triangles, N = 30 f^2
unknowns; f = 4, 16 and 32 are the sizes of the level 2, 4 and 5 spheres) whose
semi-axes come from the seed, vertices in Morton order.  Wavenumbers keep six or more
unknowns per wavelength, except where the smallest mesh is used at low frequency.
"""
import functools
import math

import numpy as np
import torch

import paper_2310_15644_amd as efie

ETA = 376.730313668
C128, C64 = "c128", "c64"
TYPES = {C128: torch.complex128, C64: torch.complex64}


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the plain method's smallest sphere: a few dozen microseconds of work, so launches count
        {"name": "assemble_fp64_n480", "kind": "assemble", "f": 4, "k": 1.0, "dtype": C128},
        # the plain method at the size of its accuracy studies
        {"name": "assemble_fp64_n7680", "kind": "assemble", "f": 16, "k": 5.0, "dtype": C128},
        # the mixed form at the largest surface in use
        {"name": "assemble_c64_n30720", "kind": "assemble", "f": 32, "k": 10.0, "dtype": C64},
        # a monostatic sweep's product: 512 plane waves against the largest matrix
        {"name": "product_c64_n30720_x512", "kind": "product", "n": 30720, "nrhs": 512, "dtype": C64},
        # an odd order and an odd column count, as block solves meet when columns converge
        {"name": "product_c64_n4317_x45", "kind": "product", "n": 4317, "nrhs": 45, "dtype": C64},
        # the FP64 products of the plain path and of true residuals, at an odd order
        {"name": "product_fp64_n7679_x64", "kind": "product", "n": 7679, "nrhs": 64, "dtype": C128},
        # right-hand sides and radar cross sections of the 16 x 32 grid of plane waves
        {"name": "sweep_n7680_x512", "kind": "sweep", "f": 16, "k": 5.0, "nwave": 512, "ndir": 512},
        # one plane wave on the smallest sphere: about a hundred short iterations
        {"name": "solve_fp64_n480", "kind": "solve", "method": "cocg", "f": 4, "k": 1.0, "nrhs": 1, "dtype": C128},
        # 64 plane waves by the preconditioned mixed path, to the accuracy of reference currents
        {"name": "solve_mixed_n4320_x64", "kind": "solve", "method": "calderon", "f": 12, "k": 5.0, "nrhs": 64,
         "dtype": C64},
        # the preconditioner with the call's default options
        {"name": "calderon_n7680", "kind": "calderon", "f": 16, "k": 5.0, "far": 0.0},
        # the shape derivative of the differentiation form: 32 directions, one plane wave
        {"name": "gradient_n7680", "kind": "gradient", "f": 16, "k": 3.0, "ndir": 32},
        # the 2-D operators at 18 nodes per wavelength, an odd node count
        {"name": "contour_n6007", "kind": "contour", "n": 6007, "k": 6007 / 18.0, "damped": False},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["assemble", "assemble", "product", "product", "product", "sweep", "solve", "calderon",
                       "gradient", "contour"])
    if kind == "assemble":
        dtype = rng.choice([C128, C64])
        f = round(_log(rng, 3, 31 if dtype == C64 else 20))
        return {"kind": kind, "f": f, "k": round(rng.uniform(0.1, 0.3 * f), 3), "dtype": dtype}
    if kind == "product":
        n = round(_log(rng, 300, 30000))
        return {"kind": kind, "n": n, "nrhs": round(_log(rng, 1, 512 if n < 16000 else 200)),
                "dtype": rng.choice([C64, C64, C128])}
    if kind == "sweep":
        return {"kind": kind, "f": round(_log(rng, 4, 20)), "k": round(rng.uniform(0.5, 4.0), 3),
                "nwave": round(_log(rng, 1, 512)), "ndir": round(_log(rng, 1, 512))}
    if kind == "solve":
        if rng.random() < 0.5:
            return {"kind": kind, "method": "cocg", "f": round(_log(rng, 3, 10)), "k": round(rng.uniform(0.5, 1.5), 3),
                    "nrhs": round(_log(rng, 1, 32)), "dtype": C128}
        return {"kind": kind, "method": "calderon", "f": round(_log(rng, 6, 14)), "k": round(rng.uniform(0.8, 2.0), 3),
                "nrhs": round(_log(rng, 9, 96)), "dtype": C64}
    if kind == "calderon":
        return {"kind": kind, "f": round(_log(rng, 3, 16)), "k": round(rng.uniform(0.3, 3.0), 3),
                "far": rng.choice([0.0, 4.0])}
    if kind == "gradient":
        return {"kind": kind, "f": round(_log(rng, 3, 18)), "k": round(rng.uniform(0.3, 2.5), 3),
                "ndir": round(_log(rng, 1, 128))}
    n = round(_log(rng, 150, 7000))
    return {"kind": kind, "n": n, "k": round(n / rng.uniform(14.0, 60.0), 3), "damped": rng.random() < 0.5}


# ------------------------------------------------------------------ surfaces
@functools.lru_cache(maxsize=16)
def _geodesic(f):
    """Unit geodesic sphere of frequency f: vertices in Morton order, outward triangles."""
    p = (1.0 + math.sqrt(5.0)) / 2.0
    c = np.array([[-1, p, 0], [1, p, 0], [-1, -p, 0], [1, -p, 0], [0, -1, p], [0, 1, p], [0, -1, -p], [0, 1, -p],
                  [p, 0, -1], [p, 0, 1], [-p, 0, -1], [-p, 0, 1]])
    d = np.linalg.norm(c[:, None] - c[None], axis=-1)
    adj = (d > 0) & (d < 2.1)
    corner = [(a, b, e) for a in range(12) for b in range(a + 1, 12) for e in range(b + 1, 12)
              if adj[a, b] and adj[b, e] and adj[a, e]]
    ij = [(i, j) for i in range(f + 1) for j in range(f + 1 - i)]
    at = {x: k for k, x in enumerate(ij)}
    lat = np.array([(i, j, f - i - j) for i, j in ij], dtype=np.float64) / f
    loc = [(at[i, j], at[i + 1, j], at[i, j + 1]) for i in range(f) for j in range(f - i)]
    loc += [(at[i + 1, j], at[i + 1, j + 1], at[i, j + 1]) for i in range(f) for j in range(f - i - 1)]
    loc = np.array(loc)
    pts, tri = [], []
    for t, e in enumerate(corner):
        pts.append(lat @ c[list(e)])
        tri.append(loc + t * len(lat))
    pts, tri = np.concatenate(pts), np.concatenate(tri)
    pts /= np.linalg.norm(pts, axis=1, keepdims=True)
    _, first, back = np.unique(np.round(pts, 8) + 0.0, axis=0, return_index=True, return_inverse=True)
    pts, tri = pts[first], back.reshape(-1)[tri]
    q = ((pts + 1.0) * 0.5 * (2 ** 20 - 1)).astype(np.int64)
    code = np.zeros(len(pts), dtype=np.int64)
    for b in range(20):
        for x in range(3):
            code |= ((q[:, x] >> b) & 1) << (3 * b + x)
    order = np.argsort(code, kind="stable")
    rank = np.empty(len(order), dtype=np.int64)
    rank[order] = np.arange(len(order))
    pts, tri = pts[order], rank[tri]
    # triangles follow their lowest vertex, so that neighbours in the list are neighbours in space
    tri = tri[np.argsort(tri.min(axis=1), kind="stable")]
    a, b, e = pts[tri[:, 0]], pts[tri[:, 1]], pts[tri[:, 2]]
    flip = np.einsum("ij,ij->i", np.cross(b - a, e - a), a + b + e) < 0
    tri[flip] = tri[flip][:, [0, 2, 1]]
    return pts, tri.astype(np.int32)


def _surface(f, seed):
    v, t = _geodesic(f)
    axes = np.random.default_rng([seed, f]).uniform(0.85, 1.15, size=3)
    return v * axes, t


def _directions(count, seed):
    rng = np.random.default_rng([seed, count, 1])
    z, ph = rng.uniform(-1, 1, count), rng.uniform(0, 2 * math.pi, count)
    s = np.sqrt(1 - z * z)
    rhat = np.stack([s * np.cos(ph), s * np.sin(ph), z], axis=1)
    that = np.stack([z * np.cos(ph), z * np.sin(ph), -s], axis=1)
    return rhat, that


def _normal(shape, seed, device="cuda"):
    g = torch.Generator(device=device).manual_seed(seed)
    return torch.complex(torch.randn(shape, generator=g, device=device, dtype=torch.float64),
                         torch.randn(shape, generator=g, device=device, dtype=torch.float64)) / math.sqrt(2.0)


def _dipoles(n, seed, dtype):
    """A matrix of the operator's kind at any order: eta j k (t_m . t_n) exp(-jkR)/(4 pi R) h^2 between
    tangential dipoles on a sphere, R^2 + h^2 in the place of R^2 (the diagonal is then the largest entry)."""
    rng = np.random.default_rng([seed, n, 2])
    i = np.arange(n) + 0.5
    z = 1 - 2 * i / n
    ph = math.pi * (1 + math.sqrt(5.0)) * i + rng.uniform(0, 2 * math.pi)
    s = np.sqrt(1 - z * z)
    r = np.stack([s * np.cos(ph), s * np.sin(ph), z], axis=1)
    t = np.cross(r, rng.standard_normal((n, 3)))
    t /= np.linalg.norm(t, axis=1, keepdims=True)
    h2, k = 4 * math.pi / n, 0.3 * math.sqrt(n / 30.0)
    r, t = (torch.as_tensor(x, device="cuda") for x in (r, t))
    Z = torch.empty((n, n), dtype=TYPES[dtype], device="cuda")
    for a in range(0, n, 4096):
        g = r[a:a + 4096] @ r.T
        R = (2.0 - 2.0 * g).clamp_(min=0.0).add_(h2).sqrt_()
        amp = (t[a:a + 4096] @ t.T) * (ETA * k * h2 / (4 * math.pi)) / R
        R *= k
        Z[a:a + 4096] = torch.complex(amp * torch.sin(R), amp * torch.cos(R)).to(Z.dtype)
    return Z


def _contour(n, seed):
    """n nodes of an ellipse, equally spaced in arc length, perimeter 2 pi; and of the circle of that perimeter."""
    aspect = np.random.default_rng([seed, n, 3]).uniform(1.2, 1.8)
    th = 2 * math.pi * np.arange(1 << 17) / (1 << 17)
    z = np.stack([aspect * np.cos(th), np.sin(th)], axis=1)
    s = np.concatenate([[0.0], np.cumsum(np.linalg.norm(np.roll(z, -1, axis=0) - z, axis=1))])
    u = np.interp(s[-1] * np.arange(n) / n, s, 2 * math.pi * np.arange(len(s)) / (1 << 17))
    c = 2 * math.pi * np.arange(n) / n
    return (np.stack([aspect * np.cos(u), np.sin(u)], axis=1) * (2 * math.pi / s[-1]),
            np.stack([np.cos(c), np.sin(c)], axis=1))


def _contour_k(case):
    return efie.ktilde(case["k"]) if case["damped"] else case["k"]


# ------------------------------------------------------------------ prepare and run
def prepare(case, seed):
    kind = case["kind"]
    if kind == "product":
        return {"case": case, "Z": _dipoles(case["n"], seed, case["dtype"]),
                "X": _normal((case["nrhs"], case["n"]), seed + 7).to(TYPES[case["dtype"]])}
    if kind == "contour":
        return {"case": case, "op": efie.Bie2d(*_contour(case["n"], seed)), "k": _contour_k(case)}
    mesh = efie.Mesh(*_surface(case["f"], seed)).upload()
    s = {"case": case, "mesh": mesh}
    if kind == "sweep":
        s["rhat"], s["that"] = _directions(max(case["nwave"], case["ndir"]), seed)
        s["J"] = _normal((case["nwave"], mesh.n), seed + 7) * 1e-3
    elif kind == "solve":
        rhat, that = _directions(case["nrhs"], seed)
        s["V"] = efie.excite_planewave(mesh, case["k"], -rhat, that)
        s["Z"] = efie.convert(efie.assemble(mesh, case["k"]), case["dtype"])
        if case["method"] == "calderon":
            cal = efie.Calderon(mesh).set_far_rule(4.0)
            s["P"] = efie.convert(cal.assemble(efie.ktilde(case["k"]), tol=1e-3, bary_dtype=C64), case["dtype"])
    elif kind == "calderon":
        s["cal"] = efie.Calderon(mesh).set_far_rule(case["far"]).upload()
        s["kt"] = efie.ktilde(case["k"])
    elif kind == "gradient":
        s["rhat"], _ = _directions(case["ndir"], seed)
        khat, pol = _directions(1, seed + 1)
        s["khat"], s["pol"] = khat[0], pol[0]
        s["J"], s["lam"] = _normal((mesh.n,), seed + 7) * 1e-3, _normal((mesh.n,), seed + 8) * 1e-3
        s["W"] = _normal((case["ndir"], 2), seed + 9)
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "assemble":
        return efie.assemble(s["mesh"], case["k"], dtype=case["dtype"])
    if kind == "product":
        return efie.zx(s["Z"], s["X"])
    if kind == "sweep":
        return {"V": efie.excite_planewave(s["mesh"], case["k"], -s["rhat"][:case["nwave"]], s["that"][:case["nwave"]]),
                "F": efie.farfield(s["mesh"], case["k"], s["J"], s["rhat"][:case["ndir"]])}
    if kind == "solve":
        # 1e-12: the currents are then those of the stored matrix, whatever the order of the sums
        if case["method"] == "calderon":
            return efie.solve_precond(s["Z"], s["P"], s["V"], tol=1e-12, max_refine=12, inner_tol=1e-3)[0]
        return efie.solve(s["Z"], s["V"], tol=1e-12, maxit=3000)[0]
    if kind == "calderon":
        return s["cal"].assemble(s["kt"])
    if kind == "gradient":
        return efie.vertex_grad(s["mesh"], case["k"], s["J"], s["lam"], s["W"], s["rhat"], s["khat"], s["pol"])
    return s["op"].assemble(s["k"])


# ------------------------------------------------------------------ work
def work(case):
    """Operations: a Green's function of two points in 3-D is counted as 40 (distance, root, sine and cosine,
    moments), a Hankel pair in 2-D as 80, a plane-wave phase at a point as 30, a complex product as 8."""
    kind = case["kind"]
    if kind == "product":
        n, m, e = case["n"], case["nrhs"], 16 if case["dtype"] == C128 else 8
        return {"bytes": e * (n * n + 2.0 * n * m), "flops": 8.0 * n * n * m}
    if kind == "contour":
        return {"bytes": 48.0 * case["n"] ** 2, "flops": 16.0 * 80 * case["n"] ** 2}
    n, t = 30 * case["f"] ** 2, 20 * case["f"] ** 2
    pairs = 49.0 * 40 * t * (t + 1) / 2
    if kind == "assemble":
        return {"bytes": n * n * (16.0 if case["dtype"] == C128 else 8.0), "flops": pairs}
    if kind == "sweep":
        return {"bytes": 16.0 * (2 * case["nwave"] * n + 2 * case["nwave"] * case["ndir"]),
                "flops": 7.0 * 30 * t * (case["nwave"] + case["ndir"]) + 16.0 * case["nwave"] * case["ndir"] * n}
    if kind == "solve":
        # no fewer than one product (two with the preconditioner) for each decade of the residual
        two = 2 if case["method"] == "calderon" else 1
        e = 16.0 if case["dtype"] == C128 else 8.0
        return {"bytes": two * e * n * n + 32.0 * n * case["nrhs"], "flops": 12 * two * 8.0 * n * n * case["nrhs"]}
    if kind == "calderon":
        return {"bytes": 16.0 * n * n, "flops": 36 * pairs}
    return {"bytes": 48.0 * n + 24.0 * n / 3, "flops": 2.5 * pairs}


# ------------------------------------------------------------------ the same in 64 bits, with torch alone
def _radon():
    s = math.sqrt(15.0)
    a1, b1, a2, b2 = (9 - 2 * s) / 21, (6 + s) / 21, (9 + 2 * s) / 21, (6 - s) / 21
    bary = [[1 / 3] * 3, [a1, b1, b1], [b1, a1, b1], [b1, b1, a1], [a2, b2, b2], [b2, a2, b2], [b2, b2, a2]]
    return bary, [9 / 40] + [(155 + s) / 1200] * 3 + [(155 - s) / 1200] * 3


class _Rwg:
    """RWG tables and 7-point data of a surface: functions numbered by their vertex pairs in lexicographic order,
    + on the triangle that runs from the lower to the higher vertex."""

    def __init__(self, v, t):
        t = t.astype(np.int64)
        a, b = t[:, [1, 2, 0]].reshape(-1), t[:, [2, 0, 1]].reshape(-1)
        pair, edge = np.unique(np.stack([np.minimum(a, b), np.maximum(a, b)], 1), axis=0, return_inverse=True)
        up = lambda x: torch.as_tensor(np.ascontiguousarray(x), device="cuda")  # noqa: E731
        self.n, self.t = len(pair), len(t)
        self.edge = up(edge.reshape(-1, 3))
        bary, w = (torch.tensor(x, dtype=torch.float64, device="cuda") for x in _radon())
        self.tri, self.x = up(t), up(v)[up(t)]                                       # (T, 3, 3)
        e = self.x[:, [2, 0, 1]] - self.x[:, [1, 2, 0]]                               # edge opposite vertex i
        nrm = torch.linalg.cross(self.x[:, 1] - self.x[:, 0], self.x[:, 2] - self.x[:, 0])
        two_a = nrm.norm(dim=1)
        self.normal, self.len = nrm / two_a[:, None], e.norm(dim=2)
        self.h = self.len.max(dim=1).values
        self.q = torch.einsum("pk,tkx->tpx", bary, self.x)                            # (T, 7, 3)
        self.w = 0.5 * two_a[:, None] * w
        sl = up(np.where(a < b, 1.0, -1.0).reshape(-1, 3)) * self.len
        self.c, self.div = sl / two_a[:, None], 2 * sl / two_a[:, None]
        self.f = self.c[:, :, None, None] * (self.q[:, None] - self.x[:, :, None])    # (T, 3, 7, 3)

    def near(self, p):
        """Sources near the test triangles p: a shared vertex, or centroids within twice the longest edge."""
        c = self.x.mean(dim=1)
        d = (c[p][:, None] - c[None]).norm(dim=2) < 2.0 * torch.maximum(self.h[p][:, None], self.h[None])
        for i in range(3):
            for j in range(3):
                d |= self.tri[p][:, None, i] == self.tri[None, :, j]
        return d

    def static(self, p, q):
        """int int f_i . f_j / (4 pi R) and the same of the charges for the pairs (p, q): the closed inner integrals
        of Wilton et al. 1984 over q, the 7-point rule over p."""
        r, n = self.q[p], self.normal[q][:, None]
        d = ((r - self.x[q][:, None, 0]) * n).sum(-1)
        rho = r - d[..., None] * n
        i0, i1 = torch.zeros_like(d), torch.zeros_like(rho)
        for e in range(3):
            a, b = self.x[q][:, None, e], self.x[q][:, None, (e + 1) % 3]
            lt = (b - a) / (b - a).norm(dim=-1, keepdim=True)
            u = torch.linalg.cross(lt, n)
            lp, lm, p0 = ((b - rho) * lt).sum(-1), ((a - rho) * lt).sum(-1), ((a - rho) * u).sum(-1)
            rp, rm, r02 = (r - b).norm(dim=-1), (r - a).norm(dim=-1), p0 * p0 + d * d
            up = torch.where(lp >= 0, rp + lp, r02 / torch.where(lp >= 0, torch.ones_like(lp), rp - lp))
            dn = torch.where(lm >= 0, rm + lm, r02 / torch.where(lm >= 0, torch.ones_like(lm), rm - lm))
            keep = r02.sqrt() >= 1e-12 * self.h[q][:, None]
            zero = torch.zeros_like(d)
            lg = torch.where(keep, torch.log(up / dn), zero)
            at = torch.where(keep, torch.atan(p0 * lp / (r02 + d.abs() * rp)) - torch.atan(p0 * lm / (r02 + d.abs() * rm)),
                             zero)
            i0 = i0 + p0 * lg - d.abs() * at
            i1 = i1 + 0.5 * (r02 * lg + lp * rp - lm * rm)[..., None] * u
        inner = self.c[q][:, :, None, None] * (i1[:, None] + (rho[:, None] - self.x[q][:, :, None]) * i0[:, None, :, None])
        ta = torch.einsum("pa,piax,pjax->pij", self.w[p], self.f[p], inner) / (4 * math.pi)
        s0 = (self.w[p] * i0).sum(-1) / (4 * math.pi)
        return ta, self.div[p][:, :, None] * self.div[q][:, None] * s0[:, None, None]

    def z(self, k):
        out = torch.zeros((self.n, self.n), dtype=torch.complex128, device="cuda")
        step = max(1, int(4e7 / (49 * self.t)))
        w_, x_ = self.w.reshape(-1), self.q.reshape(-1, 3)
        for a in range(0, self.t, step):
            p = torch.arange(a, min(self.t, a + step), device="cuda")
            near = self.near(p)
            R = ((self.q[p].reshape(-1, 1, 3) - x_) ** 2).sum(-1).sqrt()                # (7p, 7T)
            is_near = near.repeat_interleave(7, 0).repeat_interleave(7, 1)
            far = torch.where(is_near, torch.full_like(R, math.inf), R)
            far = torch.where(is_near, 0.0, 1.0 / (4 * math.pi * far)) * w_
            ph = k * R
            re, im = (far * torch.cos(ph)).reshape(-1, self.t, 7), (-far * torch.sin(ph)).reshape(-1, self.t, 7)
            del R, is_near, far, ph
            g = torch.complex(re, im)                                                   # weights of the source in it
            m0 = g.sum(-1)
            m1 = torch.stack([(g * self.q[None, :, :, x]).sum(-1) for x in range(3)], -1)
            blk = torch.empty((len(p), self.t, 3, 3), dtype=torch.complex128, device="cuda")
            m0, m1 = m0.reshape(len(p), 7, self.t), m1.reshape(len(p), 7, self.t, 3)
            s0 = (self.w[p][:, :, None] * m0).sum(1)
            wf = self.w[p][:, None, :, None] * self.f[p]                                # (p, 3, 7, 3)
            for i in range(3):
                f1 = sum((wf[:, i, :, x, None] * m1[..., x]).sum(1) for x in range(3))   # (p, T)
                f0 = [(wf[:, i, :, x, None] * m0).sum(1) for x in range(3)]
                for j in range(3):
                    ta = self.c[:, j] * (f1 - sum(f0[x] * self.x[:, j, x] for x in range(3)))
                    blk[:, :, i, j] = ETA * (1j * k * ta + self.div[p][:, i, None] * self.div[:, j] * s0 / (1j * k))
            pi, qi = near.nonzero(as_tuple=True)
            blk[pi, qi] = self._near_block(k, p[pi], qi)
            rows = torch.zeros((len(p), 3, self.n), dtype=torch.complex128, device="cuda")
            for j in range(3):
                rows.index_add_(2, self.edge[:, j], blk[:, :, :, j].permute(0, 2, 1).contiguous())
            for i in range(3):
                out.index_add_(0, self.edge[p][:, i], rows[:, i].contiguous())
        return out

    def _near_block(self, k, p, q):
        R = (self.q[p][:, :, None] - self.q[q][:, None]).norm(dim=-1)
        zero = R <= 1e-14 * self.h[p][:, None, None]
        y, Rs = k * R, torch.where(zero, torch.ones_like(R), R)
        g = torch.complex(-2 * torch.sin(0.5 * y) ** 2, -torch.sin(y)) / (4 * math.pi * Rs)
        g = torch.where(zero, torch.full_like(g, -1j * k / (4 * math.pi)), g)
        g = g * self.w[p][:, :, None] * self.w[q][:, None]
        ta = torch.stack([torch.stack([(g * (self.f[p][:, i, :, None] * self.f[q][:, j, None]).sum(-1)).sum((1, 2))
                                       for j in range(3)], -1) for i in range(3)], -2)
        tp = self.div[p][:, :, None] * self.div[q][:, None] * g.sum((1, 2))[:, None, None]
        a1, p1 = self.static(p, q)
        a2, p2 = self.static(q, p)
        ta = ta + 0.5 * (a1 + a2.transpose(1, 2))
        tp = tp + 0.5 * (p1 + p2.transpose(1, 2))
        return ETA * (1j * k * ta + tp / (1j * k))

    def planewaves(self, k, khat, pol):
        V = torch.zeros((len(khat), self.n), dtype=torch.complex128, device="cuda")
        for s in range(len(khat)):
            g = self.w * torch.exp(-1j * k * (self.q @ khat[s]))
            e = (g[:, None] * (self.f @ pol[s])).sum(-1)
            for i in range(3):
                V[s].index_add_(0, self.edge[:, i], e[:, i].contiguous())
        return V

    def farfield(self, k, J, dirs):
        z, ph = dirs[:, 2], torch.atan2(dirs[:, 1], dirs[:, 0])
        s = (1 - z * z).sqrt()
        base = torch.stack([torch.stack([z * ph.cos(), z * ph.sin(), -s], -1),
                            torch.stack([-ph.sin(), ph.cos(), torch.zeros_like(ph)], -1)], 1)
        F = torch.empty((len(J), len(dirs), 2), dtype=torch.complex128, device="cuda")
        for d in range(len(dirs)):
            R = self.planewaves(-k, dirs[d].expand(2, 3), base[d])
            F[:, d] = J @ R.T.contiguous()
        return F * (-1j * k * ETA / (4 * math.pi))


def _macdonald(w):
    """K_0 and K_1 of complex w, Re w >= 0: their power series below |w| = 4, from there the trapezoidal rule on
    K_0 = e^-w w^-1/2 int e^(-t^2) (2 + t^2/w)^-1/2 dt and K_1, which has 1 + t^2/w more (their integrals over cosh
    with t^2 = w (cosh - 1)); with steps of 1/4 its error is below 1e-16 there."""
    small = w.abs() < 4.0
    u = torch.where(small, torch.full_like(w, 4.0), w)
    k0, k1 = torch.zeros_like(w), torch.zeros_like(w)
    for i in range(27):
        a = (0.25 * i) ** 2 / u
        g = ((0.25 if i else 0.125) * 2 * math.exp(-(0.25 * i) ** 2)) / (2 + a).sqrt()
        k0 = k0 + g
        k1 = k1 + g * (1 + a)
    e = torch.exp(-u) / u.sqrt()
    k0, k1 = k0 * e, k1 * e
    u = torch.where(small, w, torch.ones_like(w))
    q, lg = u * u / 4, torch.log(u / 2)
    t0, t1 = torch.ones_like(w), u / 2
    s0, s1, har = -(lg + np.euler_gamma), 1 / u + (lg + np.euler_gamma - 0.5) * t1, 0.0
    for i in range(1, 26):
        t0, t1, har = t0 * q / i ** 2, t1 * q / (i * (i + 1)), har + 1.0 / i
        s0 = s0 + t0 * (har - np.euler_gamma - lg)
        s1 = s1 + t1 * (lg + np.euler_gamma - har - 0.5 / (i + 1))
    return torch.where(small, s0, k0), torch.where(small, s1, k1)


def _contour_exact(nodes, k):
    """S, D*, N of the polygon at k: 4 x 4 Gauss points on separate segments, an 8 x 8 Duffy rule graded to the
    shared node on neighbours, the logarithm in closed form on a segment with itself."""
    up = lambda x: torch.as_tensor(x, device="cuda", dtype=torch.float64)  # noqa: E731
    n = len(nodes)
    A = up(nodes)
    B = A.roll(-1, 0)
    L = (B - A).norm(dim=1)
    t = (B - A) / L[:, None]
    nrm = torch.stack([t[:, 1], -t[:, 0]], 1)

    def kernels(R):
        k0, k1 = _macdonald(1j * k * R)
        return k0 / (2 * math.pi), -1j * k / (2 * math.pi) * k1

    def gauss(m):
        x, w = np.polynomial.legendre.leggauss(m)
        return up(0.5 * (x + 1)), up(0.5 * w)

    hat = lambda x: (1 - x, x)  # noqa: E731
    out = [torch.zeros((n, n), dtype=torch.complex128, device="cuda") for _ in range(3)]

    def add(a, b, S, D, m0):
        """Moments (pairs,) of test segments a and sources b into the entries of their nodes."""
        LL, nn = L[a] * L[b], (nrm[a] * nrm[b]).sum(-1)
        for i in range(2):
            for j in range(2):
                s = LL * S[i][j]
                at = ((a + i) % n, (b + j) % n)
                out[0].index_put_(at, s, accumulate=True)
                out[1].index_put_(at, LL * D[i][j], accumulate=True)
                out[2].index_put_(at, (1 if i == j else -1) * m0 - k * k * nn * s, accumulate=True)

    xg, wg = gauss(4)
    every = torch.arange(n, device="cuda")
    for a0 in range(0, n, 256):
        a = every[a0:a0 + 256].repeat_interleave(n)
        b = every.repeat(min(256, n - a0))
        far = (a != b) & ((a + 1) % n != b) & ((b + 1) % n != a)
        a, b = a[far], b[far]
        S = [[0, 0], [0, 0]]
        D = [[0, 0], [0, 0]]
        m0 = 0
        for p in range(4):
            for q in range(4):
                d = A[a] + xg[p] * (B[a] - A[a]) - A[b] - xg[q] * (B[b] - A[b])
                R = d.norm(dim=1)
                G, H = kernels(R)
                w = float(wg[p] * wg[q])
                G, H = w * G, w * H * (d * nrm[a]).sum(-1) / R
                m0 = m0 + G
                for i in range(2):
                    for j in range(2):
                        c = float(hat(xg[p])[i] * hat(xg[q])[j])
                        S[i][j], D[i][j] = S[i][j] + c * G, D[i][j] + c * H
        add(a, b, S, D, m0)
    x8, w8 = gauss(8)
    for side in (1, -1):
        a, b = every, (every + side) % n
        V, Pa, Pb = (B[a], A[a], B[b]) if side == 1 else (A[a], B[a], A[b])
        S = [[0, 0], [0, 0]]
        D = [[0, 0], [0, 0]]
        m0 = 0
        for p in range(8):
            for q in range(8):
                for u, v in ((x8[p] ** 2, x8[p] ** 2 * x8[q]), (x8[p] ** 2 * x8[q], x8[p] ** 2)):
                    d = u * (Pa - V) - v * (Pb - V)
                    R = d.norm(dim=1)
                    G, H = kernels(R)
                    w = float(w8[p] * w8[q] * 2 * x8[p] ** 3)
                    G, H = w * G, w * H * (d * nrm[a]).sum(-1) / R
                    m0 = m0 + G
                    ha, hb = hat(1 - u if side == 1 else u), hat(v if side == 1 else 1 - v)
                    for i in range(2):
                        for j in range(2):
                            c = float(ha[i] * hb[j])
                            S[i][j], D[i][j] = S[i][j] + c * G, D[i][j] + c * H
        add(a, b, S, D, m0)
    S = [[0, 0], [0, 0]]
    m0 = 0
    for p in range(8):
        for q in range(8):
            R = L * abs(float(x8[p] - x8[q]))
            w = float(w8[p] * w8[q])
            if p == q:
                G = torch.ones_like(R) * (-0.25j - (np.log(k / 2) + np.euler_gamma) / (2 * math.pi))
            else:
                G = kernels(R)[0] + torch.log(R) / (2 * math.pi)
            m0 = m0 + w * G
            for i in range(2):
                for j in range(2):
                    S[i][j] = S[i][j] + w * float(hat(x8[p])[i] * hat(x8[q])[j]) * G
    for i in range(2):
        for j in range(2):
            S[i][j] = S[i][j] - (0.25 * torch.log(L) - (7 if i == j else 5) / 16) / (2 * math.pi)
    m0 = m0 - (torch.log(L) - 1.5) / (2 * math.pi)
    zero = torch.zeros_like(m0)
    add(every, every, S, [[zero, zero], [zero, zero]], m0)
    return tuple(out)


def exact(case, seed):
    """What run() computes, in 64 bits.  None for the preconditioner (its dual basis is this library's own choice among
    equivalent ones) and for the gradient (a reverse pass through the whole matrix takes too long)."""
    kind = case["kind"]
    if kind in ("calderon", "gradient"):
        return None
    if kind == "product":
        s = prepare(case, seed)
        Z, X = s["Z"], s["X"].to(torch.complex128)
        Y = torch.empty_like(X)
        for a in range(0, case["n"], 4096):
            Y[:, a:a + 4096] = X @ Z[a:a + 4096].to(torch.complex128).T.contiguous()
        return Y
    if kind == "contour":
        return _contour_exact(_contour(case["n"], seed)[0], _contour_k(case))
    m = _Rwg(*_surface(case["f"], seed))
    up = lambda x: torch.as_tensor(x, device="cuda")  # noqa: E731
    k = case["k"]
    if kind == "assemble":
        return m.z(k)
    if kind == "sweep":
        rhat, that = _directions(max(case["nwave"], case["ndir"]), seed)
        J = _normal((case["nwave"], m.n), seed + 7) * 1e-3
        return {"V": m.planewaves(k, up(-rhat[:case["nwave"]]), up(that[:case["nwave"]])),
                "F": m.farfield(k, J, up(rhat[:case["ndir"]]))}
    rhat, that = _directions(case["nrhs"], seed)
    Z = m.z(k).to(TYPES[case["dtype"]]).to(torch.complex128)
    return torch.linalg.solve(Z, m.planewaves(k, up(-rhat), up(that)).T.contiguous()).T.contiguous()
