"""Performance cases of the AGCA multigrid library: what a program that uses it has it do.

The sizes are those of the repository's workloads: lattices of n = 2^(L+1) cells per axis
(n + 1 nodes, always odd) from the 17^3 scalar diffusion problem to the 513^3 vector
viscous block, with their coefficients (an aligned cube, tanh-smoothed spherical sinkers,
sums of Gaussians in log nu), both smoothers, FP64 and FP32 multigrid with FP32 or BF16
finest coefficients.

Operations (`op`):
  apply    one product with a level's operator
  vcycle   one V-cycle, the preconditioner of every solver
  solve    a whole Krylov solve to the default tolerance
  adjoint  one step of an inverse problem: rebuild from log nu, forward solve, adjoint
           solve, gradients (paper_2511_13109_amd.autograd)
  stokes   one FGMRES cycle of the Stokes solver
  schur    the BFBT Schur approximation with the pressure multigrid

`exact` evaluates the same definitions with plain torch operations in FP64 on whole
arrays: nodal vectors are (ncomp, n+1, n+1, n+1) arrays [c, z, y, x], coefficients are
(n, n, n, 6) arrays [z, y, x, s] with s the axis order of a Kuhn simplex.
"""

import math

import numpy as np
import torch

from paper_2511_13109_amd import Hierarchy, Stokes
from paper_2511_13109_amd.autograd import solve as adjoint_solve

DEVICE = "cuda"


def listed():
    return [
        # the smallest problem of the workloads: 17^3 scalar diffusion with damped Jacobi.
        # Launches and latency are all of it.
        dict(name="vcycle_17_scalar", op="vcycle", L=3, ncomp=1, dtype="f64", smoother="jacobi",
             field="cube", contrast=1e3, count=1),
        # a product with the operator at the size of a coarsening study's inner level
        dict(name="apply_33_vector", op="apply", L=4, level=4, ncomp=3, dtype="f64", smoother="jacobi",
             field="sinkers", contrast=1e4, count=4),
        # preconditioner of the 65^3 coarsening study
        dict(name="vcycle_65_vector", op="vcycle", L=5, ncomp=3, dtype="f64", smoother="chebyshev",
             field="sinkers", contrast=1e6, count=4),
        # preconditioner of the 129^3 sinker workload, in FP64 and in the mixed form
        dict(name="vcycle_129_vector", op="vcycle", L=6, ncomp=3, dtype="f64", smoother="chebyshev",
             field="sinkers", contrast=1e6, count=8),
        dict(name="vcycle_129_mixed", op="vcycle", L=6, ncomp=3, dtype="bf16", smoother="chebyshev",
             field="sinkers", contrast=1e6, count=8),
        # scalar product above the Infinity Cache
        dict(name="apply_257_scalar", op="apply", L=7, level=7, ncomp=1, dtype="f64", smoother="jacobi",
             field="sinkers", contrast=1e6, count=16),
        # the benchmark's workload at full size: FP64 product and mixed V-cycle at 513^3
        dict(name="apply_513_vector", op="apply", L=8, level=8, ncomp=3, dtype="f64", smoother="jacobi",
             field="sinkers", contrast=1e6, count=16),
        dict(name="vcycle_513_mixed", op="vcycle", L=8, ncomp=3, dtype="bf16", smoother="chebyshev",
             field="sinkers", contrast=1e6, count=16),
        # a whole mixed solve: FP64 FCG around the FP32/BF16 V-cycle
        dict(name="solve_129_mixed", op="solve", L=6, ncomp=3, dtype="bf16", smoother="chebyshev",
             field="sinkers", contrast=1e2, count=8),
        # one training-like step of the viscosity inversion: forward and backward
        dict(name="adjoint_129", op="adjoint", L=6, ncomp=3, dtype="f64", smoother="chebyshev",
             field="gauss", contrast=1e4, count=16),
        # one FGMRES cycle of the Stokes solver with the paper's triangular preconditioner
        dict(name="stokes_129", op="stokes", L=6, ncomp=3, dtype="f64", smoother="chebyshev",
             field="sinkers", contrast=1e4, count=8, restart=30, basis="f64"),
        # the BFBT Schur approximation at the Stokes workload's size (pressure 129^3)
        dict(name="schur_257", op="schur", L=7, ncomp=3, dtype="f64", smoother="chebyshev",
             field="sinkers", contrast=1e6, count=16),
    ]


def draw(rng):
    """Sizes are uniform in L, which is uniform in the logarithm of the lattice size."""
    op = rng.choice(["apply", "apply", "vcycle", "vcycle", "vcycle", "solve", "adjoint", "stokes", "schur"])
    top = {"apply": 8, "vcycle": 8, "solve": 6, "adjoint": 6, "stokes": 6, "schur": 7}[op]
    L = rng.randint(4 if op in ("stokes", "schur") else 3, top)
    c = dict(op=op, L=L, ncomp=3 if op in ("stokes", "schur") else rng.choice([1, 3, 3]))
    c["dtype"] = "f64" if op in ("stokes", "schur", "adjoint") else rng.choice(["f64", "f32", "bf16"])
    c["smoother"] = rng.choice(["chebyshev", "chebyshev", "jacobi"])
    c["field"] = "gauss" if op == "adjoint" else rng.choice(["sinkers", "sinkers", "gauss"])
    high = {"solve": 2.0, "adjoint": 4.0, "stokes": 4.0}.get(op, 6.0)
    c["contrast"] = round(10.0 ** rng.uniform(1.0, high), 3)
    c["count"] = rng.randint(1, 16)
    if op == "apply":
        c["level"] = rng.choice([L, L, L - 1])
    elif op == "vcycle":
        c["storage"] = rng.choice(["blocks", "blocks", "mean"])
    elif op == "stokes":
        c["restart"] = rng.choice([20, 30, 48])
        c["basis"] = "f64"
    return c


# ---------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------
AXES = [(0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)]


def _centroids(n, s):
    """x, y and z coordinates of the centroids of simplex s of every cell (broadcastable)."""
    i = torch.arange(n, dtype=torch.float64, device=DEVICE)
    t = [(i + (3 - AXES[s].index(a)) / 4.0) / n for a in range(3)]
    return t[0].view(1, 1, n), t[1].view(1, n, 1), t[2].view(n, 1, 1)


def _coefficients(case, seed):
    """nu of every level 0..L, (6 n^3,) FP64 by element id: one field at all centroids."""
    rng = np.random.default_rng(seed)
    L, m = case["L"], case["count"]
    high, low = math.sqrt(case["contrast"]), 1.0 / math.sqrt(case["contrast"])
    centres = rng.uniform(0.2, 0.8, size=(m, 3))
    if case["field"] == "cube":  # the box of half-width 1/8 around the middle
        centres = np.full((1, 3), 0.5)
    spread = rng.uniform(0.05, 0.2, size=m) if case["field"] == "gauss" else np.full(m, 0.1)
    amps = rng.uniform(-1.0, 1.0, size=m)
    width = 2.0 / 2 ** (L + 1)

    def part(n, s):
        x, y, z = _centroids(n, s)
        if case["field"] == "cube":
            inside = ((x - 0.5).abs() <= 0.125) & ((y - 0.5).abs() <= 0.125) & ((z - 0.5).abs() <= 0.125)
            return torch.where(inside, 1e3, 1.0).to(torch.float64)
        acc = torch.full((n, n, n), 1.0 if case["field"] == "sinkers" else 0.0, dtype=torch.float64, device=DEVICE)
        for p, r, a in zip(centres, spread, amps):
            d2 = ((x - p[0]) ** 2 + (y - p[1]) ** 2) + (z - p[2]) ** 2
            if case["field"] == "sinkers":
                acc.mul_(d2.sqrt_().sub_(float(r)).div_(width).tanh_().add_(1.0).mul_(0.5))
            else:
                acc.add_(d2.mul_(-0.5 / float(r) ** 2).exp_(), alpha=float(a))
        return acc.mul_(low - high).add_(high) if case["field"] == "sinkers" else acc

    out = [torch.empty((2 << l, 2 << l, 2 << l, 6), dtype=torch.float64, device=DEVICE) for l in range(L + 1)]
    for l in range(L + 1):
        for s in range(6):
            out[l][..., s] = part(2 << l, s)
    if case["field"] == "gauss":  # log nu rescaled to [log low, log high] by the finest range
        lo, hi = float(out[L].min()), float(out[L].max())
        for l in range(L + 1):
            out[l] = ((out[l] - lo) * (2.0 * math.log(high) / (hi - lo)) - math.log(high)).exp_()
    return [t.reshape(-1) for t in out]


def _noise(case, seed, count, dtype=torch.float64):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return torch.randn(count, generator=g, device=DEVICE, dtype=dtype)


def _nodes(l):
    return ((2 << l) + 1) ** 3


def _vector_dtype(case):
    return torch.float64 if case["dtype"] == "f64" else torch.float32


def _inputs(case, seed):
    """The coefficient and the vectors of a case, from the seed alone."""
    nu = _coefficients(case, seed)
    L, nc = case["L"], case["ncomp"]
    v = {}
    if case["op"] == "apply":
        v["u"] = _noise(case, seed + 1, nc * _nodes(case["level"]), _vector_dtype(case))
    elif case["op"] == "vcycle":
        v["b"] = _noise(case, seed + 1, nc * _nodes(L), _vector_dtype(case))
    elif case["op"] == "schur":
        r = _noise(case, seed + 1, _nodes(L - 1))
        v["r"] = r - r.mean()
    else:
        # a buoyancy-like load: smooth in space, scaled like the integral of a body force
        n = 2 << L
        i = torch.arange(n + 1, dtype=torch.float64, device=DEVICE) / n
        k = np.random.default_rng(seed + 2).integers(1, 4, size=(nc, 3))
        w = [torch.sin(math.pi * int(a) * i).view(-1, 1, 1) * torch.sin(math.pi * int(b) * i).view(1, -1, 1) *
             torch.sin(math.pi * int(c) * i).view(1, 1, -1) for a, b, c in k]
        v["b"] = (torch.stack(w) / n ** 3).reshape(-1)
        if case["op"] == "adjoint":
            v["log_nu"] = nu[L].log()
            v["y"] = v["b"] * n ** 3 + 0.1 * _noise(case, seed + 1, nc * _nodes(L))
    return nu, v


def prepare(case, seed):
    nu, v = _inputs(case, seed)
    L = case["L"]
    mg = "f64" if case["dtype"] == "f64" else "f32"
    H = Hierarchy(L, case["ncomp"], nu[L], nu[:L], mg_dtype=mg, mg_nu_dtype=case["dtype"], smoother=case["smoother"],
                  coarse_storage=case.get("storage", "blocks"))
    s = dict(v, case=case, H=H)
    if case["op"] == "apply":
        s["out"] = torch.empty_like(v["u"])
    elif case["op"] == "vcycle":
        s["out"] = torch.empty_like(v["b"])
    elif case["op"] == "adjoint":
        s["coarse"] = nu[:L]
        s["log_nu"].requires_grad_(True)
        s["b"].requires_grad_(True)
    elif case["op"] in ("stokes", "schur"):
        s["S"] = Stokes(H)
        if case["op"] == "schur":
            s["out"] = s["S"].schur_apply(v["r"], schur="bfbt_mg", schur_iters=4)  # assembles the pressure multigrid
    return s


def run(s):
    c, H = s["case"], s["H"]
    if c["op"] == "apply":
        return H.apply(c["level"], s["u"], s["out"])
    if c["op"] == "vcycle":
        return H.vcycle(s["b"], s["out"])
    if c["op"] == "solve":
        x, _ = H.solve(s["b"], solver="pcg" if c["dtype"] == "f64" else "fcg")
        return x
    if c["op"] == "adjoint":
        u = adjoint_solve(s["log_nu"], s["b"], H, s["coarse"])
        g, w = torch.autograd.grad(u, (s["log_nu"], s["b"]), grad_outputs=s["y"])
        return u.detach(), g, w
    if c["op"] == "stokes":
        # an inexact solve: one restart cycle, whatever residual it reaches
        u, p, _ = s["S"].solve(s["b"], solver="fgmres", precond="triangular", schur="mass", restart=c["restart"],
                               max_iter=c["restart"], tol=1e-12, basis=c["basis"], raise_on_noconv=False)
        return u, p
    return s["S"].schur_apply(s["r"], schur="bfbt_mg", schur_iters=4, q=s["out"])


def work(case):
    """Bytes: inputs (vectors and the coefficient of every level used) once, outputs once.
    Flops: those of the level operators, about 234 per cell for the vector form (6 simplices
    of 9 edge differences, 6 stress sums and 24 flux updates) and 72 for the scalar one."""
    L, nc = case["L"], case["ncomp"]
    n3 = float((2 << L) ** 3)
    vec = nc * _nodes(L) * (8.0 if case["dtype"] == "f64" else 4.0)
    vec64 = nc * _nodes(L) * 8.0
    nu = 6.0 * n3 * {"f64": 8.0, "f32": 4.0, "bf16": 2.0}[case["dtype"]]
    nu_all = nu + 6.0 * n3 / 7.0 * (8.0 if case["dtype"] == "f64" else 4.0)
    per = 234.0 if nc == 3 else 72.0
    if case["op"] == "apply":
        if case["level"] < L:
            return {"bytes": (2.0 * vec + 6.0 * n3 * (8.0 if case["dtype"] == "f64" else 4.0)) / 8.0, "flops": per * n3 / 8.0}
        return {"bytes": 2.0 * vec + nu, "flops": per * n3}
    if case["op"] == "vcycle":
        return {"bytes": 2.0 * vec + nu_all, "flops": 4.0 * per * n3 * 8.0 / 7.0}
    if case["op"] == "solve":
        return {"bytes": 2.0 * vec64 + 6.0 * n3 * 8.0 + nu_all, "flops": 20.0 * 6.0 * per * n3}
    if case["op"] == "adjoint":
        return {"bytes": 4.0 * vec64 + 3.0 * nu_all, "flops": 2.0 * 15.0 * 6.0 * per * n3}
    if case["op"] == "stokes":
        return {"bytes": 2.0 * vec64 + 2.0 * _nodes(L - 1) * 8.0 + nu_all, "flops": case["restart"] * 7.0 * per * n3}
    return {"bytes": 2.0 * _nodes(L - 1) * 8.0 + nu_all + vec64, "flops": 2.0 * 4.0 * 7.0 * 130.0 * _nodes(L - 1)}


# ---------------------------------------------------------------------------------
# the same in plain torch, FP64
# ---------------------------------------------------------------------------------
def _corner(v, k, n):
    """Values at corner k = dx + 2 dy + 4 dz of every cell."""
    dx, dy, dz = k & 1, (k >> 1) & 1, k >> 2
    return v[..., dz:dz + n, dy:dy + n, dx:dx + n]


def _inner(v):
    """v with its boundary values replaced by 0."""
    o = torch.zeros_like(v)
    o[..., 1:-1, 1:-1, 1:-1] = v[..., 1:-1, 1:-1, 1:-1]
    return o


def _path(s):
    a1, a2, _ = AXES[s]
    return 0, 1 << a1, (1 << a1) | (1 << a2), 7


def _operator(nu, u):
    """A u on one level (homogeneous Dirichlet)."""
    n, nc = nu.shape[0], u.shape[0]
    u = _inner(u)
    out = torch.zeros_like(u)
    for s in range(6):
        k, w = _path(s), nu[..., s] / (6.0 * n)
        d = [[_corner(u[c], k[j + 1], n) - _corner(u[c], k[j], n) for c in range(nc)] for j in range(3)]
        for j in range(3):
            for i in range(3 if nc == 3 else 1):
                if nc == 3:  # flux of path step j in component a_i
                    c = AXES[s][i]
                    q = w * (d[j][c] + d[i][AXES[s][j]])
                else:
                    c, q = 0, w * d[j][0]
                _corner(out[c], k[j], n).sub_(q)
                _corner(out[c], k[j + 1], n).add_(q)
    return _inner(out)


def _diagonal(nu, nc):
    n = nu.shape[0]
    out = torch.zeros((nc, n + 1, n + 1, n + 1), dtype=torch.float64, device=nu.device)
    for s in range(6):
        k, w = _path(s), nu[..., s] / (6.0 * n)
        for a in range(4):
            for c in range(nc):
                lap = 1.0 if a in (0, 3) else 2.0
                g = (c == AXES[s][a - 1] if a > 0 else False) or (c == AXES[s][a] if a < 3 else False)
                _corner(out[c], k[a], n).add_(w, alpha=lap + (1.0 if g and nc == 3 else 0.0))
    return _inner(out)


def _odd(m):
    """Slices of the fine nodes of parity m and of their lower and upper coarse neighbours."""
    bits = [(m >> 2) & 1, (m >> 1) & 1, m & 1]
    fine = tuple(slice(b, None, 2) for b in bits)
    lo = tuple(slice(0, -1) if b else slice(None) for b in bits)
    hi = tuple(slice(1, None) if b else slice(None) for b in bits)
    return (Ellipsis,) + fine, (Ellipsis,) + lo, (Ellipsis,) + hi


def _prolong(e):
    n = e.shape[-1] - 1
    out = torch.zeros(e.shape[:-3] + (2 * n + 1,) * 3, dtype=torch.float64, device=e.device)
    for m in range(8):
        f, lo, hi = _odd(m)
        out[f] = 0.5 * (e[lo] + e[hi])
    return out


def _restrict(r):
    n = (r.shape[-1] - 1) // 2
    out = r[..., ::2, ::2, ::2].clone()
    for m in range(1, 8):
        f, lo, hi = _odd(m)
        out[lo] += 0.5 * r[f]
        out[hi] += 0.5 * r[f]
    return out


def _children(s):
    """(cell offset (x, y, z), axis order) of the 8 Bey children of simplex s."""
    a, b, c = AXES[s]
    one, two = [0, 0, 0], [0, 0, 0]
    one[a] = two[a] = two[b] = 1
    return [((0, 0, 0), (a, b, c)), (one, (a, b, c)), (two, (a, b, c)), ((1, 1, 1), (a, b, c)),
            (one, (b, c, a)), (one, (b, a, c)), (two, (c, a, b)), (two, (a, c, b))]


def _down(fine, how):
    """Coarse-element array from its children's: how reduces the 8 children."""
    n = fine.shape[0] // 2
    out = torch.empty((n, n, n, 6), dtype=torch.float64, device=fine.device)
    for s in range(6):
        t = [fine[o[2]::2, o[1]::2, o[0]::2, AXES.index(order)] for o, order in _children(s)]
        acc = t[0].clone()
        for x in t[1:]:
            acc = how(acc, x)
        out[..., s] = acc
    return out


class _Multigrid:
    """The hierarchy's operators and V(2,2)-cycle: per-element ratio flags with tau = 10,
    flagged elements with the mean finest coefficient (for P1 functions the Galerkin
    product of the element), damped Jacobi with 2/3 or the Chebyshev smoother."""

    def __init__(self, case, nu):
        self.nc, self.L, self.cheb = case["ncomp"], case["L"], case["smoother"] == "chebyshev"
        L = self.L
        self.nu = [t.view(2 << l, 2 << l, 2 << l, 6) for l, t in enumerate(nu)]
        mn = mx = mean = self.nu[L]
        for l in range(L - 1, -1, -1):
            mn, mx = _down(mn, torch.minimum), _down(mx, torch.maximum)
            mean = _down(mean, torch.add) / 8.0
            self.nu[l] = torch.where(mx > 10.0 * mn, mean, self.nu[l])
        self.low = list(self.nu)  # the coefficient that the V-cycle reads
        if case["dtype"] == "bf16":
            self.low[L] = self.nu[L].to(torch.bfloat16).to(torch.float64)
        self.diag = [_diagonal(t, self.nc) for t in self.nu]
        self.dinv = [torch.where(t > 0, 1.0 / t, 0.0) for t in self.diag]
        e = torch.zeros((self.nc, 3, 3, 3), dtype=torch.float64, device=DEVICE)
        a0 = []
        for c in range(self.nc):
            e.zero_()
            e[c, 1, 1, 1] = 1.0
            a0.append(_operator(self.nu[0], e)[:, 1, 1, 1])
        self.a0inv = torch.linalg.inv(torch.stack(a0, dim=1))
        self.lam = [0.0] + [self._lanczos(l) for l in range(1, L + 1)] if self.cheb else []

    def _lanczos(self, l):
        n, d = 2 << l, self.diag[l]
        i = torch.arange(n + 1, device=DEVICE)
        sign = 1.0 - 2.0 * ((i.view(1, 1, -1) + i.view(1, -1, 1) + i.view(-1, 1, 1)) % 2).to(torch.float64)
        v = _inner(sign.expand(self.nc, -1, -1, -1).contiguous())
        v = v / (v * d * v).sum().sqrt()
        old, beta, al, be = None, 0.0, [], []
        for _ in range(20):
            y = _operator(self.nu[l], v)
            a = float((v * y).sum())
            w = y * self.dinv[l] - a * v - (beta * old if old is not None else 0.0)
            al.append(a)
            beta = math.sqrt(max(0.0, float((w * d * w).sum())))
            if not beta > 1e-12 * abs(a):
                break
            be.append(beta)
            old, v = v, w / beta
        be = be[:len(al) - 1]
        t = torch.diag(torch.tensor(al, dtype=torch.float64))
        if be:
            o = torch.diag(torch.tensor(be, dtype=torch.float64), 1)
            t = t + o + o.T
        return float(torch.linalg.eigvalsh(t)[-1])

    def _smooth(self, l, b, x, sweeps, zero):
        om, old = 2.0 / 3.0, torch.zeros_like(b)
        if self.cheb:
            top = 1.1 * self.lam[l]
            theta, delta = 0.55 * top, 0.45 * top
            rho = delta / theta
        for k in range(sweeps):
            r = b if zero and k == 0 else b - _operator(self.low[l], x)
            if not self.cheb:
                x, old = x + om * self.dinv[l] * r, x
            elif k == 0:
                x, old = x + self.dinv[l] * r / theta, x
            else:
                new = 1.0 / (2.0 * theta / delta - rho)
                x, old = x + new * rho * (x - old) + (2.0 * new / delta) * self.dinv[l] * r, x
                rho = new
        return x

    def cycle(self, b, l=None):
        l = self.L if l is None else l
        b = _inner(b)
        if l == 0:
            x = torch.zeros_like(b)
            x[:, 1, 1, 1] = self.a0inv @ b[:, 1, 1, 1]
            return x
        x = self._smooth(l, b, torch.zeros_like(b), 2, True)
        r = b - _operator(self.low[l], x)
        x = x + _prolong(self.cycle(_inner(_restrict(r)), l - 1))
        return self._smooth(l, b, x, 2, False)

    def solve(self, b):
        """A^-1 b by conjugate gradients, as far as FP64 goes."""
        b = _inner(b)
        x, r, p, rz = torch.zeros_like(b), b.clone(), None, 1.0
        best, since, keep = math.inf, 0, x
        for k in range(80):
            z = self.cycle(r)
            new = float((r * z).sum())
            p = z if p is None else z + (new / rz) * p
            rz = new
            q = _operator(self.nu[self.L], p)
            x = x + (rz / float((p * q).sum())) * p
            r = b - _operator(self.nu[self.L], x)
            res = float(r.norm() / b.norm())
            if res < 0.5 * best:
                best, since, keep = res, 0, x
            else:
                since += 1
            if since >= 6 or res < 1e-15:
                break
        return keep


def _gradient_shape(s, a, c):
    """Component c of the gradient of the barycentric function of path vertex a, times h."""
    return (1 if a > 0 and AXES[s][a - 1] == c else 0) - (1 if a < 3 and AXES[s][a] == c else 0)


def _divergence(u):
    """B u: minus the integral of each pressure hat against div u."""
    n = u.shape[-1] - 1
    u, q = _inner(u), torch.zeros(u.shape[1:], dtype=torch.float64, device=u.device)
    for s in range(6):
        k = _path(s)
        div = sum(_gradient_shape(s, a, c) * _corner(u[c], k[a], n) for a in range(4) for c in range(3)
                  if _gradient_shape(s, a, c))
        for a in range(4):
            _corner(q, k[a], n).sub_(div, alpha=1.0 / (24.0 * n * n))
    return _restrict(q)


def _divergence_t(p):
    """B^T p."""
    f = _prolong(p)
    n = f.shape[-1] - 1
    out = torch.zeros((3,) + f.shape, dtype=torch.float64, device=p.device)
    for s in range(6):
        k = _path(s)
        mean = sum(_corner(f, k[a], n) for a in range(4))
        for a in range(4):
            for c in range(3):
                g = _gradient_shape(s, a, c)
                if g:
                    _corner(out[c], k[a], n).sub_(mean, alpha=g / (24.0 * n * n))
    return _inner(out)


def _exact_stokes(M, b, m):
    """One cycle of m steps of right-preconditioned GMRES, modified Gram-Schmidt."""
    n, L = 2 << M.L, M.L
    mass = torch.zeros((n + 1,) * 3, dtype=torch.float64, device=DEVICE)
    for s in range(6):
        for a in range(4):
            _corner(mass, _path(s)[a], n).add_(1.0 / M.nu[L][..., s], alpha=1.0 / (24.0 * n ** 3))
    mass = _restrict(mass)

    def precond(v):
        q = v[1] / mass
        return M.cycle(v[0] + _divergence_t(q)), -q

    def dot(v, w):
        return float((v[0] * w[0]).sum() + (v[1] * w[1]).sum())

    r = (_inner(b), torch.zeros_like(mass))
    beta = math.sqrt(dot(r, r))
    V, Z, H = [(r[0] / beta, r[1] / beta)], [], np.zeros((m + 1, m))
    for k in range(m):
        z = precond(V[k])
        Z.append(z)
        w = (_operator(M.nu[L], z[0]) + _divergence_t(z[1]), _divergence(z[0]))
        for _ in range(2):
            for i in range(k + 1):
                h = dot(w, V[i])
                H[i, k] += h
                w = (w[0] - h * V[i][0], w[1] - h * V[i][1])
        H[k + 1, k] = math.sqrt(dot(w, w))
        V.append((w[0] / H[k + 1, k], w[1] / H[k + 1, k]))
    g = np.zeros(m + 1)
    g[0] = beta
    y = np.linalg.lstsq(H, g, rcond=None)[0]
    u = sum(float(t) * z[0] for t, z in zip(y, Z))
    p = sum(float(t) * z[1] for t, z in zip(y, Z))
    return u, p - p.mean()


def _exact_schur(M, r, iters):
    """Z^-1 (B W^-1 A W^-1 B^T) Z^-1 r with W = diag(A), Z = B W^-1 B^T and each Z^-1 `iters`
    steps of CG preconditioned by one V(2,2)-cycle (damped Jacobi, 2/3) of Galerkin levels."""
    top, winv, A = M.L - 1, M.dinv[M.L], M.nu[M.L]

    def Z(l, y):
        for _ in range(l, top):
            y = _prolong(y)
        y = _divergence(winv * _divergence_t(y))
        for _ in range(l, top):
            y = _restrict(y)
        return y

    diag = []
    for l in range(top + 1):
        i = torch.arange((2 << l) + 1, device=DEVICE)
        colour = (i.view(1, 1, -1) + 34 * i.view(1, -1, 1) + 44 * i.view(-1, 1, 1)) % 65
        d = torch.zeros(colour.shape, dtype=torch.float64, device=DEVICE)
        for c in range(65):
            on = colour == c
            if bool(on.any()):
                d = torch.where(on, Z(l, on.to(torch.float64)), d)
        diag.append(d)
    e = torch.eye(27, dtype=torch.float64, device=DEVICE).view(27, 3, 3, 3)
    z0inv = torch.linalg.pinv(torch.stack([Z(0, v).reshape(-1) for v in e], dim=1), rtol=1e-10)

    def cycle(l, f):
        if l == 0:
            return (z0inv @ f.reshape(-1)).view(3, 3, 3)
        y = (2.0 / 3.0) * f / diag[l]
        y = y + (2.0 / 3.0) * (f - Z(l, y)) / diag[l]
        y = y + _prolong(cycle(l - 1, _restrict(f - Z(l, y))))
        for _ in range(2):
            y = y + (2.0 / 3.0) * (f - Z(l, y)) / diag[l]
        return y

    def solve(f):
        y, p, rz = torch.zeros_like(f), None, 1.0
        for _ in range(iters):
            z = cycle(top, f)
            new = (f * z).sum()
            p = z if p is None else z + (new / rz) * p
            rz = new
            q = Z(top, p)
            a = rz / (p * q).sum()
            y, f = y + a * p, f - a * q
        return y

    y = solve(r)
    return solve(_divergence(winv * _operator(A, winv * _divergence_t(y))))


def exact(case, seed):
    if case["op"] in ("stokes", "schur") and case["L"] > (5 if case["op"] == "stokes" else 6):
        return None  # over 20 seconds
    nu, v = _inputs(case, seed)
    L, nc = case["L"], case["ncomp"]

    def box(t, l, c=nc):
        return t.to(torch.float64).view((c,) + ((2 << l) + 1,) * 3)

    if case["op"] == "apply":
        l = case["level"]
        coef = nu[L].view((2 << L,) * 3 + (6,))
        if l < L:
            fine, coef = coef, nu[l].view((2 << l,) * 3 + (6,))
            flagged = _down(fine, torch.maximum) > 10.0 * _down(fine, torch.minimum)
            coef = torch.where(flagged, _down(fine, torch.add) / 8.0, coef)
        elif case["dtype"] == "bf16":
            coef = coef.to(torch.bfloat16).to(torch.float64)
        return _operator(coef, box(v["u"], l)).reshape(-1)
    M = _Multigrid(case, nu)
    if case["op"] == "vcycle":
        return M.cycle(box(v["b"], L)).reshape(-1)
    if case["op"] == "solve":
        return M.solve(box(v["b"], L)).reshape(-1)
    if case["op"] == "adjoint":
        u, w = M.solve(box(v["b"], L)), M.solve(box(v["y"], L))
        n = 2 << L
        g = torch.empty((n, n, n, 6), dtype=torch.float64, device=DEVICE)
        for s in range(6):  # minus w_e . A_e u_e
            k = _path(s)
            d, t = ([[_corner(f[c], k[j + 1], n) - _corner(f[c], k[j], n) for c in range(nc)] for j in range(3)]
                    for f in (u, w))
            if nc == 3:
                e = sum((d[j][AXES[s][i]] + d[i][AXES[s][j]]) * t[j][AXES[s][i]] for i in range(3) for j in range(3))
            else:
                e = sum(d[j][0] * t[j][0] for j in range(3))
            g[..., s] = -M.nu[L][..., s] / (6.0 * n) * e
        return u.reshape(-1), g.reshape(-1), w.reshape(-1)
    if case["op"] == "stokes":
        u, p = _exact_stokes(M, box(v["b"], L), case["restart"])
        return u.reshape(-1), p.reshape(-1)
    return _exact_schur(M, v["r"].view(((2 << (L - 1)) + 1,) * 3), 4).reshape(-1)
