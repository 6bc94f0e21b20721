"""Divergence and gradient of the Stokes system (csrc/k_stokes.hip, rows of 62 nodes per wavefront)
against the sums over the simplices they stand for, in torch.  Sizes: one partial row segment
(9, 33 nodes per row), one and a remainder of 3 (65), two and a remainder of 5 (129).

Tolerance: at most 45 products per value with coefficients up to 6, FP64, sums in another
order: 1e-13 of the largest entry."""

import pytest
import torch

from workloads import AlignedCube

pytestmark = pytest.mark.gpu

ORDERS = [(0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)]


def _corners(s):
    k, out = 0, [0]
    for a in ORDERS[s]:
        k |= 1 << a
        out.append(k)
    return out


def _grad(s, a, c):
    o = ORDERS[s]
    return (1 if a > 0 and c == o[a - 1] else 0) - (1 if a < 3 and c == o[a] else 0)


def _at(f, k, n):  # values at cell corner k of a field [z, y, x]
    x, y, z = k & 1, (k >> 1) & 1, k >> 2
    return f[z:z + n, y:y + n, x:x + n]


def _interpolate(pc):
    n = 2 * (pc.shape[0] - 1)
    i = torch.arange(n + 1, device=pc.device)
    lo, hi = i // 2, (i + 1) // 2
    return 0.5 * (pc[lo][:, lo][:, :, lo] + pc[hi][:, hi][:, :, hi])


def _restrict(qf):
    """P^T: the transpose of _interpolate."""
    n = qf.shape[0] - 1
    i = torch.arange(n + 1, device=qf.device)
    out = torch.zeros((n // 2 + 1,) * 3, dtype=qf.dtype, device=qf.device)
    for j in (i // 2, (i + 1) // 2):
        idx = (j[:, None, None] * (n // 2 + 1) + j[None, :, None]) * (n // 2 + 1) + j[None, None, :]
        out.view(-1).index_add_(0, idx.reshape(-1), 0.5 * qf.reshape(-1))
    return out


@pytest.mark.parametrize("L", [2, 4, 5, 6])
def test_div_and_grad(L):
    from paper_2511_13109_amd import Hierarchy, Stokes, coefficients_from_field
    print(f"\n[stokes rows L={L}]", flush=True)
    nu = coefficients_from_field(AlignedCube(), L)
    H = Hierarchy(L, 3, nu[L], nu[:L])
    try:
        S = Stokes(H)
        n = H.n(L)
        g = torch.Generator(device="cuda")
        g.manual_seed(9)
        u = torch.randn(3, n + 1, n + 1, n + 1, generator=g, dtype=torch.float64, device="cuda")
        pc = torch.randn(n // 2 + 1, n // 2 + 1, n // 2 + 1, generator=g, dtype=torch.float64, device="cuda")
        inside = torch.zeros(n + 1, n + 1, n + 1, dtype=torch.float64, device="cuda")
        inside[1:-1, 1:-1, 1:-1] = 1.0
        ui = u * inside  # boundary values of the velocity are not part of the input
        w = (1.0 / n) ** 2 / 24.0
        qf = torch.zeros(n + 1, n + 1, n + 1, dtype=torch.float64, device="cuda")
        v = torch.zeros_like(u)
        pf = _interpolate(pc)
        for s in range(6):
            ks = _corners(s)
            d = sum(_grad(s, b, c) * _at(ui[c], ks[b], n) for b in range(4) for c in range(3) if _grad(s, b, c))
            m = sum(_at(pf, ks[b], n) for b in range(4))
            for a in range(4):
                _at(qf, ks[a], n).sub_(w * d)
                for c in range(3):
                    if _grad(s, a, c):
                        _at(v[c], ks[a], n).sub_(w * _grad(s, a, c) * m)
        v *= inside
        q = _restrict(qf)
        got_q, got_v = S.div(u.reshape(-1).contiguous()).view_as(q), S.grad(pc.reshape(-1).contiguous()).view_as(v)
        for name, a, b in (("div", got_q, q), ("grad", got_v, v)):
            err = float((a - b).abs().max() / b.abs().max())
            print(f"{name} {err:.2e}", flush=True)
            assert err <= 1e-13, name
    finally:
        H.close()
