"""V-cycles whose smoothing passes run two operator products per launch (csrc/k_smooth2.hip)
against the same cycle composed in Python from the library's single operations (residual,
restriction, prolongation, each its own kernel and checked against the oracle elsewhere) and
torch vector updates.  Sizes cover one partial tile (17^3), full tiles with remainders in x
and y and several z chunks (65^3, 129^3).  Boundary slots of b hold NaN: they are not part of
the input.

Tolerances: both sides evaluate the same formula in the same precision with sums in another
order.  FP64 as for the other V-cycle tests (1e-12); FP32 the same multiple of the unit
roundoff would be 5e-4, 2e-5 is used (300 roundings)."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _hierarchy(L, ncomp, dtype, smoother, pre, post, storage):
    from paper_2511_13109_amd import Hierarchy, coefficients_from_field
    from workloads import Sinkers
    field = Sinkers(4, 2, radius=0.15, width=2.0 / 2 ** (L + 1), contrast=1e6)
    nu = coefficients_from_field(field, L)
    return Hierarchy(L, ncomp, nu[L], nu[:L], mg_dtype="f64" if dtype == "f64" else "f32", mg_nu_dtype=dtype,
                     smoother=smoother, pre=pre, post=post, coarse_storage=storage)


def _passes(H, l, b, x, count, dinv, zero):
    """count smoothing passes on level l (Section 4's Chebyshev iteration or damped Jacobi)."""
    om = 2.0 / 3.0
    if H.cfg.smoother == 1:
        top = 1.1 * H.query(l)["lambda_max"]
        theta, delta = 0.55 * top, 0.45 * top
        rho = delta / theta
    old = torch.zeros_like(b)
    for k in range(count):
        r = b if zero and k == 0 else H.residual(l, b, x)
        if H.cfg.smoother != 1:
            x, old = x + om * dinv * r, x
        elif k == 0:
            x, old = x + dinv * r / theta, x
        else:
            new = 1.0 / (2.0 * theta / delta - rho)
            x, old = x + new * rho * (x - old) + (2.0 * new / delta) * dinv * r, x
            rho = new
    return x


def _cycle(H, l, b, pre, post):
    if l == 0:
        cols = []
        for c in range(H.ncomp):
            e = H.vec(0)
            e[27 * c + 13] = 1.0
            cols.append(H.apply(0, e).view(H.ncomp, 27)[:, 13])
        x = torch.zeros(H.ncomp, 27, dtype=torch.float64, device=b.device)
        x[:, 13] = torch.linalg.solve(torch.stack(cols, dim=1), b.double().view(H.ncomp, 27)[:, 13])
        return x.reshape(-1).to(b.dtype)
    d = torch.from_numpy(H.diagonal(l)).to(b.device)
    dinv = torch.where(d > 0, 1.0 / d, torch.zeros_like(d)).to(b.dtype)
    x = _passes(H, l, b, torch.zeros_like(b), pre, dinv, True)
    rc = H.restrict(l, H.residual(l, b, x))
    x = H.prolong_add(l - 1, _cycle(H, l - 1, rc, pre, post), x)
    return _passes(H, l, b, x, post, dinv, False)


CASES = [(3, 1, "f64"), (3, 3, "bf16"), (4, 1, "f32"), (4, 3, "f32"), (5, 3, "f64"), (5, 1, "bf16"), (6, 3, "f64"),
         (6, 3, "bf16")]


@pytest.mark.parametrize("L,ncomp,dtype", CASES)
@pytest.mark.parametrize("smoother,pre,post", [("chebyshev", 2, 2), ("jacobi", 2, 2), ("chebyshev", 2, 3),
                                               ("jacobi", 1, 2), ("jacobi", 3, 2)])
def test_vcycle_composed(L, ncomp, dtype, smoother, pre, post):
    print(f"\n[two products L={L} ncomp={ncomp} {dtype} {smoother} V({pre},{post})]", flush=True)
    H = _hierarchy(L, ncomp, dtype, smoother, pre, post, "mean" if pre == 1 else "blocks")
    try:
        n1 = H.n(L) + 1
        g = torch.Generator(device="cuda")
        g.manual_seed(5)
        t = torch.float64 if dtype == "f64" else torch.float32
        b = torch.zeros(ncomp, n1, n1, n1, dtype=t, device="cuda")
        b[:, 1:-1, 1:-1, 1:-1] = torch.randn(ncomp, n1 - 2, n1 - 2, n1 - 2, generator=g, dtype=t, device="cuda")
        ref = _cycle(H, L, b.reshape(-1), pre, post)
        if pre == 2:  # one pass from zero alone multiplies the boundary slots by D^-1 = 0
            junk = torch.full_like(b, float("nan"))
            junk[:, 1:-1, 1:-1, 1:-1] = b[:, 1:-1, 1:-1, 1:-1]
            b = junk
        x = H.vcycle(b.reshape(-1).contiguous())
        x2 = H.vcycle(b.reshape(-1).contiguous())
        assert torch.equal(x, x2)
        v = x.view(ncomp, n1, n1, n1)
        for face in (v[:, 0], v[:, -1], v[:, :, 0], v[:, :, -1], v[..., 0], v[..., -1]):
            assert not face.any()
        err = float((x.double() - ref.double()).abs().max() / ref.double().abs().max())
        print(f"error {err:.2e}", flush=True)
        assert err <= (1e-12 if dtype == "f64" else 2e-5)
    finally:
        H.close()
