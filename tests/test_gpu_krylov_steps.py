"""The Krylov loop against the same steps composed in Python from the library's single operations
(apply, residual, V-cycle) and torch vector updates.  Its scalars never leave the device: the kernels
that use them sum the partial sums themselves, or read a sum formed before where the product
has more than 2048 workgroups (257^3 scalar: 2340).  FP64 V-cycles only: a mixed solve rounds r to
FP32 before the V-cycle, which turns one FP64 rounding of difference into 6e-8 of an entry.  Sizes: one workgroup of partial sums
(3^3 scalar) up to that.  Steps with and without a residual replacement (r.r halved since the last
one) are among them.

Tolerance: k steps of the same recurrence with sums in another order, FP64.  A relative
perturbation of a few 1e-16 per step grows by at most the ratio of consecutive residuals, which
here is below 10 per step: 1e-16 * 10^4 after four steps, 1e-10 asked."""

import pytest
import torch

from workloads import Sinkers

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,ncomp", [(1, 1), (2, 3), (4, 1), (5, 3), (7, 1)])
def test_steps(L, ncomp):
    from paper_2511_13109_amd import Hierarchy, coefficients_from_field
    print(f"\n[krylov steps L={L} ncomp={ncomp}]", flush=True)
    nu = coefficients_from_field(Sinkers(4, 2, radius=0.15, width=2.0 / 2 ** (L + 1), contrast=1e2), L)
    H = Hierarchy(L, ncomp, nu[L], nu[:L], smoother="chebyshev")
    try:
        n1 = H.n(L) + 1
        g = torch.Generator(device="cuda")
        g.manual_seed(3)
        b = torch.zeros(ncomp, n1, n1, n1, dtype=torch.float64, device="cuda")
        b[:, 1:-1, 1:-1, 1:-1] = torch.randn(ncomp, n1 - 2, n1 - 2, n1 - 2, generator=g, dtype=torch.float64, device="cuda")
        b = b.reshape(-1)

        steps = 1 if L == 1 else 4  # 3^3 scalar: one unknown, solved by the first step
        x = torch.zeros_like(b)
        r = b.clone()
        bn = float(torch.linalg.vector_norm(b))
        anchor = float(torch.linalg.vector_norm(r))
        z = H.vcycle(r)
        p = z.clone()
        rz = torch.dot(z, r)
        replaced = 0
        for k in range(steps):
            q = H.apply(L, p)
            pq = torch.dot(p, q)
            alpha = rz / pq
            x = x + alpha * p
            r = r - alpha * q
            if k + 1 == steps:
                break
            if float(torch.linalg.vector_norm(r)) <= 0.5 * anchor:
                r = H.residual(L, b, x)
                anchor = float(torch.linalg.vector_norm(r))
                replaced += 1
            z = H.vcycle(r)
            rz = torch.dot(z, r)
            p = z - (torch.dot(z, q) / pq) * p
        y, stats = H.solve(b, solver="pcg", tol=1e-14, max_iter=steps, raise_on_noconv=False)
        err = float((y - x).abs().max() / x.abs().max())
        true = float(torch.linalg.vector_norm(H.residual(L, b, y))) / bn
        print(f"error {err:.2e}, {replaced} replacements, residual {true:.3e}", flush=True)
        assert stats["iterations"] == steps
        assert err <= 1e-10
        assert abs(true - stats["rel_residual"]) <= 1e-9 * max(true, 1e-6)
    finally:
        H.close()
