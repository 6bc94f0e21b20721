"""The Krylov loop with an FP32 V-cycle (FP64 recurrences, r rounded to FP32 before the cycle, z widened
in the dot products and the direction update), step by step against the same steps composed in Python from the
library's single operations and torch vector updates; and the residual replacements of both
kinds of solve.

Tolerance.  The two sides differ by FP64 roundings, which now and then round an entry of r to the
other FP32 neighbour.  Cycles of inputs that differ in the last FP32 bit differ by at most the
cycle's own rounding, 2e-5 of the largest entry (the bound of the composed FP32 cycles), in
each of at most four steps: 1e-4 of the largest entry of x.  A cycle on the r (or with the z) of
the step before misses it: composed with that mistake from the second step on, x is off by more than 1e-3."""

import pytest
import torch

from workloads import Sinkers

pytestmark = pytest.mark.gpu


def _steps(H, L, b, steps, mixed, stale=False):
    """x after `steps` iterations of flexible CG from zero, and the replacements taken."""
    def cycle(r):
        return H.vcycle(r.float()).double() if mixed else H.vcycle(r)
    x = torch.zeros_like(b)
    r = b.clone()
    anchor = float(torch.linalg.vector_norm(r))
    z = cycle(r)
    p = z.clone()
    rz = torch.dot(z, r)
    replaced = 0
    for k in range(steps):
        q = H.apply(L, p)
        pq = torch.dot(p, q)
        alpha = rz / pq
        x = x + alpha * p
        r_old, r = r, r - alpha * q
        if k + 1 == steps:
            break
        if float(torch.linalg.vector_norm(r)) <= 0.5 * anchor:
            r = H.residual(L, b, x)
            anchor = float(torch.linalg.vector_norm(r))
            replaced += 1
        z = cycle(r_old if stale and k > 0 else r)
        rz = torch.dot(z, r)
        p = z - (torch.dot(z, q) / pq) * p
    return x, replaced


# size, precision, steps, replacements before the last one: every case has steps with a
# replacement, all but the first also one without
CASES = [(2, 1, "bf16", 3, 2), (4, 3, "f32", 4, 2), (5, 3, "bf16", 4, 2), (6, 1, "f32", 4, 2), (5, 3, "f64", 4, 2), (4, 1, "f64", 4, 2)]


@pytest.mark.parametrize("L,ncomp,dtype,steps,replacements", CASES)
def test_steps(L, ncomp, dtype, steps, replacements):
    from paper_2511_13109_amd import Hierarchy, coefficients_from_field
    mixed = dtype != "f64"
    print(f"\n[krylov steps L={L} ncomp={ncomp} {dtype}]", flush=True)
    nu = coefficients_from_field(Sinkers(4, 2, radius=0.15, width=2.0 / 2 ** (L + 1), contrast=1e2), L)
    H = Hierarchy(L, ncomp, nu[L], nu[:L], mg_dtype="f32" if mixed else "f64", mg_nu_dtype=dtype, smoother="chebyshev")
    try:
        n1 = H.n(L) + 1
        g = torch.Generator(device="cuda")
        g.manual_seed(3)
        b = torch.zeros(ncomp, n1, n1, n1, dtype=torch.float64, device="cuda")
        b[:, 1:-1, 1:-1, 1:-1] = torch.randn(ncomp, n1 - 2, n1 - 2, n1 - 2, generator=g, dtype=torch.float64, device="cuda")
        b = b.reshape(-1)
        x, replaced = _steps(H, L, b, steps, mixed)
        y, stats = H.solve(b, solver="fcg" if mixed else "pcg", tol=1e-14, max_iter=steps, raise_on_noconv=False)
        top = float(x.abs().max())
        err = float((y - x).abs().max()) / top
        wrong, _ = _steps(H, L, b, steps, mixed, stale=True)
        off = float((wrong - x).abs().max()) / top
        print(f"error {err:.2e}, {replaced} replacements (library {stats['replacements']}), a stale residual {off:.2e}", flush=True)
        assert stats["iterations"] == steps
        assert replaced == replacements
        assert stats["replacements"] - replaced in (0, 1)  # the last step may take one
        assert err <= (1e-4 if mixed else 1e-10)
        assert off > 1e-3
    finally:
        H.close()
