"""FP32 V-cycles at the ends of the type's range, with the element loop, its two-product passes
(csrc/k_smooth2.hip) and the scalar seven-point form (csrc/k_scalar.hip) on the fine levels."""

import pytest
import torch

from workloads import Sinkers

pytestmark = pytest.mark.gpu


def _make(L, ncomp, nud, factor=1.0, **kw):
    from paper_2511_13109_amd import Hierarchy, coefficients_from_field
    nu = coefficients_from_field(Sinkers(4, 2, radius=0.15, width=2.0 / 2 ** (L + 1), contrast=1e4), L)
    nu = [v * factor for v in nu]
    H = Hierarchy(L, ncomp, nu[L], nu[:L], mg_dtype="f32", mg_nu_dtype=nud, **kw)
    n1 = H.n(L) + 1
    g = torch.Generator(device="cuda")
    g.manual_seed(8)
    b = torch.zeros(ncomp, n1, n1, n1, dtype=torch.float32, device="cuda")
    b[:, 1:-1, 1:-1, 1:-1] = torch.randn(ncomp, n1 - 2, n1 - 2, n1 - 2, generator=g, dtype=torch.float32, device="cuda")
    return H, b.reshape(-1)


@pytest.mark.parametrize("ncomp,nud", [(1, "f32"), (3, "f32"), (3, "bf16")])
def test_damping_below_fp32(ncomp, nud):
    """A damping factor that is 0 in FP32: every pass is without effect and the cycle is the
    interpolated level-0 solution.  Tolerance: FP32 sums of at most 15 terms on five levels."""
    L = 4
    print(f"\n[damping below FP32 ncomp={ncomp} {nud}]", flush=True)
    H, b = _make(L, ncomp, nud, smoother="jacobi", omega=1e-60)
    try:
        r = b
        for l in range(L, 0, -1):
            r = H.restrict(l, r)
        cols = []
        for c in range(ncomp):
            e = H.vec(0)
            e[27 * c + 13] = 1.0
            cols.append(H.apply(0, e).view(ncomp, 27)[:, 13])
        x = torch.zeros(ncomp, 27, dtype=torch.float64, device="cuda")
        x[:, 13] = torch.linalg.solve(torch.stack(cols, dim=1), r.double().view(ncomp, 27)[:, 13])
        x = x.reshape(-1).float()
        for l in range(L):
            x = H.prolong_add(l, x, torch.zeros(ncomp * H.nodes(l + 1), dtype=torch.float32, device="cuda"))
        z = H.vcycle(b)
        err = float((z.double() - x.double()).abs().max() / x.double().abs().max())
        print(f"error {err:.2e}", flush=True)
        assert err <= 2e-5
    finally:
        H.close()


@pytest.mark.parametrize("L,ncomp,nud", [(4, 1, "f32"), (4, 3, "f32"), (6, 1, "bf16"), (6, 3, "f32"), (6, 3, "bf16")])
def test_large_right_hand_side(L, ncomp, nud):
    """One entry of 2^124: the sums of A x are of that size, but 6 n times larger without the factor h/6
    of the element matrices, beyond the largest FP32 number 2^128.  Powers of two are exact: the cycle of
    2^k b is 2^k times that of b, bit for bit."""
    print(f"\n[large right-hand side L={L} ncomp={ncomp} {nud}]", flush=True)
    # the coefficient at least 2^9: no iterate is larger than b
    H, b = _make(L, ncomp, nud, factor=2.0 ** 16, smoother="chebyshev")
    try:
        n1 = H.n(L) + 1
        b.zero_()
        m = n1 // 2 - 3
        b.view(ncomp, n1, n1, n1)[-1, m, m, m] = 1.0
        z = H.vcycle(b)
        big = H.vcycle(b * 2.0 ** 124)
        print(f"max {float(big.abs().max()):.3e}", flush=True)
        assert torch.isfinite(big).all()
        # entries below the normal range of the small cycle aside
        normal = z.abs() >= 2.0 ** -126
        assert torch.equal(big[normal], z[normal] * 2.0 ** 124)
    finally:
        H.close()
