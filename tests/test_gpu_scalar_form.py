"""The scalar levels' seven-point form (csrc/k_scalar.hip) and the one-workgroup cycle of the small
levels (csrc/k_coarse_cycle.hip) against the element loop, which the same hierarchy runs when
a memory limit leaves no room for the edge weights.  Sizes: the one-workgroup cycle alone
(5^3, 9^3, 17^3), under one and two more levels, and the marching kernels from 65^3 on.

Tolerances: both sides evaluate the same operator in the same precision with sums in another
order.  FP64 1e-12, FP32 2e-5 (300 roundings), of the largest entry."""

import pytest
import torch

from workloads import Sinkers

pytestmark = pytest.mark.gpu


def _make(L, dtype, smoother, limit=0):
    from paper_2511_13109_amd import Hierarchy, coefficients_from_field
    nu = coefficients_from_field(Sinkers(4, 2, radius=0.15, width=2.0 / 2 ** (L + 1), contrast=1e6), L)
    return Hierarchy(L, 1, nu[L], nu[:L], mg_dtype="f64" if dtype == "f64" else "f32", mg_nu_dtype=dtype,
                     smoother=smoother, mem_limit_bytes=limit)


def _weight_bytes(L, dtype):
    return sum(3 * (2 ** (l + 1) + 1) ** 3 * (8 if dtype == "f64" else 12) for l in range(L + 1))


@pytest.mark.parametrize("L", [1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
@pytest.mark.parametrize("smoother", ["chebyshev", "jacobi"])
def test_forms_agree(L, dtype, smoother):
    print(f"\n[scalar form L={L} {dtype} {smoother}]", flush=True)
    A = _make(L, dtype, smoother)
    B = _make(L, dtype, smoother, A.device_bytes() - 1)
    try:
        assert A.device_bytes() - B.device_bytes() == _weight_bytes(L, dtype)
        tol = 1e-12 if dtype == "f64" else 2e-5
        t = torch.float64 if dtype == "f64" else torch.float32
        n1 = A.n(L) + 1
        g = torch.Generator(device="cuda")
        g.manual_seed(7)

        def vec(dt, edge=0.0):
            v = torch.full((n1, n1, n1), edge, dtype=dt, device="cuda")
            v[1:-1, 1:-1, 1:-1] = torch.randn(n1 - 2, n1 - 2, n1 - 2, generator=g, dtype=dt, device="cuda")
            return v.reshape(-1)

        b, u = vec(t), vec(t)
        # boundary slots of the input are not part of it
        uj = u.clone().view(n1, n1, n1)
        for face in (uj[0], uj[-1], uj[:, 0], uj[:, -1], uj[..., 0], uj[..., -1]):
            face.fill_(float("nan"))
        uj = uj.reshape(-1)
        results = []
        for H in (A, B):
            r = {"apply": H.apply(L, uj), "residual": H.residual(L, b, uj), "cycle": H.vcycle(b),
                 "smooth 1": H.smooth(L, b, u.clone(), 1), "smooth 3": H.smooth(L, b, u.clone(), 3)}
            r["apply f64"] = H.apply(L, uj.double())
            results.append(r)
        for k, x in results[0].items():
            y = results[1][k].double()
            err = float((x.double() - y).abs().max() / y.abs().max())
            print(f"{k}: {err:.2e}", flush=True)
            assert err <= (1e-12 if k == "apply f64" else tol), k
            v = x.view(n1, n1, n1)
            for face in (v[0], v[-1], v[:, 0], v[:, -1], v[..., 0], v[..., -1]):
                assert not face.any(), k
    finally:
        A.close()
        B.close()


@pytest.mark.parametrize("edge", ["least", "most"])
def test_solve_gives_up_weights_for_its_vectors(edge):
    """A limit that holds the weights or the solver's four vectors, but not both: the solve
    runs, without the weights."""
    L = 4
    vectors = 4 * 8 * (2 ** (L + 1) + 1) ** 3
    room = vectors - _weight_bytes(L, "f64") if edge == "least" else vectors - 1
    assert room >= 0
    A = _make(L, "f64", "jacobi")
    full = A.device_bytes()
    B = _make(L, "f64", "jacobi", full + room)
    try:
        assert B.device_bytes() == full
        n1 = A.n(L) + 1
        b = torch.zeros(n1, n1, n1, dtype=torch.float64, device="cuda")
        b[1:-1, 1:-1, 1:-1] = 1.0
        b = b.reshape(-1)
        sa, sb = A.solve(b, tol=1e-10)[1], B.solve(b, tol=1e-10)[1]
        assert A.device_bytes() == full + vectors
        assert B.device_bytes() == full + vectors - _weight_bytes(L, "f64")
        assert sa["converged"] and sb["converged"] and abs(sa["iterations"] - sb["iterations"]) <= 1
    finally:
        A.close()
        B.close()
