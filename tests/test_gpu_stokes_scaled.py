"""The scaled forms of the Stokes divergence and gradient (csrc/k_stokes.hip: B (s u) and s (in - B^T p),
which only the BFBT Schur approximation calls) against the unscaled ones, which have tests of their own.
Boundary entries of u and s are not part of the input of the divergence; on the boundary the gradient
returns its input.  Called below the C ABI.

Tolerance: the divergence forms the same products of s u (the same bits); the gradient's sum may round
once more, 4 roundings of the largest entry."""

import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4, 32, 64, 128])
@pytest.mark.parametrize("in_place", [False, True])
def test_scaled_forms(n, in_place):
    from paper_2511_13109_amd import _lib
    print(f"\n[stokes scaled n={n}]", flush=True)
    lib = _lib.load()
    div = getattr(lib, "_ZN4agca22launch_stokes_div_fineEiPKdS1_PdP12ihipStream_t")
    div.restype, div.argtypes = C.c_int, [C.c_int] + 4 * [C.c_void_p]
    grad = getattr(lib, "_ZN4agca18launch_stokes_gradEiPKdS1_S1_PdP12ihipStream_t")
    grad.restype, grad.argtypes = C.c_int, [C.c_int] + 5 * [C.c_void_p]
    st = torch.cuda.current_stream().cuda_stream
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    opts = dict(generator=g, dtype=torch.float64, device="cuda")
    u, b = torch.randn(3, n + 1, n + 1, n + 1, **opts), torch.randn(3, n + 1, n + 1, n + 1, **opts)
    s = 0.5 + torch.rand(3, n + 1, n + 1, n + 1, **opts)
    p = torch.randn(n // 2 + 1, n // 2 + 1, n // 2 + 1, **opts)
    edge = torch.ones(n + 1, n + 1, n + 1, dtype=torch.bool, device="cuda")
    edge[1:-1, 1:-1, 1:-1] = False

    su, sn, un = s * u, s.clone(), u.clone()
    sn[:, edge] = float("nan")
    un[:, edge] = float("nan")
    q, q1 = (torch.empty(n + 1, n + 1, n + 1, dtype=torch.float64, device="cuda") for _ in range(2))
    assert div(n, su.data_ptr(), None, q.data_ptr(), st) == 0
    assert div(n, un.data_ptr(), sn.data_ptr(), q1.data_ptr(), st) == 0
    assert torch.equal(q, q1)

    v = torch.empty_like(u)
    assert grad(n, p.data_ptr(), b.data_ptr(), None, v.data_ptr(), st) == 0
    want = torch.where(edge, b, s * v)
    out = b.clone() if in_place else torch.empty_like(b)
    assert grad(n, p.data_ptr(), out.data_ptr() if in_place else b.data_ptr(), sn.data_ptr(), out.data_ptr(), st) == 0
    err = float((out - want).abs().max() / want.abs().max())
    print(f"gradient {err:.2e}", flush=True)
    assert err <= 4 * 2.0 ** -53
    assert torch.equal(out[:, edge], b[:, edge])
    none = torch.empty_like(b)  # in = 0
    zero = torch.zeros_like(b)
    assert grad(n, p.data_ptr(), None, s.data_ptr(), none.data_ptr(), st) == 0
    assert grad(n, p.data_ptr(), zero.data_ptr(), s.data_ptr(), out.data_ptr(), st) == 0
    assert torch.equal(none, out)
