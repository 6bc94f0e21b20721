"""Passes whose output buffer is also an input read at the same node: a residual written over its
right-hand side (agca_residual refuses r = x only), and Chebyshev passes of degree 3, which write over the
iterate before the current one.  Scalar levels below and above the marching kernel's 64 cells
(csrc/k_scalar.hip), and a vector level.  The bits are those of separate buffers."""

import pytest
import torch

from test_gpu_two_products import _cycle, _hierarchy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,ncomp,dtype", [(4, 1, "f64"), (5, 1, "f32"), (6, 1, "f64"), (4, 3, "f64")])
def test_output_over_input(L, ncomp, dtype):
    print(f"\n[in place L={L} ncomp={ncomp} {dtype}]", flush=True)
    H = _hierarchy(L, ncomp, dtype, "chebyshev", 3, 3, "mean")
    try:
        n1 = H.n(L) + 1
        t = torch.float64 if dtype == "f64" else torch.float32
        g = torch.Generator(device="cuda")
        g.manual_seed(4)
        b, x = (torch.zeros(ncomp, n1, n1, n1, dtype=t, device="cuda") for _ in range(2))
        for v in (b, x):
            v[:, 1:-1, 1:-1, 1:-1] = torch.randn(ncomp, n1 - 2, n1 - 2, n1 - 2, generator=g, dtype=t, device="cuda")
        b, x = b.reshape(-1), x.reshape(-1)
        r = H.residual(L, b, x)
        over = b.clone()
        assert torch.equal(H.residual(L, over, x, over), r)
        ref = _cycle(H, L, b, 3, 3)
        err = float((H.vcycle(b).double() - ref.double()).abs().max() / ref.double().abs().max())
        print(f"error {err:.2e}", flush=True)
        assert err <= (1e-12 if dtype == "f64" else 2e-5)
    finally:
        H.close()
