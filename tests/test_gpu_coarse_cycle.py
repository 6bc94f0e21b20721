"""The one-workgroup cycle of the small levels (csrc/k_coarse_cycle.hip) against the same cycle composed
in Python from the library's single operations: as the whole cycle (3^3 .. 9^3 vector, up to 17^3
scalar), below one more level, and switched off (a finest coefficient in BF16, more passes than
it takes), with no passes before or after the correction among them.

Tolerances as for the other composed cycles: FP64 1e-12, FP32 2e-5 of the largest entry."""

import pytest
import torch

from test_gpu_two_products import _cycle, _hierarchy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L,ncomp,dtype", [(1, 3, "f64"), (1, 3, "f32"), (1, 3, "bf16"), (2, 3, "f64"), (2, 3, "f32"),
                                           (2, 3, "bf16"), (3, 3, "f64"), (3, 3, "f32"), (1, 1, "f64"), (2, 1, "bf16"),
                                           (3, 1, "f64"), (3, 1, "f32"), (4, 1, "f64")])
@pytest.mark.parametrize("smoother,pre,post", [("chebyshev", 2, 2), ("chebyshev", 3, 1), ("jacobi", 1, 0), ("jacobi", 0, 2),
                                               ("jacobi", 8, 8), ("jacobi", 9, 1)])
def test_cycle(L, ncomp, dtype, smoother, pre, post):
    print(f"\n[coarse cycle L={L} ncomp={ncomp} {dtype} {smoother} V({pre},{post})]", flush=True)
    H = _hierarchy(L, ncomp, dtype, smoother, pre, post, "mean")
    try:
        n1 = H.n(L) + 1
        g = torch.Generator(device="cuda")
        g.manual_seed(6)
        t = torch.float64 if dtype == "f64" else torch.float32
        b = torch.zeros(ncomp, n1, n1, n1, dtype=t, device="cuda")
        b[:, 1:-1, 1:-1, 1:-1] = torch.randn(ncomp, n1 - 2, n1 - 2, n1 - 2, generator=g, dtype=t, device="cuda")
        b = b.reshape(-1)
        ref = _cycle(H, L, b, pre, post)
        x = H.vcycle(b)
        err = float((x.double() - ref.double()).abs().max() / ref.double().abs().max())
        print(f"error {err:.2e}", flush=True)
        assert err <= (1e-12 if dtype == "f64" else 2e-5)
        assert torch.equal(x, H.vcycle(b))
        v = x.view(ncomp, n1, n1, n1)
        for face in (v[:, 0], v[:, -1], v[:, :, 0], v[:, :, -1], v[..., 0], v[..., -1]):
            assert not face.any()
    finally:
        H.close()
