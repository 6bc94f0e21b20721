"""The pressure multigrid's 65-offset product (csrc/k_zmg.hip) where one row of nodes takes more than 64
KB of LDS, the largest lattices (from 325 nodes per axis; 513 is the pressure lattice of a 1025^3
velocity one), and at the size before: against sums of shifted arrays with random stencils.
Called below the C ABI, which reaches these sizes with vectors of a hundred gigabytes only.

Tolerance: 65 products per node in another order, entries below 1: 1e-13 of the largest entry."""

import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu


def _upper_offsets():
    o = [(x, y, z) for z in range(-2, 3) for y in range(-2, 3) for x in range(-2, 3)
         if max(x, y, z, 0) - min(x, y, z, 0) <= 2]
    assert len(o) == 65
    return o[32:]


@pytest.mark.parametrize("n", [323, 324, 512])
def test_product(n):
    from paper_2511_13109_amd import _lib
    print(f"\n[z product n={n}]", flush=True)
    fn = getattr(_lib.load(), "_ZN4agca15launch_zstencilEiiPKdS1_S1_dPdP12ihipStream_t")
    fn.restype, fn.argtypes = C.c_int, [C.c_int, C.c_int, C.c_void_p, C.c_void_p, C.c_void_p, C.c_double, C.c_void_p, C.c_void_p]
    n1, m = n + 1, n + 5
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    opts = dict(generator=g, dtype=torch.float64, device="cuda")
    x = torch.randn(n1, n1, n1, **opts)
    S = torch.zeros(33, m, m, m, dtype=torch.float64, device="cuda")
    ref = torch.zeros_like(x)

    def part(d):  # nodes whose neighbour at distance d lies on the lattice, and those neighbours
        return slice(max(0, -d), n1 - max(0, d)), slice(max(0, d), n1 + min(0, d))

    for j, (dx, dy, dz) in enumerate(_upper_offsets()):
        a, b = zip(part(dz), part(dy), part(dx))
        inner = S[j, 2:2 + n1, 2:2 + n1, 2:2 + n1]
        w = torch.rand(ref[a].shape, **opts)
        inner[a] = w
        ref[a] += w * x[b]
        if j:
            ref[b] += w * x[a]
        del w
    r = torch.randn(n1, n1, n1, **opts)
    out = torch.empty_like(x)
    st = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    for mode in (0, 1, 2):
        assert fn(mode, n, S.data_ptr(), x.data_ptr(), r.data_ptr(), 0.5, out.data_ptr(), st) == 0
        want = ref if mode == 0 else r - ref if mode == 1 else x + 0.5 * (r - ref) / S[0, 2:2 + n1, 2:2 + n1, 2:2 + n1]
        err = float((out - want).abs().max() / want.abs().max())
        print(f"mode {mode}: {err:.2e}", flush=True)
        assert err <= 1e-13
