"""Calls that find no device memory: what the hierarchy can do without is given up (the scalar
levels' edge weights, until a rebuild finds room for them; in a rebuild the stored Galerkin blocks), and a rebuild that fails all the same
leaves the hierarchy as it was, a solve what a later one needs.  Weights that a captured graph reads stay.

The test runs in a process of its own, in which hipMalloc is a function that refuses on demand (a shared
library in the global scope, before the HIP runtime): refuse until something is freed, or always."""

import os
import shutil
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SHIM = r"""
#include <dlfcn.h>
#include <stddef.h>
static int mode, refused, pass;  // mode 1: refuse until a hipFree, 2: refuse, after `pass` more calls
static void* real(const char* name) {
    void* lib = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
    return lib ? dlsym(lib, name) : 0;
}
extern "C" void refuse(int m, int after) { mode = m; refused = 0; pass = after; }
extern "C" int refusals() { return refused; }
extern "C" int hipMalloc(void** p, size_t n) {
    if (mode && pass-- <= 0) { ++refused; return 2; }  // hipErrorOutOfMemory
    return ((int (*)(void**, size_t))real("hipMalloc"))(p, n);
}
extern "C" int hipFree(void* p) {
    if (mode == 1) mode = 0;
    return ((int (*)(void*))real("hipFree"))(p);
}
"""

CHILD = r"""
import ctypes, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
ncomp, what = int(sys.argv[2]), sys.argv[3]
import numpy as np, torch
from paper_2511_13109_amd import AGCAError, Hierarchy, Stokes, coefficients_from_field
from workloads import Sinkers
L = 4
first, second = (coefficients_from_field(Sinkers(3, seed, radius=0.15, width=2.0 / 32, contrast=1e6), L) for seed in (2, 7))
F, G = Hierarchy(L, ncomp, first[L], first[:L]), Hierarchy(L, ncomp, second[L], second[:L])
H = Hierarchy(L, ncomp, first[L], first[:L])
g = torch.Generator(device="cuda")
g.manual_seed(5)
n1 = H.n(L) + 1
u = torch.zeros(ncomp, n1, n1, n1, dtype=torch.float64, device="cuda")
u[:, 1:-1, 1:-1, 1:-1] = torch.randn(ncomp, n1 - 2, n1 - 2, n1 - 2, generator=g, dtype=torch.float64, device="cuda")
u = u.reshape(-1)

def same(A, B):
    for op in (lambda X: X.apply(L, u), lambda X: X.vcycle(u)):
        a, b = op(A), op(B)
        torch.cuda.synchronize()  # the two may have streams of their own
        err = float((a - b).abs().max() / b.abs().max())
        assert err <= 1e-12, err
    for l in range(L):
        assert np.array_equal(A.flags(l), B.flags(l))
        assert np.array_equal(A.blocks(l), B.blocks(l))

def refused(call):
    try:
        call()
    except AGCAError as e:
        return "AGCA_E_OOM" in str(e)
    return False

full = H.device_bytes()
if what == "rebuild":
    # the weights or the blocks make room
    shim.refuse(1, 0)
    H.set_nu(second[L], second[:L])
    assert shim.refusals() > 0
    same(H, G)
    # and are there again
    assert H.device_bytes() == G.device_bytes()
    assert torch.equal(H.apply(L, u), G.apply(L, u))
elif what == "blocks":
    if ncomp == 1:
        shim.refuse(1, 0)
        got = H.blocks(1)
        assert shim.refusals() > 0
        assert H.device_bytes() < full
        assert np.array_equal(got, F.blocks(1))
        H.set_nu(first[L], first[:L])
        assert H.device_bytes() == full
        assert torch.equal(H.apply(L, u), F.apply(L, u))
    else:  # nothing to give up
        shim.refuse(2, 0)
        assert refused(lambda: H.blocks(1))
        shim.refuse(0, 0)
    same(H, F)
elif what == "solve":
    # the first solve (and the first Stokes operation), refused at each of its allocations, then again
    b = u
    want = F.solve(b, tol=1e-8)[0]
    M = Hierarchy(L, ncomp, first[L], first[:L], mg_dtype="f32")
    mixed = M.solve(b, solver="fcg", tol=1e-8)[0]
    M.close()
    for kind in ("f64", "f32") + (("stokes",) if ncomp == 3 else ()):
        for after in range(12):
            X = Hierarchy(L, ncomp, first[L], first[:L], mg_dtype="f32" if kind == "f32" else "f64")
            y = torch.empty_like(b)
            if kind == "stokes":
                S, q = Stokes(X), torch.empty((X.n(L - 1) + 1) ** 3, dtype=torch.float64, device="cuda")
                call = lambda: S.div(b, q)
            else:
                call = lambda: X.solve(b, y, solver="pcg" if kind == "f64" else "fcg", tol=1e-8)
            shim.refuse(2, after)
            failed = refused(call)
            assert failed == (shim.refusals() > 0)
            shim.refuse(0, 0)
            y.zero_()
            call()
            if kind == "stokes":
                assert torch.equal(q, Stokes(F).div(b))
            else:
                ref = want if kind == "f64" else mixed
                assert float((y - ref).abs().max()) <= 1e-6 * float(ref.abs().max())
            X.close()
            if not failed:
                break
        assert not failed and after > 0
elif what == "captured":
    # weights that a captured cycle reads are not given up; its replays follow a rebuild
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        C = Hierarchy(L, 1, first[L], first[:L], stream=st)
        x = torch.empty_like(u)
        C.vcycle(u, x)
        graph = torch.cuda.CUDAGraph()
        st.synchronize()
        with torch.cuda.graph(graph, stream=st):
            C.vcycle(u, x)
        held = C.device_bytes()
        shim.refuse(1, 0)
        assert refused(lambda: C.blocks(1))
        shim.refuse(0, 0)
        assert C.device_bytes() == held
        for X, nu in ((F, first), (G, second), (F, first)):
            C.set_nu(nu[L], nu[:L])
            for _ in range(2):
                x.zero_()
                graph.replay()
                st.synchronize()
                assert torch.equal(x, C.vcycle(u))
            same(C, X)
    C.close()
else:
    # every allocation of a rebuild in turn is the first that is refused
    for after in range(30):
        shim.refuse(2, after)
        version = H.version
        failed = refused(lambda: H.set_nu(second[L], second[:L]))
        assert failed == (shim.refusals() > 0)
        shim.refuse(0, 0)
        assert H.version != version  # what a backward pass goes by
        # the old operators or the new ones, with their flags and blocks
        old = all(np.array_equal(H.flags(l), F.flags(l)) for l in range(L))
        same(H, F if old else G)
        print("refused after", after, "failed" if failed else "done", "old" if old else "new", flush=True)
        if not failed:
            assert not old and after > 0
            break
        H.close()
        H = Hierarchy(L, ncomp, first[L], first[:L])
    assert not failed
for X in (F, G, H):
    X.close()
print("child ok")
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("shim")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run([gxx, "-O1", "-shared", "-fPIC", str(d / "shim.cpp"), "-o", str(d / "shim.so"), "-ldl"], check=True)
    return str(d / "shim.so")


@pytest.mark.parametrize("what,ncomp", [("rebuild", 1), ("rebuild", 3), ("blocks", 1), ("blocks", 3), ("failed rebuild", 1),
                                        ("failed rebuild", 3), ("solve", 1), ("solve", 3), ("captured", 1)])
def test_no_memory(shim, what, ncomp):
    print(f"\n[low memory {what} ncomp={ncomp}]", flush=True)
    r = subprocess.run([sys.executable, "-c", CHILD, shim, str(ncomp), what], cwd=ROOT, capture_output=True, text=True,
                       timeout=100)
    print(r.stdout, flush=True)
    assert r.returncode == 0 and "child ok" in r.stdout, r.stdout + r.stderr
