"""The operators, which keep one coefficient per flagged element (its descendants' mean), against the
product formed from the stored Galerkin blocks: blocks come from the element-wise recursion (2.7), which knows
nothing of the means.  At 129^3, on levels whose flagged elements are many; every block also equals its
element's mean times the unit element matrix.

Tolerances: FP64 sums of up to 8^5 finest elements' entries, in other orders: 1e-12 of the largest entry, as in the
comparison with the oracle."""

import numpy as np
import pytest
import torch

from oracle import agca
from workloads import workload
from workloads.lattice import element_centroids

pytestmark = pytest.mark.gpu
ORDERS = [(0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)]
L, NC = 6, 3


@pytest.fixture(scope="module")
def case():
    from paper_2511_13109_amd import Hierarchy
    field = workload("sinker129").make_field()
    nu = [torch.from_numpy(np.ascontiguousarray(field.nu(element_centroids(l)))).cuda() for l in range(L + 1)]
    H = Hierarchy(L, NC, nu[L], nu[:L])
    yield H, nu
    H.close()


def _vertices(n, ids):
    """Node indices of the elements `ids`, (elements, 4) in path order."""
    s, cell = ids % 6, ids // 6
    x, y, z = cell % n, (cell // n) % n, cell // (n * n)
    step = torch.tensor(ORDERS, device=ids.device)[s]
    p = torch.stack([x, y, z], dim=1)
    out = []
    for a in range(4):
        out.append(p[:, 0] + (n + 1) * (p[:, 1] + (n + 1) * p[:, 2]))
        if a < 3:
            p = p + torch.nn.functional.one_hot(step[:, a], 3)
    return torch.stack(out, dim=1)


def _product(n, ids, mats, u):
    """Sum over the elements of matrix times u, with rows (c, a) = 4 c + a; u (NC, nodes)."""
    v = _vertices(n, ids)
    ue = u[:, v].permute(1, 0, 2).reshape(len(ids), 4 * NC)
    ye = (mats * ue[:, None, :]).sum(dim=2).view(len(ids), NC, 4)
    y = torch.zeros_like(u)
    for c in range(NC):
        y[c].index_add_(0, v.reshape(-1), ye[:, c].reshape(-1))
    return y


@pytest.mark.parametrize("level", [2, 3, 4])
def test_product_with_blocks(case, level):
    H, nu = case
    n = H.n(level)
    print(f"\n[blocks product level {level}]", flush=True)
    unit = torch.from_numpy(np.stack([agca.unit_element_matrix_path(1.0 / n, NC, o) for o in ORDERS])).cuda()
    flagged = torch.from_numpy(H.flags(level).astype(np.int64)).cuda()
    blocks = torch.from_numpy(H.blocks(level)).cuda().reshape(len(flagged), 4 * NC, 4 * NC)
    assert len(flagged) > 0
    g = torch.Generator(device="cuda")
    g.manual_seed(9)
    u = torch.zeros(NC, n + 1, n + 1, n + 1, dtype=torch.float64, device="cuda")
    u[:, 1:-1, 1:-1, 1:-1] = torch.randn(NC, n - 1, n - 1, n - 1, generator=g, dtype=torch.float64, device="cuda")
    u = u.reshape(NC, -1)
    y = _product(n, flagged, blocks, u)
    plain = torch.ones(6 * n ** 3, dtype=torch.bool, device="cuda")
    plain[flagged] = False
    plain = plain.nonzero()[:, 0]
    for ids in plain.split(1 << 18):
        y += _product(n, ids, unit[ids % 6] * nu[level][ids][:, None, None], u)
    y = y.view(NC, n + 1, n + 1, n + 1)
    ref = torch.zeros_like(y)
    ref[:, 1:-1, 1:-1, 1:-1] = y[:, 1:-1, 1:-1, 1:-1]
    got = H.apply(level, u.reshape(-1)).view_as(ref)
    err = float((got - ref).abs().max() / ref.abs().max())
    # the means, from the blocks' first diagonal entries
    mean = blocks[:, 0, 0] / unit[flagged % 6, 0, 0]
    off = (blocks - mean[:, None, None] * unit[flagged % 6]).abs().amax(dim=(1, 2)) / blocks.abs().amax(dim=(1, 2))
    print(f"{len(flagged)} flagged, product {err:.2e}, blocks {float(off.max()):.2e}", flush=True)
    assert err <= 1e-12
    assert float(off.max()) <= 1e-12
