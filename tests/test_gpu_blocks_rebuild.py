"""Stored Galerkin blocks are formed when they are first read: they follow every coefficient
rebuild, whether or not they were read before it, and the operators do not depend on them."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ncomp", [1, 3])
@pytest.mark.parametrize("read_before", [False, True])
def test_blocks_follow_rebuild(ncomp, read_before):
    from paper_2511_13109_amd import Hierarchy, coefficients_from_field
    from workloads import Sinkers
    L = 4
    first, second = (coefficients_from_field(Sinkers(3, seed, radius=0.15, width=2.0 / 32, contrast=1e6), L)
                     for seed in (2, 7))
    H = Hierarchy(L, ncomp, first[L], first[:L])
    F = Hierarchy(L, ncomp, second[L], second[:L])
    M = Hierarchy(L, ncomp, second[L], second[:L], coarse_storage="mean")
    try:
        if read_before:
            for l in range(L):
                assert H.blocks(l).shape[0] == H.query(l)["flagged"]
        H.set_nu(second[L], second[:L])
        for l in range(L):
            assert np.array_equal(H.flags(l), F.flags(l))
            assert np.array_equal(H.blocks(l), F.blocks(l))
            u = torch.randn(ncomp * H.nodes(l), dtype=torch.float64, device="cuda")
            assert torch.equal(H.apply(l, u), M.apply(l, u))
    finally:
        H.close()
        F.close()
        M.close()
