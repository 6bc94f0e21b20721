"""The edge-flux form of the cell operator (csrc/cube_math.h, cell_flux), compiled for the
host, against the oracle's element matrices (eq. (2.3) / (3.5)) summed over the cell's six
simplices."""

import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import agca

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2511_13109_amd", "csrc")
ORDERS = [(0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)]


@pytest.mark.parametrize("ncomp", [1, 3])
@pytest.mark.parametrize("only", [None, 0, 1, 2, 3, 4, 5])
def test_cell_flux(tmp_path, ncomp, only):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    out = str(tmp_path / "host_flux")
    subprocess.run([gxx, "-std=c++17", "-O1", "-Wall", "-Wno-unknown-pragmas", "-Werror", "-I", CSRC,
                    os.path.join(HERE, "host_flux.cpp"), "-o", out], check=True)
    rng = np.random.default_rng(ncomp)
    U = rng.standard_normal((8, ncomp))
    w = np.exp(rng.uniform(-7.0, 7.0, size=6)) if only is None else np.eye(6)[only]
    txt = f"{ncomp} " + " ".join(f"{v:.17g}" for v in np.concatenate([U.ravel(), w]))
    r = subprocess.run([out], input=txt, capture_output=True, text=True, check=True)
    got = np.array([float(v) for v in r.stdout.split()]).reshape(8, ncomp)
    ref = np.zeros((8, ncomp))
    for s, order in enumerate(ORDERS):
        K = agca.unit_element_matrix_path(1.0, ncomp, order) * 6.0  # row 4 c + a, without h/6
        corners = [0]
        for ax in order:
            corners.append(corners[-1] | (1 << ax))
        v = w[s] * (K @ U[corners].T.ravel())
        for c in range(ncomp):
            for a in range(4):
                ref[corners[a], c] += v[4 * c + a]
    # at most 10 roundings on any sum, each relative 1.1e-16 of the largest term
    assert np.abs(got - ref).max() <= 1e-14 * w.max() * np.abs(U).max() * 4
