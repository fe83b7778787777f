"""Nonconforming faces whose two triangles border on tetrahedra of different
impedance (the blocks of either side then enter with factors of their own):
material drawn per tetrahedron, contrasts up to 1.1 and up to 100, against the
oracle; bounds as for hybrid meshes (relative L2, FP64 1e-12, FP32 1e-5)."""
import numpy as np
import pytest

from paper_1607_03399_amd import inputs
from parity import TOL
from test_gpu_hybrid import _compare_rhs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("contrast", [1.1, 100.0])
@pytest.mark.parametrize("bits", [64, 32])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5])
def test_rhs_across_a_diagonal(N, bits, contrast):
    v, w, t, c, rho = inputs.split_columns(inputs.layered_config(3, 3, 0.3, seed=N), [2, 7, 11])
    rng = np.random.default_rng(N)
    half = 0.5 * np.log(contrast)
    rho = rho * np.exp(rng.uniform(-half, half, len(rho)))  # impedances by as much, wave speeds as they were
    for bc, flux in (("rigid", "upwind"), ("dirichlet", "central")):
        assert _compare_rhs((v, w, t, c, rho), N, bits, bc, flux, 30 + N) <= TOL[bits]
