"""Tetrahedron counts around the stage kernel's chunk of 8 (part of one, one
more than one, whole ones) on both tetrahedron kernels, beside wedges across
nonconforming faces; bounds as for hybrid meshes (relative L2, FP64 1e-12,
FP32 1e-5)."""
import pytest

from paper_1607_03399_amd import inputs
from parity import TOL
from test_gpu_hybrid import _compare_rhs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [64, 32])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5])
def test_rhs_around_a_chunk(N, bits):
    for layers in (1, 3, 8):  # 3, 9 and 24 tetrahedra
        mesh = inputs.split_columns(inputs.layered_config(1, layers, 0.3, seed=N), [0])
        assert len(mesh[2]) == 3 * layers
        assert _compare_rhs(mesh, N, bits, "rigid", "upwind", layers) <= TOL[bits]
