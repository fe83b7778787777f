"""Lengths far from one in FP32: a mesh scaled by s has the right-hand side of
the mesh itself divided by s (no other number of the problem has a length in
it).  At 1e-12 the mass weights (volumes) are near the smallest normal number;
at 4e12 near the largest.  Against the FP64 oracle on the unscaled mesh,
relative L2 1e-5 as everywhere in FP32."""
import numpy as np
import pytest

from oracle import dg
from paper_1607_03399_amd import inputs
from paper_1607_03399_amd import wdg
from parity import TOL, check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("split", [False, True])
@pytest.mark.parametrize("N", [1, 2, 3, 4, 5])
def test_rhs_of_a_scaled_mesh(N, split):
    m = inputs.layered_config(3, 4, 0.3, seed=N)
    tets = None
    v, w, c, rho = m.verts, m.wedges, m.c, m.rho
    if split:
        v, w, tets, c, rho = inputs.split_columns(m, [1, 4])
    om = dg.Mesh(v, w, c, rho, "rigid", "upwind", tets=tets)
    mask = dg.node_mask(om, N)
    U = np.random.default_rng(N).standard_normal((om.K, 4, mask.shape[1])) * mask[:, None, :]
    ref = dg.rhs(dg.build_operators(om, N), U)
    lift = None
    for scale in (1.0, 1e-12, 2e-12, 1e-10, 4e12):
        s = wdg.Solver(N, 32, device=0)
        s.set_mesh(v * scale, w, tets)
        s.set_material(c, rho)
        got = s.eval_rhs(U[:, :, :s.NPmax]) * scale
        check(got, ref[:, :, :got.shape[2]], TOL[32], f"N={N} scale {scale}")
        L = s.element_data()[1] * scale ** 3  # one over a volume
        s.close()
        lift = L if lift is None else lift
        check(L, lift, TOL[32], f"N={N} scale {scale} lift")
