"""The adjoint stage over its launch shapes: gradients against the FP64 oracle
(complex step of the whole solve) at every order and precision, on meshes with
part chunks and rotated vertex lists.  Bounds as for the other gradients
against the oracle: relative L2 1e-12 in FP64, 1e-5 in FP32."""
import numpy as np
import pytest

from oracle import adjoint, dg
from paper_1607_03399_amd import inputs
from paper_1607_03399_amd import wdg
from parity import TOL, rel

pytestmark = pytest.mark.gpu

# elements per chunk: 64 lanes / (N + 1) levels, whole lines at N = 2, LDS at N = 5 in FP64
CHUNK = {(1, 32): 32, (1, 64): 32, (2, 32): 20, (2, 64): 20, (3, 32): 16, (3, 64): 16, (4, 32): 12, (4, 64): 12,
         (5, 32): 10, (5, 64): 9}


def _mesh(K, seed):
    """The first K wedges of a layered mesh (removed neighbours become walls),
    every vertex list rotated by a random amount: neighbours then see each
    other's triangular faces through vertex permutations."""
    m = inputs.layered_config(3, 4, 0.3, seed=seed)
    rng = np.random.default_rng(seed)
    w = np.array([np.concatenate([np.roll(q[:3], -r), np.roll(q[3:], -r)])
                  for q, r in zip(m.wedges[:K], rng.integers(3, size=K))])
    used = np.unique(w)
    ids = np.zeros(len(m.verts), dtype=np.int64)
    ids[used] = np.arange(len(used))
    return inputs.WedgeMesh(m.verts[used], ids[w], m.c[:K], m.rho[:K], m.layers, "cut")


@pytest.mark.parametrize("N,bits", sorted(CHUNK))
def test_gradient_around_a_chunk(N, bits):
    nsteps, flux = 3, "upwind"
    for K, bc in ((CHUNK[N, bits] - 1, "dirichlet"), (CHUNK[N, bits] + 1, "rigid")):
        m = _mesh(K, N)
        om = dg.Mesh(m.verts, m.wedges, m.c, m.rho, bc, flux)
        x = dg.node_coords(om, N)
        U0 = np.stack([np.cos(3 * x[..., 0] + x[..., 2]), np.sin(2 * x[..., 1]), np.cos(x[..., 0] - 2 * x[..., 1]),
                       np.sin(3 * x[..., 2])], axis=1)
        centre = m.verts[m.wedges].mean(axis=1)
        rec, src = centre[[0, K // 2, K - 1]], (centre[K // 3].tolist(), 4.0, 0.15, 1.0)
        dt = dg.stable_dt(om, N, 0.5)
        w = np.random.default_rng(K).standard_normal((nsteps, len(rec)))
        base = adjoint.solve_traces(om, N, U0, dt, nsteps, src, rec)
        elems = np.array([0, 1, K // 2, K - 2, K - 1])
        _, gc_ref, gr_ref = adjoint.gradient_complex_step(om, N, U0, dt, nsteps, src, rec, base - w, elems=elems)
        s = wdg.Solver(N, bits, device=0)
        s.set_mesh(m.verts, m.wedges)
        s.set_material(m.c, m.rho)
        s.set_boundary(bc)
        s.set_flux(flux)
        s.add_ricker_source(*src)
        s.set_receivers(rec)
        s.set_fields(U0)
        gc, gr = s.adjoint_gradient(nsteps, dt, w, checkpoint_every=2)
        s.close()
        assert rel(gc[elems], gc_ref) <= TOL[bits], f"N={N} {bits} K={K} c"
        assert rel(gr[elems], gr_ref) <= TOL[bits], f"N={N} {bits} K={K} rho"
