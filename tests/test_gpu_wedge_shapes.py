"""Edges of the level-lane wedge kernel's launch shapes and of the rules that
choose a kernel or a cache policy by the mesh size: element counts around a
block's chunk against the FP64 oracle (relative L2 1e-12 in FP64, 1e-5 in
FP32), the line between the wedge kernels, a batch on both sides of it, and a
state whose residual alone is streamed past the caches against the FP64 solve
(10 steps add the rounding of 50 stages, below 1e-5 as a single right-hand
side's)."""
import numpy as np
import pytest

from oracle import dg
from paper_1607_03399_amd import inputs
from paper_1607_03399_amd import wdg
from parity import TOL, check, rel

pytestmark = pytest.mark.gpu

# elements per chunk: 64 lanes / (N + 1) levels, whole lines at N = 2, LDS at N = 5 in FP64
CHUNK = {(1, 32): 32, (1, 64): 32, (2, 32): 20, (2, 64): 20, (3, 32): 16, (3, 64): 16, (4, 32): 12, (4, 64): 12,
         (5, 32): 10, (5, 64): 9}


def _cut(K, seed):
    """The first K wedges of a layered mesh (removed neighbours become walls)."""
    m = inputs.layered_config(3, 4, 0.3, seed=seed)
    used = np.unique(m.wedges[:K])
    ids = np.zeros(len(m.verts), dtype=np.int64)
    ids[used] = np.arange(len(used))
    return inputs.WedgeMesh(m.verts[used], ids[m.wedges[:K]], m.c[:K], m.rho[:K], m.layers, "cut")


def _solver(m, N, bits, wedge="level", mass="exact"):
    s = wdg.Solver(N, bits, device=0)
    s.set_mesh(m.verts, m.wedges)
    s.set_material(m.c, m.rho)
    s.set_wedge_kernel(wedge)
    s.set_mass(mass)
    return s


@pytest.mark.parametrize("mass", ["exact", "lumped"])
@pytest.mark.parametrize("N,bits", sorted(CHUNK))
def test_rhs_around_a_chunk(N, bits, mass):
    for K in (CHUNK[N, bits] - 1, CHUNK[N, bits], CHUNK[N, bits] + 1, 2 * CHUNK[N, bits] + 1):
        m = _cut(K, N)
        U = np.random.default_rng(K).standard_normal((K, 4, (N + 1) ** 2 * (N + 2) // 2))
        ops = dg.build_operators(dg.Mesh(m.verts, m.wedges, m.c, m.rho, "rigid", "upwind"), N, lumped=mass == "lumped")
        s = _solver(m, N, bits, mass=mass)
        check(s.eval_rhs(U), dg.rhs(ops, U), TOL[bits], f"N={N} {bits} K={K} {mass}")
        s.close()


@pytest.mark.parametrize("N", [4, 5])
def test_default_kernel_by_mesh_size(N):
    """Fewer than 32 wedges run on the node-lane kernel, others on the level-lane one."""
    for K, kernel in ((31, "node"), (32, "level")):
        m = _cut(K, 2)
        U = np.random.default_rng(K).standard_normal((K, 4, (N + 1) ** 2 * (N + 2) // 2))
        out = []
        for wedge in ("auto", kernel):
            s = _solver(m, N, 32, wedge)
            out.append(s.eval_rhs(U))
            s.close()
        assert np.array_equal(*out)


def test_batch_on_both_kernels_of_an_order():
    """Problems of one order on both sides of the line: each ends as it does alone."""
    batch = wdg.Batch(32, device=0)
    solvers, fields, alone = [], [], []
    for i, K in enumerate((24, 60)):
        m = _cut(K, 3 + i)
        U = 0.1 * np.random.default_rng(i).standard_normal((K, 4, 75))
        for bucket in (solvers, alone):
            s = _solver(m, 4, 32, "auto")
            s.set_fields(U)
            bucket.append(s)
        batch.add(solvers[-1], 1e-3)
    batch.prepare()
    assert {t[0] for t in batch.trials(4)} == {"level"}
    batch.step(4)
    for s, r in zip(solvers, alone):
        r.step(4, 1e-3)
        assert np.array_equal(s.get_fields(), r.get_fields())
    batch.close()
    for s in solvers + alone:
        s.close()


def test_streamed_residual_alone():
    """114 688 wedges at N = 3 in FP32 (220 MiB of state and residual: the
    residual streams, the states stay cached) against the FP64 solve."""
    m = inputs.layered_config(64, 14, 0.3, seed=2)
    out = []
    for bits in (64, 32):
        s = _solver(m, 3, bits)
        U = np.zeros((s.K, 4, s.NPmax))
        U[:, 0] = inputs.gaussian_pulse(s.node_coords(), width=0.2)
        s.set_fields(U)
        s.step(10, s.stable_dt(0.5))
        out.append(s.get_fields())
        s.close()
    assert rel(out[1], out[0]) <= TOL[32]
