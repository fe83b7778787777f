"""The node-lane kernel's operator exists where that kernel runs: a default
mesh holds no second operator per wedge, and choosing the kernel before or
after the mesh, or around a batch, gives the same results bit for bit."""
import numpy as np
import pytest
import torch

from paper_1607_03399_amd import inputs
from paper_1607_03399_amd import wdg

pytestmark = pytest.mark.gpu


def _solver(m, N, before=None, after=None, bits=32):
    s = wdg.Solver(N, bits, device=0)
    if before:
        s.set_wedge_kernel(before)
    s.set_mesh(m.verts, m.wedges)
    s.set_material(m.c, m.rho)
    if after:
        s.set_wedge_kernel(after)
    return s


@pytest.mark.parametrize("N", [4, 5])
def test_device_memory_of_a_default_mesh(N):
    """States, residual, geometry (FP32), FP64 weights, connectivity and the
    packed inverse mass; 24 MiB for everything that does not grow with the mesh
    and the allocator's rounding.  The second operator would be 28 and 55 MiB."""
    m = inputs.layered_config(32, 16, 0.3, seed=1)
    NT = (N + 1) * (N + 2) // 2
    per = 3 * 16 * NT * (N + 1) + 4 * (40 + (NT * (NT + 1) // 2 + 3) // 4 * 4) + 64 + 32 + 8
    torch.cuda.init()
    _solver(inputs.layered_config(2, 2, 0.3, seed=1), N).close()  # code objects are loaded
    free = torch.cuda.mem_get_info(0)[0]
    s = _solver(m, N)
    used = free - torch.cuda.mem_get_info(0)[0]
    s.close()
    assert used <= m.K * per + (24 << 20)


@pytest.mark.parametrize("N", [4, 5])
def test_kernel_chosen_before_or_after_the_mesh(N):
    for nx, layers in ((2, 3), (4, 4)):  # 24 and 128 wedges: node-lane and level-lane by default
        m = inputs.layered_config(nx, layers, 0.3, seed=3)
        U = None
        out = {}
        for before, after in ((None, "node"), ("node", None), ("level", "node"), ("node", "level"), (None, "level")):
            s = _solver(m, N, before, after)
            U = np.random.default_rng(0).standard_normal((s.K, 4, s.NPmax)) if U is None else U
            out[before, after] = s.eval_rhs(U)
            s.close()
        assert np.array_equal(out[None, "node"], out["node", None])
        assert np.array_equal(out[None, "node"], out["level", "node"])
        assert np.array_equal(out["node", "level"], out[None, "level"])


def test_batch_keeps_its_kernel_over_a_new_mesh():
    """A batch prepared with the node-lane kernel; then the problem's kernel
    and mesh are set again (same size): the batch still runs, as the
    node-lane kernel does alone."""
    m = inputs.layered_config(4, 4, 0.3, seed=3)
    m2 = inputs.layered_config(4, 4, 0.2, seed=4)
    s, r = _solver(m, 4, "node"), _solver(m2, 4, "node")
    U = 0.1 * np.random.default_rng(1).standard_normal((s.K, 4, s.NPmax))
    batch = wdg.Batch(32, device=0)
    s.set_fields(U)
    batch.add(s, 1e-3)
    batch.prepare(autotune=False)
    s.set_wedge_kernel("level")
    s.set_mesh(m2.verts, m2.wedges)
    s.set_material(m2.c, m2.rho)
    s.set_fields(U)
    batch.step(3)
    r.set_fields(U)
    r.step(3, 1e-3)
    assert np.array_equal(s.get_fields(), r.get_fields())
    batch.close()
    s.close()
    r.close()


@pytest.mark.parametrize("N,nx,layers", [(4, 4, 5), (4, 24, 24), (5, 4, 5), (5, 24, 20)])
def test_batch_of_both_kernels(N, nx, layers):
    """Problems below and above 32 wedges in one launch (few blocks) and in two
    (more than 1200): each ends as it does alone."""
    batch = wdg.Batch(32, device=0)
    solvers, alone = [], []
    for i, (n, lay) in enumerate(((2, 3), (nx, layers), (1, 1))):
        m = inputs.layered_config(n, lay, 0.3, seed=i)
        for bucket in (solvers, alone):
            s = _solver(m, N)
            s.set_boundary("dirichlet" if i == 0 else "rigid")
            U = np.zeros((s.K, 4, s.NPmax))
            U[:, 0] = inputs.gaussian_pulse(s.node_coords(), width=0.3)
            s.set_fields(U)
            bucket.append(s)
        batch.add(solvers[-1], 1e-4 * (i + 1))
    batch.prepare()
    batch.step(2)
    for i, (s, r) in enumerate(zip(solvers, alone)):
        r.step(2, 1e-4 * (i + 1))
        assert np.array_equal(s.get_fields(), r.get_fields())
    batch.close()
    for s in solvers + alone:
        s.close()
