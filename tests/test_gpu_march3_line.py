"""F64 boxes on both sides of the line from which they are stored as ten numbers per
node (more than 2048 segments of 64 nodes along x, or 110,000 nodes): every step
equals, bit for bit, the same step from the populations, which a checkpoint
before each step forces, and the oracle within the parity bound."""
import numpy as np
import pytest

from oracle import d3q27 as o3
from paper_2501_16000_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,eq", [
    (45, 45, 45, "guided"),     # 2025 segments
    (46, 46, 46, "guided"),     # 2116
    (37, 53, 43, "poly2"),      # ragged tiles and chunks
    (64, 64, 33, "poly2"),
    (300, 1, 500, "guided"),    # flat in y: a tile wraps onto itself
    (251, 600, 1, "guided"),    # one plane: its own neighbour
    (100, 35, 33, "guided"),    # 115,500 nodes
])
def test_steps_equal_steps_from_checkpoints(nx, ny, nz, eq):
    from paper_2501_16000_amd import oreg3
    print(f"[march3 line] {nx}x{ny}x{nz} {eq}", flush=True)
    shape, steps = (nz, ny, nx), 3
    rho = 1.0 + 0.1 * workloads.noise(shape, nx)
    f0 = o3.init(eq, 1 / 3, rho, *[0.05 * workloads.noise(shape, nx + k) for k in (1, 2, 3)])
    f0 = f0 * (1.0 + workloads.noise(f0.shape, nx + 4, 0.02))
    with oreg3.Lattice3(nx, ny, nz, 0.7, equilibrium=eq) as A, \
            oreg3.Lattice3(nx, ny, nz, 0.7, equilibrium=eq) as B:
        A.set_populations(f0)
        A.step(steps)
        B.set_populations(f0)
        for _ in range(steps):
            B.step(1)
            B.set_populations(B.populations())
        fa = A.populations()
        np.testing.assert_array_equal(fa, B.populations())
        np.testing.assert_array_equal(A.moments(), B.moments())
        np.testing.assert_array_equal(A.diagnostics(), B.diagnostics())
    ref = o3.run(f0, steps, 0.7, 1 / 3, eq)
    assert float(np.max(np.abs(fa - ref) / np.abs(ref))) <= 1e-12
