"""FP64 strips, which store five numbers per node and have launches of every length,
against the single-step sweep on nine populations: a lattice that repeats a smaller
one equals it node by node, bit for bit."""
import numpy as np
import pytest

from paper_2501_16000_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,copies_x,copies_y,steps", [
    (211, 233, 3, 3, 9),       # 442,467 nodes; ragged strips and row blocks
    (211, 233, 3, 3, 1),
    (40, 7001, 2, 1, 8),       # one strip and a part
    (541, 547, 4, 4, 10),      # 4.7 M nodes
    (276, 548, 20, 10, 9),     # buffers above 2 GiB: addresses from 64-bit pointers
])
@pytest.mark.parametrize("eq", ["guided", "poly2"])
def test_strips_equal_single_sweeps_of_the_period(nx, ny, copies_x, copies_y, steps, eq):
    from paper_2501_16000_amd import oreg
    print(f"[strip control] {copies_x}x{copies_y} of {nx}x{ny} {eq} {steps}", flush=True)
    f = [workloads.noise((ny, nx), nx + k, 0.05) for k in range(3)]
    f[0] = 1.0 + f[0]
    tile = lambda a: np.tile(a, (1,) * (a.ndim - 2) + (copies_y, copies_x))
    with oreg.Lattice(nx, ny, 0.6, equilibrium=eq, fuse_steps=1) as small:
        small.init(*f)
        small.step(steps)
        m, p = small.moments(), small.populations()
    with oreg.Lattice(nx * copies_x, ny * copies_y, 0.6, equilibrium=eq) as large:
        large.init(*[tile(a) for a in f])
        large.step(steps)
        np.testing.assert_array_equal(large.moments(), tile(m))
        if copies_x * copies_y <= 16:
            np.testing.assert_array_equal(large.populations(), tile(p))
