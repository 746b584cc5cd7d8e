"""Results that come back through the pinned block (up to 16 KiB a call, from the
second one on) and just above it, from calls that follow each other: the same numbers
as the device holds."""
import numpy as np
import pytest

from paper_2501_16000_amd import workloads

pytestmark = pytest.mark.gpu


def lattice(nx, ny):
    from paper_2501_16000_amd import oreg
    L = oreg.Lattice(nx, ny, 0.7)
    rho = 1.0 + 0.1 * workloads.noise((ny, nx), nx)
    L.init(rho, *[0.05 * workloads.noise((ny, nx), nx + k) for k in (1, 2)])
    return L


@pytest.mark.parametrize("nx,ny", [(1, 1), (455, 1), (456, 1), (682, 1), (683, 1), (1365, 1),
                                   (1366, 1), (35, 39), (2048, 1), (2049, 1), (4096, 1),
                                   (4097, 1)])
def test_results_around_the_block(nx, ny):
    import torch
    print(f"[small results] {nx}x{ny}", flush=True)
    with lattice(nx, ny) as L:
        out = torch.empty((3, ny, nx), dtype=torch.float64, device="cuda")
        sums = torch.empty(6, dtype=torch.float64, device="cuda")
        for steps in (0, 3, 9):
            L.step(steps)
            # one after another: each takes the block over from the one before
            m, d, p, f, m2 = L.moments(), L.diagnostics(), L.density_profile(), L.populations(), L.moments()
            L.moments(out)
            L.diagnostics_device_noalloc(sums)
            L.sync()
            np.testing.assert_array_equal(m, out.cpu().numpy())
            np.testing.assert_array_equal(m2, m)
            np.testing.assert_array_equal(d, sums.cpu().numpy())
            # sums of nine populations and of ny densities, in any order
            np.testing.assert_allclose(p, m[0].mean(0), rtol=1e-14 * (ny + 1))
            np.testing.assert_allclose(f.sum(0), m[0], rtol=1e-14)


def test_box_sums():
    from paper_2501_16000_amd import oreg3
    shape = (5, 7, 9)
    with oreg3.Lattice3(9, 7, 5, 0.7) as L:
        L.init(1.0 + 0.1 * workloads.noise(shape, 1), *[0.05 * workloads.noise(shape, k) for k in (2, 3, 4)])
        for steps in (0, 2):
            L.step(steps)
            d, m = L.diagnostics(), L.moments()
            np.testing.assert_allclose(d[:4], [m[0].sum(), *[(m[0] * m[k]).sum() for k in (1, 2, 3)]],
                                       rtol=0, atol=1e-12)
