"""Multi-step launches (tile, block and strip sweeps) against one sweep launch
per step, bit for bit, at the sizes where their regions and halos have edges.

Both paths evaluate the same per-node update on the same stored values, so the
populations are equal exactly; no tolerance applies."""
import numpy as np
import pytest

import oracle
from paper_2501_16000_amd import workloads

pytestmark = pytest.mark.gpu

STORAGES = ("f64", "f32s", "f16s", "bf16s")


def populations(eq, theta, ny, nx, seed):
    rho = 1.0 + 0.1 * workloads.noise((ny, nx), seed)
    ux, uy = (0.05 * workloads.noise((ny, nx), seed + k) for k in (1, 2))
    f = oracle.init(eq, theta, rho, ux, uy)
    return f * (1.0 + workloads.noise(f.shape, seed + 3, 0.02))


CASES = [
    # nx, ny, steps, eq, collision, boundary
    (1, 1, 300, "guided", "oreg", "periodic"),       # one node, several launches of 128 steps
    (3, 2, 130, "poly2", "oreg", "periodic"),        # halos as deep as the lattice never wrap twice
    (7, 5, 40, "guided", "bgk", "bounceback"),
    (32, 32, 50, "guided", "oreg", "periodic"),      # tiles smaller than their halos
    (33, 31, 7, "guided", "oreg", "bounceback"),
    (1, 5000, 100, "guided", "oreg", "periodic"),    # tiles that wrap across x
    (800, 1, 131, "guided", "oreg", "bounceback"),   # tiles that wrap across y
    (1030, 36, 33, "poly2", "bgk", "periodic"),
    (2, 90000, 40, "guided", "oreg", "periodic"),    # flat, more tiles than fit at once
    (286, 286, 17, "guided", "oreg", "periodic"),    # below and above the tile sweep's size
    (287, 287, 17, "guided", "oreg", "periodic"),
    (64, 1025, 13, "guided", "bgk", "bounceback"),
    (37, 2000, 11, "poly2", "oreg", "periodic"),     # blocks wider than the lattice
    (777, 523, 21, "guided", "oreg", "bounceback"),
    (547, 548, 15, "guided", "oreg", "periodic"),    # the last F64 size before strips
    (548, 548, 15, "guided", "oreg", "periodic"),
    (1500, 1499, 13, "guided", "oreg", "periodic"),  # many rounds of blocks
    (1500, 1499, 5, "poly2", "bgk", "bounceback"),
]


@pytest.mark.parametrize("storage", STORAGES)
@pytest.mark.parametrize("nx,ny,steps,eq,coll,bc", CASES)
def test_multi_step_launches_equal_single_steps(nx, ny, steps, eq, coll, bc, storage):
    from paper_2501_16000_amd import oreg
    print(f"[multistep] {nx}x{ny} {steps} {eq} {coll} {bc} {storage}", flush=True)
    f0 = populations(eq, 1 / 3, ny, nx, seed=13 * nx + ny)
    out = []
    for fuse in (0, 1):
        with oreg.Lattice(nx, ny, 0.7, equilibrium=eq, storage=storage, collision=coll,
                          boundary_x=bc, fuse_steps=fuse) as L:
            L.set_populations(f0)
            L.step(steps - 3)
            L.step(1)
            L.step(2)
            assert L.time == steps
            out.append(L.populations())
    np.testing.assert_array_equal(out[0], out[1])
