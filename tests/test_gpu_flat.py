"""Long flat lattices, whose tiles cover the short side and wrap across it, against
one sweep launch per step: the same update on the same values, so every bit."""
import numpy as np
import pytest

from paper_2501_16000_amd import workloads

pytestmark = pytest.mark.gpu

CASES = [
    # nx, ny, steps, equilibrium, collision, boundary
    (1048583, 1, 75, "guided", "oreg", "periodic"),   # two launches and a part of one
    (1, 1000003, 35, "poly2", "oreg", "periodic"),
    (500009, 2, 33, "guided", "bgk", "bounceback"),   # walls in the first and last tile
    (2, 600011, 21, "guided", "oreg", "bounceback"),  # nothing but walls
    (200003, 7, 19, "poly2", "bgk", "periodic"),
    (11, 100003, 23, "guided", "oreg", "periodic"),
    (33, 40009, 13, "guided", "oreg", "bounceback"),
    (50021, 33, 13, "guided", "oreg", "periodic"),
    (64, 20011, 11, "guided", "bgk", "periodic"),
    (10007, 127, 11, "guided", "oreg", "periodic"),
]


@pytest.mark.parametrize("storage", ["f64", "f32s", "f16s", "bf16s"])
@pytest.mark.parametrize("nx,ny,steps,eq,coll,bc", CASES)
def test_flat_lattices_equal_single_steps(nx, ny, steps, eq, coll, bc, storage):
    import torch
    from paper_2501_16000_amd import oreg
    print(f"[flat] {nx}x{ny} {steps} {eq} {coll} {bc} {storage}", flush=True)
    u = [0.03 * torch.from_numpy(workloads.noise((ny, nx), nx + k)).cuda() for k in (0, 1)]
    out = []
    for fuse in (0, 1):
        with oreg.Lattice(nx, ny, 0.7, equilibrium=eq, storage=storage, collision=coll,
                          boundary_x=bc, fuse_steps=fuse) as L:
            L.init(1.0 + u[0], u[0], u[1])
            L.step(steps - 1)
            L.step(1)
            out.append(L.populations())
    np.testing.assert_array_equal(out[0], out[1])
