"""16-bit lattices whose rows fill strips of 244 columns badly run strips of one
wavefront (52 columns), F32S ones blocks: against one sweep launch per step, the
same update on the same values, so every bit."""
import numpy as np
import pytest

from paper_2501_16000_amd import workloads

pytestmark = pytest.mark.gpu

CASES = [
    # nx, ny, steps, storage, equilibrium, collision, boundary
    (37, 121700, 9, "bf16s", "guided", "oreg", "periodic"),     # narrower than a strip
    (52, 90007, 12, "f16s", "poly2", "oreg", "periodic"),       # exactly one
    (53, 90007, 11, "f16s", "guided", "oreg", "periodic"),      # one column in the second
    (105, 43003, 6, "bf16s", "guided", "oreg", "bounceback"),
    (200, 23003, 8, "f16s", "guided", "bgk", "periodic"),       # 6 steps, then a block of 2
    (300, 15101, 17, "bf16s", "poly2", "oreg", "periodic"),     # 6 + 6 + 5 steps
    (97003, 48, 11, "bf16s", "guided", "oreg", "periodic"),     # few rows
    (1500, 3101, 7, "bf16s", "guided", "oreg", "periodic"),     # 6 + 1 steps
    (300, 15101, 13, "f32s", "guided", "oreg", "periodic"),
]


@pytest.mark.parametrize("nx,ny,steps,storage,eq,coll,bc", CASES)
def test_narrow_strips_equal_single_steps(nx, ny, steps, storage, eq, coll, bc):
    import torch
    from paper_2501_16000_amd import oreg
    print(f"[narrow strips] {nx}x{ny} {steps} {storage} {eq} {coll} {bc}", flush=True)
    u = [0.03 * torch.from_numpy(workloads.noise((ny, nx), nx + k)).cuda() for k in (0, 1)]
    out = []
    for fuse in (0, 1):
        with oreg.Lattice(nx, ny, 0.7, equilibrium=eq, storage=storage, collision=coll,
                          boundary_x=bc, fuse_steps=fuse) as L:
            L.init(1.0 + u[0], u[0], u[1])
            L.step(steps)
            out.append(L.populations())
    np.testing.assert_array_equal(out[0], out[1])
