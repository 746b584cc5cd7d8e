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


NUMBER_CASES = [
    # nx, ny, steps, equilibrium: F64 lattices large enough for strips, which
    # store five numbers per node after every launch
    (548, 548, 15, "guided"),        # 7 + 7 + 1 steps
    (701, 613, 10, "poly2"),         # ragged strips and row blocks
    (40, 8000, 9, "guided"),         # narrower than a strip
    (8000, 40, 6, "poly2"),
]


@pytest.mark.parametrize("nx,ny,steps,eq", NUMBER_CASES)
def test_steps_from_numbers_equal_steps_from_populations(nx, ny, steps, eq):
    """A step that starts from the five numbers of every node equals, bit for
    bit, one that starts from the populations, which a checkpoint forces."""
    from paper_2501_16000_amd import oreg
    print(f"[numbers] {nx}x{ny} {steps} {eq}", flush=True)
    f0 = populations(eq, 1 / 3, ny, nx, seed=nx + 3 * ny)
    with oreg.Lattice(nx, ny, 0.7, equilibrium=eq) as A, \
            oreg.Lattice(nx, ny, 0.7, equilibrium=eq) as B:
        A.set_populations(f0)
        A.step(steps)
        B.set_populations(f0)
        for _ in range(steps):
            B.step(1)
            B.set_populations(B.populations())
        fa = A.populations()
        np.testing.assert_array_equal(fa, B.populations())
        # A holds five numbers per node, B populations
        np.testing.assert_array_equal(A.moments(), B.moments())
        np.testing.assert_array_equal(A.diagnostics(), B.diagnostics())
        np.testing.assert_array_equal(A.density_profile(), B.density_profile())
        ref = oracle.run(f0, steps, 0.7, 1 / 3, eq)
        assert float(np.max(np.abs(fa - ref) / np.abs(ref))) <= 1e-12
        m = oracle.moments(ref)
        np.testing.assert_allclose(A.moments(), m, rtol=0, atol=1e-12)
        np.testing.assert_allclose(A.density_profile(), m[0].mean(0), rtol=1e-12)
        np.testing.assert_allclose(A.diagnostics()[:5], oracle.diagnostics(ref, 1 / 3)[:5],
                                   rtol=1e-11, atol=1e-9)


SHARED_CASES = [
    # nx, ny, steps, storage, equilibrium, collision, boundary: 32- and 16-bit
    # lattices whose strips of 256 columns are shared by a workgroup; and
    # remainders that run as block launches, in every storage
    (4881, 931, 11, "f32s", "guided", "oreg", "periodic"),   # last strip one column wide, 6 + 5 steps
    (37, 121700, 9, "f16s", "guided", "oreg", "periodic"),   # narrower than a strip
    (121700, 37, 14, "bf16s", "poly2", "oreg", "periodic"),
    (2200, 2101, 8, "f16s", "poly2", "bgk", "periodic"),
    (2001, 2300, 13, "bf16s", "guided", "oreg", "bounceback"),
    (2300, 2003, 6, "f32s", "poly2", "bgk", "bounceback"),
    (2300, 2003, 5, "f32s", "guided", "bgk", "periodic"),
    (2200, 2101, 11, "f16s", "guided", "bgk", "periodic"),   # 6 + 4 + 1 steps
    (701, 613, 12, "f64", "guided", "bgk", "periodic"),      # 7 + 5 steps
    (640, 601, 6, "f64", "poly2", "oreg", "bounceback"),
    (40, 8000, 9, "f64", "guided", "bgk", "bounceback"),
    (8000, 40, 4, "f64", "poly2", "bgk", "periodic"),
]


@pytest.mark.parametrize("nx,ny,steps,storage,eq,coll,bc", SHARED_CASES)
def test_shared_strips_equal_single_steps(nx, ny, steps, storage, eq, coll, bc):
    """The same update on the same values, so equality is exact."""
    import torch
    from paper_2501_16000_amd import oreg
    print(f"[shared strips] {nx}x{ny} {steps} {storage} {eq} {coll} {bc}", flush=True)
    u = [0.03 * torch.from_numpy(workloads.noise((ny, nx), nx + k)).cuda() for k in (0, 1)]
    with oreg.Lattice(nx, ny, 0.7, equilibrium=eq, storage=storage, collision=coll,
                      boundary_x=bc) as A, \
            oreg.Lattice(nx, ny, 0.7, equilibrium=eq, storage=storage, collision=coll,
                         boundary_x=bc) as B:
        for L in (A, B):
            L.init(1.0 + u[0], u[0], u[1])
        A.step(steps)
        for _ in range(steps):
            B.step(1)
        np.testing.assert_array_equal(A.populations(), B.populations())


def test_captured_steps_follow_a_new_init():
    """A captured graph of steps replayed on a state that was initialized after
    the capture: the kernels read the buffers' format on the device."""
    import torch
    from paper_2501_16000_amd import oreg
    n = 560
    stream = torch.cuda.Stream()
    f = [workloads.shear_wave(n, u) for u in (0.02, 0.03)]
    with torch.cuda.stream(stream), oreg.Lattice(n, n, 0.7, stream=stream) as A, \
            oreg.Lattice(n, n, 0.7, stream=stream) as B:
        A.init(*f[0])
        A.step(14)
        A.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            A.step(14)
        for fields in f:
            A.init(*fields)
            B.init(*fields)
            for k in range(3):
                graph.replay()
                torch.cuda.synchronize()
                B.step(14)
                np.testing.assert_array_equal(A.populations(), B.populations(), err_msg=str(k))


REPLAY_CASES = [
    # nx, ny, storage, collision, boundary, steps: calls that return to the buffer
    # they started from: two launches of 7 (FP64) or 6 steps from 48^2 nodes up, a
    # remainder counted once (periodic OReg) or per step, and single steps below
    (32, 32, "f64", "oreg", "periodic", 50),
    (800, 1, "f64", "oreg", "bounceback", 90),
    (128, 128, "f64", "oreg", "periodic", 14),
    (128, 128, "f64", "oreg", "periodic", 22),
    (300, 200, "f32s", "bgk", "periodic", 12),
    (300, 200, "f32s", "oreg", "bounceback", 29),   # 4 x 6 + 5 steps: nine launches
    (300, 200, "f32s", "oreg", "bounceback", 28),
    (777, 523, "f16s", "oreg", "periodic", 24),
    (700, 600, "f64", "oreg", "periodic", 28),
    (700, 600, "f64", "bgk", "periodic", 16),
    (700, 600, "f64", "bgk", "periodic", 10),
    (2200, 2101, "bf16s", "oreg", "periodic", 24),
    (2200, 2101, "bf16s", "bgk", "periodic", 11),   # 6 + 5 steps: six launches
]


@pytest.mark.parametrize("nx,ny,storage,coll,bc,steps", REPLAY_CASES)
def test_captured_calls_replay(nx, ny, storage, coll, bc, steps):
    """Which calls can be replayed (those of an even number of launches by the
    rule above) does not depend on the plan; every replay equals the eager call."""
    import torch
    from paper_2501_16000_amd import oreg
    print(f"[replay] {nx}x{ny} {storage} {coll} {bc} {steps}", flush=True)
    K = 7 if storage == "f64" else 6
    rest = steps % K if coll == "bgk" or bc == "bounceback" else (steps % K > 0)
    launches = steps if nx * ny < 2304 else steps // K + rest
    stream = torch.cuda.Stream()
    rho = np.ones((ny, nx))
    u = [0.03 * workloads.noise((ny, nx), nx + k) for k in (0, 1)]
    opts = dict(storage=storage, collision=coll, boundary_x=bc, stream=stream)
    with torch.cuda.stream(stream), oreg.Lattice(nx, ny, 0.7, **opts) as A, \
            oreg.Lattice(nx, ny, 0.7, **opts) as B:
        for L in (A, B):
            L.init(rho, *u)
            L.step(2)
            L.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            A.step(steps)
            if launches % 2:
                A.step(steps)
        for k in range(3):
            graph.replay()
            torch.cuda.synchronize()
            for _ in range(1 + launches % 2):
                B.step(steps)
            np.testing.assert_array_equal(A.moments(), B.moments(), err_msg=str(k))
