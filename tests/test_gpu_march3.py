"""D3Q27 boxes stored as ten numbers per node (F64 from 60,000 nodes, F32S from
300,000): every step equals, bit for bit, the same step from the populations,
which a checkpoint before each step forces; and FP64 equals the oracle.

The checkpoint round trip is exact in both formats, and both paths form every
population by the same operations, so no tolerance applies; against the oracle
the repository's parity bound of 1e-12 relative does."""
import numpy as np
import pytest

from oracle import d3q27 as o3
from paper_2501_16000_amd import workloads

pytestmark = pytest.mark.gpu

CASES = [
    # nx, ny, nz, storage, equilibrium: tiles of at most 512 columns with a
    # halo, chunks of planes
    (64, 32, 30, "f64", "guided"),      # whole tiles
    (37, 41, 43, "f64", "poly2"),       # ragged tiles and chunks
    (300, 1, 211, "f64", "guided"),     # flat in y: a tile wraps onto itself
    (1, 250, 250, "f64", "guided"),     # flat in x
    (251, 250, 1, "f64", "poly2"),      # one plane: its own neighbour
    (2, 3, 10007, "f64", "guided"),     # a single tile, many chunks
    (64, 64, 80, "f32s", "guided"),
    (71, 73, 59, "f32s", "poly2"),
    (500, 2, 307, "f32s", "guided"),
]


def populations(eq, shape, seed):
    rho = 1.0 + 0.1 * workloads.noise(shape, seed)
    us = [0.05 * workloads.noise(shape, seed + k) for k in (1, 2, 3)]
    f = o3.init(eq, 1 / 3, rho, *us)
    return f * (1.0 + workloads.noise(f.shape, seed + 4, 0.02))


@pytest.mark.parametrize("nx,ny,nz,storage,eq", CASES)
def test_steps_equal_steps_from_checkpoints(nx, ny, nz, storage, eq):
    from paper_2501_16000_amd import oreg3
    print(f"[march3] {nx}x{ny}x{nz} {storage} {eq}", flush=True)
    shape, steps = (nz, ny, nx), 4
    f0 = populations(eq, shape, 3 * nx + ny)
    with oreg3.Lattice3(nx, ny, nz, 0.7, equilibrium=eq, storage=storage) as A, \
            oreg3.Lattice3(nx, ny, nz, 0.7, equilibrium=eq, storage=storage) as B:
        A.set_populations(f0)
        A.step(steps)
        B.set_populations(f0)
        for _ in range(steps):
            B.step(1)
            B.set_populations(B.populations())
        fa = A.populations()
        np.testing.assert_array_equal(fa, B.populations())
        # A holds ten numbers per node, B populations
        np.testing.assert_array_equal(A.moments(), B.moments())
        np.testing.assert_array_equal(A.diagnostics(), B.diagnostics())
        # reading changes nothing
        A.step(1)
        B.step(1)
        np.testing.assert_array_equal(A.populations(), B.populations())
    if storage == "f64":
        ref = o3.run(f0, steps, 0.7, 1 / 3, eq)
        assert float(np.max(np.abs(fa - ref) / np.abs(ref))) <= 1e-12


PACKED_CASES = [
    # nx, ny, nz, copies along x: wavefronts of 64 consecutive nodes, against a
    # box of whole 64-node segments that repeats the first one
    (17, 28, 101, 64),
    (2, 3, 8001, 32),     # many rows and layers in one wavefront, a last one not full
    (65, 2, 401, 64),
    (200, 5, 47, 8),
]


@pytest.mark.parametrize("nx,ny,nz,copies", PACKED_CASES)
@pytest.mark.parametrize("storage,eq,coll", [("bf16s", "guided", "oreg"), ("f16s", "poly2", "oreg"),
                                             ("f64", "poly2", "bgk"), ("f32s", "guided", "bgk"),
                                             ("f32s", "guided", "oreg")])
def test_packed_nodes_equal_rows(nx, ny, nz, copies, storage, eq, coll):
    """The same update on the same values, so equality is exact."""
    from paper_2501_16000_amd import oreg3
    print(f"[packed] {nx}x{ny}x{nz} {storage} {eq} {coll}", flush=True)
    f = [workloads.noise((nz, ny, nx), nx + k, 0.03) for k in range(4)]
    f[0] = 1.0 + f[0]
    with oreg3.Lattice3(nx, ny, nz, 0.7, equilibrium=eq, storage=storage, collision=coll) as A, \
            oreg3.Lattice3(nx * copies, ny, nz, 0.7, equilibrium=eq, storage=storage,
                           collision=coll) as B:
        A.init(*f)
        B.init(*[np.tile(v, (1, 1, copies)) for v in f])
        for L in (A, B):
            L.step(3)
        np.testing.assert_array_equal(np.tile(A.moments(), (1, 1, 1, copies)), B.moments())


def test_captured_steps_follow_a_new_init():
    """A captured graph of steps replayed on a state that was initialized after
    the capture: the kernels read the buffers' format on the device."""
    import torch
    from paper_2501_16000_amd import oreg3
    n = 40
    stream = torch.cuda.Stream()
    f = [workloads.shear_wave3(n, u) for u in (0.02, 0.03)]
    with torch.cuda.stream(stream), oreg3.Lattice3(n, n, n, 0.7, stream=stream) as A, \
            oreg3.Lattice3(n, n, n, 0.7, stream=stream) as B:
        A.init(*f[0])
        A.step(2)
        A.sync()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            A.step(2)
        for fields in f:
            A.init(*fields)
            B.init(*fields)
            for k in range(3):
                graph.replay()
                torch.cuda.synchronize()
                B.step(2)
                np.testing.assert_array_equal(A.populations(), B.populations(), err_msg=str(k))
