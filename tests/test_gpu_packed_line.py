"""D3Q27 boxes on both sides of the lines between rows, rows in one round of
wavefronts and packed nodes: the box equals, bit for bit, a longer one of whole 64-node segments that repeats it."""
import numpy as np
import pytest

from paper_2501_16000_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [31, 33, 40, 41, 45, 46])   # 961 to 2116 segments
@pytest.mark.parametrize("storage,coll", [("f64", "bgk"), ("f32s", "oreg"), ("bf16s", "oreg")])
def test_boxes_equal_whole_segments(n, storage, coll):
    from paper_2501_16000_amd import oreg3
    print(f"[packed line] {n}^3 {storage} {coll}", flush=True)
    copies = 64 if n % 2 else 32
    f = [workloads.noise((n, n, n), n + k, 0.03) for k in range(4)]
    f[0] = 1.0 + f[0]
    with oreg3.Lattice3(n, n, n, 0.7, storage=storage, collision=coll) as A, \
            oreg3.Lattice3(n * copies, n, n, 0.7, storage=storage, collision=coll) as B:
        A.init(*f)
        B.init(*[np.tile(v, (1, 1, copies)) for v in f])
        for L in (A, B):
            L.step(3)
        np.testing.assert_array_equal(np.tile(A.moments(), (1, 1, 1, copies)), B.moments())
