"""Populations in and out: sizes at the edges of the pieces that a result is
copied in (1 MiB, from 1.5 MB on), and input that is refused leaves the state as
it was.  In FP64 a checkpoint comes back bit for bit; no tolerance."""
import numpy as np
import pytest

import oracle
from oracle import d3q27 as o3
from paper_2501_16000_amd import workloads

pytestmark = pytest.mark.gpu

SIZES = [(31, 17), (144, 144), (146, 142), (256, 256), (512, 257), (571, 613)]


def populations(ny, nx):
    rho = 1.0 + 0.1 * workloads.noise((ny, nx), nx)
    u = [0.05 * workloads.noise((ny, nx), nx + k) for k in (1, 2)]
    return oracle.init("guided", 1 / 3, rho, *u)


@pytest.mark.parametrize("nx,ny", SIZES)
@pytest.mark.parametrize("storage", ["f64", "f32s"])
def test_checkpoint_comes_back(nx, ny, storage):
    from paper_2501_16000_amd import oreg
    print(f"[checkpoint] {nx}x{ny} {storage}", flush=True)
    f = populations(ny, nx)
    with oreg.Lattice(nx, ny, 0.7, storage=storage) as L:
        L.set_populations(f)
        got = L.populations()
        if storage == "f64":
            np.testing.assert_array_equal(got, f)
        else:
            L.set_populations(got)  # representable now
            np.testing.assert_array_equal(L.populations(), got)
        m = L.moments()
        out = np.stack([got.sum(0)])
        # 9 terms of at most 0.5, summed in another order
        np.testing.assert_allclose(m[0], out[0], rtol=0, atol=9 * 2.0 ** -52)


@pytest.mark.parametrize("fault,text", [("nan", "population 7 of node 1290 is not finite"),
                                        ("inf", "population 7 of node 1290 is not finite"),
                                        ("negative", "node 1290 has sum_i f_i <= 0")])
def test_refused_populations_leave_the_state(fault, text):
    from paper_2501_16000_amd import oreg, oreg3
    f = populations(571, 613)
    f3 = o3.init("guided", 1 / 3, np.ones((40, 40, 40)), *[np.zeros((40, 40, 40))] * 3)
    for lat, good in ((oreg.Lattice(613, 571, 0.7), f), (oreg3.Lattice3(40, 40, 40, 0.7), f3)):
        with lat as L:
            L.set_populations(good)
            L.step(3)
            before = L.populations()
            bad = good.copy()
            flat = bad.reshape(len(bad), -1)
            flat[7, 1290] = {"nan": np.nan, "inf": np.inf, "negative": -5.0}[fault]
            flat[3, 2000] = np.nan  # a later node is not the one that is named
            with pytest.raises(Exception, match=text):
                L.set_populations(bad)
            assert L.time == 3
            np.testing.assert_array_equal(L.populations(), before)
            L.step(1)
            assert np.isfinite(L.populations()).all()
