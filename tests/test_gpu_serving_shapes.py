"""Served lattices while the resident set, and with it the split of a launch
into tiles or strips, changes under them: each result equals lb_step on the
same lattice bit for bit (the same update on the same values; no tolerance)."""
import numpy as np
import pytest

from paper_2501_16000_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f64", "f32s", "f16s", "bf16s"])
def test_results_do_not_depend_on_the_split(storage):
    from paper_2501_16000_amd import oreg, serve
    print(f"[serve shapes] {storage}", flush=True)
    # 33 lattices of 500^2 (8.25 M nodes: strips in the 16-bit formats), which
    # finish one after the other down to a few small ones (blocks)
    sizes = [500] * 33 + [33, 64, 129, 300]
    steps = [6 + 2 * k for k in range(33)] + [150, 160, 171, 133]
    got = {}
    with serve.Server(memory_budget=4 << 30, pinned_bytes=512 << 20, storage=storage) as srv:
        fields = {n: workloads.shear_wave(n, 0.03) for n in set(sizes)}
        for tag, (n, k) in enumerate(zip(sizes, steps)):
            assert srv.submit(tag, *fields[n], 0.6 + 0.01 * tag, k)
        while len(got) < len(sizes):
            srv.step(1)
            while (res := srv.poll()) is not None:
                got[res.tag] = srv.fetch(res)
    for tag in (0, 1, 16, 32, 33, 34, 35, 36):
        with oreg.Lattice(sizes[tag], sizes[tag], 0.6 + 0.01 * tag, storage=storage) as L:
            L.init(*fields[sizes[tag]])
            L.step(steps[tag])
            np.testing.assert_array_equal(got[tag], L.moments())
