"""The longest lattice there is: a row of 2^31 - 1 nodes, where a column plus a
halo, or the row rounded up to whole workgroups, passes the largest int."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

N, TAU, STEPS = 2 ** 31 - 1, 0.8, 6


def test_one_row_of_the_most_nodes():
    """F16S, default launches and one sweep launch per step: the same bits at both
    ends and in the middle, and there the oracle within the rounding of the
    storage (a stored |f - w rho0| <= 0.03 rounds by 2^-11 of itself in each of
    six stores and nine populations: below 1e-3)."""
    import torch
    from paper_2501_16000_amd import oreg
    if torch.cuda.get_device_properties(0).total_memory < 240 * 2 ** 30:
        pytest.skip("needs a GPU with 240 GiB")
    m = 4000  # nodes looked at: both ends (they are neighbours) and the middle
    pieces = [slice(0, m), slice(N // 2, N // 2 + m), slice(N - m, N)]
    fields = [0.05 * np.sin(np.arange(m) / 7 + k) for k in range(3)]
    got = []
    for fuse in (0, 1):
        print(f"[longest] {N}x1 f16s fuse_steps={fuse}", flush=True)
        with oreg.Lattice(N, 1, TAU, 1 / 3, storage="f16s", fuse_steps=fuse) as L:
            ux = torch.zeros((1, N), dtype=torch.float64, device="cuda")
            for p, f in zip(pieces, fields):
                ux[0, p] = torch.from_numpy(f).cuda()
            L.init(torch.ones_like(ux), ux, torch.zeros_like(ux))
            del ux
            torch.cuda.empty_cache()
            L.step(STEPS)
            out = torch.empty((3, 1, N), dtype=torch.float64, device="cuda")
            L.moments(out)
            L.sync()
            got.append([out[:, 0, p].cpu().numpy() for p in pieces])
            del out
        torch.cuda.empty_cache()
    for a, b in zip(*got):
        np.testing.assert_array_equal(a, b)
    # the two ends in one piece (the seam in its middle), and the middle
    for f, g in ((np.concatenate([fields[2], fields[0]]), np.concatenate([got[0][2], got[0][0]], axis=1)),
                 (fields[1], got[0][1])):
        one = np.ones((1, len(f)))
        ref = oracle.run(oracle.init("guided", 1 / 3, one, f[None], 0 * one), STEPS, TAU, 1 / 3)
        inner = slice(STEPS, len(f) - STEPS)
        assert np.max(np.abs(g[:, inner] - oracle.moments(ref)[:, 0, inner])) < 1e-3
