"""Reductions of the per-tile correlator partials (time-block closes and open
sums) at the tile counts where their split changes: one tile, the largest
count one workgroup sums and the next, one range per workgroup and its
neighbours, several tiles per range.  The correlators of one sample of the
state are compared with the same sums over the populations in numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [1, 2, 16, 64, 65, 255, 256, 257, 600, 4099])
@pytest.mark.parametrize("block", [0, 1])
def test_sums_of_every_tile_count(flb, tiles, block):
    # 64 x 4 tiles, the last one ragged.  Tolerance: each sum of n ~ 1e6 terms
    # in FP64 carries at most n eps ~ 2e-10 of its absolute terms and in
    # practice sqrt(n) eps ~ 2e-13; 1e-11 of the largest entry.
    nx, ny = 61, 4 * tiles - 1
    L = flb.Lattice(flb.make_params(nx, ny, precision=flb.FP64, ux0=0.05, kT=1e-4, seed=tiles,
                                    init=flb.INIT_THERMAL, sample_every=1, block_steps=block))
    L.step(2)
    h = L.populations().reshape(9, -1)
    w = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)
    vx = np.array([0, 1, 0, -1, 0, 1, -1, -1, 1.0])
    f0 = w * (1 + 3 * vx * 0.05 + 4.5 * (vx * 0.05) ** 2 - 1.5 * 0.05 ** 2)
    h = h - f0[:, None]
    L.reset_stats()
    L.step(1)
    for _ in range(2):  # reading leaves the sums as they are
        c = L.covariance()
        assert c["nsamples"] == nx * ny and c["nblocks"] == block
        mean = h.mean(1)
        cov = h @ h.T / (nx * ny) - np.outer(mean, mean)
        assert np.abs(c["mean_df"] - mean).max() <= 1e-11 * np.sqrt(cov.max())
        assert np.abs(c["cov_f"] - cov).max() <= 1e-11 * cov.max()
    L.close()
