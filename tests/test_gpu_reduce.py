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


def test_requests_that_close_together(flb):
    """More requests than one launch lists, of tile counts on both sides of
    one range per tile, closing at the same steps and at their own: each
    request's correlators are its lattice's."""
    ps = []
    for k in range(70):
        tiles = [1, 5, 255, 256, 257, 300, 600][k % 7]
        ps.append(flb.make_params(50 + k % 5, 4 * tiles - 1, ux0=0.3 if k % 9 == 4 else 0.05,
                                  kT=1e-4, seed=k, sample_every=1 + k % 2,
                                  block_steps=3 + (k % 10 == 9)))
    S = flb.Server(256 << 20, max_slots=70, chunk_steps=8, threaded=False)
    for k, p in enumerate(ps):
        S.submit(p, 30, tag=k)
    S.drain()
    res = {r["tag"]: r for r in S.poll(80)}
    S.close()
    assert len(res) == len(ps)
    for k, p in enumerate(ps):
        L = flb.Lattice(p)
        L.step(30)
        want, got = L.covariance(), res[k]["cov"]
        L.close()
        assert got["nblocks"] == want["nblocks"] > 0
        for key in ("mean_df", "cov_f", "se_cov_f"):
            np.testing.assert_array_equal(got[key], want[key], err_msg="%d %s" % (k, key))
