"""FP64 D3Q19 steps on both sides of one tile per compute unit (256), where
the launcher goes over to two wavefronts per SIMD for one relaxation time and
for steps with sums, against the oracle: populations to 1e-12 of the largest
after every step (both phases), the sums of all steps to 1e-10, the bounds of
the smaller lattices' tests (each sum has fewer than 1e5 terms: n eps = 2e-11 of
its absolute terms at most)."""
import numpy as np
import pytest

from oracle import d3q19 as D
from test_gpu_d3q19 import TAUS, perturbed

pytestmark = pytest.mark.gpu

# rows and columns that leave lanes and wavefronts of every tile empty
TILES = {256: (13, 5, 128), 258: (13, 5, 129), 270: (40, 33, 30)}


@pytest.mark.parametrize("tiles", sorted(TILES))
@pytest.mark.parametrize("basis", [0, 1])
@pytest.mark.parametrize("tau", ["one", "mixed"])
@pytest.mark.parametrize("every", [0, 1, 2])
def test_fp64_steps_match_oracle(flb, tiles, basis, tau, every):
    nx, ny, nz = TILES[tiles]
    assert -(-nx // 64) * -(-ny // 4) * nz == tiles
    kw = dict(ux0=0.1, uy0=-0.05, uz0=0.03, kT=1e-4, seed=tiles + every,
              tau=TAUS if tau == "mixed" else (0.8,) * 15, sample_every=every)
    # the library's blocks are counted in samples, the oracle's in steps
    g = flb.Lattice3(flb.make_params3(nx, ny, nz, precision=flb.FP64, basis=basis, block_steps=2,
                                      **kw))
    o = D.Lattice(D.make_params(nx, ny, nz, basis=basis, block_steps=2 * every, **kw))
    f = perturbed(nx, ny, nz, (0.1, -0.05, 0.03), seed=4)
    g.set_populations(f)
    o.set_populations(f)
    for n in (1, 1, 3) if tiles < 270 else (1, 1):
        g.step(n)
        o.step(n)
        fg, fo = g.populations(), o.populations()
        assert np.abs(fg - fo).max() <= 1e-12 * np.abs(fo).max(), o.t
    if every:
        cg, co = g.covariance(), o.covariance()
        assert cg["nsamples"] == co["nsamples"] > 0 and cg["nblocks"] == co["nblocks"]
        for k in ("mean_df", "cov_f"):
            assert np.abs(cg[k] - co[k]).max() <= 1e-10 * np.abs(co[k]).max(), k
    g.close()
