"""Ensembles beyond the last-level cache whose steps without sums use another
tile shape than those with: every member is bit for bit its own lattice."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,n,chunk", [(256, 99, 350, 0), (256, 99, 350, 12),
                                           (1000, 63, 130, 12)])
def test_members_equal_lattices(flb, nx, ny, n, chunk):
    ps = [flb.make_params(nx, ny, ux0=0.3 if k % 9 == 4 else 0.0003 * k, kT=1e-4, seed=k,
                          sample_every=3 * (k % 2), block_steps=4) for k in range(n)]
    E = flb.Ensemble(ps, graph_chunk=chunk)
    for steps in (12, 7, 29):
        E.step(steps)
    for k in (0, 4, 13, n // 2, n - 1):
        L = flb.Lattice(ps[k])
        L.set_launch(1, 0)
        L.step(48)
        np.testing.assert_array_equal(E.populations(k), L.populations())
        ce, cl = E.covariance(k), L.covariance()
        for key, v in ce.items():
            np.testing.assert_array_equal(v, cl[key], err_msg=key)
        L.close()
    E.close()
