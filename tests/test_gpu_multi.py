"""Several steps per launch (small lattices) against one step per launch: a
forced launch shape makes a lattice take single steps, and everything has to
be the same bit for bit: populations, correlator sums, time blocks,
structure factors, the step of an error.  Sides at the edges of the kernel's
tiles and halos (narrower than a halo, one wavefront wide and its
neighbours, several tiles with a ragged last one)."""
import numpy as np
import pytest

from paper_1204_6734_amd import inputs as I

pytestmark = pytest.mark.gpu

SIDES = [(3, 3), (5, 4), (21, 21), (32, 32), (33, 7), (63, 9), (64, 64), (65, 5), (70, 22),
         (127, 3), (130, 61), (256, 40), (300, 33)]


def pair(flb, nx, ny, stream=None, **kw):
    a = flb.Lattice(flb.make_params(nx, ny, **kw))
    b = flb.Lattice(flb.make_params(nx, ny, **kw))
    b.set_launch(1, 0)
    return a, b


def same(a, b, sk=False):
    np.testing.assert_array_equal(a.populations(), b.populations())
    ca, cb = a.covariance(), b.covariance()
    for k, v in ca.items():
        np.testing.assert_array_equal(v, cb[k], err_msg=k)
    if sk:
        for w in range(5):
            np.testing.assert_array_equal(a.structure_factor(w), b.structure_factor(w))


@pytest.mark.parametrize("nx,ny", SIDES)
@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp32 fast flow"])
def test_several_steps_equal_single_steps(flb, nx, ny, prec):
    kw = dict(precision=flb.FP64 if prec == "fp64" else flb.FP32_SHIFTED,
              ux0=0.3 if "fast" in prec else 0.1, uy0=-0.03, kT=1e-4, seed=nx + ny,
              init=flb.INIT_THERMAL)
    # no samples, one relaxation time
    a, b = pair(flb, nx, ny, **kw)
    for n in (4, 2, 9, 8, 23):
        a.step(n)
        b.step(n)
        np.testing.assert_array_equal(a.populations(), b.populations())
    # samples of every step and every third, blocks that end inside launches
    for every, block in ((1, 7), (3, 4)):
        a, b = pair(flb, nx, ny, tau=I.mixed_taus(2), sample_every=every, block_steps=block,
                    **kw)
        for n in (12, 5, 32):
            a.step(n)
            b.step(n)
            same(a, b)


@pytest.mark.parametrize("basis", [0, 1, 2])
@pytest.mark.parametrize("nx,ny", [(32, 32), (96, 40)])
def test_structure_factors_and_graphs(flb, basis, nx, ny):
    for prec in (flb.FP64, flb.FP32_SHIFTED):
        for sk in (10, 5, 2):
            kw = dict(precision=prec, basis=basis, ux0=0.1, kT=1e-4, seed=3, sample_every=2,
                      sk_every=sk, block_steps=9)
            a, b = pair(flb, nx, ny, **kw)
            g = flb.Lattice(flb.make_params(nx, ny, **kw))
            g.set_graph_chunk(20)
            for n in (30, 7, 43, 40):
                for L in (a, b, g):
                    L.step(n)
                same(a, b, sk=True)
                same(g, b, sk=True)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_ensembles(flb, prec):
    """Replicas of both compute classes, replayed and eager."""
    ps = [flb.make_params(70, 18, precision=flb.FP64 if prec == "fp64" else flb.FP32_SHIFTED,
                          ux0=u, kT=1e-4, seed=9 + k, sample_every=5, block_steps=4)
          for k, u in enumerate([0.1, 0.3, 0.0, 0.27])]
    one = flb.Ensemble(ps)
    one.set_launch(1, 0)
    for chunk in (0, 10):
        E = flb.Ensemble(ps, graph_chunk=chunk)
        E.step(93)
        if chunk == 0:
            one.step(93)
        for i in range(len(ps)):
            np.testing.assert_array_equal(E.populations(i), one.populations(i))
            ce, co = E.covariance(i), one.covariance(i)
            for k, v in ce.items():
                np.testing.assert_array_equal(v, co[k], err_msg=k)


def test_replicas_in_two_graph_branches_equal_alone(flb):
    """Enough tiles that a captured chunk advances two halves side by side
    (and, with an odd count, unequal ones), in both compute classes."""
    ps = [flb.make_params(128, 120, ux0=0.3 if k % 7 == 3 else 0.01 * k, kT=1e-4, seed=k,
                          sample_every=3, block_steps=5) for k in range(35)]
    E = flb.Ensemble(ps, graph_chunk=12)
    for n in (24, 7, 29):  # replays between eager steps
        E.step(n)
        E.sync()
    for i in (0, 3, 16, 17, 18, 34):
        L = flb.Lattice(ps[i])
        L.step(60)
        np.testing.assert_array_equal(E.populations(i), L.populations())
        ce, cl = E.covariance(i), L.covariance()
        for k, v in ce.items():
            np.testing.assert_array_equal(v, cl[k], err_msg=k)


def test_an_error_has_the_same_step(flb):
    kw = dict(precision=flb.FP32_SHIFTED, kT=0.05, seed=7, init=flb.INIT_THERMAL)
    a, b = pair(flb, 40, 40, **kw)
    for L in (a, b):
        L.step(60)
        with pytest.raises(flb.FlbError) as e:
            L.sync()
        assert e.value.code == flb.E_INVALID_VELOCITY
    assert a.error_step == b.error_step


@pytest.mark.parametrize("prec,side,n", [("fp32", 32, 24), ("fp32", 32, 32), ("fp32", 32, 64),
                                         ("fp32", 21, 80), ("fp32", 128, 4), ("fp64", 12, 9), ("fp64", 16, 11), ("fp64", 32, 16),
                                         ("fp64", 32, 32), ("fp64", 21, 40)])
def test_fewer_steps_as_the_chip_fills(flb, prec, side, n):
    """Tile counts at which a launch goes from six or four steps to two and to
    one, with the sums of every third step between the launches."""
    ps = [flb.make_params(side, side, precision=flb.FP64 if prec == "fp64" else flb.FP32_SHIFTED,
                          ux0=0.1, kT=1e-4, seed=k, sample_every=3 * (k % 2), block_steps=5)
          for k in range(n)]
    a, b = flb.Ensemble(ps), flb.Ensemble(ps)
    b.set_launch(1, 0)
    for steps in (13, 28):
        a.step(steps)
        b.step(steps)
    for i in (0, 1, n - 1):
        np.testing.assert_array_equal(a.populations(i), b.populations(i))
        if i % 2:
            ca, cb = a.covariance(i), b.covariance(i)
            for k, v in ca.items():
                np.testing.assert_array_equal(v, cb[k], err_msg=k)
