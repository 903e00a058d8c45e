"""Launches of several steps where the side under test is known to take them
(pass_steps counts the steps), against single steps bit for bit: lattices and
ensembles of both compute classes, structure factors and restarts at odd times
between passes over memory, and the sides of the other tests' cases."""
import numpy as np
import pytest

from paper_1204_6734_amd import inputs as I
from test_gpu_march import HERMITE, SIDES
from test_zz_no_alloc import one_call

pytestmark = pytest.mark.gpu


def same_cov(a, b):
    for k, v in a.items():
        np.testing.assert_array_equal(v, b[k], err_msg=k)


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp32 fast flow"])
@pytest.mark.parametrize("nx,ny", [(3, 3), (5, 4), (12, 12), (16, 15), (17, 9), (21, 21), (31, 3),
                                   (32, 32), (33, 40), (64, 64), (65, 5), (130, 61), (255, 30),
                                   (256, 128)])
def test_lattices_take_several_steps(flb, nx, ny, prec):
    """FP64 collisions do on up to 32 columns, FP32 ones on all these sides."""
    fp64 = prec != "fp32"
    kw = dict(precision=flb.FP64 if prec == "fp64" else flb.FP32_SHIFTED,
              ux0=0.3 if "fast" in prec else 0.1, kT=1e-4, seed=nx, init=flb.INIT_THERMAL,
              tau=I.mixed_taus(2))
    for every, block in ((0, 0), (1, 5), (3, 4)):
        ps = flb.make_params(nx, ny, sample_every=every, block_steps=block, **kw)
        a, b, g = (flb.Lattice(ps) for _ in range(3))
        b.set_launch(1, 0)
        g.set_graph_chunk(12)
        for n in (24, 13, 36):
            for L in (a, b, g):
                L.step(n)
        assert b.pass_steps() == 0
        assert (a.pass_steps() > 20) == (g.pass_steps() > 20) == (not fp64 or nx <= 32)
        for L in (a, g):
            np.testing.assert_array_equal(L.populations(), b.populations())
            same_cov(L.covariance(), b.covariance())


@pytest.mark.parametrize("nx,ny,n", [(21, 18, 4), (32, 32, 6), (12, 9, 11), (5, 7, 20)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("chunk", [0, 20])
def test_ensembles_of_both_compute_classes(flb, nx, ny, n, prec, chunk):
    ps = [flb.make_params(nx, ny, precision=flb.FP64 if prec == "fp64" else flb.FP32_SHIFTED,
                          ux0=[0.1, 0.3, 0.0, 0.27, 0.31][k % 5], kT=1e-4, seed=9 + k,
                          sample_every=[5, 0, 2][k % 3], block_steps=4) for k in range(n)]
    E = flb.Ensemble(ps, graph_chunk=chunk)
    for steps in (40, 13, 40):
        E.step(steps)
    assert E.pass_steps() >= 40
    for i in range(n):
        L = flb.Lattice(ps[i])
        L.set_launch(1, 0)
        L.step(93)
        np.testing.assert_array_equal(E.populations(i), L.populations())
        same_cov(E.covariance(i), L.covariance())


@pytest.mark.parametrize("nx,ny,basis", [(x, y, b) for x, y in SIDES for b in (0, 1, 2)] +
                         [(x, y, 1) for x, y in HERMITE] +
                         [(3000, 2950, 0), (1024, 1024, 1), (4096, 4096, 0)])
def test_large_lattices_take_two_steps_a_pass(flb, nx, ny, basis):
    L = flb.Lattice(flb.make_params(nx, ny, basis=basis, kT=1e-4))
    L.step(5)  # two passes of two, and one step
    assert L.pass_steps() == 4
    L.step(8)  # one step at the odd time, a pair of passes, three steps
    assert L.pass_steps() == 8
    L.sync()


def test_members_take_two_steps_a_pass(flb):
    E = flb.Ensemble([flb.make_params(1003, 1001, ux0=0.01 * m, kT=1e-4, seed=m,
                                      sample_every=6 if m % 2 else 0) for m in range(9)])
    E.step(33)
    assert E.pass_steps() > 8


@pytest.mark.parametrize("nx,ny,basis", [(1024, 1024, 1), (4096, 4096, 0)])
def test_structure_factors_and_odd_restarts_between_passes(flb, nx, ny, basis):
    kw = dict(basis=basis, ux0=0.1, uy0=-0.03, kT=1e-4, seed=4, init=flb.INIT_THERMAL,
              sample_every=12, sk_every=6)
    a, b = flb.Lattice(flb.make_params(nx, ny, **kw)), flb.Lattice(flb.make_params(nx, ny, **kw))
    b.set_launch(1, 0)

    def compare():
        for y in (0, ny // 2 - 20, ny - 40):
            np.testing.assert_array_equal(a.rows(y, 40), b.rows(y, 40))
        for w in range(5):
            np.testing.assert_array_equal(a.structure_factor(w), b.structure_factor(w))
        same_cov(a.covariance(), b.covariance())

    for L in (a, b):
        L.step(25)
    compare()
    blob = a.checkpoint()  # of time 25
    for L in (a, b):
        L.step(14)
        L.restore(blob)
        L.step(22)
    compare()
    if nx == 1024:
        f = a.populations()
        for L in (a, b):
            L.set_populations(f, 33)
            L.step(21)
        compare()
    assert a.pass_steps() >= 28 and b.pass_steps() == 0


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
def test_noalloc_step_across_tile_shapes(flb, prec):
    """256 x 1 tiles in both precisions (FP32 takes them above 65536 sites with
    a full last tile), then 64 x 4."""
    import torch
    precision = flb.FP32_SHIFTED if prec == "fp32" else flb.FP64
    one_call(flb, torch, 1024, 80, precision, 41)
    one_call(flb, torch, 70, 9, precision, 24)
