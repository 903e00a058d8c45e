"""Readouts through page-locked staging: pieces around the sizes where the
staging changes (small area, straight, two halves filled in turn), several
readouts in a row, and from several threads at once."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# 9 nx ny doubles: below, at and above 256 KiB; above 8 and 16 MiB; 37 MB
@pytest.mark.parametrize("nx,ny", [(10, 7), (64, 56), (64, 57), (64, 58), (400, 300), (500, 480),
                                   (1000, 520)])
def test_whole_readout_equals_row_readouts(flb, nx, ny):
    L = flb.Lattice(flb.make_params(nx, ny, precision=flb.FP64, ux0=0.1, kT=1e-4, seed=nx,
                                    init=flb.INIT_THERMAL, sample_every=1))
    L.step(3)
    rows = np.concatenate([L.rows(y, min(37, ny - y)) for y in range(0, ny, 37)], axis=1)
    for _ in range(3):
        np.testing.assert_array_equal(L.populations(), rows)
        blob = L.checkpoint()
    L.step(2)
    L.restore(blob)
    np.testing.assert_array_equal(L.populations(), rows)
    L.close()


@pytest.mark.parametrize("nx,ny", [(21, 21), (32, 9), (9, 64), (64, 33)])
def test_structure_factors_are_symmetric(flb, nx, ny):
    L = flb.Lattice(flb.make_params(nx, ny, precision=flb.FP64, ux0=0.1, kT=1e-4, seed=5,
                                    init=flb.INIT_THERMAL, sk_every=1))
    L.step(4)
    for w in range(5):
        s = L.structure_factor(w)
        m = np.roll(s[::-1, ::-1], (1, 1), (0, 1))  # the value at -k
        own = np.ones((ny, nx), bool)
        own[:, 0] = False
        if nx % 2 == 0:
            own[:, nx // 2] = False
        np.testing.assert_array_equal(s[own], -m[own] if w == flb.SK_JXJY_IM else m[own])
    L.close()


@pytest.mark.parametrize("nx,ny", [(8, 8), (8, 2048), (16, 64), (512, 8), (512, 1024), (128, 30),
                                   (1024, 16), (64, 4)])
@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_structure_factors_equal_numpy(flb, nx, ny, prec):
    """One sample of a known state at the edges of the transforms' ranges:
    the two-kernel one takes powers of two up to 512 x 2048."""
    fp64 = prec == "fp64"
    L = flb.Lattice(flb.make_params(nx, ny, precision=flb.FP64 if fp64 else flb.FP32_SHIFTED,
                                    ux0=0.1, uy0=-0.02, kT=1e-4, seed=9, init=flb.INIT_THERMAL,
                                    sk_every=1))
    L.step(2)
    f = L.populations()
    L.reset_stats()
    L.step(1)
    vx = np.array([0, 1, 0, -1, 0, 1, -1, -1, 1.0])
    vy = np.array([0, 0, 1, 0, -1, 1, 1, -1, -1.0])
    r = f.sum(0) - 1.0
    jx = np.tensordot(vx, f, 1) - 0.1
    jy = np.tensordot(vy, f, 1) + 0.02
    a, b, c = (np.fft.fft2(x) for x in (r, 3 ** .5 * (jx - 0.1 * r), 3 ** .5 * (jy + 0.02 * r)))
    x = b * c.conj()
    want = [abs(a) ** 2, abs(b) ** 2, abs(c) ** 2, x.real, x.imag]
    # FP32: fields and transform carry 2^-24 each, ~log2(n) roundings of the
    # transform; squares double it.  FP64 the same with 2^-53 (and the fields'
    # difference from 1: 2^-53 of 1 against fluctuations of 1e-2).
    tol = 1e-11 if fp64 else 5e-6
    for w in range(5):
        got = L.structure_factor(w) * (nx * ny)
        assert np.abs(got - want[w]).max() <= tol * max(np.abs(want[k]).max() for k in (0, 1, 2))
    L.close()


def test_readouts_from_several_threads(flb):
    """Threads reading their own lattices share the staging or copy straight."""
    lats = [flb.Lattice(flb.make_params(300 + 40 * k, 200, kT=1e-4, seed=k, ux0=0.02 * k,
                                        init=flb.INIT_THERMAL, sample_every=1))
            for k in range(4)]
    want = []
    for L in lats:
        L.step(5)
        want.append((L.populations(), L.covariance()["cov_f"]))
    bad = []

    def work(k):
        for _ in range(10):
            f, c = lats[k].populations(), lats[k].covariance()["cov_f"]
            if not (np.array_equal(f, want[k][0]) and np.array_equal(c, want[k][1])):
                bad.append(k)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


@pytest.mark.parametrize("lattice,blocks", [("d2q9", 500), ("d2q9", 700), ("d2q9", 1023),
                                            ("d3q19", 150), ("d3q19", 600), ("d3q19", 1023)])
def test_correlators_behind_steps_equal_those_after_a_wait(flb, lattice, blocks):
    """Closed blocks below and above 256 KiB, read while their steps run."""
    def make():
        if lattice == "d2q9":
            return flb.Lattice(flb.make_params(16, 12, kT=1e-4, seed=3, init=flb.INIT_THERMAL,
                                               sample_every=1, block_steps=1))
        return flb.Lattice3(flb.make_params3(8, 5, 4, kT=1e-4, seed=3, sample_every=1,
                                             block_steps=1))

    a, b = make(), make()
    for _ in range(3):
        a.step(blocks // 3)
        b.step(blocks // 3)
        b.sync()
        got, want = a.covariance(), b.covariance()
        assert got["nblocks"] == want["nblocks"] > 0
        for k in want:
            np.testing.assert_array_equal(got[k], want[k])
