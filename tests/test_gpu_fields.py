"""Density, velocity and the sums over nodes at the sizes where their kernels
can go wrong: fewer nodes than a wavefront, a partial last run, more runs
than groups, tiles and column marches with remainders, axes shorter than a
derivative's reach, and every lag tiling of the x-correlation."""
import ctypes

import numpy as np
import pytest

from oracle import statistics as ost
from paper_1507_02518_amd import inputs, kbc
from paper_1507_02518_amd.kbc import AA, F16_DEV, F32_DEV, F32_DEV_X, F64, PULL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (5, 3, 2), (70, 9, 33), (33, 16, 65), (64, 64, 66)])
@pytest.mark.parametrize("dtype,streaming,steps", [
    (F64, PULL, 3), (F64, AA, 2), (F64, AA, 3), (F32_DEV, PULL, 2), (F32_DEV_X, AA, 3),
    (F16_DEV, AA, 2), (F16_DEV, PULL, 3)])
def test_fields_and_sums_match_oracle(orc, shape, dtype, streaming, steps):
    with kbc.Box(shape, 2e-3, dtype, streaming=streaming) as b:
        b.init_velocity(inputs.smooth_random(shape, 0.05, seed=3))
        b.step(steps)
        f = b.populations()
        if not np.isfinite(f).all():    # a box this small and rough leaves FP16's range
            for call in (b.moments, b.energy, b.enstrophy):
                with pytest.raises(kbc.KbcError) as e:
                    call()
                assert e.value.code == kbc.KBC_EUNSTABLE
            return
        rho, u = b.moments()
        k, w2 = b.energy(), b.enstrophy()
    orho, ou = orc.macros(f)
    # two sums of 27 terms below 0.3 and, for the deviation forms, one more
    # rounding of each population: below 27 * 2^-54 each
    assert np.abs(rho - orho).max() <= 4e-15 and np.abs(u - ou).max() <= 4e-15
    # sums over nodes of the same u, 64-bit: 1e-12 of the value, and the
    # rounding of u itself where the flow is uniform
    assert k == pytest.approx(orc.energy(u), rel=1e-12, abs=1e-30)
    assert w2 == pytest.approx(orc.enstrophy(u), rel=1e-12, abs=1e-28)


@pytest.mark.parametrize("shape", [(5, 3, 2), (70, 9, 33), (64, 64, 66)])
def test_energy_keeps_its_digits_on_a_mean_flow(shape):
    """Perturbations of 1e-6 on a uniform flow of 0.1: u is rounded at 1.4e-17
    and kept to a few of these, 1e-10 of the perturbation."""
    u0 = inputs.smooth_random(shape, 1e-6, seed=5)
    u0 += np.array([0.1, -0.07, 0.05])[:, None, None, None]
    with kbc.Box(shape, 2e-3) as b:
        b.init_velocity(u0)
        b.step(1)
        k, (_, u) = b.energy(), b.moments()
    d = u.astype(np.longdouble).reshape(3, -1)
    d = d - d.mean(axis=1, keepdims=True)
    assert k == pytest.approx(float(0.5 * (d * d).sum(axis=0).mean()), rel=1e-10)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("node", [0, 63, 64, 70 * 9 * 33 - 1])
def test_one_node_that_is_not_finite_is_reported(orc, bad, node):
    shape = (70, 9, 33)
    f = orc.init_feq(inputs.smooth_random(shape, 0.05, seed=3))
    f.reshape(27, -1)[13, node] = bad      # the population at rest: the velocity may stay finite
    with kbc.Box(shape, 2e-3) as b:
        b.set_populations(f)
        for call in (b.energy, b.moments, b.enstrophy):
            with pytest.raises(kbc.KbcError) as e:
                call()
            assert e.value.code == kbc.KBC_EUNSTABLE


@pytest.mark.parametrize("order", [2, 8])
@pytest.mark.parametrize("shape", [(3, 2, 5), (33, 9, 33), (64, 17, 32), (31, 8, 70)])
def test_gradient_statistics_on_ragged_tiles(shape, order):
    with kbc.Box(shape, 2e-3) as b:
        b.init_velocity(inputs.smooth_random(shape, 0.05, seed=9))
        b.step(2)
        got = b.statistics(order)
        _, u = b.moments()
    ref = ost.statistics(u, 2e-3, order)
    for key in ("k", "omega", "epsilon", "div2"):
        assert got[key] == pytest.approx(ref[key], rel=1e-12), key
    for n in range(2, 7):
        # odd moments cancel: their rounding is that of the terms
        scale = ref["dudx_moments"][2] ** (n / 2)
        assert got["dudx_moments"][n] == pytest.approx(ref["dudx_moments"][n], rel=1e-11,
                                                       abs=1e-11 * scale), n


@pytest.mark.parametrize("shape,rmax", [
    ((1, 5, 3), 0), ((5, 3, 2), 4), ((13, 70, 3), 12), ((40, 12, 10), 0), ((64, 16, 130), 7),
    ((64, 16, 5), 8), ((600, 3, 2), 599), ((1100, 2, 1), 1030)])
def test_correlation_tilings_match_oracle(shape, rmax):
    with kbc.Box(shape, 2e-3) as b:
        u0 = inputs.smooth_random(shape, 0.05, seed=21)
        b.init_velocity(u0)
        b.step(1)
        r11, r22 = b.correlation(rmax)
        _, u = b.moments()
    o11, o22 = ost.correlation_x(u, rmax)
    assert np.abs(r11 - o11).max() < 1e-13 and np.abs(r22 - o22).max() < 1e-13


@pytest.mark.parametrize("shape", [(5, 3, 2), (70, 9, 33), (48, 20, 36)])
@pytest.mark.parametrize("n", [1, 2, 17, 20])
@pytest.mark.parametrize("dtype,streaming,variant", [
    (F64, PULL, kbc.S_DTQ), (F64, AA, kbc.S_CDT), (F32_DEV, PULL, kbc.S_DQ), (F32_DEV_X, AA, kbc.S_D),
    (F16_DEV, AA, kbc.S_DTQ), (F16_DEV, PULL, kbc.S_CDTQ)])
def test_series_is_the_energy_after_each_step(shape, n, dtype, streaming, variant):
    _check_series(shape, n, dtype, streaming, variant)


@pytest.mark.parametrize("dtype,streaming,variant", [
    (F64, PULL, kbc.S_DTQ), (F64, AA, kbc.S_CD), (F32_DEV, PULL, kbc.S_CDTQ), (F32_DEV, AA, kbc.S_DTQ),
    (F32_DEV_X, PULL, kbc.S_D), (F32_DEV_X, AA, kbc.S_CDT)])
def test_steps_that_store_through_the_caches_give_the_same_bits(dtype, streaming, variant):
    """Lattices between the L2s' and the last-level cache's size: the single
    steps store through the caches, those of the series past them."""
    _check_series((97, 64, 80), 5, dtype, streaming, variant)


def test_series_with_fewer_states_at_once():
    """A box large enough that its states are added up in smaller numbers."""
    _check_series((192, 160, 132), 21, F32_DEV, AA, kbc.S_DTQ)


def _check_series(shape, n, dtype, streaming, variant):
    u = inputs.smooth_random(shape, 0.02, seed=3)
    ks = np.empty(n)
    with kbc.Box(shape, 2e-2, dtype, streaming=streaming, variant=variant) as b:
        b.init_velocity(u)
        b.step(1)
        rc = kbc.load().kbc_energy_series(b.h, n, ks.ctypes.data_as(ctypes.POINTER(ctypes.c_double)))
        t, f = b.t, b.populations()
    kr = np.full(n, np.nan)     # where the state has left the range of FP16
    with kbc.Box(shape, 2e-2, dtype, streaming=streaming, variant=variant) as b:
        b.init_velocity(u)
        b.step(1)
        for j in range(n):
            b.step(1)
            try:
                kr[j] = b.energy()
            except kbc.KbcError as e:
                assert e.code == kbc.KBC_EUNSTABLE
        g = b.populations()
    good = np.isfinite(kr)
    assert dtype == F16_DEV or good.all()
    assert rc == (kbc.KBC_OK if good.all() else kbc.KBC_EUNSTABLE)
    # the same bits
    assert t == n + 1 and np.array_equal(ks[good], kr[good])
    assert np.array_equal(f, g, equal_nan=True)
