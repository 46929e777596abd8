"""Two steps per sweep on the planes layout (pull lattices of 4 GiB and more): the bits of
single steps, and in FP64 the oracle.  The start repeats a smaller box along every
axis, so the oracle evolves that one."""
import numpy as np
import pytest

from paper_1507_02518_amd import inputs, kbc

pytestmark = pytest.mark.gpu


# rows of whole 64 bytes (the last tile half empty in y); every plane at an odd
# node; FP32 with the longest rows that take pairs, the last tile partly empty
@pytest.mark.parametrize("small,times,dtype,variant", [
    ((72, 69, 64), 4, kbc.F64, kbc.S_DTQ), ((91, 91, 91), 3, kbc.F64, kbc.S_CDTQ),
    ((88, 87, 90), 4, kbc.F32_DEV, kbc.S_DTQ)])
def test_pairs_on_planes(orc, small, times, dtype, variant):
    shape = tuple(times * n for n in small)
    nodes = shape[0] * shape[1] * shape[2]
    assert 27 * nodes * (8 if dtype == kbc.F64 else 4) >= 1 << 32
    print(f"pairs on planes {shape} dtype={dtype} variant={variant}", flush=True)
    us = inputs.smooth_random(small, 0.04, seed=5)
    u = np.tile(us, (1, times, times, times))
    rng = np.random.default_rng(2)
    at = np.concatenate([[0, shape[0] - 1, nodes - 1, nodes - shape[0]], rng.integers(0, nodes, 100000)])
    nu, steps = 1e-2, 5
    got = []
    for single in (False, True):
        with kbc.Box(shape, nu, dtype, variant=variant) as b:
            b.init_velocity(u)
            if single:
                for _ in range(steps):
                    b.step(1)
            else:
                b.step(steps)      # two pairs and a single step
            got.append((b.sample(at), *b.moments()))
    for a, c in zip(*got):
        assert np.array_equal(a, c)
    if dtype == kbc.F64:
        F = orc.run(orc.init_feq(us), orc.beta_from_nu(nu), steps, variant=variant)
        x, y, z = at % shape[0], at // shape[0] % shape[1], at // (shape[0] * shape[1])
        ref = F[:, z % small[2], y % small[1], x % small[0]].T
        # the bound of the ragged-box parity tests
        assert np.abs(got[0][0] - ref).max() <= 1e-13
