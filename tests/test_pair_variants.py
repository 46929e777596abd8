"""Two steps per sweep in every variant and with a fixed stabilizer: the bits of single
steps and, in FP64, the oracle."""
import numpy as np
import pytest

from paper_1507_02518_amd import inputs, kbc

pytestmark = pytest.mark.gpu

F64, F32 = kbc.F64, kbc.F32_DEV
ALL = (kbc.S_D, kbc.S_DT, kbc.S_DQ, kbc.S_DTQ, kbc.S_CD, kbc.S_CDT, kbc.S_CDQ, kbc.S_CDTQ)
NATURAL = ALL[:4]


# the shapes take pairs in these variants (test_pair_sweep: 112 x 96 x 33 with the
# dearest one); LBGK and a regularised gamma in one natural and one central variant
CASES = [((112, 96, 33), F64, v, None) for v in ALL] + [((160, 160, 160), F32, v, None) for v in NATURAL]
CASES += [(shape, dtype, v, g) for g in (2.0, 1.3)
          for shape, dtype, v in (((112, 96, 33), F64, kbc.S_DTQ), ((112, 96, 33), F64, kbc.S_CD),
                                  ((160, 160, 160), F32, kbc.S_DT))]


@pytest.mark.parametrize("shape,dtype,variant,gamma", CASES)
def test_pairs_in_every_variant_and_with_fixed_gamma(orc, shape, dtype, variant, gamma):
    print(f"pairs {shape} dtype={dtype} variant={variant} gamma={gamma}", flush=True)
    u = inputs.smooth_random(shape, 0.03, seed=7)
    nu, steps = 1e-2, 2
    got = []
    for runs in ((steps,), (1,) * steps):
        with kbc.Box(shape, nu, dtype, variant=variant, gamma=gamma) as b:
            b.init_velocity(u)
            for n in runs:
                b.step(n)
            got.append(b.populations())
    assert np.array_equal(*got)
    if dtype == F64:
        mode = {} if gamma is None else {"gamma": gamma}
        F = orc.run(orc.init_feq(u), orc.beta_from_nu(nu), steps, variant=variant, **mode)
        # the bound of the ragged-box parity tests
        assert np.abs(got[0] - F).max() <= 1e-13
