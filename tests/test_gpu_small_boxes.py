"""The workgroup of a step follows the box: one wavefront, two or four.  Boxes
on both sides of each line (64 and 128 nodes for each of 256 CUs), with ragged
last workgroups, against the oracle."""
import numpy as np
import pytest

from paper_1507_02518_amd import inputs, kbc
from paper_1507_02518_amd.kbc import AA, F32_DEV_X, F64, PULL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(64, 16, 16), (65, 9, 28), (5, 29, 113), (128, 16, 16), (33, 32, 31),
                                   (300, 10, 11), (3, 105, 105)])
@pytest.mark.parametrize("streaming", [PULL, AA])
@pytest.mark.parametrize("variant", [kbc.S_DTQ, kbc.S_CD])
def test_small_boxes_match_oracle(orc, shape, streaming, variant):
    u = inputs.smooth_random(shape, 0.03, seed=4)
    nu, steps = 2e-2, 5
    F = orc.run(orc.init_feq(u), orc.beta_from_nu(nu), steps, variant=variant)
    with kbc.Box(shape, nu, F64, streaming=streaming, variant=variant) as b:
        b.init_velocity(u)
        b.step(steps)
        f = b.populations()
    # the bound of the ragged-box parity tests
    assert np.abs(f - F).max() <= 1e-13
    with kbc.Box(shape, nu, F32_DEV_X, streaming=streaming, variant=variant) as b:
        b.init_velocity(u)
        b.step(steps)
        f = b.populations()
    # five roundings to FP32 of deviations below 0.03 (each 2^-25 of it), and
    # FP32 relaxation of a non-equilibrium that is smaller still
    assert np.abs(f - F).max() <= 5e-8
