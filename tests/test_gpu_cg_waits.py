"""What a conjugate-gradient solve reports and returns when it does not end as it should:
a residual that overflows, and workgroups that give up waiting for each other."""
import math

import numpy as np
import pytest
import torch

import synth as S
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# one workgroup, several, the two-kernel iteration
@pytest.mark.parametrize("n", [(20, 18), (24, 20, 12), (99, 91, 95)])
def test_a_residual_that_is_not_a_number_is_reported(n):
    """||res_0||^2 of values around 1e200 overflows, so relres = inf / inf: the solve does
    not iterate and must not read as converged, whichever field of the batch it was."""
    from paper_2604_18536_amd import Solver

    lo, hi = S.channel_box(n)
    s = Solver(n, batch=3, lo=lo, hi=hi, bc="walls", pressure="cg")
    for bad in range(3):
        r = np.stack([S.random_scalar(n, 8 + b) for b in range(3)])
        r[bad] *= 1e200
        s.poisson_solve(dev(r))
        assert math.isnan(s.cg_info()[1]), bad
    s.poisson_solve(dev(np.stack([S.random_scalar(n, 8 + b) for b in range(3)])))
    assert 0.0 < s.cg_info()[1] <= 1e-10
    s.close()
