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


# 2 and 6 cells per thread in 2D; 2, 4, 6, 8, 10, 12, 16 and 20 in 3D
WAIT_SIZES = [(96, 77), (400, 400), (24, 20, 12), (50, 49, 47), (53, 52, 50), (66, 61, 50), (66, 81, 48), (71, 70, 70),
              (73, 72, 72), (79, 77, 80)]


@pytest.mark.parametrize("polls", [0, 1, 6, 1 << 21])
@pytest.mark.parametrize("n", WAIT_SIZES)
def test_workgroups_that_give_up_leave_a_solved_field(n, polls):
    """With no poll every workgroup gives up at its first wait; with a few some get
    further than others. The field is then solved by one workgroup: the oracle's iterates
    within the rounding that the several-workgroup solve (with polls enough) is held to."""
    from oracle import walls as W
    from paper_2604_18536_amd import Solver
    from paper_2604_18536_amd import _lib as L
    from tests.gpu_util import host, max_rel

    lo, hi = S.channel_box(n)
    h = S.spacing(n, lo, hi)
    s = Solver(n, batch=2, nu=0.01, lo=lo, hi=hi, bc="walls", pressure="cg")
    L.call("ins_cg_set_wait", s._ctx, polls)
    r = np.stack([S.random_scalar(n, 7), S.random_scalar(n, 8)])
    for k in (1, 7):
        s.cg_set(rtol=0.0, maxiter=k, check_every=0)
        x = host(s.poisson_solve(dev(r)))
        for b in range(2):
            xo, ito, rel = W.cg_solve(r[b], h, rtol=0.0, maxiter=k)
            assert max_rel(x[b], xo) < 1e-11
        assert s.cg_info()[0] == k
    s.cg_set(rtol=1e-9, maxiter=5000)
    s.poisson_solve(dev(r))
    assert 0.0 < s.cg_info()[1] <= 1e-9
    s.close()


@pytest.mark.parametrize("n,walls", [((70, 63), False), ((42, 35, 20), False), ((42, 35, 20), True)])
def test_workgroups_that_give_up_on_a_stretched_grid(n, walls):
    from oracle import stretched as ST
    from paper_2604_18536_amd import Solver
    from paper_2604_18536_amd import _lib as L
    from tests.gpu_util import host, max_rel

    lo, hi = [0.0] * len(n), [2.0] * len(n)
    faces = [S.tanh_faces(n[a], lo[a], hi[a], 0.8 + 0.2 * a) for a in range(len(n))]
    s = Solver(n, nu=0.01, lo=lo, hi=hi, bc="walls" if walls else "periodic")
    for a, f in enumerate(faces):
        s.set_faces(a, f)
    L.call("ins_cg_set_wait", s._ctx, 0)
    o = ST.StretchedGrid(faces, ywalls=walls)
    r = S.random_scalar(n, 3)
    for k in (1, 7):
        s.cg_set(rtol=0.0, maxiter=k, check_every=0)
        x = host(s.poisson_solve(dev(r)))
        xo, ito, rel = o.cg_solve(r, rtol=0.0, maxiter=k)
        assert max_rel(x, xo) < 1e-11 and s.cg_info()[0] == k
        assert abs(s.cg_info()[1] - rel) <= 1e-10 * rel
    # waits as long as it takes: the usual solve
    L.call("ins_cg_set_wait", s._ctx, 1 << 21)
    x = host(s.poisson_solve(dev(r)))
    assert max_rel(x, xo) < 1e-11
    s.close()
