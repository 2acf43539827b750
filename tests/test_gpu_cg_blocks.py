"""Single-launch conjugate-gradient solve: every split of a field over threads and
workgroups (and the two-kernel iteration of fields that do not fit) vs the oracle's CG
iterates, on the channel and on grids stretched in every direction."""
import numpy as np
import pytest
import torch

import synth as S
from oracle import stretched as ST
from oracle import walls as W
from tests.gpu_util import dev, host, max_rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# one workgroup: 256 and 512 threads, full and partial runs; several workgroups: 2, 4, 8,
# 10 and 20 cells per thread, blocks that divide the grid and that do not, one
# block across a direction; too large: the two-kernel iteration
CHANNEL = [(33, 5, 7), (16, 16, 16), (64, 64), (1, 30), (66, 63), (300, 41), (4, 1100), (24, 20, 12), (33, 31, 29),
           (50, 49, 47), (66, 61, 50), (66, 81, 48), (71, 66, 60), (79, 77, 80), (99, 91, 95)]


@pytest.mark.parametrize("n", [n for n in CHANNEL if n[0] > 1])
def test_channel_iterates(n):
    from paper_2604_18536_amd import Solver

    lo, hi = S.channel_box(n)
    h = S.spacing(n, lo, hi)
    s = Solver(n, nu=0.01, lo=lo, hi=hi, bc="walls", pressure="cg")
    r = S.random_scalar(n, 7)
    for k in (1, 2, 7):
        s.cg_set(rtol=0.0, maxiter=k, check_every=0)
        x = host(s.poisson_solve(dev(r)))
        xo, ito, rel = W.cg_solve(r, h, rtol=0.0, maxiter=k)
        assert ito == k and s.cg_info()[0] == k
        # the same recurrence from the same r: rounding, grown over k iterations
        assert max_rel(x, xo) < 1e-11
        assert abs(s.cg_info()[1] - rel) <= 1e-10 * rel
    s.close()


@pytest.mark.parametrize("n,walls", [((24, 18), False), ((64, 64), False), ((70, 63), False), ((70, 63), True),
                                     ((16, 14, 10), False), ((42, 35, 20), False), ((42, 35, 20), True)])
def test_stretched_iterates(n, walls):
    from paper_2604_18536_amd import Solver

    lo, hi = [0.0] * len(n), [2.0] * len(n)
    faces = [S.tanh_faces(n[a], lo[a], hi[a], 0.8 + 0.2 * a) for a in range(len(n))]
    s = Solver(n, nu=0.01, lo=lo, hi=hi, bc="walls" if walls else "periodic")
    for a, f in enumerate(faces):
        s.set_faces(a, f)
    o = ST.StretchedGrid(faces, ywalls=walls)
    r = S.random_scalar(n, 3)
    for k in (1, 2, 7):
        s.cg_set(rtol=0.0, maxiter=k, check_every=0)
        x = host(s.poisson_solve(dev(r)))
        xo, ito, rel = o.cg_solve(r, rtol=0.0, maxiter=k)
        assert ito == k and s.cg_info()[0] == k
        assert max_rel(x, xo) < 1e-11
    s.cg_set(rtol=1e-9, maxiter=5000)
    s.poisson_solve(dev(r))
    it, rel = s.cg_info()
    assert abs(it - o.cg_solve(r, rtol=1e-9)[1]) <= 1 and rel <= 1e-9
    s.close()


@pytest.mark.parametrize("n", [(20, 18), (40, 33, 28)])
def test_batch_fields_are_bitwise_those_alone(n):
    from paper_2604_18536_amd import Solver

    lo, hi = S.channel_box(n)
    r = np.stack([S.random_scalar(n, 8 + b) for b in range(3)])
    r[1] = 0.25  # a constant right-hand side: no iteration
    s = Solver(n, batch=3, lo=lo, hi=hi, bc="walls", pressure="cg")
    s.cg_set(rtol=1e-9, maxiter=5000)
    a = s.poisson_solve(dev(r))
    assert not host(a[1]).any()
    one = Solver(n, lo=lo, hi=hi, bc="walls", pressure="cg")
    one.cg_set(rtol=1e-9, maxiter=5000, check_every=0)
    for b in range(3):
        assert torch.equal(one.poisson_solve(dev(r[b])), a[b])
    s.close()
    one.close()
