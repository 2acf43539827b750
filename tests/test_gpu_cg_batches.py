"""Batches of fields solved by the single-launch conjugate gradients: side by side on the
whole chip, in several launches where it does not hold all of them, from two streams at
once, and replayed from graphs. Every field must be, bit for bit, the field alone."""
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


def _solver(n, batch):
    from paper_2604_18536_amd import Solver

    lo, hi = S.channel_box(n)
    s = Solver(n, batch=batch, lo=lo, hi=hi, bc="walls", pressure="cg")
    s.cg_set(rtol=0.0, maxiter=30, check_every=0)
    return s


# (sizes, batch): one launch and several, the last one partly filled; 2, 4, 8 and 20 cells per thread
BATCHES = [((17, 17, 17), 150), ((128, 128), 33), ((41, 40, 40), 7), ((70, 63, 54), 6), ((79, 77, 80), 5)]


@pytest.mark.parametrize("n,batch", BATCHES)
def test_fields_of_a_batch_are_those_alone(n, batch):
    few = [S.random_scalar(n, 8 + b) for b in range(3)]
    r = dev(np.stack([few[b % 3] for b in range(batch)]))
    s, one = _solver(n, batch), _solver(n, 1)
    a = s.poisson_solve(r)
    alone = [one.poisson_solve(dev(f)) for f in few]
    for b in range(batch):
        assert torch.equal(a[b], alone[b % 3]), b
    s.close()
    one.close()


def test_solves_on_two_streams_at_once():
    n, batch = (70, 63, 54), 4  # each launch fills the chip
    r = dev(np.stack([S.random_scalar(n, 8 + b) for b in range(batch)]))
    s = [_solver(n, batch) for _ in range(2)]
    ref = s[0].poisson_solve(r)
    out = [[torch.empty_like(r) for _ in range(3)] for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for k in range(3):
        for i in range(2):
            with torch.cuda.stream(streams[i]):
                s[i].poisson_solve(r, out=out[i][k])
    torch.cuda.synchronize()
    for i in range(2):
        for k in range(3):
            assert torch.equal(out[i][k], ref), (i, k)
        s[i].close()


@pytest.mark.parametrize("n,batch", [((17, 17, 17), 60), ((70, 63, 54), 5)])
def test_batches_replay_from_a_graph(n, batch):
    """Several replays, with eager solves and host work between them."""
    s = _solver(n, batch)
    r = dev(np.stack([S.random_scalar(n, 8 + b % 3) for b in range(batch)]))
    ref = s.poisson_solve(r)
    x = torch.empty_like(r)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        s.poisson_solve(r, out=x)
    for rep in range(3):
        x.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(x, ref), rep
        assert torch.equal(s.poisson_solve(r), ref)
    s.close()
