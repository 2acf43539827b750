"""z-marches cut into chunks of planes: a field alone and in a large batch is cut
differently (1 to nz chunks); steps and pullbacks of both vs the oracle, and on the
channel vs each other (each within the channel tests' tolerance of the oracle)."""
import pytest
import torch

import oracle as O
import synth as S
from tests.gpu_util import dev, host, max_rel
from tests.test_gpu_channel_fft import TOL as TOL_CHANNEL
from tests.test_gpu_parity import TOL64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


SIZES = [(70, 20, 36), (32, 9, 50), (128, 8, 7)]
NB, B, NU, DT = 40, 20, 0.02, 5e-3


def _batch(u):
    us = torch.stack([u * (1 + 0.01 * k) for k in range(NB)])
    us[B] = u
    return us


@pytest.mark.parametrize("scheme", ["rk4", "wray3"])
@pytest.mark.parametrize("n", SIZES)
def test_periodic(n, scheme):
    from paper_2604_18536_amd import Solver

    h = S.spacing(n)
    step, vjp = (O.step_rk4, O.step_rk4_vjp) if scheme == "rk4" else (O.step_wray3, O.step_wray3_vjp)
    u0, ub = S.random_field(n, 3), S.random_field(n, 4)
    ref, gref = step(u0, h, NU, DT), vjp(u0, ub, h, NU, DT)
    u, b = dev(u0), dev(ub)
    one, many = Solver(n, nu=NU), Solver(n, nu=NU, batch=NB)
    us, bs = _batch(u), _batch(b)
    assert max_rel(host(one.step(u, DT, scheme=scheme)), ref) < TOL64
    assert max_rel(host(many.step(us, DT, scheme=scheme)[B]), ref) < TOL64
    assert max_rel(host(one.step_vjp(u, b, DT, scheme=scheme)), gref) < TOL64
    assert max_rel(host(many.step_vjp(us, bs, DT, scheme=scheme)[B]), gref) < TOL64


@pytest.mark.parametrize("n", SIZES)
def test_channel(n):
    from paper_2604_18536_amd import Solver

    u, b = dev(S.channel_random(n, 3)), dev(S.channel_random(n, 4))
    one, many = Solver(n, nu=NU, bc="walls"), Solver(n, nu=NU, bc="walls", batch=NB)
    us, bs = _batch(u), _batch(b)
    assert max_rel(host(many.step(us, DT)[B]), host(one.step(u, DT))) < 2 * TOL_CHANNEL
    assert max_rel(host(many.step_vjp(us, bs, DT)[B]), host(one.step_vjp(u, b, DT))) < 2 * TOL_CHANNEL
