"""Float32 reverse stages on 64 x 8 and 32 x 8 tiles: widths around the multiples of 32
where the tile changes, ragged y and z, one and several z chunks, vs the float64 oracle."""
import pytest
import torch

import oracle as O
import synth as S
from tests.gpu_util import dev, f32, host, l2_rel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("scheme", ["rk4", "wray3"])
@pytest.mark.parametrize("n", [(4, 6, 2), (32, 9, 5), (36, 9, 5), (64, 7, 4), (70, 10, 35), (100, 16, 3), (128, 5, 6)])
def test_step_pullback_fp32(n, scheme):
    from paper_2604_18536_amd import Solver

    nu, dt = 0.02, 5e-3
    s = Solver(n, nu=nu, precision="fp32")
    u0, ub = f32(S.random_field(n, 11)), f32(S.random_field(n, 12))
    vjp = O.step_rk4_vjp if scheme == "rk4" else O.step_wray3_vjp
    g = host(s.step_vjp(dev(u0, torch.float32), dev(ub, torch.float32), dt, scheme=scheme))
    assert l2_rel(g, vjp(u0, ub, S.spacing(n), nu, dt)) < 1e-5
    s.close()
