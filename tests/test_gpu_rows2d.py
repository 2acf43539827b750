"""2D periodic steps and pullbacks in blocks of rows: the smallest grids, rows that do
not divide into blocks, every radix, the longest rows and the most blocks that the
fused kernels take and the next larger ones, fields of a batch, vs the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
import synth as S
from tests.gpu_util import dev, host, l2_rel, max_rel
from tests.test_gpu_parity import TOL64

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


STEP = {"rk4": (O.step_rk4, O.step_rk4_vjp), "wray3": (O.step_wray3, O.step_wray3_vjp)}


# (n_x, n_y), fields: blocks of 4 rows; rows <= 256 and <= 256 blocks are fused
@pytest.mark.parametrize("scheme", ["rk4", "wray3"])
@pytest.mark.parametrize("n,batch", [((4, 4), 1), ((4, 6), 3), ((6, 7), 2), ((8, 9), 1), ((14, 27), 1), ((30, 50), 2),
                                     ((98, 21), 1), ((162, 5), 1), ((250, 18), 3), ((256, 14), 1), ((32, 1024), 1),
                                     ((32, 1029), 1), ((256, 30), 32), ((256, 30), 33), ((270, 12), 1)])
def test_step_and_pullback(n, batch, scheme):
    from paper_2604_18536_amd import Solver

    nu, dt, h = 0.02, 5e-3, S.spacing(n)
    step, vjp = STEP[scheme]
    u0 = np.stack([S.random_field(n, 50 + b) for b in range(batch)])
    ub = np.stack([S.random_field(n, 90 + b) for b in range(batch)])
    one = (lambda v: v[0]) if batch == 1 else (lambda v: v)
    for precision, tol in (("fp64", TOL64), ("fp32", 1e-5)):
        s = Solver(n, nu=nu, precision=precision, batch=batch)
        t = torch.float64 if precision == "fp64" else torch.float32
        du, db = dev(one(u0)).to(t), dev(one(ub)).to(t)
        kept = s.stage_buffers(scheme)
        u1, g = s.step(du, dt, scheme=scheme), s.step_vjp(du, db, dt, scheme=scheme)
        assert torch.equal(u1, s.step(du, dt, scheme=scheme, keep=kept))
        assert torch.equal(g, s.step_vjp(du, db, dt, scheme=scheme, kept=kept))
        v = du.clone()
        assert torch.equal(u1, s.step(v, dt, scheme=scheme, out=v))
        u1, g = (host(x).astype(np.float64).reshape(u0.shape) for x in (u1, g))
        err = max_rel if precision == "fp64" else l2_rel
        for b in sorted({0, batch // 2, batch - 1}):
            assert err(u1[b], step(u0[b], h, nu, dt)) < tol
            assert err(g[b], vjp(u0[b], ub[b], h, nu, dt)) < tol
        s.close()
