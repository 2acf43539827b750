"""The learned closure's kernels where their blocks, rows and GELU branches end: the
smallest grids, blocks that stick out of the grid in y and z, one and several blocks
along x, and pre-activations far beyond the centre of GELU, layer by layer vs the oracle
(the bounds of tests/closure_check.py)."""
import numpy as np
import pytest
import torch

import synth as S
from tests.closure_check import check_closure_layers
from tests.gpu_util import dev, f32, host
from tests.test_gpu_closure import _layout, _solver, _theta

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("n,batch,scale", [((32, 2, 2), 1, 2.0), ((32, 3, 2), 2, 2.0), ((32, 5, 3), 1, 12.0),
                                           ((64, 9, 7), 2, 2.0), ((96, 4, 5), 1, 12.0), ((32, 10, 14), 1, 0.5)])
def test_layers(n, batch, scale):
    s = _solver(n, batch=batch)
    th = _theta(3, scale)
    s.set_closure(torch.tensor(th, dtype=torch.float32, device="cuda"))
    u = np.stack([f32(S.random_field(n, 4 + b)) for b in range(batch)])
    mbar = np.stack([f32(S.random_field(n, 24 + b)) for b in range(batch)])
    if batch == 1:
        u1, mbar1 = u[0], mbar[0]
    else:
        u1, mbar1 = u, mbar
    m_fwd = host(s.cnn_forward(dev(u1, torch.float32)))
    ub, tb = s.cnn_backward(dev(u1, torch.float32), dev(mbar1, torch.float32))
    t = {k: _layout(s.cnn_saved(w), batch, n)
         for w, k in enumerate(("x0", "z1", "a1", "z2", "a2", "gm", "gz2", "gz1"))}
    t["m"] = host(s.cnn_saved(8)).reshape(u.shape)
    assert np.array_equal(m_fwd.reshape(u.shape), t["m"])
    ff, fb = check_closure_layers(u, th, mbar, t, host(ub).reshape(u.shape), host(tb).astype(np.float64))
    hidden = u.size // 3 * 32 * 2
    if scale > 10:
        # far below zero GELU is smaller than its own float32 error bound, and nearly every
        # value there may round either way (a float32 erf flips a tenth of these): no count
        assert np.abs(t["z1"]).max() > 8 and np.abs(t["z2"]).max() > 8
    else:
        assert ff < 1e-3 * hidden + 2 and fb < 1e-3 * hidden + 2
    s.close()
