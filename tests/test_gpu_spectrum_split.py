"""Energy spectrum summed by several workgroups per field (partial shell rows) vs the oracle."""
import numpy as np
import pytest
import torch

import oracle as O
import synth as S
from tests.gpu_util import dev, host, max_rel

pytestmark = pytest.mark.gpu


# one workgroup and the smallest scratch; ragged rows over several workgroups;
# fewer bins than shells; more bins than shells; odd n_y, n_z
@pytest.mark.parametrize("n,batch,nbins", [((4, 2), 1, None), ((4, 2, 2), 3, None), ((90, 84), 2, None),
                                           ((70, 63, 45), 2, None), ((48, 40, 50), 1, 7), ((48, 40, 50), 2, 300)])
def test_split_shell_sums(n, batch, nbins):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2604_18536_amd import Solver

    s = Solver(n, batch=batch)
    u = np.stack([S.random_field(n, 3 + b) for b in range(batch)])
    for _ in range(2):  # overwritten, not accumulated
        e = host(s.energy_spectrum(dev(u), nbins))
    for b in range(batch):
        ref = O.energy_spectrum(u[b])
        k = min(len(ref), e.shape[1])
        # a DFT of N values and a sum of positive terms: about log2(N) rounding errors
        assert max_rel(e[b][:k], ref[:k]) < 1e-13 and not e[b][k:].any()
    s.close()
