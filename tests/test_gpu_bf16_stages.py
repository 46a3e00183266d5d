"""The stages of the BF16-gradient pipelines (k_lr16_grad_pipe, k_lr16_logp_pipe)
at few rows: less than a sub-tile, one, and one short of, at and past the
sub-tiles of one and of two stages (1, 2 or 4 sub-tiles of 32 rows, by width),
where copies past the end repeat the last sub-tile.  The large run is past the
few-chain kernels' line and takes the pipelines; the same first chains alone take
the few-chain kernels, whose matrix products are the same in the same order: all
outputs agree bit for bit."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import gpu_available, to_np

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

from paper_2002_01184_amd import hmc  # noqa: E402


def _step(w, C):
    s = hmc.sampler_for(w, grad_bf16=True, num_chains=C)
    s.set_state(torch.from_numpy(np.ascontiguousarray(w.x0[:C])).cuda(), None, 2)
    g = {k: to_np(v) for k, v in s.step(want_proposal=True).items()}
    s.close()
    return g


@pytest.mark.parametrize("D,big", [(30, 25000), (64, 25000), (100, 25000), (190, 25000), (256, 25000), (300, 16500),
                                   (500, 16500)])
@pytest.mark.parametrize("N", [1, 31, 32, 33, 64, 65, 96, 127, 129, 200, 257])
def test_pipeline_stages_bitwise_as_few_chains(N, D, big):
    if N > 256 and D > 256:
        pytest.skip("129 tiles of 128 chains take one row split there, the small run two: other FP32 sums")
    w = W.logreg(N, D, big, L=2, step_size=0.02, bf16=True, init=0.1, seed=N + D)
    ref, g = _step(w, big), _step(w, 40)
    for k in g:
        assert np.array_equal(g[k], ref[k][:40]), k
