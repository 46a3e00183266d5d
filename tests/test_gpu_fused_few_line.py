"""The element-wise kernels on both sides of the few-chain line with a lane per chain
(49152 chains): a run's chains are bitwise those of a larger run, whichever kernel
either takes.
"""
import pytest

import workloads as W
from gpu_helpers import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

from paper_2002_01184_amd import hmc  # noqa: E402


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("dim", [1, 4])
def test_both_sides_of_the_line(dim, dtype):
    outs = []
    for C in (49152, 49153, 65600):
        w = W.std_normal_1d(num_chains=65600, dim=dim, state_dtype=dtype, L=3, step_size=0.4, seed=dim)
        s = hmc.sampler_for(w, num_chains=C)
        outs.append(s.sample_chain(5, 8, adapt=True))
        s.close()
    for k in ("samples", "step_size", "is_accepted", "target_log_prob"):
        assert torch.equal(outs[0][k], outs[2][k][:, :49152]), k
        assert torch.equal(outs[1][k], outs[2][k][:, :49153]), k
