"""A resumed run of the plain and graph forms on logistic regression equals the
uninterrupted one bit for bit: set_state rebuilds the gradient and the
log-probability that the last transition left.

Edges: up to 32 dims, where set_state has a kernel of its own for the fused
form, and past them; X stored FP32 and BF16; BF16 gradients; a fused-form
context's own set_state beside them is not held to this (its chains carry the
fused kernel's own gradient).
"""
import pytest

import workloads as W
from gpu_helpers import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

from paper_2002_01184_amd import hmc  # noqa: E402


@pytest.mark.parametrize("form", [hmc.HMC_FORM_PLAIN, hmc.HMC_FORM_GRAPH])
@pytest.mark.parametrize("N,D,bf16x,grad16", [
    (1500, 1, False, False), (1500, 12, False, False), (2000, 25, True, False), (90, 32, False, False),
    (1500, 33, False, False), (1500, 70, True, False), (1500, 70, True, True)])
def test_resume_is_bitwise(N, D, bf16x, grad16, form):
    w = W.logreg(N, D, 70, L=4, step_size=0.02, seed=N + D, bf16=bf16x, init=0.2)

    def sampler():
        return hmc.sampler_for(w, form=form, grad_bf16=grad16)
    s = sampler()
    full = s.sample_chain(14, 0)
    s.close()
    s = sampler()
    s.sample_chain(6, 0)
    x, e, t = s.get_state()
    s.close()
    assert t == 6
    s = sampler()
    s.set_state(x, e, t)
    rest = s.sample_chain(8, 0)
    s.close()
    for k in ("samples", "target_log_prob", "log_accept_ratio", "is_accepted"):
        assert torch.equal(rest[k], full[k][6:]), k
