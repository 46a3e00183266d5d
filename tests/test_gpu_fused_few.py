"""The few-chain form of the fused element-wise kernel (k_fused_elem_few) against
the kernel for many chains: chains are independent and both do the same
arithmetic on the same random numbers, so the first chains of a large run and a
run of those chains alone agree bit for bit, over transitions that cross blocks
of draws, with adaptation of both kinds, and under a transform.

Edges: every lane-group class (1, 4, 16, 64 lanes; 1, 2, 4 blocks per lane), one
and two dims of a block, a block cut by D, one chain, chain counts that leave the
last workgroup short and the largest of the class (65536 lanes).  The exchange
inside the launch is covered by the replica-exchange tests, which compare it with
single transitions.
"""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

from paper_2002_01184_amd import hmc  # noqa: E402


def _run(w, C, adapt, scale, R, B):
    s = hmc.sampler_for(w, num_chains=C)
    if scale:
        s.set_transform_scale(np.linspace(0.6, 1.5, w.dim))
    o = s.sample_chain(R, B, adapt=adapt)
    x, eps, t = s.get_state()
    s.close()
    assert t == R + B
    return {**o, "state": x[None], "eps": eps[None]}


@pytest.mark.parametrize("dim,dtype,big,few,adapt,scale", [
    (1, "f64", 65600, (1, 100, 65536), False, False), (1, "f32", 65600, (257,), "simple", False),
    (2, "f64", 65600, (300,), True, False), (3, "f64", 65600, (77,), True, True), (4, "f32", 65600, (513,), True, False),
    (5, "f64", 16400, (1, 16384), False, False), (13, "f32", 16400, (900,), True, True),
    (16, "f64", 16400, (31,), "simple", False), (17, "f64", 4100, (333,), True, False), (37, "f64", 4100, (4096,), False, True),
    (64, "f32", 4100, (70,), True, False), (65, "f64", 1030, (1024,), True, False), (256, "f32", 1030, (10,), False, False),
    (257, "f64", 1030, (40,), True, True), (333, "f32", 1030, (1000,), True, False), (512, "f64", 1030, (3,), False, False),
    (513, "f32", 1030, (1, 600), True, False), (1023, "f32", 1030, (260,), False, True)])
def test_few_chains_bitwise_as_among_many(dim, dtype, big, few, adapt, scale):
    w = W.gauss_diag(dim=dim, num_chains=big, L=4, step_size=0.3, seed=dim, state_dtype=dtype, lam_lo=0.3, lam_hi=3.0)
    R, B = 6, 70 if dim < 5 else 9
    ref = _run(w, big, adapt, scale, R, B)
    for C in few:
        o = _run(w, C, adapt, scale, R, B)
        for k in o:
            assert torch.equal(o[k], ref[k][:, :C]), (C, k)
