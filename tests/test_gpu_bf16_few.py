"""The few-chain kernels of the BF16-gradient form (k_lr16_grad_few,
k_lr16_logp_few) against the kernels for many chains: chains are independent and
both sequences of matrix products are the same, so the first chains of a large
run and a run of those chains alone agree bit for bit.

Edges: every padded width (32, 64, 128, 192, 256, 384, 512 dims) with the last
width's first and last dim, rows read by less than 4 floats, at odd alignments
and whole; one chain, one short of, at and past a 16-chain tile, the smallest
counts of the 32- and 64-chain workgroups; one, a ragged and a whole number of
stages and sub-tiles per split.
"""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import gpu_available, to_np

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

from paper_2002_01184_amd import hmc  # noqa: E402


def _step(w, C, t):
    s = hmc.sampler_for(w, grad_bf16=True, num_chains=C)
    s.set_state(torch.from_numpy(np.ascontiguousarray(w.x0[:C])).cuda(), None, t)
    g = {k: to_np(v) for k, v in s.step(want_proposal=True).items()}
    s.close()
    return g


# (N, D, chains of the large run, chains of the small ones): the large run is past
# the few-chain kernels' line (more than 384 workgroups of 64 chains) and has the
# same row splits
@pytest.mark.parametrize("N,D,big,few", [
    (1100, 1, 4096, (1, 17)), (1030, 3, 4096, (16,)), (2085, 31, 4096, (15, 700)), (1100, 32, 4096, (513,)),
    (1500, 33, 4096, (40,)), (4100, 61, 4096, (16, 1030)), (1024, 100, 4096, (33,)), (1333, 128, 4096, (520,)),
    (2000, 150, 4096, (200,)), (1217, 192, 4096, (1025,)), (1300, 250, 4096, (64,)), (1029, 256, 4096, (600,)),
    (1100, 257, 2100, (17,)), (1190, 383, 2100, (530,)), (1100, 400, 2100, (31, 1026)), (1027, 511, 2100, (16,)),
    (1060, 512, 2100, (515,)), (40, 20, 25000, (5, 300)), (300, 70, 13000, (9,))])
def test_few_chains_bitwise_as_among_many(N, D, big, few):
    w = W.logreg(N, D, big, L=3, step_size=0.02, bf16=True, init=0.1, seed=N + D)
    ref = _step(w, big, 3)
    for C in few:
        g = _step(w, C, 3)
        for k in g:
            assert np.array_equal(g[k], ref[k][:C]), (C, k)
