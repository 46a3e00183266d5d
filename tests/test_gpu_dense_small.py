"""The dense Gaussian's bootstrap gradient at D <= 32 (k_dense_grad's direct form)
at the edges of its tiles, through one transition from a set state, against the
FP64 oracle: one dim, one short of, at and past 16 dims, the last width; rows of
three floats and less; one chain, a short last chain tile.

Bar: per chain ||x_L - ref|| / ||ref|| and the same for p_L at most 1e-5, that of
the dense Gaussian's one-step parity elsewhere here."""
import numpy as np
import pytest

import oracle
import workloads as W
from gpu_helpers import gpu_available, oracle_target, rel_err_rows, to_np

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

from paper_2002_01184_amd import hmc  # noqa: E402


@pytest.mark.parametrize("form", [hmc.HMC_FORM_PLAIN, hmc.HMC_FORM_AUTO])
@pytest.mark.parametrize("D,C", [(1, 1), (2, 17), (3, 40), (8, 300), (15, 16), (16, 33), (17, 31), (31, 15), (32, 130)])
def test_dense_small_edges(D, C, form):
    w = W.gauss_dense(dim=D, num_chains=C, L=3, step_size=0.08, seed=D)
    s = hmc.sampler_for(w, form=form)
    s.set_state(torch.from_numpy(w.x0).cuda(), None, 4)
    g = {k: to_np(v) for k, v in s.step(want_proposal=True).items()}
    s.close()
    chains = list(range(C))
    o = oracle.step_chains(oracle_target(w), 3, w.seed, 4, w.step_size, w.x0.astype(np.float64), chains)
    e = np.maximum(rel_err_rows(g["proposed_state"], o["x_prop"]), rel_err_rows(g["proposed_momentum"], o["p_prop"]))
    assert e.max() <= 1e-5
