"""GPU parity of the dense Gaussian gradient beyond D = 128 (k_dense_grad) at the
edges of its tiles, against the FP64 oracle in one-step mode.

Edges: one row past each 64-row group and 16-row tile; contractions of a whole
number of 16-k-step chunks and with a remainder; rows of P and x that are only
element-aligned (D odd); one chain and both chain-tile widths (the second needs
two workgroups per CU); one leapfrog step, where the last step is the first, and
an even and an odd number of them, between which the position's buffer changes.

Bar: per chain ||x_L - ref|| / ||ref|| and the same for p_L at most 1e-5, that of
the dense Gaussian's one-step parity elsewhere here.
"""
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


@pytest.mark.parametrize("D,C,L", [(129, 17, 1), (144, 16, 2), (161, 33, 3), (192, 1, 4), (193, 40, 5), (256, 31, 2),
                                   (257, 15, 3), (129, 5500, 2), (133, 5461, 3), (515, 20, 1), (1024, 18, 2)])
def test_dense_wide_edges(D, C, L):
    w = W.gauss_dense(dim=D, num_chains=C, L=L, step_size=0.08, seed=D)
    s = hmc.sampler_for(w)
    assert s.form == "plain"
    t = 6
    s.set_state(torch.from_numpy(w.x0).cuda(), None, t)
    g = {k: to_np(v) for k, v in s.step(want_proposal=True).items()}
    # the same transition in the graph form, bitwise
    sg = hmc.sampler_for(w, form=hmc.HMC_FORM_GRAPH)
    sg.set_state(torch.from_numpy(w.x0).cuda(), None, t)
    gg = {k: to_np(v) for k, v in sg.step().items()}
    x, xg = s.get_state()[0], sg.get_state()[0]
    s.close()
    sg.close()
    chains = sorted({0, C - 1, C // 2, min(15, C - 1), min(16, C - 1), min(31, C - 1), min(32, C - 1)})
    o = oracle.step_chains(oracle_target(w), L, w.seed, t, w.step_size, w.x0[chains].astype(np.float64), chains)
    e = np.maximum(rel_err_rows(g["proposed_state"][chains], o["x_prop"]),
                   rel_err_rows(g["proposed_momentum"][chains], o["p_prop"]))
    print(f"dense D={D} C={C} L={L}: rel err max {e.max():.2e}")
    assert e.max() <= 1e-5
    assert torch.equal(x, xg)
    for k in gg:
        assert np.array_equal(g[k], gg[k]), k
