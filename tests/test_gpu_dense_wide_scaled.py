"""The dense Gaussian beyond D = 128 (k_begin_drift, k_dense_grad) under a diagonal
transform and at an inverse temperature, alone and together, against the FP64 oracle in
one-step mode: the drift carries the scale, the kicks the scale and the temperature.

Edges: one leapfrog step, an even and an odd number of them (the position changes its
buffer between them); both chain-tile widths.  Bar 1e-5, that of the dense Gaussian's
one-step parity elsewhere here.
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


@pytest.mark.parametrize("scaled,beta", [(True, 1.0), (False, 0.4), (True, 0.4)])
@pytest.mark.parametrize("D,C,L", [(129, 20, 1), (150, 33, 2), (200, 17, 3), (133, 5461, 2)])
def test_dense_wide_scaled(D, C, L, scaled, beta):
    w = W.gauss_dense(dim=D, num_chains=C, L=L, step_size=0.08, seed=D)
    scale = np.linspace(0.5, 1.5, D) if scaled else np.ones(D)
    s = hmc.sampler_for(w, form=hmc.HMC_FORM_PLAIN)
    if scaled:
        s.set_transform_scale(scale)
    if beta != 1.0:
        s.set_inverse_temperature(torch.full((C,), beta, dtype=torch.float64, device="cuda"))
    t = 5
    s.set_state(torch.from_numpy(w.x0).cuda(), None, t)
    g = {k: to_np(v) for k, v in s.step(want_proposal=True).items()}
    s.close()
    some = sorted({0, 1, C // 2, C - 1, min(16, C - 1)})
    tz = oracle_target(w).tempered(beta).transformed(scale)
    o = oracle.step_chains(tz, L, w.seed, t, w.step_size, w.x0[some].astype(np.float64) / scale, some)
    e = np.maximum(rel_err_rows(g["proposed_state"][some], o["x_prop"] * scale),
                   rel_err_rows(g["proposed_momentum"][some], o["p_prop"]))
    print(f"dense D={D} C={C} L={L} scaled={scaled} beta={beta}: rel err max {e.max():.2e}")
    assert e.max() <= 1e-5
