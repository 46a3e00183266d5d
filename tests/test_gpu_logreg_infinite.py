"""One infinite coordinate of a position in the FP32 logistic step: rows with a
non-zero entry there have infinite logits, the other coordinates' gradients stay
finite, as in FP32 arithmetic, and the proposal is rejected.

Edges: X stored FP32 and BF16 (entries that need one BF16 term, and three); rows one
short of, at and one past the 32 of a stage, whose missing rows are zeros; up to 32
dims and beyond.  Reference in 64 bits; bar 1e-5, that of every FP32 logistic path.
"""
import numpy as np
import pytest

import oracle
import workloads as W
from gpu_helpers import gpu_available, rel_err_rows, to_np

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

from paper_2002_01184_amd import hmc  # noqa: E402


@pytest.mark.parametrize("bf16x", [False, True])
@pytest.mark.parametrize("N,D", [(90, 40), (95, 7), (96, 70), (97, 300)])
def test_one_infinite_coordinate(N, D, bf16x):
    w = W.logreg(N, D, 20, L=1, step_size=0.01, bf16=bf16x, init=0.2, seed=N)
    w.X[:, 1] = 1.0                                   # an intercept: exact in one BF16 term
    if bf16x:
        w.X_bf16[:, 1] = 0x3F80
    eps, far, C = 10.0, 1, w.num_chains
    scale = np.full(D, 1e-3)
    scale[far] = 1e38
    s = hmc.Sampler(w.kind, D, C, 1, eps, torch.from_numpy(w.x0).cuda(),
                    X=torch.from_numpy(w.X_bf16.view(np.int16) if bf16x else w.X).cuda(),
                    y=torch.from_numpy(w.y).cuda(), x_bf16=bf16x, seed=w.seed, form=hmc.HMC_FORM_PLAIN)
    s.set_transform_scale(scale)
    s.set_state(torch.from_numpy(w.x0).cuda(), None, 2)
    g = {k: to_np(v) for k, v in s.step(want_proposal=True).items()}
    s.close()
    X, y = w.X.astype(np.float64), w.y.astype(np.float64)
    iv = 1.0 / w.prior_scale ** 2

    def grad(x):
        with np.errstate(over="ignore"):
            return (y - 1.0 / (1.0 + np.exp(-(x @ X.T)))) @ X - iv * x
    x1 = g["proposed_state"].astype(np.float64)
    assert np.isinf(x1[:, far]).all()
    near = [d for d in range(D) if d != far]
    assert np.isfinite(x1[:, near]).all()
    p = oracle.momentum(w.seed, C, 2, D) + 0.5 * eps * scale * (grad(w.x0.astype(np.float64)) + grad(x1))
    e = rel_err_rows(g["proposed_momentum"][:, near], p[:, near])
    print(f"{N}x{D} bf16x={bf16x}: rel err of the finite coordinates {e.max():.1e}")
    assert e.max() <= 1e-5
    assert not g["is_accepted"].any() and np.isneginf(g["log_accept_ratio"]).all()
