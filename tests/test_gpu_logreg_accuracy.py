"""Accuracy of the FP32 logistic steps against 64 bits over many rows, where
errors of one sign add up.

The bars count roundings: a term of the log-probability is good to 2^-24 or so,
and N of them that round independently are off by sqrt(N) 2^-24 together; the
bars allow four times that.
"""
import math

import numpy as np
import pytest

import oracle
import workloads as W
from gpu_helpers import gpu_available, oracle_target, to_np

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

from paper_2002_01184_amd import hmc  # noqa: E402


def _step(w, L, eps):
    s = hmc.Sampler(w.kind, w.dim, w.num_chains, L, eps, torch.from_numpy(w.x0).cuda(),
                    X=torch.from_numpy(w.X_bf16.view(np.int16) if w.X_bf16 is not None else w.X).cuda(),
                    y=torch.from_numpy(w.y).cuda(), x_bf16=w.X_bf16 is not None, seed=w.seed,
                    form=hmc.HMC_FORM_PLAIN)
    s.set_state(torch.from_numpy(np.ascontiguousarray(w.x0)).cuda(), None, 3)
    g = {k: to_np(v).astype(np.float64) for k, v in s.step(want_proposal=True).items()}
    s.close()
    return g


@pytest.mark.parametrize("bf16x", [False, True])
@pytest.mark.parametrize("N,D", [(100000, 5), (60000, 31), (30000, 40)])
def test_energy_change(N, D, bf16x):
    # both ends' log-probabilities come from one arithmetic: what they share cancels
    w = W.logreg(N, D, 64, L=2, step_size=0.001, bf16=bf16x, init=0.1, seed=N + D)
    g = _step(w, 2, 1.0 / math.sqrt(N * D))
    tg = oracle_target(w)
    l0, l1 = (oracle.logp_grad(tg, x)[0] for x in (w.x0.astype(np.float64), g["proposed_state"]))
    p0 = oracle.momentum(w.seed, w.num_chains, 3, D)
    dh = l0 - l1 + 0.5 * ((g["proposed_momentum"] ** 2).sum(1) - (p0 ** 2).sum(1))
    err = math.sqrt(np.mean((g["delta_h"] - dh) ** 2))
    bar = 4.0 * math.sqrt(2.0 * N) * 2.0 ** -24
    print(f"{N}x{D} bf16x={bf16x}: energy change off by {err:.1e} (bar {bar:.1e})")
    assert err <= bar


@pytest.mark.parametrize("bf16x", [False, True])
@pytest.mark.parametrize("N,D,C,splits", [(100000, 2, 64, 64), (100000, 31, 64, 64), (60000, 100, 64, 64),
                                          (100000, 130, 4000, 8), (30000, 300, 64, 64)])
def test_gradient(N, D, C, splits, bf16x):
    # A split's sums round once a stage of 32 rows, independently, 2^-24 of a sum that is
    # half grown on average; four more roundings on the way into the momentum.  The chains
    # start far enough from the mode that the rows' terms do not cancel.
    w = W.logreg(N, D, C, L=1, step_size=0.001, bf16=bf16x, init=0.1, seed=N + D)
    eps = 20.0 / math.sqrt(N)
    g = _step(w, 1, eps)
    some = np.arange(0, C, max(1, C // 8))
    tg = oracle_target(w)
    g0, g1 = (oracle.logp_grad(tg, x[some])[1] for x in (w.x0.astype(np.float64), g["proposed_state"]))
    kick = 0.5 * eps * (g0 + g1)
    err = np.linalg.norm(g["proposed_momentum"][some] - oracle.momentum(w.seed, C, 3, D)[some] - kick)
    err /= np.linalg.norm(kick)
    bar = (0.5 * math.sqrt(math.ceil(N / splits / 32)) + 4.0) * 2.0 ** -24
    print(f"{N}x{D} C={C} bf16x={bf16x}: gradient off by {err:.1e} (bar {bar:.1e})")
    assert err <= bar


@pytest.mark.parametrize("bf16x", [False, True])
@pytest.mark.parametrize("N,D", [(100000, 2), (100000, 5), (60000, 31), (60000, 100)])
def test_log_probability(N, D, bf16x):
    w = W.logreg(N, D, 64, L=1, step_size=0.001, bf16=bf16x, init=0.1, seed=N + D)
    g = _step(w, 1, 1e-3 / math.sqrt(N * D))                 # every proposal is accepted
    assert g["is_accepted"].all()
    lp = oracle.logp_grad(oracle_target(w), g["proposed_state"])[0]
    err = math.sqrt(np.mean((g["target_log_prob"] - lp) ** 2))
    bar = 4.0 * math.sqrt(N) * 2.0 ** -24
    print(f"{N}x{D} bf16x={bf16x}: log-probability off by {err:.1e} (bar {bar:.1e})")
    assert err <= bar


@pytest.mark.parametrize("D", [3, 5, 16])
def test_gradient_near_the_mode(D):
    # There the rows' terms, N of about 0.3, cancel to sqrt(N) of them, and an error of one
    # sign in every term stands out in the mean over chains.  Terms good to 2^-24 that
    # round either way leave about 2^-24 of the gradient; the bar allows twice that.  The
    # middle gradient of two steps is formed without the log-probability; its position is
    # the end of one step.
    N, C = 60000, 192
    w = W.logreg(N, D, C, L=2, step_size=0.001, init=1.0 / math.sqrt(N), seed=N + D)
    eps = 1.0 / math.sqrt(N)
    one, two = _step(w, 1, eps), _step(w, 2, eps)
    tg = oracle_target(w)
    g0, g1, g2 = (oracle.logp_grad(tg, x)[1] for x in (w.x0.astype(np.float64), one["proposed_state"],
                                                       two["proposed_state"]))
    kick = 0.5 * g0 + g1 + 0.5 * g2
    err = (two["proposed_momentum"] - oracle.momentum(w.seed, C, 3, D)) / eps - kick
    err = np.linalg.norm(err.mean(0)) / math.sqrt(np.mean((kick ** 2).sum(1)))
    bar = 2.0 * 2.0 ** -24
    print(f"{N}x{D}: mean gradient off by {err:.1e} (bar {bar:.1e})")
    assert err <= bar
