"""GPU parity of the split FP32 gradient of logistic regression (k_lr32_step:
operands cut into three BF16 terms) at the edges of its tiles, against the FP64
oracle in one-step mode.

Edges: the k-step counts of 32 dims it is compiled for and one dim past each;
rows one short of, at and one past a 32-row sub-tile, fewer rows than one; the
last 8-column unit of the last row, which is read element by element; 64-chain
tiles one short, full and one past; rows of X at an address that is only
element-aligned; more than eight row splits.

Bar: per chain ||x_L - ref|| / ||ref|| and the same for p_L at most 1e-5, that
of every FP32 logistic path here (a gradient is a sum of products exact to
2^-23 accumulated in FP32, about 1e-6 after three steps).
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


def _sampler(w, shift=0):
    """A plain-form sampler whose X starts `shift` elements into its allocation."""
    dev = torch.device("cuda")
    X = torch.from_numpy(w.X_bf16.view(np.int16)) if w.X_bf16 is not None else torch.from_numpy(w.X)
    buf = torch.zeros(X.numel() + shift, dtype=X.dtype, device=dev)
    buf[shift:] = X.reshape(-1).to(dev)
    Xd = buf[shift:].view(*X.shape)
    return hmc.Sampler(w.kind, w.dim, w.num_chains, w.num_leapfrog_steps, w.step_size, torch.from_numpy(w.x0).to(dev),
                       X=Xd, y=torch.from_numpy(w.y).to(dev), x_bf16=w.X_bf16 is not None, seed=w.seed,
                       form=hmc.HMC_FORM_PLAIN)


def _step(s, x, t):
    s.set_state(torch.from_numpy(np.ascontiguousarray(x)).cuda(), None, t)
    return {k: to_np(v) for k, v in s.step(want_proposal=True).items()}


@pytest.mark.parametrize("bf16x", [False, True])
@pytest.mark.parametrize("N,D,C,shift", [
    (1, 1, 1, 0), (31, 32, 63, 0), (32, 33, 64, 1), (33, 31, 65, 1), (65, 64, 17, 0), (127, 65, 16, 3),
    (97, 129, 70, 1), (160, 161, 130, 0), (1300, 193, 40, 1), (95, 225, 66, 2), (64, 256, 64, 0), (90, 289, 20, 1),
    (61, 353, 33, 0), (70, 385, 48, 1), (40, 449, 65, 1), (33, 511, 16, 1), (2100, 12, 1, 0)])
def test_split_gradient_edges(N, D, C, shift, bf16x):
    w = W.logreg(N, D, C, L=3, step_size=0.02, bf16=bf16x, init=0.2, seed=N + D)
    s = _sampler(w, shift)
    t = 4
    g = _step(s, w.x0, t)
    s.close()
    o = oracle.step(oracle_target(w), w.num_leapfrog_steps, w.seed, t, w.step_size, w.x0.astype(np.float64))
    e = np.maximum(rel_err_rows(g["proposed_state"], o["x_prop"]), rel_err_rows(g["proposed_momentum"], o["p_prop"]))
    dh = np.abs(g["delta_h"] - o["delta_h"])
    print(f"logreg {N}x{D} C={C} shift={shift} bf16x={bf16x}: rel err max {e.max():.2e}, dH err max {dh.max():.2e}")
    assert e.max() <= 1e-5


@pytest.mark.parametrize("bf16x", [False, True])
def test_diverged_chain_is_rejected_and_leaves_the_others(bf16x):
    w = W.logreg(300, 50, 40, L=3, step_size=0.02, bf16=bf16x, init=0.2, seed=3)
    s = _sampler(w)
    ref = _step(s, w.x0, 2)
    x = w.x0.copy()
    x[5, 7], x[6, 0], x[21, :] = np.inf, np.nan, -np.inf
    g = _step(s, x, 2)
    s.close()
    bad = [5, 6, 21]
    ok = [c for c in range(40) if c not in bad]
    assert not g["is_accepted"][bad].any()
    assert not np.isfinite(g["proposed_momentum"][bad]).all(axis=1).any()
    for k in ("proposed_state", "proposed_momentum", "delta_h", "is_accepted"):
        assert np.array_equal(g[k][ok], ref[k][ok]), k
