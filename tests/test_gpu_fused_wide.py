"""The fused element-wise kernel in FP64 beyond 1024 dims, whose state is loaded a
block of four dims at a time, against the FP64 oracle over whole runs.

Edges: one dim past 1024; a last block of 1, 2, 3 and 4 dims, with rows that are then
only element-aligned; the largest D; both Gaussian targets; a transform.  Bar: 1e-11 of
the samples' size (about 2000 terms a sum, a few transitions in FP64).
"""
import numpy as np
import pytest

import oracle
import workloads as W
from gpu_helpers import gpu_available, oracle_target, to_np

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2002_01184_amd import hmc  # noqa: E402


@pytest.mark.parametrize("scaled", [False, True])
@pytest.mark.parametrize("kind,D", [("diag", 1025), ("std", 1026), ("diag", 1359), ("diag", 1500), ("std", 2047),
                                    ("diag", 2048)])
def test_wide_fp64_runs(kind, D, scaled):
    C = 9
    if kind == "std":
        w = W.std_normal_1d(num_chains=C, dim=D, L=3, step_size=0.1, seed=D)
        w.x0 = np.random.default_rng(D).standard_normal((C, D))
    else:
        w = W.gauss_diag(dim=D, num_chains=C, L=3, step_size=0.05, seed=D, state_dtype="f64", lam_lo=0.5, lam_hi=2.0)
    s = hmc.sampler_for(w, form=hmc.HMC_FORM_FUSED)
    scale = np.linspace(0.7, 1.4, D)
    if scaled:
        s.set_transform_scale(scale)
    g = s.sample_chain(4, 2)
    s.close()
    x0 = w.x0.astype(np.float64)
    args = (w.num_leapfrog_steps, w.seed, x0, w.step_size, 2, 4)
    o = (oracle.transformed_sample_chain(oracle_target(w), scale, None, *args) if scaled
         else oracle.sample_chain(oracle_target(w), *args))
    assert np.array_equal(to_np(g["is_accepted"]).astype(bool), o["is_accepted"])
    err = np.max(np.abs(to_np(g["samples"]) - o["samples"])) / np.max(np.abs(o["samples"]))
    print(f"{kind} D={D} scaled={scaled}: off by {err:.1e}")
    assert err <= 1e-11
