"""Which BF16 logistic requests of one class share launches in the server: a few of
few chains run side by side, on the kernel that each runs alone; many share.  Either
way each request's results are bitwise those of its own sample_chain.
"""
import pytest

import workloads as W
from gpu_helpers import gpu_available

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import torch  # noqa: E402

from paper_2002_01184_amd import hmc  # noqa: E402


def _served(reqs):
    srv = hmc.Server(2 << 30, transitions_per_tick=5)
    preps = [srv.prepare(w, grad_bf16=True) for w in reqs]
    outs = [srv.wait(i)[0] for i in [srv.submit_prepared(p) for p in preps]]
    st = srv.stats()
    srv.close()
    for w, o in zip(reqs, outs):
        s = hmc.sampler_for(w, grad_bf16=True)
        ref = s.sample_chain(w.num_results, w.num_burnin, adapt=w.adapt)
        for k in ("samples", "is_accepted", "step_size", "target_log_prob"):
            assert torch.equal(o[k], ref[k]), (w.name, k)
        s.close()
    return st


def _requests(n, N, D, C, T):
    return [W.logreg(N, D, C + 3 * i, L=3, step_size=0.003, burnin=T, results=4, seed=50 + i, bf16=True, init=0.05)
            for i in range(n)]


# pairs of 16, 32 and 64 chains a workgroup; three with row splits of 16 sub-tiles and more
@pytest.mark.parametrize("n,N,D,C", [(2, 5000, 100, 100), (2, 2000, 400, 700), (3, 5000, 60, 60)])
def test_few_run_side_by_side(n, N, D, C):
    st = _served(_requests(n, N, D, C, 60))
    assert st["max_active"] == n and st["batched_plain_transitions"] == 0


# more than there are streams; a pair whose chains nearly fill a round of the many-chain
# kernel each, at a size past one workgroup per CU (C * D > 2^19: the sums of the partials
# alone are read 16 bytes at a time); three bound by their launches
@pytest.mark.parametrize("n,N,D,C", [(6, 2000, 100, 100), (2, 3000, 240, 3000), (3, 1500, 60, 60)])
def test_many_share(n, N, D, C):
    st = _served(_requests(n, N, D, C, 200))
    assert st["batched_plain_transitions"] >= 1


# alone in its class a request takes the kernels of sample_chain, a tick at a time, down to
# a last tick of one transition; beside another of its class a ragged launch
@pytest.mark.parametrize("kind,D,C,dtype", [("std", 1, 100, "f64"), ("std", 3, 700, "f32"), ("diag", 37, 200, "f32"),
                                            ("diag", 333, 300, "f32")])
@pytest.mark.parametrize("n", [1, 2])
def test_element_wise_requests(kind, D, C, dtype, n):
    if kind == "std":
        reqs = [W.std_normal_1d(num_chains=C, dim=D, state_dtype=dtype, L=4, step_size=0.4, burnin=20, results=11,
                                seed=70 + i) for i in range(n)]
    else:
        reqs = [W.gauss_diag(dim=D, num_chains=C, L=4, step_size=0.05, burnin=20, results=11, seed=70 + i)
                for i in range(n)]
    srv = hmc.Server(1 << 30, transitions_per_tick=5)
    preps = [srv.prepare(w) for w in reqs]
    outs = [srv.wait(i)[0] for i in [srv.submit_prepared(p) for p in preps]]
    srv.close()
    for w, o in zip(reqs, outs):
        s = hmc.sampler_for(w)
        ref = s.sample_chain(w.num_results, w.num_burnin, adapt=w.adapt)
        for k in ("samples", "is_accepted", "step_size", "target_log_prob"):
            assert torch.equal(o[k], ref[k]), (w.name, k)
        s.close()
