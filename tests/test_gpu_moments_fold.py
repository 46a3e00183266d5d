"""The moments fold (k_moments) against the same recurrences in numpy on the kept
draws of the same chain: each half's mean follows mu += (x - mu) / n with every
operation correctly rounded, so it agrees bit for bit, also where the fold forms
the quotient from a reciprocal; the batch sums add draws in order, a chunk's part
at a time, and agree bit for bit; the squared deviations may be contracted to
fused multiply-adds, n terms of one rounding each, bounded by n 2^-52 relative.

Edges: draws past the reciprocals' table (256), chunks that no block of eight
divides, a half that ends inside a chunk, batches across chunks, one draw a
chunk, draws equal to the mean (repeated rejections), and a chain so far out that
every proposal is rejected and the quotients are beyond the table's range."""
import numpy as np
import pytest

import workloads as W
from gpu_helpers import gpu_available, to_np

pytestmark = pytest.mark.gpu

if not gpu_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2002_01184_amd import hmc  # noqa: E402


@pytest.mark.parametrize("dtype,R,ring,blen", [
    ("f64", 600, 600, 40), ("f32", 600, 97, 40), ("f64", 602, 301, 7), ("f32", 50, 1, 25), ("f64", 18, 5, 1), ("f32", 2, 9, 2)])
def test_fold_matches_recurrence(dtype, R, ring, blen):
    w = W.gauss_diag(dim=7, num_chains=45, L=3, step_size=0.9, seed=6, state_dtype=dtype)
    if dtype == "f64":
        w.x0[3] = 1e280
    s = hmc.sampler_for(w)
    g = s.sample_chain_moments(R, 0, ring_rows=ring, batch_len=blen)
    s.close()
    s = hmc.sampler_for(w)
    x = to_np(s.sample_chain(R, 0)["samples"]).astype(np.float64)
    s.close()
    assert np.any(x[1:] == x[:-1])                     # some draws repeat
    h = R // 2
    bsum = np.zeros((R // blen,) + x.shape[1:])
    for k, part in enumerate((x[:h], x[h:])):
        mu, ss = np.zeros(x.shape[1:]), np.zeros(x.shape[1:])
        with np.errstate(over="ignore"):
            for n, v in enumerate(part, 1):
                d = v - mu
                mu = mu + d / n
                ss = ss + d * (v - mu)
        assert np.array_equal(to_np(g["mean"])[k], mu)
        assert np.allclose(to_np(g["m2"])[k], ss, rtol=R * 2.0 ** -52, atol=0)
    for r0 in range(0, R, ring):
        acc = {}
        for r in range(r0, min(r0 + ring, R)):
            acc[r // blen] = acc.get(r // blen, np.zeros(x.shape[1:])) + x[r]
        for b, v in acc.items():
            bsum[b] += v
    assert np.array_equal(to_np(g["batch_sum"]), bsum)
