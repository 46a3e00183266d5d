"""Timed work of the sampler: what user programs have it do, through its public entry points.

listed() gives the named cases, draw(rng) one more case of the same ranges, prepare(case, seed) what a program
holds before the call, run(state) one pass, work(case) the bytes and operations a pass cannot do without, and
exact(case, seed) the pass's outputs in 64-bit arithmetic, written here with torch alone.

Kinds of a case:
  chain    sample_chain: burn-in and kept transitions, samples and traces stored
  remc     replica-exchange sample_chain on a ladder of inverse temperatures
  moments  sample_chain with the kept states folded into streaming moments
  nuts     No-U-Turn sample_chain
  step     a program's own sweep around the kernel (HMC within Gibbs, delayed acceptance): it sets every chain's
           state, takes one transition and reads the end of every trajectory, position and momentum, which it
           decides on by itself
"""
from __future__ import annotations

import ctypes
import math

import numpy as np
import torch

import paper_2002_01184_amd.hmc as H

KINDS = {"std": H.HMC_TGT_STD_NORMAL, "diag": H.HMC_TGT_GAUSS_DIAG, "dense": H.HMC_TGT_GAUSS_DENSE,
         "logreg": H.HMC_TGT_LOGREG}
ADAPT_TARGET = 0.8


def listed():
    return [
        # the paper's introductory example, whole: 100 chains on N(0, 1) in FP64, 300 burn-in and 100 kept
        # transitions; the smallest call there is, one launch whose chains leave almost all of the chip idle
        dict(name="example_1d", kind="chain", target="std", dim=1, chains=100, leapfrog=3, eps=1.5, burnin=300,
             results=100, dtype="f64", adapt=False),
        # a ragged diagonal Gaussian in FP64 under replica exchange: four temperatures, 83 chains each
        dict(name="diag_37_remc", kind="remc", target="diag", dim=37, chains=332, leapfrog=10, eps=0.1, burnin=50,
             results=50, dtype="f64", adapt=False, replicas=4),
        # many chains of a wide diagonal Gaussian, the element-wise workload that fills the chip
        dict(name="diag_1000", kind="chain", target="diag", dim=1000, chains=16384, leapfrog=10, eps=0.1, burnin=10,
             results=10, dtype="f32", adapt=False),
        # a run too long to store: streaming moments over a ring of kept states
        dict(name="diag_333_moments", kind="moments", target="diag", dim=333, chains=1000, leapfrog=10, eps=0.1,
             burnin=64, results=256, dtype="f32", adapt=False, ring=64),
        # Bayesian logistic regression 1000 x 25 with dual averaging, sampled in one launch
        dict(name="logreg_1000x25", kind="chain", target="logreg", rows=1000, dim=25, chains=1024, leapfrog=10,
             eps=0.05, burnin=100, results=100, dtype="f32", x="f32", grad="f32", adapt=True),
        # the No-U-Turn sampler on the same model
        dict(name="logreg_1000x25_nuts", kind="nuts", target="logreg", rows=1000, dim=25, chains=1024, eps=0.05,
             leapfrog=1, burnin=0, results=20, dtype="f32", x="f32", grad="f32", adapt=False, depth=10),
        # the ill-conditioned dense Gaussian at its configured size
        dict(name="dense_100", kind="step", target="dense", dim=100, chains=4096, leapfrog=20, eps=0.1, dtype="f32"),
        # a dense Gaussian beyond 128 dimensions
        dict(name="dense_300", kind="step", target="dense", dim=300, chains=1000, leapfrog=20, eps=0.1, dtype="f32"),
        # a served request of few chains: ragged rows and dims, X in BF16, BF16 gradients
        dict(name="logreg_20011x150_bf16", kind="step", target="logreg", rows=20011, dim=150, chains=200, leapfrog=10,
             eps=0.011, dtype="f32", x="bf16", grad="bf16"),
        # full-precision gradients on a data set beyond one workgroup, X in FP32
        dict(name="logreg_10000x25", kind="step", target="logreg", rows=10000, dim=25, chains=1024, leapfrog=10,
             eps=0.015, dtype="f32", x="f32", grad="f32"),
        # the large model, 100000 x 256 with X in BF16: full-precision gradients at 2048 chains
        dict(name="logreg_100000x256", kind="step", target="logreg", rows=100000, dim=256, chains=2048, leapfrog=10,
             eps=0.005, dtype="f32", x="bf16", grad="f32"),
        # and as it is benchmarked: BF16 gradients at 8192 chains, the largest work
        dict(name="logreg_100000x256_bf16", kind="step", target="logreg", rows=100000, dim=256, chains=8192,
             leapfrog=10, eps=0.005, dtype="f32", x="bf16", grad="bf16"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: sizes over the ranges of the listed ones (about 1 to 2048 dimensions element-wise, 2 to 512
    dense and logistic; 1 to 16384 chains; 60 to 100000 rows), bounded by the cost of the largest listed case."""
    kind = rng.choice(["chain", "chain", "chain", "remc", "moments", "nuts", "dense", "dense", "logreg", "logreg",
                       "logreg", "logreg"])
    if kind in ("chain", "remc", "moments"):
        if kind == "chain" and rng.random() < 0.3:      # small logistic regression, adapted, in one launch
            rows = _log_int(rng, 60, 1000)
            return dict(kind="chain", target="logreg", rows=rows, dim=rng.randint(2, 32),
                        chains=_log_int(rng, 20, 2048), leapfrog=rng.randint(3, 15), eps=1.6 / math.sqrt(rows),
                        burnin=rng.randint(20, 100), results=rng.randint(20, 100), dtype="f32",
                        x=rng.choice(["f32", "bf16"]), grad="f32", adapt=True)
        dim = _log_int(rng, 1, 1500)
        chains = _log_int(rng, 20, max(40, min(16384, 4000000 // dim)))
        n = rng.randint(10, 60) if dim * chains < 400000 else rng.randint(4, 10)
        c = dict(kind=kind, target=rng.choice(["std", "diag"]), dim=dim, chains=chains, leapfrog=rng.randint(2, 20),
                 eps=0.1, burnin=n, results=n, dtype=rng.choice(["f64", "f32"]), adapt=False)
        if kind == "remc":
            c["replicas"] = rng.choice([2, 4])
            c["chains"] = max(1, chains // c["replicas"]) * c["replicas"]
            c["dtype"] = "f64"
        if kind == "moments":
            c["ring"] = rng.choice([16, 64])
            c["results"] = 2 * n
        return c
    if kind == "nuts":
        if rng.random() < 0.5:
            return dict(kind="nuts", target=rng.choice(["std", "diag"]), dim=_log_int(rng, 1, 300),
                        chains=_log_int(rng, 20, 2000), eps=0.1, leapfrog=1, burnin=0, results=rng.randint(5, 15),
                        dtype="f64", adapt=False, depth=10)
        rows = _log_int(rng, 60, 3000)
        return dict(kind="nuts", target="logreg", rows=rows, dim=rng.randint(2, 32), chains=_log_int(rng, 20, 1024),
                    eps=1.6 / math.sqrt(rows), leapfrog=1, burnin=0, results=rng.randint(4, 10), dtype="f32",
                    x=rng.choice(["f32", "bf16"]), grad="f32", adapt=False, depth=10)
    if kind == "dense":
        dim = _log_int(rng, 2, 512)
        return dict(kind="step", target="dense", dim=dim, chains=_log_int(rng, 20, min(16384, 1000000 // dim)),
                    leapfrog=_log_int(rng, 3, 40), eps=0.1, dtype="f32")
    # logistic regression beyond one workgroup, over the served stream's mix: the shape of rows, dims and chains
    # is drawn until a step costs no more than the largest listed one's
    x = rng.choice(["f32", "bf16", "bf16"])
    grad = rng.choice(["f32", "bf16"]) if x == "bf16" else "f32"
    most = 100000 * 256 * (8192 if grad == "bf16" else 2048)
    while True:
        rows, dim, chains = _log_int(rng, 1100, 100000), _log_int(rng, 5, 512), _log_int(rng, 20, 8192)
        if rows * dim * chains <= most:
            break
    return dict(kind="step", target="logreg", rows=rows, dim=dim, chains=chains, leapfrog=rng.randint(3, 10),
                eps=1.6 / math.sqrt(rows) * min(1.0, 5.0 / math.sqrt(dim)), dtype="f32", x=x, grad=grad)


# ---- inputs -----------------------------------------------------------------------------------------------------
def _inputs(case, seed):
    """Target arrays and the initial state on the GPU, made from the seed alone."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(1000003 * int(seed) + 17)
    dt = torch.float64 if case["dtype"] == "f64" else torch.float32
    C, D = case["chains"], case["dim"]
    o = dict(prec=None, X=None, y=None)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device=dev, dtype=torch.float64)

    if case["target"] == "std":
        o["x0"] = torch.zeros(C, D, dtype=dt, device=dev) if D == 1 else normal(C, D).to(dt)
    elif case["target"] == "diag":
        # variances log-spaced over four decades; the chains start at draws of the target
        lam = torch.logspace(-2, 2, D, dtype=torch.float64, device=dev)
        o["prec"] = (1.0 / lam).to(dt)
        o["x0"] = (normal(C, D) * lam.sqrt()).to(dt)
    elif case["target"] == "dense":
        # covariance Q diag(lambda) Q^T, lambda log-spaced over four decades, Q Haar
        r = np.random.default_rng([int(seed), 21])
        q, t = np.linalg.qr(r.standard_normal((D, D)))
        q = q * np.sign(np.diag(t))[None, :]
        lam = np.logspace(-2, 2, D)
        p = ((q / lam[None, :]) @ q.T).astype(np.float32)
        p = np.triu(p) + np.triu(p, 1).T
        o["prec"] = torch.from_numpy(np.ascontiguousarray(p)).to(dev)
        root = torch.from_numpy(np.ascontiguousarray((q * np.sqrt(lam)[None, :]).T)).to(dev)
        o["x0"] = (normal(C, D) @ root).to(dt)
    else:
        # X and the generating weights N(0, 1), labels Bernoulli; the chains start near those weights
        N = case["rows"]
        X = torch.randn(N, D, generator=gen, device=dev, dtype=torch.float32)
        if case["x"] == "bf16":
            X = X.to(torch.bfloat16)
        w = normal(D)
        p = torch.sigmoid(X.double() @ w)
        o["y"] = (torch.rand(N, generator=gen, device=dev, dtype=torch.float64) < p).to(torch.uint8)
        o["X"] = X
        jitter = 0.05 if N > 3000 else 0.3
        o["x0"] = (w + jitter * (2.0 * torch.rand(C, D, generator=gen, device=dev, dtype=torch.float64) - 1.0)).to(dt)
    return o


def _ladder(case):
    """beta of every chain, replica-major: geometric from 1 to 0.1."""
    K = case["replicas"]
    b = 0.1 ** (torch.arange(K, dtype=torch.float64, device="cuda") / (K - 1))
    return b.repeat_interleave(case["chains"] // K).contiguous()


def prepare(case, seed):
    o = _inputs(case, seed)
    X = o["X"]
    x_bf16 = X is not None and X.dtype == torch.bfloat16
    s = H.Sampler(KINDS[case["target"]], case["dim"], case["chains"], case["leapfrog"], case["eps"], o["x0"],
                  prec=o["prec"], X=X.view(torch.int16) if x_bf16 else X, y=o["y"], x_bf16=x_bf16, seed=int(seed),
                  grad_bf16=case.get("grad") == "bf16")
    state = dict(case=case, sampler=s, x0=o["x0"])
    if case["kind"] == "remc":
        s.set_inverse_temperature(_ladder(case))
    if case["kind"] == "step":
        state["position"] = torch.empty_like(o["x0"])
        state["momentum"] = torch.empty_like(o["x0"])
        state["out"] = H.hmc_step_out(None, None, None, ctypes.c_void_p(state["position"].data_ptr()),
                                      ctypes.c_void_p(state["momentum"].data_ptr()), None)
    return state


def run(state):
    case, s = state["case"], state["sampler"]
    kind = case["kind"]
    if kind == "step":
        H.hmc_set_state(s.ctx, ctypes.c_void_p(state["x0"].data_ptr()), None, 0)
        H.hmc_step(s.ctx, state["out"])
        return dict(position=state["position"], momentum=state["momentum"])
    if kind == "nuts":
        return s.nuts_sample_chain(case["results"], case["burnin"], max_depth=case["depth"])
    kw = dict(adapt=case["adapt"], target_accept=ADAPT_TARGET)
    if kind == "remc":
        return s.remc_sample_chain(case["replicas"], case["results"], case["burnin"], **kw)
    if kind == "moments":
        r = s.sample_chain_moments(case["results"], case["burnin"], ring_rows=case["ring"], **kw)
        return {k: v for k, v in r.items() if k not in ("ring", "batch_sum")}
    return s.sample_chain(case["results"], case["burnin"], **kw)


def work(case):
    C, D, L = case["chains"], case["dim"], case["leapfrog"]
    es = 8 if case["dtype"] == "f64" else 4
    N = case.get("rows", 0)
    # one gradient of all chains, and the drift and kick around it
    grad = C * {"std": D, "diag": D, "dense": 2 * D * D, "logreg": 4 * N * D}[case["target"]] + 4 * C * D
    data = {"std": 0, "diag": es * D, "dense": es * D * D,
            "logreg": N * D * (2 if case.get("x") == "bf16" else 4) + N}[case["target"]]
    if case["kind"] == "step":
        # the state in, both ends of the trajectory out; a gradient at the new state and one per leapfrog step
        return dict(bytes=data + 3 * C * D * es, flops=(L + 1) * grad)
    T = case["burnin"] + case["results"]
    traces = {"chain": 25, "remc": 26, "moments": 25, "nuts": 16}[case["kind"]] * C * case["results"]
    kept = 4 * C * D * 8 if case["kind"] == "moments" else case["results"] * C * D * es
    steps = 7 * T if case["kind"] == "nuts" else L * T     # a tree of NUTS here is rarely below three doublings
    return dict(bytes=data + 2 * C * D * es + kept + traces, flops=steps * grad)


# ---- 64-bit reference -------------------------------------------------------------------------------------------
_M32 = 0xFFFFFFFF


def _mulhilo(a, b):
    """High and low words of the 32 x 32-bit products a b (a an int, b an int64 tensor of 32-bit values)."""
    lo = (a * b) & _M32
    hi = (a * (b >> 16) + ((a * (b & 0xFFFF)) >> 16)) >> 16
    return hi, lo


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 (Salmon et al., SC'11) on int64 tensors of 32-bit words."""
    k0, k1 = seed & _M32, (seed >> 32) & _M32
    c0, c1, c2, c3 = torch.broadcast_tensors(c0, c1, c2, c3)
    for _ in range(10):
        h0, l0 = _mulhilo(0xD2511F53, c0)
        h1, l1 = _mulhilo(0xCD9E8D57, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return c0, c1, c2, c3


def _i64(*v):
    return [torch.as_tensor(x, dtype=torch.int64, device="cuda") for x in v]


def _momentum(seed, C, D, t):
    """The standard-normal momenta [C, D] of transition t: Box-Muller on the word pairs of block d / 4, tag 0."""
    nb = (D + 3) // 4
    chain = torch.arange(C, device="cuda").view(C, 1)
    block = torch.arange(nb, device="cuda").view(1, nb)
    w = _philox(chain, _i64(t)[0], block, _i64(0)[0], seed)
    u = [((x >> 9).double() + 0.5) * 2.0 ** -23 for x in w]
    z = []
    for a, b in ((u[0], u[1]), (u[2], u[3])):
        r = torch.sqrt(-2.0 * torch.log(a))
        z += [r * torch.cos(2.0 * math.pi * b), r * torch.sin(2.0 * math.pi * b)]
    return torch.stack(z, dim=2).reshape(C, 4 * nb)[:, :D].contiguous()


def _log_uniform(seed, chain, t, tag):
    w0, w1, _, _ = _philox(chain, *_i64(t, 0, tag), seed)
    return torch.log((((w0 >> 6).double() * 67108864.0 + (w1 >> 6).double()) + 0.5) * 2.0 ** -52)


def _gradient(case, o):
    """x -> gradient of the log-probability, in 64 bits."""
    if case["target"] == "std":
        return lambda x: -x
    if case["target"] == "diag":
        prec = o["prec"].double()
        return lambda x: -prec * x
    if case["target"] == "dense":
        prec = o["prec"].double()
        return lambda x: -(x @ prec)
    y = o["y"].double()

    def logistic(x):
        g = -x
        for r0 in range(0, y.numel(), 8192):            # rows at a time: the logits of all would not fit
            X = o["X"][r0:r0 + 8192].double()
            g = g + (y[r0:r0 + 8192] - torch.sigmoid(x @ X.T.contiguous())) @ X
        return g
    return logistic


def exact(case, seed):
    kind = case["kind"]
    if kind == "nuts" or case.get("adapt"):
        return None     # trees and adapted step sizes feed rounding back until 64-bit runs part company as well
    o = _inputs(case, seed)
    C, D, L, eps = case["chains"], case["dim"], case["leapfrog"], case["eps"]
    grad = _gradient(case, o)
    beta = _ladder(case) if kind == "remc" else torch.ones(C, dtype=torch.float64, device="cuda")
    bcol = beta.view(C, 1)
    x = o["x0"].double()
    g = grad(x)

    def trajectory(x, g, t):
        p0 = _momentum(int(seed), C, D, t)
        p = p0 + 0.5 * eps * bcol * g
        for k in range(L):
            x = x + eps * p
            g = grad(x)
            p = p + (0.5 if k == L - 1 else 1.0) * eps * bcol * g
        return p0, x, p, g

    if kind == "step":
        _, xn, pn, _ = trajectory(x, g, 0)
        return dict(position=xn, momentum=pn)

    chain = torch.arange(C, device="cuda")
    logp = 0.5 * (x * g).sum(1)
    R, B = case["results"], case["burnin"]
    out = dict(step_size=torch.full((R, C), float(eps), dtype=torch.float64, device="cuda"),
               is_accepted=torch.empty(R, C, dtype=torch.uint8, device="cuda"),
               log_accept_ratio=torch.empty(R, C, dtype=torch.float64, device="cuda"),
               target_log_prob=torch.empty(R, C, dtype=torch.float64, device="cuda"))
    if kind == "moments":
        mean = torch.zeros(2, C, D, dtype=torch.float64, device="cuda")
        m2 = torch.zeros_like(mean)
    else:
        out["samples"] = torch.empty(R, C, D, dtype=torch.float64, device="cuda")
    if kind == "remc":
        out["swapped"] = torch.zeros(R, C, dtype=torch.uint8, device="cuda")
    for i in range(B + R):
        p0, xn, pn, gn = trajectory(x, g, i)
        ln = 0.5 * (xn * gn).sum(1)
        ratio = beta * (ln - logp) + 0.5 * ((p0 * p0).sum(1) - (pn * pn).sum(1))
        acc = _log_uniform(int(seed), chain, i, 1) < ratio
        x = torch.where(acc.view(C, 1), xn, x)
        g = torch.where(acc.view(C, 1), gn, g)
        logp = torch.where(acc, ln, logp)
        r = i - B
        if r >= 0:
            out["is_accepted"][r] = acc.to(torch.uint8)
            out["log_accept_ratio"][r] = ratio
            out["target_log_prob"][r] = logp
        if kind == "remc":
            K = case["replicas"]
            M = C // K
            src = torch.arange(C, device="cuda")
            for k in range(i % 2, K - 1, 2):
                a, b = chain[k * M:(k + 1) * M], chain[(k + 1) * M:(k + 2) * M]
                swap = _log_uniform(int(seed), a, i, 2) < (beta[a] - beta[b]) * (logp[b] - logp[a])
                src[a], src[b] = torch.where(swap, b, a), torch.where(swap, a, b)
            x, g, logp = x[src], g[src], logp[src]
            if r >= 0:
                out["swapped"][r] = (src != chain).to(torch.uint8)
        if r >= 0 and kind == "moments":
            h = 0 if r < R // 2 else 1
            n = r + 1 if h == 0 else r - R // 2 + 1
            delta = x - mean[h]
            mean[h] += delta / n
            m2[h] += delta * (x - mean[h])
        elif r >= 0:
            out["samples"][r] = x
    if kind == "moments":
        out.update(mean=mean, m2=m2)
    return out
