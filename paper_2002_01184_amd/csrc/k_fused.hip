// k_fused.hip -- fused persistent form: each workgroup owns a tile of chains
// and runs whole transitions (momentum, L leapfrog steps, energy, accept,
// select, dual averaging, sample and trace writes) with the chain state in
// registers and LDS.  HBM traffic per transition is the kept sample and
// trace rows; target data stays in registers/LDS/L2.
//
//   elementwise  N(0, I), diagonal Gaussian: G lanes per chain, 4-dim Philox
//                blocks per lane, reductions across the lane group
//   dense        g = -P x on v_mfma_f32_16x16x4f32; 16 chains per workgroup,
//                P held in VGPRs as A operands, x^T staged in LDS (double
//                buffered, one barrier per leapfrog step)
//   logreg       see k_fused_logreg.hip
#include "hmc_internal.hpp"

namespace hmc {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// Per-chain bookkeeping at the end of a transition, executed identically by
// every lane that holds a part of the chain.
struct ChainCtl {
    double logp, eps;
    DualAvg da;
};

// dual_avg_apply with its fused multiply-adds written out (as the compiler
// contracts it where the factors are computed in place), so that every kernel
// here rounds alike.
__device__ __forceinline__ double dual_avg_apply_fma(DualAvg& s, const DaConst& c, double alpha, double delta) {
    s.hbar = fma(1.0 - c.w, s.hbar, c.w * (delta - alpha));
    const double log_eps = fma(-c.k, s.hbar, s.mu);
    s.log_eps_bar = fma(1.0 - c.eta, s.log_eps_bar, c.eta * log_eps);
    return log_eps;
}

template <bool OUT, typename DaOf>
__device__ __forceinline__ void after_decision(const FusedRun& r, int64_t C, int64_t c, int64_t i, bool acc,
                                               double lar, double dh, double lp_new, ChainCtl& s, bool writer,
                                               DaOf da_of) {
    const double eps_used = s.eps;
    if (r.adapt && i < r.n_burnin) {
        const double alpha = lar < 0.0 ? exp(lar) : 1.0;
        if (r.adapt_kind == HMC_ADAPT_SIMPLE) {
            s.eps = simple_adapt(s.eps, alpha, r.target_accept, r.rate);
        } else {
            const int64_t m = r.m_offset + i + 1;
            const double log_eps = dual_avg_apply_fma(s.da, da_of(m), alpha, r.target_accept);
            s.eps = (m < r.adapt_total) ? exp(log_eps) : exp(s.da.log_eps_bar);
        }
    }
    if (!writer) return;
    if (i >= r.n_burnin) {
        const int64_t k = (i - r.n_burnin) * C + c;
        if (r.trace.step_size) r.trace.step_size[k] = eps_used;
        if (r.trace.is_accepted) r.trace.is_accepted[k] = acc ? 1 : 0;
        if (r.trace.log_accept_ratio) r.trace.log_accept_ratio[k] = lar;
        if (r.trace.target_log_prob) r.trace.target_log_prob[k] = lp_new;
    }
    if (!OUT) return;
    if (r.out.is_accepted) r.out.is_accepted[c] = acc ? 1 : 0;
    if (r.out.log_accept_ratio) r.out.log_accept_ratio[c] = lar;
    if (r.out.target_log_prob) r.out.target_log_prob[c] = lp_new;
    if (r.out.delta_h) r.out.delta_h[c] = dh;
}

// ---------------------------------------------------------------------------
// Elementwise targets.  NB blocks of 4 dims per lane; lane j of a group owns
// blocks j, j + G, ...
// ---------------------------------------------------------------------------
// EX: a transform and / or the replica exchange inside the launch (a template
// parameter, so that plain runs carry neither).  With the exchange, lane group
// (slot) s holds replica s % K of chain index s / K; K divides the 64 / G slots
// of a wavefront, so the two chains of every pair exchange by shuffles G lanes
// apart.
// Transformed kernel (x = shift + scale z, EX): the chain runs in z = x / scale,
// whose precision is prec scale^2; states are converted at load and store.
// ND: dims of a block held (4, or the dims themselves where they are fewer).
// WIDE (FP64 beyond 1024 dims): x, g, the precisions, the trajectory and its gradient
// would take 640 of 512 registers.  The new gradient is formed again where it is used
// after the trajectory (one product an element, the same bits), the code of a leapfrog
// step stands once, and the state is loaded a block at a time: N(0, I) D = 2048, 3000
// chains, 20 transitions 752 -> 616 us, one 108 -> 95; D = 1358 675 -> 570, 92 -> 84.
template <typename T, int G, int NB, bool EX, int ND = 4>
struct ElemChain {
    static constexpr bool WIDE = NB * sizeof(T) > 32;
    struct __attribute__((packed, aligned(sizeof(T)))) T4 { T v[ND]; };   // rows are at least element-aligned
    T x[NB][ND], g[NB][ND], pr[NB][ND];
    bool ok[NB][ND];
    ChainCtl s;
    double bt;               // inverse temperature of the chain
    int lane, nrep, krep;
    int64_t c, cc;
    bool active;
    const double* sc;        // the transform's scale, or NULL
    const T* sc_lds;         // and in the state's precision, staged in LDS for the stores of x

    // slot: the lane group's index over the whole launch
    __device__ __forceinline__ void load(const PlainArgs& a, const FusedRun& r, int64_t slot, int lane_,
                                         const T* sc_lds_) {
        lane = lane_;
        nrep = EX ? r.remc_K : 0;
        krep = nrep > 1 ? (int)(slot % nrep) : 0;
        c = nrep > 1 ? krep * r.remc_M + slot / nrep : slot;
        active = slot < a.C;                  // with the exchange: chain index slot / K < M
        cc = active ? c : 0;
        sc = EX ? a.ws.scale : nullptr;
        sc_lds = sc_lds_;
        const int64_t D = a.tg.D;
        const bool diag = a.tg.kind == HMC_TGT_GAUSS_DIAG;
        const T* X = (const T*)a.ws.x;
        const T* Gr = (const T*)a.ws.g;
        const T* prec = (const T*)a.tg.prec;
        if constexpr (WIDE) {
#pragma unroll
            for (int k = 0; k < NB; ++k)
#pragma unroll
                for (int j = 0; j < ND; ++j) ok[k][j] = active && 4 * (lane + (int64_t)G * k) + j < D;
            // whole blocks in a loop of their own: one loop for both kinds loses half the gain
#pragma unroll
            for (int k = 0; k < NB; ++k)
                if (ok[k][ND - 1]) {
                    const int64_t d = 4 * (lane + (int64_t)G * k);
                    const T4 xv = *(const T4*)(X + cc * D + d), gv = *(const T4*)(Gr + cc * D + d);
                    T4 pv;
                    if (diag) pv = *(const T4*)(prec + d);
#pragma unroll
                    for (int j = 0; j < ND; ++j) {
                        x[k][j] = xv.v[j];
                        g[k][j] = gv.v[j];
                        pr[k][j] = diag ? pv.v[j] : (T)1;
                    }
                }
        }
#pragma unroll
        for (int k = 0; k < NB; ++k)
#pragma unroll
            for (int j = 0; j < ND; ++j) {
                const int64_t d = 4 * (lane + (int64_t)G * k) + j;
                if (!WIDE) ok[k][j] = active && d < D;
                if (!(WIDE && ok[k][ND - 1])) {
                    x[k][j] = ok[k][j] ? X[cc * D + d] : (T)0;
                    g[k][j] = ok[k][j] ? Gr[cc * D + d] : (T)0;
                    pr[k][j] = ok[k][j] ? (diag ? prec[d] : (T)1) : (T)0;
                }
                if (sc && ok[k][j]) {
                    const double sd = sc[d];
                    pr[k][j] = (T)((double)pr[k][j] * sd * sd);
                    x[k][j] = (T)((double)x[k][j] / sd);
                    g[k][j] = (T)((double)g[k][j] * sd);
                }
            }
        s.logp = a.ws.logp[cc];
        s.eps = a.ws.eps[cc];
        s.da = a.ws.da[cc];
        bt = a.ws.beta ? a.ws.beta[cc] : 1.0;
    }

    // Transition i of the launch, t of the run.  Random numbers and the
    // dual-averaging factors through draw(k, z) (momenta of block k), accept(lar)
    // (log of the accept uniform < lar), swap(b_side, thr) (log of the exchange
    // uniform of this chain's pair < thr) and da_of(m), so that they can be computed
    // here or taken from LDS.
    // OUT: the outputs of hmc_step may be asked for (single transitions).
    template <bool OUT, typename Draw, typename Accept, typename Swap, typename DaOf>
    __device__ __forceinline__ void transition(const PlainArgs& a, const FusedRun& r, int64_t i, uint32_t t, Draw draw,
                                               Accept accept, Swap swap, DaOf da_of) {
        const int64_t D = a.tg.D;
        const bool trs = sc != nullptr;
        const T eps = (T)s.eps;                   // drift
        const T half = (T)(0.5 * s.eps * bt);     // kicks: beta eps (replica exchange; beta = 1 otherwise)
        const T keps = (T)(s.eps * bt);
        T xn[NB][ND], pn[NB][ND], gk[WIDE ? 1 : NB][ND];
        auto gn = [&](int k, int j) { return WIDE ? -pr[k][j] * xn[k][j] : gk[WIDE ? 0 : k][j]; };
        // dk and lp are summed without their factor 1/2 (exact in binary, applied below)
        double dk = 0.0;
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            T z[4];
            draw(k, z);
#pragma unroll
            for (int j = 0; j < ND; ++j) {
                const T p0 = ok[k][j] ? z[j] : (T)0;
                dk = fma(-(double)p0, (double)p0, dk);
                xn[k][j] = x[k][j];
                pn[k][j] = fma(half, g[k][j], p0);
            }
        }
        auto leap = [&](T ke) {
#pragma unroll
            for (int k = 0; k < NB; ++k)
#pragma unroll
                for (int j = 0; j < ND; ++j) {
                    xn[k][j] = fma(eps, pn[k][j], xn[k][j]);
                    const T gv = -pr[k][j] * xn[k][j];
                    if (!WIDE) gk[WIDE ? 0 : k][j] = gv;
                    pn[k][j] = fma(ke, gv, pn[k][j]);
                }
        };
        // The last step apart: in FP64 the choice of the factor in the chain of
        // dependent operations is not free (D = 1 run 158 -> 154 us, D = 37 135 ->
        // 128); in FP32 the shorter code is (D = 1000, 1000 chains 907 against 934).
        if constexpr (sizeof(T) == 8 && !WIDE) {
            for (int l = 1; l < a.L; ++l) leap(keps);
            leap(half);
        } else {
            for (int l = 0; l < a.L; ++l) leap(l == a.L - 1 ? half : keps);
        }
        double lp = 0.0;
#pragma unroll
        for (int k = 0; k < NB; ++k)
#pragma unroll
            for (int j = 0; j < ND; ++j) {
                dk = fma((double)pn[k][j], (double)pn[k][j], dk);
                lp = fma((double)xn[k][j], (double)gn(k, j), lp);
            }
        dk = 0.5 * group_sum<G>(dk);
        lp = 0.5 * group_sum<G>(lp);
        const double dh = -(bt * lp) + bt * s.logp + dk;
        const double lar = log_accept_ratio_of(dh);
        const bool acc = accept(lar);
        if (acc) {
#pragma unroll
            for (int k = 0; k < NB; ++k)
#pragma unroll
                for (int j = 0; j < ND; ++j) {
                    x[k][j] = xn[k][j];
                    g[k][j] = gn(k, j);
                }
            s.logp = lp;
        }
        // four dims of a row at p + d, as one store where the block is whole
        auto store4 = [&](T* p, int k, const T (&v)[ND]) {
            if (ok[k][ND - 1]) {
                T4 o;
#pragma unroll
                for (int j = 0; j < ND; ++j) o.v[j] = v[j];
                *(T4*)p = o;
            } else {
#pragma unroll
                for (int j = 0; j < ND - 1; ++j)
                    if (ok[k][j]) p[j] = v[j];
            }
        };
        // kept sample and proposal outputs of this transition
        auto store_outputs = [&]() {
            int l4 = 4 * lane;
            // an index the compiler cannot see through keeps the LDS reads of the scale
            // here: hoisted out of the transition loop they would hold NB 4 registers
            // for the whole run
            if (EX) asm volatile("" : "+v"(l4));
            auto scaled = [&](int k, const T (&v)[ND], T (&o)[ND]) {
#pragma unroll
                for (int j = 0; j < ND; ++j) o[j] = (EX && trs) ? v[j] * sc_lds[l4 + 4 * G * k + j] : v[j];
            };
            if (r.samples && i >= r.n_burnin) {
                T* smp = (T*)r.samples + ((i - r.n_burnin) * a.C + c) * D;
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    T o[ND];
                    scaled(k, x[k], o);
                    store4(smp + 4 * (lane + (int64_t)G * k), k, o);
                }
            }
            if (OUT && (r.out.proposed_state || r.out.proposed_momentum)) {
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    const int64_t d = c * D + 4 * (lane + (int64_t)G * k);
                    if (r.out.proposed_state) {
                        T o[ND];
                        scaled(k, xn[k], o);
                        store4((T*)r.out.proposed_state + d, k, o);
                    }
                    if (r.out.proposed_momentum) store4((T*)r.out.proposed_momentum + d, k, pn[k]);
                }
            }
        };
        if (EX) {
            // traces and adaptation record the transition; the exchange follows
            // it, and the kept sample is the state after the exchange
            if (active) after_decision<OUT>(r, a.C, c, i, acc, lar, dh, s.logp, s, lane == 0, da_of);
            if (nrep > 1) {
                const int par = (int)(t & 1u);
                const bool a_side = krep >= par && ((krep - par) & 1) == 0 && krep + 1 < nrep;
                const bool b_side = krep >= par + 1 && ((krep - 1 - par) & 1) == 0;
                const int wl = threadIdx.x & 63;
                const int src = a_side ? wl + G : (b_side ? wl - G : wl);
                const double lp_o = __shfl(s.logp, src, 64);
                const double bt_o = __shfl(bt, src, 64);
                bool swp = false;
                if (active && (a_side || b_side)) {
                    const double la = a_side ? s.logp : lp_o, lb = a_side ? lp_o : s.logp;
                    const double ba = a_side ? bt : bt_o, bb = a_side ? bt_o : bt;
                    swp = swap(b_side, (ba - bb) * (lb - la));
                }
#pragma unroll
                for (int k = 0; k < NB; ++k)
#pragma unroll
                    for (int j = 0; j < ND; ++j) {
                        const T xo = __shfl(x[k][j], src, 64), go = __shfl(g[k][j], src, 64);
                        if (swp) {
                            x[k][j] = xo;
                            g[k][j] = go;
                        }
                    }
                if (swp) s.logp = lp_o;
                if (active && r.swapped && i >= r.n_burnin && lane == 0)
                    r.swapped[(i - r.n_burnin) * a.C + c] = swp ? 1 : 0;
            }
            if (active) store_outputs();
        } else if (active) {
            store_outputs();
            after_decision<OUT>(r, a.C, c, i, acc, lar, dh, s.logp, s, lane == 0, da_of);
        }
    }

    __device__ __forceinline__ void store(const PlainArgs& a) {
        if (!active) return;
        const int64_t D = a.tg.D;
        const bool trs = sc != nullptr;
        T* X = (T*)a.ws.x;
        T* Gr = (T*)a.ws.g;
        // a fresh read of the scale: reusing the values loaded before the loop
        // would hold them in registers for the whole run
        if (EX) asm volatile("" ::: "memory");
#pragma unroll
        for (int k = 0; k < NB; ++k)
#pragma unroll
            for (int j = 0; j < ND; ++j)
                if (ok[k][j]) {
                    const int64_t d = 4 * (lane + (int64_t)G * k) + j;
                    X[c * D + d] = (EX && trs) ? (T)((double)x[k][j] * sc[d]) : x[k][j];
                    Gr[c * D + d] = (EX && trs) ? (T)((double)g[k][j] / sc[d]) : g[k][j];
                }
        if (lane == 0) {
            a.ws.logp[c] = s.logp;
            a.ws.eps[c] = s.eps;
            a.ws.da[c] = s.da;
        }
    }
};

// the scale in the state's precision, staged once in LDS for the stores of x (a
// lane group covers 4 G NB >= D dims)
template <typename T, bool EX>
__device__ __forceinline__ void elem_stage_scale(const PlainArgs& a, T* sc_lds) {
    if (!EX) return;
    if (a.ws.scale)
        for (int64_t d = threadIdx.x; d < a.tg.D; d += blockDim.x) sc_lds[d] = (T)a.ws.scale[d];
    __syncthreads();
}

template <typename T, int G, int NB, bool EX>
__device__ __forceinline__ void fused_elem_body(const PlainArgs& a, const FusedRun& r, int64_t lblock) {
    const int64_t gid = lblock * blockDim.x + threadIdx.x;
    __shared__ T sc_lds[EX ? 4 * G * NB : 1];
    elem_stage_scale<T, EX>(a, sc_lds);
    ElemChain<T, G, NB, EX> ch;
    ch.load(a, r, gid / G, (int)(threadIdx.x % G), sc_lds);
    const int64_t D = a.tg.D;
    for (int64_t i = 0; i < r.n_transitions; ++i) {
        const uint32_t t = (uint32_t)(r.t_begin + i);
        ch.template transition<true>(
            a, r, i, t,
            [&](int k, T (&z)[4]) {
                momentum4<T>(a.key, (uint32_t)ch.cc, t, (uint32_t)(ch.lane + G * k), z,
                             4 * (ch.lane + (int64_t)G * k) + 2 < D);
            },
            [&](double lar) { return accept_below(a.key, (uint32_t)ch.cc, t, lar); },
            [&](bool b_side, double thr) {
                return log_uniform52_below(a.key, (uint32_t)(b_side ? ch.c - r.remc_M : ch.c), t, TAG_SWAP, thr);
            },
            [&](int64_t m) { return dual_avg_const((double)m, r.gamma, r.t0, r.kappa); });
    }
    ch.store(a);
}

// ---------------------------------------------------------------------------
// Few chains: when the lane groups of all chains are at most a wavefront per
// SIMD, a run's time is one wavefront's instruction stream, and two thirds of it
// are draws (Philox, FP64 logarithms, Box-Muller) that do not depend on the
// chain.  Here a workgroup of 8 waves owns `chains` chains, as few as spread all
// of them over the 256 CUs; its first waves run the transitions with momenta,
// accept and exchange uniforms and dual-averaging factors read from LDS, while
// the others draw those of the next block of transitions, every lane a different
// (transition, chain, block).  The arithmetic is that of fused_elem_body on the
// same numbers: results are bitwise the same.  Whole runs, before and after: N(0,
// 1) FP64, 100 chains, 400 transitions 485 -> 154 us; diagonal D = 37 FP64, 332
// chains in 4 replicas, 100 transitions 311 -> 130; D = 333 FP32, 1000 chains, 64
// transitions 178 -> 103 (there the draws bound it on either side); N(0, I) D = 3
// FP64, 16384 chains, 80 transitions 159 -> 68.
// ---------------------------------------------------------------------------
constexpr int EF_THREADS = 512;
struct ElemFew {
    int32_t chains;          // per workgroup
    int32_t bt;              // transitions per block of draws
};
// LDS doubles per chain and transition besides the momenta: accept and exchange uniform; three more per transition
template <typename T, int G, int NB>
constexpr size_t elem_few_lds(int chains, int bt) {
    return (size_t)2 * bt * ((size_t)chains * G * NB * 4 * sizeof(T) + (2 * chains + 4) * sizeof(double));
}

template <typename T, int G, int NB, bool EX, int ND>
__global__ __launch_bounds__(EF_THREADS) void k_fused_elem_few(PlainArgs a, FusedRun r, ElemFew f) {
    extern __shared__ __align__(16) uint8_t few_lds[];
    __shared__ T sc_lds[EX ? 4 * G * NB : 1];
    elem_stage_scale<T, EX>(a, sc_lds);
    struct __attribute__((aligned(16))) Z4 { T v[4]; };
    const int lw = f.chains * G;                            // owner lanes (<= 256)
    const int nw = (lw + 63) & ~63;                         // owner threads, whole waves
    Z4* zb = (Z4*)few_lds;                                  // [2][bt][NB][lw]
    double* lub = (double*)(zb + (size_t)2 * f.bt * NB * lw);       // [2][bt][chains] log accept uniforms
    double* swb = lub + (size_t)2 * f.bt * f.chains;        // [2][bt][chains] log exchange uniforms
    double* dab = swb + (size_t)2 * f.bt * f.chains;        // [2][bt][4] dual-averaging factors
    const int64_t D = a.tg.D, T0 = r.n_transitions;
    const int64_t slot0 = (int64_t)blockIdx.x * f.chains;
    const int nrep = EX ? r.remc_K : 0;
    auto chain_of = [&](int s) -> int64_t {
        const int64_t slot = slot0 + s;
        if (slot >= a.C) return -1;
        return nrep > 1 ? (slot % nrep) * r.remc_M + slot / nrep : slot;
    };
    // A thread's tasks of a block of draws: me, me + n, ... as (transition q, chain
    // cs, part p of np), stepped without divisions.
    struct Task {
        int q, cs, p, dq, dcs, dp, np, nc;
        __device__ __forceinline__ void init(int me, int n, int np_, int nc_) {
            np = np_;
            nc = nc_;
            p = me % np; cs = me / np % nc; q = me / np / nc;
            dp = n % np; dcs = n / np % nc; dq = n / np / nc;
        }
        __device__ __forceinline__ void next() {
            p += dp;
            const int c1 = p >= np ? 1 : 0;
            p -= c1 ? np : 0;
            cs += dcs + c1;
            const int c2 = cs >= nc ? 1 : 0;
            cs -= c2 ? nc : 0;
            q += dq + c2;
        }
    };
    const int nblk = (int)((D + 3) / 4);
    // draws of transitions i0 .. i0 + bt - 1 into half b, by threads me of n: one block
    // of four dims per task, and the uniforms by threads of their own (zt counts from
    // the first thread, ut from the last)
    auto produce = [&](int64_t i0, int b, Task zt, Task ut, int mine, int n) {
        const int nt = T0 - i0 < f.bt ? (int)(T0 - i0) : f.bt;
        for (; zt.q < nt; zt.next()) {
            const int64_t c = chain_of(zt.cs);
            if (c >= 0) {
                Z4 z;
                momentum4<T>(a.key, (uint32_t)c, (uint32_t)(r.t_begin + i0 + zt.q), (uint32_t)zt.p, z.v,
                             4 * (int64_t)zt.p + 2 < D);
                zb[((size_t)b * f.bt + zt.q) * (NB * lw) + (zt.p / G) * lw + zt.cs * G + zt.p % G] = z;
            }
        }
        for (; ut.q < nt; ut.next()) {
            const int64_t c = chain_of(ut.cs);
            if (c < 0) continue;
            const uint32_t t = (uint32_t)(r.t_begin + i0 + ut.q);
            lub[((size_t)b * f.bt + ut.q) * f.chains + ut.cs] = log_accept_uniform(a.key, (uint32_t)c, t);
            if (EX && nrep > 1)
                swb[((size_t)b * f.bt + ut.q) * f.chains + ut.cs] = log_uniform52(a.key, (uint32_t)c, t, TAG_SWAP);
        }
        if (r.adapt && r.adapt_kind != HMC_ADAPT_SIMPLE)
            for (int q = mine; q < nt; q += n)
                if (i0 + q < r.n_burnin) {
                    const DaConst o = dual_avg_const((double)(r.m_offset + i0 + q + 1), r.gamma, r.t0, r.kappa);
                    double* d = dab + ((size_t)b * f.bt + q) * 4;
                    d[0] = o.w;
                    d[1] = o.k;
                    d[2] = o.eta;
                }
    };
    const int tid = (int)threadIdx.x;
    const bool owner = tid < lw;
    ElemChain<T, G, NB, EX, ND> ch;
    if (owner) ch.load(a, r, slot0 + tid / G, tid % G, sc_lds);
    {
        Task zt, ut;
        zt.init(tid, EF_THREADS, nblk, f.chains);
        ut.init(EF_THREADS - 1 - tid, EF_THREADS, 1, f.chains);
        produce(0, 0, zt, ut, EF_THREADS - 1 - tid, EF_THREADS);
    }
    Task zt, ut;
    const int np = EF_THREADS - nw, me = tid >= nw ? tid - nw : 0;
    zt.init(me, np, nblk, f.chains);
    ut.init(np - 1 - me, np, 1, f.chains);
    __syncthreads();
    int b = 0;
    for (int64_t i0 = 0; i0 < T0; i0 += f.bt, b ^= 1) {
        if (tid >= nw) {
            if (i0 + f.bt < T0) produce(i0 + f.bt, b ^ 1, zt, ut, np - 1 - me, np);
        } else if (owner) {
            const int nt = T0 - i0 < f.bt ? (int)(T0 - i0) : f.bt;
            const Z4* zq = zb + (size_t)b * f.bt * (NB * lw) + tid;
            const double* lq = lub + (size_t)b * f.bt * f.chains + tid / G;
            const double* sq = swb + (size_t)b * f.bt * f.chains + tid / G;
            const double* dq = dab + (size_t)b * f.bt * 4;
            // the draws of a transition are read during the one before it
            Z4 zc[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) zc[k] = zq[k * lw];
            double lc = *lq;
            for (int q = 0; q < nt; ++q) {
                const int more = q + 1 < nt ? 1 : 0;
                zq += more * (NB * lw);
                lq += more * f.chains;
                Z4 zn[NB];
#pragma unroll
                for (int k = 0; k < NB; ++k) zn[k] = zq[k * lw];
                const double ln = *lq;
                const double own = EX ? sq[q * f.chains] : 0.0, below = EX ? sq[q * f.chains - 1] : 0.0;
                ch.template transition<false>(
                    a, r, i0 + q, (uint32_t)(r.t_begin + i0 + q),
                    [&](int k, T (&z)[4]) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) z[j] = zc[k].v[j];
                    },
                    [&](double lar) { return lc < lar; },
                    [&](bool b_side, double thr) { return (b_side ? below : own) < thr; },
                    [&](int64_t) { return DaConst{dq[4 * q], dq[4 * q + 1], dq[4 * q + 2]}; });
#pragma unroll
                for (int k = 0; k < NB; ++k) zc[k] = zn[k];
                lc = ln;
            }
        }
        __syncthreads();
    }
    if (owner) ch.store(a);
}

template <typename T, int G, int NB, bool EX>
__global__ __launch_bounds__(256) void k_fused_elem(PlainArgs a, FusedRun r) {
    fused_elem_body<T, G, NB, EX>(a, r, blockIdx.x);
}

// Several requests of one shape class in one grid: block b runs job j with
// jobs[j].block_begin <= b < jobs[j + 1].block_begin.
template <typename T, int G, int NB>
__global__ __launch_bounds__(256) void k_fused_elem_multi(const ElemJob* __restrict__ jobs, int njobs) {
    int lo = 0, hi = njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].block_begin <= (int64_t)blockIdx.x) lo = mid;
        else hi = mid - 1;
    }
    const PlainArgs a = jobs[lo].a;
    const FusedRun r = jobs[lo].r;
    fused_elem_body<T, G, NB, false>(a, r, (int64_t)blockIdx.x - jobs[lo].block_begin);
}

// ---------------------------------------------------------------------------
// Dense Gaussian on MFMA.  16 chains per workgroup (the N dimension), 8 waves
// (two per SIMD, so that one wave's MFMAs cover the other's LDS and barrier
// waits), wave w owns M-tiles w, w + NW, ...; lane (g4 = lane/16, i16 = lane%16) holds rows
// 16 mt + 4 g4 + v (v = 0..3) of chain i16 -- exactly the 4 dims of Philox
// block 4 mt + g4, so each lane draws its own momenta.
//
// NT = ceil(D / 16) tiles is a template parameter, so the contraction over
// the 4 NT k-steps is fully unrolled with no guards: P is zero-padded in the
// A operands and rows D .. 16 NT of x stay exactly zero, so the padding adds
// zeros.  Every wave runs MT tiles (a wave's tiles past NT multiply zeros on
// its own SIMD while the other SIMDs finish theirs), and each tile keeps two
// accumulators (even / odd k-steps) so that consecutive MFMAs are independent.
//
// The contraction index is assigned as k = g4 KM + ks (lane group g4 supplies
// dims g4 KM .. g4 KM + KM - 1 over the k-steps ks), so with x staged chain-
// major in LDS ([16 chains][16 NT + 4], the pad making the 16 chains of a
// lane group hit distinct bank quads) each lane fetches the B operands of 4
// consecutive k-steps with one ds_read_b128 and writes its own 4 dims of a
// tile with one ds_write_b128.
// ---------------------------------------------------------------------------
constexpr int DENSE_NW = 8;                 // waves per workgroup (2 per SIMD)

// EX: a transform and / or the replica exchange inside the launch (a template
// parameter, so that plain runs carry neither).  With the exchange, slot i16
// of the workgroup holds replica i16 % K of chain m = 16 / K * block + i16 / K,
// so the two chains of every pair sit in neighbouring lanes of one wavefront
// and exchange by shuffles.
template <int NT, bool EX>
__global__ __launch_bounds__(64 * DENSE_NW) void k_fused_dense(PlainArgs a, FusedRun r) {
    constexpr int MT = (NT + DENSE_NW - 1) / DENSE_NW;
    constexpr int KM = 4 * NT;
    extern __shared__ float lds[];
    const int64_t D = a.tg.D;
    const int ntiles = NT;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i16 = lane & 15, g4 = lane >> 4;
    const int nrep = EX ? r.remc_K : 0;
    const int krep = nrep > 1 ? i16 % nrep : 0;
    const int64_t mrep = nrep > 1 ? (int64_t)blockIdx.x * (16 / nrep) + i16 / nrep : 0;
    const int64_t c = nrep > 1 ? krep * r.remc_M + mrep : (int64_t)blockIdx.x * 16 + i16;
    const bool cvalid = nrep > 1 ? mrep < r.remc_M : c < a.C;
    const int64_t cc = cvalid ? c : 0;
    constexpr int XS = 16 * NT + 4;                 // floats per chain row in LDS
    float* xs0 = lds;                               // [16][XS] x 2 buffers
    float* xs1 = lds + 16 * XS;
    double* red = (double*)(lds + 2 * 16 * XS);     // [2][NW][16] (dk, lp)
    const float* P = (const float*)a.tg.prec;
    float* X = (float*)a.ws.x;
    float* Gr = (float*)a.ws.g;

    // Transformed kernel (x = shift + scale z, EX): the chain runs in
    // z = x / scale, whose precision matrix is S P S (S = diag(scale)); states
    // are converted at load and store.
    const double* sc = EX ? a.ws.scale : nullptr;
    const bool trs = sc != nullptr;
    __shared__ float sc_lds[EX ? 16 * NT : 1];     // the scale, for the stores of x
    if (EX) {
        if (trs)
            for (int d = threadIdx.x; d < D; d += blockDim.x) sc_lds[d] = (float)sc[d];
        __syncthreads();
    }
    // P as A operands: pa[m][ks] = P[16 mt + i16][g4 KM + ks]
    float pa[MT][KM];
    bool tile_ok[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int mt = w + DENSE_NW * m;
        tile_ok[m] = mt < ntiles;
        const int64_t row = 16 * mt + i16;
#pragma unroll
        for (int ks = 0; ks < KM; ++ks) {
            const int64_t col = (int64_t)g4 * KM + ks;
            const bool in = tile_ok[m] && row < D && col < D;
            pa[m][ks] = in ? P[row * D + col] : 0.f;
            if (sc && in) pa[m][ks] = (float)((double)pa[m][ks] * sc[row] * sc[col]);
        }
    }
    float x[MT][4], g[MT][4];
    bool ok[MT][4];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int64_t d = 16 * (w + DENSE_NW * m) + 4 * g4 + v;
            ok[m][v] = tile_ok[m] && cvalid && d < D;
            x[m][v] = ok[m][v] ? X[cc * D + d] : 0.f;
            g[m][v] = ok[m][v] ? Gr[cc * D + d] : 0.f;
            if (sc && ok[m][v]) {
                x[m][v] = (float)((double)x[m][v] / sc[d]);
                g[m][v] = (float)((double)g[m][v] * sc[d]);
            }
        }
    ChainCtl s;
    s.logp = a.ws.logp[cc];
    s.eps = a.ws.eps[cc];
    s.da = a.ws.da[cc];
    const double bt = a.ws.beta ? a.ws.beta[cc] : 1.0;   // inverse temperature of the chain
    int buf = 0;

    for (int64_t i = 0; i < r.n_transitions; ++i) {
        const uint32_t t = (uint32_t)(r.t_begin + i);
        const float eps = (float)s.eps, half = (float)(0.5 * s.eps * bt), keps = (float)(s.eps * bt);
        float xn[MT][4], pn[MT][4], gn[MT][4];
        double dk = 0.0;
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            float z[4];
            momentum4<float>(a.key, (uint32_t)cc, t, (uint32_t)(4 * (w + DENSE_NW * m) + g4), z);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float p0 = ok[m][v] ? z[v] : 0.f;
                dk -= 0.5 * (double)p0 * (double)p0;
                xn[m][v] = x[m][v];
                pn[m][v] = fmaf(half, g[m][v], p0);
                gn[m][v] = 0.f;
            }
        }
        for (int l = 0; l < a.L; ++l) {
            const float ke = (l == a.L - 1) ? half : keps;
            float* xs = buf ? xs1 : xs0;
#pragma unroll
            for (int m = 0; m < MT; ++m) {
#pragma unroll
                for (int v = 0; v < 4; ++v) xn[m][v] = fmaf(eps, pn[m][v], xn[m][v]);
                if (tile_ok[m])
                    *(floatx4*)(xs + i16 * XS + 16 * (w + DENSE_NW * m) + 4 * g4) =
                        floatx4{xn[m][0], xn[m][1], xn[m][2], xn[m][3]};
            }
            __syncthreads();
            floatx4 bq[NT];
#pragma unroll
            for (int q = 0; q < NT; ++q) bq[q] = *(const floatx4*)(xs + i16 * XS + g4 * KM + 4 * q);
            floatx4 acc[MT][2];
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                acc[m][0] = floatx4{0.f, 0.f, 0.f, 0.f};
                acc[m][1] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int ks = 0; ks < KM; ++ks) {
                const float bv = bq[ks >> 2][ks & 3];
#pragma unroll
                for (int m = 0; m < MT; ++m)
                    acc[m][ks & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(pa[m][ks], bv, acc[m][ks & 1], 0, 0, 0);
            }
            // all operand reads first (one LDS latency per step), then the MFMAs
            __builtin_amdgcn_sched_group_barrier(0x100, NT, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, KM * MT, 0);
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    gn[m][v] = -(acc[m][0][v] + acc[m][1][v]);
                    pn[m][v] = fmaf(ke, gn[m][v], pn[m][v]);
                }
            buf ^= 1;
        }
        double lp = 0.0;
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (ok[m][v]) {
                    dk += 0.5 * (double)pn[m][v] * (double)pn[m][v];
                    lp += 0.5 * (double)xn[m][v] * (double)gn[m][v];
                }
        dk += __shfl_xor(dk, 16, 64);
        dk += __shfl_xor(dk, 32, 64);
        lp += __shfl_xor(lp, 16, 64);
        lp += __shfl_xor(lp, 32, 64);
        double* rb = red + (i & 1) * (2 * DENSE_NW * 16);
        if (g4 == 0) {
            rb[(2 * w) * 16 + i16] = dk;
            rb[(2 * w + 1) * 16 + i16] = lp;
        }
        __syncthreads();
        dk = 0.0;
        lp = 0.0;
#pragma unroll
        for (int ww = 0; ww < DENSE_NW; ++ww) {
            dk += rb[(2 * ww) * 16 + i16];
            lp += rb[(2 * ww + 1) * 16 + i16];
        }
        const double dh = -(bt * lp) + bt * s.logp + dk;
        const double lar = log_accept_ratio_of(dh);
        const bool acc = accept_below(a.key, (uint32_t)cc, t, lar);
        if (acc) {
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    x[m][v] = xn[m][v];
                    g[m][v] = gn[m][v];
                }
            s.logp = lp;
        }
        // traces and adaptation record the transition; the exchange follows it,
        // and the kept sample is the state after the exchange
        if (cvalid)
            after_decision<true>(r, a.C, c, i, acc, lar, dh, s.logp, s, w == 0 && g4 == 0, [&](int64_t m) {
                return dual_avg_const((double)m, r.gamma, r.t0, r.kappa);
            });
        if (EX && nrep > 1) {
            const int par = (int)(t & 1u);
            const bool a_side = krep >= par && ((krep - par) & 1) == 0 && krep + 1 < nrep;
            const bool b_side = krep >= par + 1 && ((krep - 1 - par) & 1) == 0;
            const int src = a_side ? lane + 1 : (b_side ? lane - 1 : lane);
            const double lp_o = __shfl(s.logp, src, 64);
            const double bt_o = __shfl(bt, src, 64);
            bool swp = false;
            if (cvalid && (a_side || b_side)) {
                const int64_t ca = a_side ? c : c - r.remc_M;
                const double la = a_side ? s.logp : lp_o, lb = a_side ? lp_o : s.logp;
                const double ba = a_side ? bt : bt_o, bb = a_side ? bt_o : bt;
                swp = log_uniform52_below(a.key, (uint32_t)ca, t, TAG_SWAP, (ba - bb) * (lb - la));
            }
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float xo = __shfl(x[m][v], src, 64), go = __shfl(g[m][v], src, 64);
                    if (swp) {
                        x[m][v] = xo;
                        g[m][v] = go;
                    }
                }
            if (swp) s.logp = lp_o;
            if (cvalid && r.swapped && i >= r.n_burnin && w == 0 && g4 == 0)
                r.swapped[(i - r.n_burnin) * a.C + c] = swp ? 1 : 0;
        }
        if (cvalid) {
            const bool want_smp = r.samples && i >= r.n_burnin;
            int q = 16 * w + 4 * g4;                 // opaque: keeps the LDS reads of the scale here
            if (EX) asm volatile("" : "+v"(q));
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (ok[m][v]) {
                        const int64_t d = 16 * (w + DENSE_NW * m) + 4 * g4 + v;
                        const float sd = (EX && trs) ? sc_lds[q + 16 * DENSE_NW * m + v] : 1.f;
                        if (want_smp)
                            ((float*)r.samples)[((i - r.n_burnin) * a.C + c) * D + d] =
                                (EX && trs) ? x[m][v] * sd : x[m][v];
                        if (r.out.proposed_state)
                            ((float*)r.out.proposed_state)[c * D + d] = (EX && trs) ? xn[m][v] * sd : xn[m][v];
                        if (r.out.proposed_momentum) ((float*)r.out.proposed_momentum)[c * D + d] = pn[m][v];
                    }
        }
    }
    if (!cvalid) return;
    if (EX) asm volatile("" ::: "memory");   // a fresh read of the scale (see the element-wise kernel)
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (ok[m][v]) {
                const int64_t d = 16 * (w + DENSE_NW * m) + 4 * g4 + v;
                X[c * D + d] = sc ? (float)((double)x[m][v] * sc[d]) : x[m][v];
                Gr[c * D + d] = sc ? (float)((double)g[m][v] / sc[d]) : g[m][v];
            }
    if (w == 0 && g4 == 0) {
        a.ws.logp[c] = s.logp;
        a.ws.eps[c] = s.eps;
        a.ws.da[c] = s.da;
    }
}

// ---------------------------------------------------------------------------
// Launch selection
// ---------------------------------------------------------------------------
bool fused_logreg_supported(const PlainArgs& a);
hipError_t launch_fused_logreg(const PlainArgs& a, const FusedRun& r, hipStream_t s);

static int elem_nb(int64_t D, int* G) {
    // lanes per chain and 4-blocks per lane
    const int64_t nblk = (D + 3) / 4;
    if (nblk <= 1) { *G = 1; return 1; }
    if (nblk <= 4) { *G = 4; return 1; }
    if (nblk <= 16) { *G = 16; return 1; }
    if (nblk <= 64) { *G = 64; return 1; }
    if (nblk <= 128) { *G = 64; return 2; }
    if (nblk <= 256) { *G = 64; return 4; }
    if (nblk <= 512) { *G = 64; return 8; }
    *G = 0;
    return 0;
}

bool fused_supported(const PlainArgs& a) {
    switch (a.tg.kind) {
    case HMC_TGT_STD_NORMAL:
    case HMC_TGT_GAUSS_DIAG: {
        int G;
        return elem_nb(a.tg.D, &G) > 0;
    }
    case HMC_TGT_GAUSS_DENSE:
        return !a.f64 && a.tg.D <= 128;
    case HMC_TGT_LOGREG:
        return fused_logreg_supported(a);
    }
    return false;
}

static int elem_class_of(int G, int NB) {
    if (G == 1) return 0;
    if (G == 4) return 1;
    if (G == 16) return 2;
    return NB == 1 ? 3 : (NB == 2 ? 4 : (NB == 4 ? 5 : 6));
}

// lanes per chain G and 4-blocks per lane NB, after the tuned multiplier
// (doubling G halves NB when the blocks still cover D)
static int elem_shape(const PlainArgs& a, int* G) {
    int NB = elem_nb(a.tg.D, G);
    if (NB == 0) return 0;
    if (a.tune.elem_gmult == 2 && *G < 64) *G = *G == 1 ? 4 : 4 * *G;   // next wider lane group
    return NB;
}

int elem_class(const PlainArgs& a) {
    if (a.tg.kind != HMC_TGT_STD_NORMAL && a.tg.kind != HMC_TGT_GAUSS_DIAG) return -1;
    int G;
    const int NB = elem_shape(a, &G);
    if (NB == 0) return -1;
    return (a.f64 ? 8 : 0) + elem_class_of(G, NB);
}

int64_t elem_blocks(const PlainArgs& a) {
    int G;
    elem_shape(a, &G);
    return (a.C * G + 255) / 256;
}

bool fused_remc_inline(const PlainArgs& a, int64_t K) {
    if (K < 2 || a.C % K != 0 || !fused_supported(a)) return false;
    if (a.tg.kind == HMC_TGT_GAUSS_DENSE) return 16 % K == 0;
    if (a.tg.kind == HMC_TGT_STD_NORMAL || a.tg.kind == HMC_TGT_GAUSS_DIAG) {
        int G;
        elem_shape(a, &G);
        return G <= 64 && (64 / G) % K == 0;       // a pair's two lane groups in one wavefront
    }
    if (a.tg.kind == HMC_TGT_LOGREG) return 4 % K == 0;   // 4 chains per workgroup
    return false;
}

#define HMC_ELEM_DISPATCH(CLS, MACRO)                  \
    switch ((CLS) & 7) {                               \
    case 0: MACRO(1, 1); break;                        \
    case 1: MACRO(4, 1); break;                        \
    case 2: MACRO(16, 1); break;                       \
    case 3: MACRO(64, 1); break;                       \
    case 4: MACRO(64, 2); break;                       \
    case 5: MACRO(64, 4); break;                       \
    default: MACRO(64, 8); break;                      \
    }

// The few-chain kernel: the lanes of all chains fill at most one wavefront per
// SIMD (65536 lanes: 256 owner threads of a workgroup's 512 on 256 CUs), and the
// owners' state fits the registers of 8 waves per CU.  With a lane per chain, whose
// transitions are short beside their draws, only up to three quarters of that.  40
// transitions at L = 3 (10), without and with: N(0, I) D = 4 FP64, 49152 chains 68.8,
// 69.3 us, 65536 chains 70.6, 77.2 (81.5, 83.1); FP32 48.0, 45.0 and 48.7, 52.7 (59.1,
// 52.3); D = 16 FP64, 16384 chains of four lanes 72.3, 66.9; D = 250 FP64, 1024
// chains of 64 lanes 70.3, 68.0.
template <typename T, int G, int NB>
static bool launch_elem_few(const PlainArgs& a, const FusedRun& r, hipStream_t s) {
    if constexpr (NB * sizeof(T) > 16) {
        return false;
    } else {
        if (a.C * G > (G == 1 ? 49152 : 65536) || r.n_transitions < 2) return false;
        const int64_t unit = r.remc_K > 1 ? r.remc_K : 1;              // a pair's chains share a wavefront
        int64_t chains = (a.C + 255) / 256;
        chains = (chains + unit - 1) / unit * unit;
        if (chains * G > 256) return false;
        if (unit > 1 && (64 / G) % unit != 0) return false;
        ElemFew f;
        f.chains = (int32_t)chains;
        const int64_t zbytes = chains * G * NB * 4 * (int64_t)sizeof(T);
        int64_t bt = 32768 / zbytes;
        f.bt = (int32_t)(bt > 64 ? 64 : (bt < 1 ? 1 : bt));
        const size_t lds = elem_few_lds<T, G, NB>(f.chains, f.bt);
        const dim3 grid((unsigned)((a.C + chains - 1) / chains));
        if (r.out.is_accepted || r.out.log_accept_ratio || r.out.target_log_prob || r.out.delta_h ||
            r.out.proposed_state || r.out.proposed_momentum)
            return false;
        auto go = [&](auto kern) {
            if (lds > 65536)
                (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            hipLaunchKernelGGL(kern, grid, dim3(EF_THREADS), lds, s, a, r, f);
        };
        const bool ex = a.ws.scale || r.remc_K > 1;
        if constexpr (G == 1) {
            if (a.tg.D <= 2) {
                if (a.tg.D == 1) ex ? go(k_fused_elem_few<T, 1, 1, true, 1>) : go(k_fused_elem_few<T, 1, 1, false, 1>);
                else ex ? go(k_fused_elem_few<T, 1, 1, true, 2>) : go(k_fused_elem_few<T, 1, 1, false, 2>);
                return true;
            }
        }
        if (ex) go(k_fused_elem_few<T, G, NB, true, 4>);
        else go(k_fused_elem_few<T, G, NB, false, 4>);
        return true;
    }
}

template <typename T>
static hipError_t launch_elem(const PlainArgs& a, const FusedRun& r, hipStream_t s) {
    const int cls = elem_class(a);
    const dim3 grid((unsigned)elem_blocks(a));
    if (r.remc_K > 1 && !fused_remc_inline(a, r.remc_K)) return hipErrorInvalidValue;
#define HMC_ELEM_FEW(GG, NN) if (launch_elem_few<T, GG, NN>(a, r, s)) return hipGetLastError()
    HMC_ELEM_DISPATCH(cls, HMC_ELEM_FEW)
#undef HMC_ELEM_FEW
    if (a.ws.scale || r.remc_K > 1) {
#define HMC_ELEM(GG, NN) hipLaunchKernelGGL((k_fused_elem<T, GG, NN, true>), grid, dim3(256), 0, s, a, r)
        HMC_ELEM_DISPATCH(cls, HMC_ELEM)
#undef HMC_ELEM
    } else {
#define HMC_ELEM(GG, NN) hipLaunchKernelGGL((k_fused_elem<T, GG, NN, false>), grid, dim3(256), 0, s, a, r)
        HMC_ELEM_DISPATCH(cls, HMC_ELEM)
#undef HMC_ELEM
    }
    return hipGetLastError();
}

hipError_t launch_fused_elem_multi(int cls, const ElemJob* jobs_dev, int njobs, int64_t total_blocks,
                                   hipStream_t s) {
    const dim3 grid((unsigned)total_blocks);
    if (cls & 8) {
#define HMC_ELEM_M(GG, NN) hipLaunchKernelGGL((k_fused_elem_multi<double, GG, NN>), grid, dim3(256), 0, s, jobs_dev, njobs)
        HMC_ELEM_DISPATCH(cls, HMC_ELEM_M)
#undef HMC_ELEM_M
    } else {
#define HMC_ELEM_M(GG, NN) hipLaunchKernelGGL((k_fused_elem_multi<float, GG, NN>), grid, dim3(256), 0, s, jobs_dev, njobs)
        HMC_ELEM_DISPATCH(cls, HMC_ELEM_M)
#undef HMC_ELEM_M
    }
    return hipGetLastError();
}

static hipError_t launch_dense_fused(const PlainArgs& a, const FusedRun& r, hipStream_t s) {
    const int ntiles = (int)((a.tg.D + 15) / 16);
    const size_t lds = (size_t)2 * 16 * (16 * ntiles + 4) * sizeof(float) + 2 * 2 * DENSE_NW * 16 * sizeof(double);
    if (r.remc_K > 1 && (!fused_remc_inline(a, r.remc_K) || r.remc_K * r.remc_M != a.C)) return hipErrorInvalidValue;
    const int64_t per = r.remc_K > 1 ? 16 / r.remc_K : 16;      // values of m (or chains) per workgroup
    const int64_t units = r.remc_K > 1 ? r.remc_M : a.C;
    const dim3 grid((unsigned)((units + per - 1) / per));
    const bool ex = a.ws.scale || r.remc_K > 1;
    switch (ntiles) {
#define HMC_DENSE_NT(N)                                                                   \
    case N:                                                                               \
        if (ex) hipLaunchKernelGGL((k_fused_dense<N, true>), grid, dim3(64 * DENSE_NW), lds, s, a, r); \
        else hipLaunchKernelGGL((k_fused_dense<N, false>), grid, dim3(64 * DENSE_NW), lds, s, a, r);            \
        break;
        HMC_DENSE_NT(1) HMC_DENSE_NT(2) HMC_DENSE_NT(3) HMC_DENSE_NT(4)
        HMC_DENSE_NT(5) HMC_DENSE_NT(6) HMC_DENSE_NT(7) HMC_DENSE_NT(8)
#undef HMC_DENSE_NT
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_fused(const PlainArgs& a, const FusedRun& r, hipStream_t s) {
    switch (a.tg.kind) {
    case HMC_TGT_STD_NORMAL:
    case HMC_TGT_GAUSS_DIAG:
        return a.f64 ? launch_elem<double>(a, r, s) : launch_elem<float>(a, r, s);
    case HMC_TGT_GAUSS_DENSE:
        return launch_dense_fused(a, r, s);
    case HMC_TGT_LOGREG:
        return launch_fused_logreg(a, r, s);
    }
    return hipErrorNotSupported;
}

}  // namespace hmc
