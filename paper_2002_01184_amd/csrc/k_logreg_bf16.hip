// k_logreg_bf16.hip -- mixed-precision gradient of Bayesian logistic
// regression for large data sets (X stored BF16): both contractions of each
// leapfrog step on v_mfma_f32_16x16x32_bf16 with FP32 accumulation,
//     S  = X theta              (M = rows, N = chains, K = dims)
//     G^T = R^T X,  R = y - sigmoid(S)   (M = chains, N = dims, K = rows)
// and an accurate-logit pass for the log-probability that enters dH: theta is
// split into three BF16 terms (hi + mid + lo), so X theta is formed from exact
// BF16 x BF16 products with FP32 accumulation, and the softplus terms are
// summed in FP64.  The gradient is a deterministic function of position, so
// the trajectory stays reversible and volume preserving; with dH taken from the
// accurate log-probability the accept test keeps detailed balance.
//
// Data: at init the context builds zero-padded copies of the target in its
// workspace -- X as [NP, DP] and X^T as [DP, NP] (BF16), y as [NP] bytes, with
// NP = N rounded up to 32 rows and DP = 32 KS dims -- so every sub-tile of 32
// rows is whole and rows are 16-byte aligned.  Padded rows and dims are zero
// in X: they add nothing to S or G (their residuals multiply zeros), and the
// log-probability pass skips rows >= N.
//
// Work decomposition: a workgroup (NW waves) owns 16 NW CS chains and a chunk
// of rows; each wave computes S and G^T for its own 16 CS chains, so the
// residuals never leave registers.  theta (drifted) stays in registers as the B
// operands of the first contraction, beside the G^T accumulators; every LDS
// operand fragment feeds CS MFMAs.  32-row sub-tiles of X and X^T are copied global ->
// LDS by the load-to-LDS instructions (global_load_lds_dwordx4: lane i of an
// instruction writes bytes 16 i .. 16 i + 15 of a 1 KB block) into rings of
// buffers, a few sub-tiles ahead, with no staging registers; the barrier
// between sub-tiles waits for LDS only, each wave first waiting (vmcnt) for its
// own copies of the sub-tile it is about to read.  Row chunks are mapped
// XCD-aware: blocks on the same XCD work on the same chunk, so the 32 CUs of
// an XCD stream X through their shared L2 together.  Partials per chunk are
// summed in a fixed order by k_logreg_finish / k_lr16_lp_sum.
//
// Lane layouts (v_mfma_f32_16x16x32_bf16, checked on gfx950): A[i][k] at lane
// i + 16 (k / 8), element k % 8; B[k][j] at lane j + 16 (k / 8), element k % 8;
// D[i][j] in VGPR i % 4 of lane j + 16 (i / 4).
#include "hmc_internal.hpp"

namespace hmc {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx8 __attribute__((ext_vector_type(8)));
typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8v __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4v __attribute__((ext_vector_type(4)));

constexpr int LB_NW = 4;      // waves per workgroup
constexpr int LB_RS = 32;     // rows per sub-tile
constexpr int LD_YB = 256;    // LDS bytes reserved for the labels of a sub-tile (32 used)

__device__ __forceinline__ float sigmoid_hw(float s) {
    const float e = __builtin_amdgcn_exp2f(-1.4426950408889634f * s);
    return __builtin_amdgcn_rcpf(1.0f + e);
}

// softplus(s) = max(s, 0) + log(1 + e), e = exp(-|s|), in three parts that a kernel
// can spread over its MFMAs.  Both forms of the logarithm are made and one is
// selected: a branch a value costs more than the polynomial.  The median with 0
// and +inf is the maximum with 0 without the compiler's quieting of a NaN (the
// logarithm's NaN carries on).
__device__ __forceinline__ float softplus_exp(float s) {
    return __builtin_amdgcn_exp2f(-1.4426950408889634f * fabsf(s));
}
__device__ __forceinline__ float softplus_log(float e) { return __builtin_amdgcn_logf(1.0f + e); }
__device__ __forceinline__ float softplus_sum(float s, float e, float lg) {
    const float big = 0.69314718055994531f * lg;
    const float small = e * (1.0f - e * (0.5f - e * 0.33333333f));
    return __builtin_amdgcn_fmed3f(s, 0.f, INFINITY) + (e >= 0x1p-10f ? big : small);
}
__device__ __forceinline__ float softplus_hw(float s) {
    const float e = softplus_exp(s);
    return softplus_sum(s, e, softplus_log(e));
}

// eight floats to BF16, round to nearest even (v_cvt_pk_bf16_f32)
__device__ __forceinline__ bf16x8 pack_bf16(floatx8 f) {
    return __builtin_bit_cast(bf16x8, __builtin_convertvector(f, bf16x8v));
}
// four floats to BF16, packed in two dwords
__device__ __forceinline__ uint2 pack4_bf16(floatx4 f) {
    return __builtin_bit_cast(uint2, __builtin_convertvector(f, bf16x4v));
}

// block -> (chain tile, row chunk): blocks b and b + 8k run on the same XCD
__device__ __forceinline__ void lb_map(int b, int ntile, int nsplit, int* tile, int* split) {
    if (nsplit <= 8 && (8 % nsplit) == 0 && ((ntile * nsplit) % 8) == 0) {
        const int xcd = b & 7, idx = b >> 3;
        *split = xcd % nsplit;
        *tile = idx * (8 / nsplit) + xcd / nsplit;
    } else {
        *split = b % nsplit;
        *tile = b / nsplit;
    }
}

// s_waitcnt vmcnt(n) leaving the other counters unconstrained (gfx9 encoding)
template <int n>
__device__ __forceinline__ void wait_vmcnt() {
    static_assert(n >= 0 && n < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8));
}

// workgroup barrier that orders LDS accesses only (in-flight global->LDS copies
// of later sub-tiles stay in flight)
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

typedef __attribute__((address_space(3))) void lds_void_t;

// ---------------------------------------------------------------------------
// Tile layouts in LDS (16-byte slots, XOR-swizzled so that the operand reads
// of the MFMAs spread over the LDS banks):
//   X   [32 rows][SR = DP / 8 slots]: slot c of row r at position c ^ xsw(r),
//       xsw(r) = (r & 3) | (bit 3 of r) << 2  (r & 3 when SR = 4)
//   X^T [DP dims][4 slots of 8 rows]: slot c of dim d at position c ^ ((d >> 1) & 3)
// The S halves take rows in the order 8 q + 4 mt + v (lane position i = 4 q + v
// of half mt), so lane group g holds the residuals of rows 8 g .. 8 g + 7 --
// rows 8 g + v from half 0, 8 g + 4 + v from half 1 -- which is the K order of
// the second contraction: its X^T operand is the one 16-byte slot g of a dim.
// ---------------------------------------------------------------------------
template <int SR>
__device__ __forceinline__ int lb_xsw(int r) {
    return SR >= 8 ? ((r & 3) | (((r >> 3) & 1) << 2)) : (r & 3);
}

// Copy of 1 KB block i of an X sub-tile (rows of the padded copy, stride DP)
// into xbase: lane ln writes position 64 i + ln of the tile's slot grid.
template <int KS>
__device__ __forceinline__ void lb_copy_x_block(const char* xsrc_t, uint8_t* __restrict__ xbase, int i, int ln) {
    constexpr int DP = 32 * KS, SR = DP / 8;
    const int q = i * 64 + ln;
    const int row = q / SR, c = (q % SR) ^ lb_xsw<SR>(row);
    const uint32_t off = (uint32_t)(row * (DP * 2) + 16 * c);
    __builtin_amdgcn_global_load_lds((const void*)(xsrc_t + off), (lds_void_t*)(xbase + i * 1024), 16, 0, 0);
}

// per-lane fragment offsets of the two S halves (even / odd k-step): row
// rho = 8 (l16 >> 2) + 4 mt + (l16 & 3), slot (4 ks + g) ^ xsw(rho) =
// 8 (ks >> 1) + 4 ((ks & 1) ^ rb) + (g ^ (sw & 3)) with sw = xsw(rho), rb = bit 2 of sw
template <int KS>
__device__ __forceinline__ void lb_xfrag_offsets(int l16, int g, uint32_t (&xoff)[2][2]) {
    constexpr int DP = 32 * KS, SR = DP / 8;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        const int row = 8 * (l16 >> 2) + 4 * mt + (l16 & 3);
        const int sw = lb_xsw<SR>(row);
        const int rb = (sw >> 2) & 1, gg = g ^ (sw & 3);
#pragma unroll
        for (int e = 0; e < 2; ++e) xoff[mt][e] = (uint32_t)(row * (DP * 2) + 16 * (4 * (e ^ rb) + gg));
    }
}

// theta (drifted when drift) of chain c as B operands B[k][j] = theta[j][k]:
// the 8 dims 32 ks + 8 g .. + 7 of k-step ks (zeros past D and for c >= C)
template <int KS>
__device__ __forceinline__ void lb_load_theta(const PlainArgs& a, const float* __restrict__ xsrc,
                                              const float* __restrict__ psrc, int drift, int64_t c, int g,
                                              floatx8 (&v)[KS]) {
    const int64_t D = a.tg.D;
    const bool cok = c < a.C;
    const float eps = cok ? (float)a.ws.eps[c] : 0.f;
    const float* xr = xsrc + (cok ? c : 0) * D;
    const float* pr = drift ? psrc + (cok ? c : 0) * D : nullptr;
    const bool vec = (D % 4) == 0;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const int d0 = 32 * ks + 8 * g;
        floatx8 t = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (cok && vec && d0 + 8 <= D) {
            const float4 x0 = *(const float4*)(xr + d0), x1 = *(const float4*)(xr + d0 + 4);
            t = floatx8{x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
            if (drift) {
                const float4 p0 = *(const float4*)(pr + d0), p1 = *(const float4*)(pr + d0 + 4);
                const floatx8 pv = {p0.x, p0.y, p0.z, p0.w, p1.x, p1.y, p1.z, p1.w};
#pragma unroll
                for (int e = 0; e < 8; ++e) t[e] = fmaf(eps, pv[e], t[e]);
            }
        } else if (cok) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int d = d0 + e;
                float u = 0.f;
                if (d < D) {
                    u = xr[d];
                    if (drift) u = fmaf(eps, pr[d], u);
                }
                t[e] = u;
            }
        }
        v[ks] = t;
    }
}

// ---------------------------------------------------------------------------
// Gradient partials, software-pipelined: 16 CS chains per wave, NW waves per
// workgroup (LbGrad: 256 chains per workgroup up to D = 256, so at 8192 chains
// 32 chain tiles x 8 row splits = one workgroup per CU with each split on its
// own XCD; two waves per SIMD from D = 33 on).  A sub-tile s is one sequence of
// 4 KS steps of CS MFMAs: S of its rows 0..15, G^T += R^T X^T of sub-tile s - 1, S
// of its rows 16..31.  A step also reads the operand fragment of the step PD later,
// does a slice of the residuals (rows 16..31 of s - 1 in the first part, rows 0..15
// of s in the second) and, every few steps, issues one copy; scheduling barriers
// keep the steps apart, since the scheduler, short of registers, had gathered the
// reads of the G part one by one in front of their MFMAs.
// Copies and waves meet once per stage of SUBS sub-tiles: one stage is read while
// the next is copied.  X^T of sub-tile s - 1 is still read in s, so the X^T tiles
// sit in a ring of one buffer more than the X tiles (beyond D = 256 two X tiles and
// three X^T tiles of 32 KB fill the 160 KB).  The labels of a sub-tile are copied
// beside its X^T tile, or (beyond D = 256) read from global memory by each lane.
//
// What bounds it: power and the matrix cores.  At D = 256, N = 100000, 8192 chains
// the MFMAs fill 54% -> 60% of the clocks (3800 -> 3340 a sub-tile), and the clock
// falls with it, 2.20 -> 2.12 GHz: 704 -> 656 us a gradient (1.28 PFLOP/s).  With
// half the CUs (50000 rows, 4000 chains) 356 -> 304 us, D = 128 214 -> 190, D = 100
// (4096 chains) 194 -> 157, D = 500 399 -> 385 (gradient and its finish).
// ---------------------------------------------------------------------------
template <int KS>
struct LbGrad {
    // waves per workgroup and 16-chain tiles per wave: eight waves (two per SIMD, so that
    // one's residual work overlaps the other's MFMAs) of 32 chains from D = 33 to 256 and
    // of 16 beyond (theta and G^T of wider chains fill the registers); up to D = 32, whose
    // sub-tile has too few copies for eight waves, four of 64
    static constexpr int NW = KS >= 2 ? 8 : 4;
    static constexpr int CS = KS == 1 ? 4 : (KS <= 8 ? 2 : 1);
    static constexpr int CT = NW * 16 * CS;               // chains per workgroup
    static constexpr int SUBS = KS <= 4 ? 4 : (KS <= 8 ? 2 : 1);          // sub-tiles per stage
    static constexpr int NBX = 2 * SUBS;                  // X buffers
    static constexpr int NBT = NBX + 1;                   // X^T buffers
    static constexpr bool YLDS = KS <= 8;                 // labels copied to LDS
    static constexpr int DP = 32 * KS;
    static constexpr int XB = LB_RS * DP * 2;             // bytes of an X (or X^T) sub-tile
    static constexpr int TBY = XB + (YLDS ? LD_YB : 0);   // X^T sub-tile + labels
    static constexpr int XI = XB / 1024;                  // 1 KB copy blocks of a tile
    static constexpr int JW = (2 * XI) / NW;              // tile copies per wave
    static constexpr int J = JW + (YLDS ? 1 : 0);         // copy instructions per wave and sub-tile
    static constexpr int LDS = NBX * XB + NBT * TBY;
};

template <int KS>
__device__ __forceinline__ void lr16_grad_body(const PlainArgs& a, const float* __restrict__ xsrc,
                                               const float* __restrict__ psrc, int drift, int64_t rows_per_split,
                                               int nsplit, int blk) {
    using P = LbGrad<KS>;
    constexpr int CS = P::CS, CT = P::CT, NT = 2 * KS, DP = P::DP, XB = P::XB, TBY = P::TBY, XI = P::XI;
    constexpr int JW = P::JW, J = P::J, SUBS = P::SUBS, NBX = P::NBX, NBT = P::NBT, NW = P::NW;
    static_assert((2 * XI) % NW == 0, "copies must split evenly over the waves");
    static_assert(P::LDS <= 160 * 1024, "LDS");
    extern __shared__ __align__(16) uint8_t ldsb[];
    uint8_t* xring = ldsb;                      // [NBX][XB]
    uint8_t* tring = ldsb + NBX * XB;           // [NBT][TBY]

    const int64_t D = a.tg.D, C = a.C, NP = (a.tg.N + LB_RS - 1) / LB_RS * LB_RS;
    const int ntile = (int)((C + CT - 1) / CT);
    int tile, split;
    lb_map(blk, ntile, nsplit, &tile, &split);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int64_t cw = (int64_t)tile * CT + 16 * CS * w;
    const uint16_t* Xp = (const uint16_t*)a.ws.xp;
    const uint16_t* Xt = (const uint16_t*)a.ws.xt;
    const uint8_t* Yp = (const uint8_t*)a.ws.yp;

    bf16x8 thb[CS][KS];
#pragma unroll
    for (int cs = 0; cs < CS; ++cs) {
        floatx8 v[KS];
        lb_load_theta<KS>(a, xsrc, psrc, drift, cw + 16 * cs + l16, g, v);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) thb[cs][ks] = pack_bf16(v[ks]);
    }

    const int64_t r_begin = (int64_t)split * rows_per_split;
    int64_t r_end = r_begin + rows_per_split;
    if (r_end > NP) r_end = NP;
    const int nsub = r_begin < r_end ? (int)((r_end - r_begin) / LB_RS) : 0;

    // copy k of a wave's J for sub-tile sidx (the last one past the end): X into
    // xbase, X^T and, as the last copy, the labels into tbase
    auto copy_k = [&](int sidx, int k, uint8_t* __restrict__ xbase, uint8_t* __restrict__ tbase) {
        if (sidx >= nsub) sidx = nsub - 1;
        const int64_t r0 = r_begin + (int64_t)sidx * LB_RS;
        // the lane index through an empty asm: the per-lane offsets are recomputed
        // for every copy instead of being hoisted out of the loop (and spilled: a
        // reload's wait would also wait for the copies in flight)
        int ln = lane;
        asm volatile("" : "+v"(ln));
        if (k == JW) {
            __builtin_amdgcn_global_load_lds((const void*)(Yp + r0 + 4 * (ln & 7)), (lds_void_t*)(tbase + XB), 4, 0,
                                             0);
            return;
        }
        const int i = w + NW * k;
        const bool isx = (XI % NW == 0) ? (k < XI / NW) : (i < XI);
        if (isx) {
            // with SR dividing 64 the row of lane ln in copy k is A + (64 NW / SR) k, A
            // below, with no carry from A's low bits into bit 3, so its swizzle depends
            // on k only through bit 3 of (64 NW / SR) k
            constexpr int SR = DP / 8;
            constexpr bool POW2 = (64 % SR) == 0;
            constexpr int KSTR = 64 * NW / SR;
            static_assert(!POW2 || KSTR % 8 == 0 || (KSTR == 4 && NW == 4), "row stride of the copies");
            const char* src = (const char*)(Xp + r0 * DP);
            if constexpr (POW2) {
                const int arow = (64 / SR) * w + ln / SR, par = ((KSTR * k) >> 3) & 1;
                const int sw = SR >= 8 ? ((arow & 3) | ((((arow >> 3) & 1) ^ par) << 2)) : (arow & 3);
                const uint32_t xo = (uint32_t)(ln / SR) * (uint32_t)(DP * 2) + 16u * (uint32_t)((ln % SR) ^ sw);
                __builtin_amdgcn_global_load_lds((const void*)(src + (uint32_t)i * 1024u + xo),
                                                 (lds_void_t*)(xbase + i * 1024), 16, 0, 0);
            } else {
                lb_copy_x_block<KS>(src, xbase, i, ln);
            }
        } else {
            const int ii = i - XI;
            const uint32_t toff = (uint32_t)(ln >> 2) * (uint32_t)NP * 2u + 16u * (uint32_t)((ln & 3) ^ ((ln >> 3) & 3));
            __builtin_amdgcn_global_load_lds(
                (const void*)((const char*)(Xt + r0) + (uint32_t)(16 * ii) * (uint32_t)NP * 2u + toff),
                (lds_void_t*)(tbase + ii * 1024), 16, 0, 0);
        }
    };
    // labels of the lane's rows 8 g .. 8 g + 7 of sub-tile sidx
    auto labels = [&](int sidx, const uint8_t* tb) {
        if constexpr (P::YLDS) return *(const uint2*)(tb + XB + 8 * g);
        else return *(const uint2*)(Yp + r_begin + (int64_t)sidx * LB_RS + 8 * g);
    };

    uint32_t xoff[2][2];
    lb_xfrag_offsets<KS>(l16, g, xoff);
    const uint32_t toff_f = (uint32_t)(l16 * 64 + 16 * (g ^ ((l16 >> 1) & 3)));
    auto xfrag = [&](const uint8_t* xb, const uint32_t* o2, int ks) {
        return *(const bf16x8*)(xb + o2[ks & 1] + 128 * (ks >> 1));
    };
    // residuals of one 16-row half (the lane's rows 8 g + 4 mt + v)
    auto resid = [&](floatx4 sv, uint32_t yw) {
        floatx4 r;
#pragma unroll
        for (int v = 0; v < 4; ++v) r[v] = (float)((yw >> (8 * v)) & 0xffu) - sigmoid_hw(sv[v]);
        return pack4_bf16(r);
    };
    // The part of step `st` of n in the same residuals of CS halves, one element a lane
    // after the other from step `first` on, over `span` steps: the exponential, the
    // reciprocal and the difference in three consecutive steps (the last step takes
    // what is left); r[cs] holds the values between.
    auto resid_slice = [&](int st, int n, int first, int span, const floatx4* sv, uint32_t yw, floatx4* r) {
        constexpr int E = 4 * CS;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int cs = e / 4, v = e % 4;
            auto at = [&](int k) { const int t = first + e * span / E + k; return (t < n ? t : n - 1) == st; };
            if (at(0)) r[cs][v] = __builtin_amdgcn_exp2f(-1.4426950408889634f * sv[cs][v]);
            if (at(1)) r[cs][v] = __builtin_amdgcn_rcpf(1.0f + r[cs][v]);
            if (at(2)) r[cs][v] = (float)((yw >> (8 * v)) & 0xffu) - r[cs][v];
        }
    };
    constexpr int PD = KS == 1 ? 2 : 4;                                  // fragments read ahead of the MFMAs
    // S of one half from fragments read ahead (all of them up to KS = 8, else
    // eight in flight)
    constexpr int FA = KS < 8 ? KS : 8;
    auto sphase = [&](const uint8_t* __restrict__ xb, const uint32_t* o2, floatx4* sacc) {
        bf16x8 xa[FA];
#pragma unroll
        for (int ks = 0; ks < FA; ++ks) xa[ks] = xfrag(xb, o2, ks);
#pragma unroll
        for (int cs = 0; cs < CS; ++cs) sacc[cs] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 ax = xa[ks % FA];
            if (ks + FA < KS) xa[ks % FA] = xfrag(xb, o2, ks + FA);
#pragma unroll
            for (int cs = 0; cs < CS; ++cs)
                sacc[cs] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ax, thb[cs][ks], sacc[cs], 0, 0, 0);
        }
    };

    floatx4 gacc[CS][NT];
#pragma unroll
    for (int cs = 0; cs < CS; ++cs)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) gacc[cs][nt] = floatx4{0.f, 0.f, 0.f, 0.f};

    // G^T += R^T X^T of the sub-tile in tb with residual operands ra
    auto gphase = [&](const uint8_t* __restrict__ tb, const bf16x8* ra, uint32_t to) {
        auto tfrag = [&](int nt) { return *(const bf16x8*)(tb + to + 1024 * nt); };
        bf16x8 tf0 = tfrag(0), tf1 = tfrag(1);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const bf16x8 bx = tf0;
            tf0 = tf1;
            if (nt + 2 < NT) tf1 = tfrag(nt + 2);
#pragma unroll
            for (int cs = 0; cs < CS; ++cs)
                gacc[cs][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ra[cs], bx, gacc[cs][nt], 0, 0, 0);
        }
    };

    // pipeline registers: S of rows 16..31 of the previous sub-tile, the packed
    // residuals of its rows 0..15 and its labels of rows 16..31
    floatx4 s1p[CS];
    uint2 lo_p[CS];
    uint32_t yp1 = 0u;
    // the first sub-tile: no G of a previous one
    auto head = [&](const uint8_t* __restrict__ xb, const uint8_t* __restrict__ tcur) {
        const uint2 yl = labels(0, tcur);
        floatx4 s0[CS];
        sphase(xb, xoff[0], s0);
#pragma unroll
        for (int cs = 0; cs < CS; ++cs) lo_p[cs] = resid(s0[cs], yl.x);
        sphase(xb, xoff[1], s1p);
        yp1 = yl.y;
    };
    // copies of sub-tile sn, one every few steps of another's MFMAs: the address units
    // take 16 clocks a copy, and in a burst behind the barrier the waves stood at them
    // for 600 clocks a sub-tile (D = 256)
    auto spread_copy = [&](int st, int sn, uint8_t* xw, uint8_t* tw) {
        static_assert(J <= 2 * KS, "one copy a step");
        const int k = (st * J + 2 * KS - 1) / (2 * KS);
        if (k < J && (k * 2 * KS) / J == st) copy_k(sn, k, xw + (sn % NBX) * XB, tw + (sn % NBT) * TBY);
    };
    // One sub-tile, and the copies of the sub-tile SUBS later into buffers that no
    // wave reads before the next stage's barrier (past the end, the last sub-tile
    // again).  The copies write through xw and tw and the sub-tile reads through xr
    // and tr, which are restrict: the LDS reads need not wait for the copies in
    // flight (the vmcnt wait and the barrier between stages order them).
    auto step = [&](int sidx, uint8_t* __restrict__ xw, uint8_t* __restrict__ tw, const uint8_t* __restrict__ xr,
                    const uint8_t* __restrict__ tr) {
        const uint8_t* xb = xr + (sidx % NBX) * XB;
        const uint8_t* tprev = tr + ((sidx + NBT - 1) % NBT) * TBY;
        const uint8_t* tcur = tr + (sidx % NBT) * TBY;
        const uint2 yl = labels(sidx, tcur);
        // a phase's base offsets pass through one empty asm at its start, so that a
        // register per offset plus immediate offsets address its fragments
        uint32_t o1[2] = {xoff[0][0], xoff[0][1]}, o2[2] = {xoff[1][0], xoff[1][1]}, ot = toff_f;
        auto frag = [&](int st) {
            if (st < KS) return xfrag(xb, o1, st);
            if (st < 3 * KS) return *(const bf16x8*)(tprev + ot + 1024 * (st - KS));
            return xfrag(xb, o2, st - 3 * KS);
        };
        asm volatile("" : "+v"(o1[0]), "+v"(o1[1]));
        bf16x8 fr[PD];
#pragma unroll
        for (int st = 0; st < PD; ++st) {
            if (st == KS) asm volatile("" : "+v"(ot));
            if (st == 3 * KS) asm volatile("" : "+v"(o2[0]), "+v"(o2[1]));
            fr[st] = frag(st);
        }
        floatx4 s0[CS], hi[CS], lo[CS];
        bf16x8 rp[CS];
#pragma unroll
        for (int st = 0; st < 4 * KS; ++st) {
            const bf16x8 f = fr[st % PD];
            // the wave in its G phase goes before the SIMD's other one
            if (KS <= 8 && st == KS) __builtin_amdgcn_s_setprio(1);
            if (KS <= 8 && st == 3 * KS) __builtin_amdgcn_s_setprio(0);
#pragma unroll
            for (int cs = 0; cs < CS; ++cs) {
                const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
                if (st < KS)
                    s0[cs] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, thb[cs][st], st == 0 ? zero : s0[cs], 0, 0, 0);
                else if (st < 3 * KS)
                    gacc[cs][st - KS] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(rp[cs], f, gacc[cs][st - KS], 0, 0, 0);
                else
                    s1p[cs] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, thb[cs][st - 3 * KS],
                                                                      st == 3 * KS ? zero : s1p[cs], 0, 0, 0);
            }
            if (st + PD < 4 * KS) {
                if (st + PD == KS) asm volatile("" : "+v"(ot));
                if (st + PD == 3 * KS) asm volatile("" : "+v"(o2[0]), "+v"(o2[1]));
                fr[st % PD] = frag(st + PD);
            }
            if (st < KS) {
                resid_slice(st, KS, 0, KS > 3 ? KS - 3 : 1, s1p, yp1, hi);
                if (st == KS - 1)
#pragma unroll
                    for (int cs = 0; cs < CS; ++cs) {
                        const uint2 h = pack4_bf16(hi[cs]);
                        rp[cs] = __builtin_bit_cast(bf16x8, make_uint4(lo_p[cs].x, lo_p[cs].y, h.x, h.y));
                    }
            } else if (st < 3 * KS) {
                resid_slice(st - KS, 2 * KS, 1, KS > 1 ? 2 * KS - 3 : 1, s0, yl.x, lo);
                if (st == 3 * KS - 1)
#pragma unroll
                    for (int cs = 0; cs < CS; ++cs) lo_p[cs] = pack4_bf16(lo[cs]);
            }
            spread_copy(st, sidx + SUBS, xw, tw);
            if (KS > 1 && (st & 1)) __builtin_amdgcn_sched_barrier(0);
        }
        yp1 = yl.y;
    };
    if (nsub > 0) {
#pragma unroll
        for (int u = 0; u <= SUBS; ++u) {
#pragma unroll
            for (int k = 0; k < J; ++k) copy_k(u, k, xring + (u % NBX) * XB, tring + (u % NBT) * TBY);
            if (u == SUBS - 1) {
                wait_vmcnt<0>();       // the only copies outstanding are the first stage's
                lds_barrier();
            }
        }
        head(xring, tring);
    }
    for (int sidx = 1; sidx < nsub; ++sidx) {
        if (sidx % SUBS == 0) {
            wait_vmcnt<0>();
            lds_barrier();
        }
        step(sidx, xring, tring, xring, tring);
    }
    wait_vmcnt<0>();                   // no copy may land in LDS after the end
    if (nsub > 0) {
        bf16x8 rp[CS];
#pragma unroll
        for (int cs = 0; cs < CS; ++cs) {
            const uint2 hi = resid(s1p[cs], yp1);
            rp[cs] = __builtin_bit_cast(bf16x8, make_uint4(lo_p[cs].x, lo_p[cs].y, hi.x, hi.y));
        }
        gphase(tring + ((nsub - 1) % NBT) * TBY, rp, toff_f);
    }
#pragma unroll
    for (int cs = 0; cs < CS; ++cs)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t c = cw + 16 * cs + 4 * g + v;
                const int64_t d = 16 * nt + l16;
                if (c < C && d < D) a.ws.part_g[((int64_t)split * C + c) * D + d] = gacc[cs][nt][v];
            }
}

// ---------------------------------------------------------------------------
// Accurate log-probability partials: theta = hi + mid + lo (three BF16 terms,
// smallest first), 16 chains per wave, each X fragment feeding 3 MFMAs; the
// softplus terms summed per chain in FP64.  Steps like the gradient's: the terms of
// one 16-row half are formed in slices between the MFMAs of the next one (before,
// with a branch a value, MFMAs and terms took turns: 3500 clocks a sub-tile, 1540
// of them MFMAs).  D = 256, N = 100000, 8192 chains 1150 -> 1010 us, D = 128
// 393 -> 317 us.
// ---------------------------------------------------------------------------
template <int KS>
struct LbLogp {
    // eight waves of 16 chains (two waves per SIMD)
    static constexpr int NW = 8;
    static constexpr int CT = NW * 16;
    static constexpr int SUBS = 2;                        // sub-tiles per stage
    static constexpr int NB = 2 * SUBS;
    static constexpr int DP = 32 * KS;
    static constexpr int XB = LB_RS * DP * 2;
    static constexpr int BUF = XB + LD_YB;
    static constexpr int XI = XB / 1024;
    static constexpr int JW = (XI + NW - 1) / NW;         // X copy instructions per wave (a wave may repeat one)
    static constexpr int J = JW + 1;                      // plus the labels
    static constexpr int LDS = NB * BUF;
};

// theta = hi + mid + lo in BF16
__device__ __forceinline__ void lb_split_theta(floatx8 v, bf16x8& hi, bf16x8& mid, bf16x8& lo) {
    floatx8 r1, r2;
    hi = pack_bf16(v);
#pragma unroll
    for (int e = 0; e < 8; ++e) r1[e] = v[e] - bf16_to_f32((uint16_t)hi[e]);
    mid = pack_bf16(r1);
#pragma unroll
    for (int e = 0; e < 8; ++e) r2[e] = r1[e] - bf16_to_f32((uint16_t)mid[e]);
    lo = pack_bf16(r2);
}

template <int KS>
__device__ __forceinline__ void lr16_logp_body(const PlainArgs& a, const float* __restrict__ xsrc,
                                               int64_t rows_per_split, int nsplit, int blk) {
    using P = LbLogp<KS>;
    constexpr int CT = P::CT, SUBS = P::SUBS, NB = P::NB, XB = P::XB, BUF = P::BUF, XI = P::XI, JW = P::JW, J = P::J;
    constexpr int DP = P::DP;
    static_assert(P::LDS <= 160 * 1024, "LDS");
    extern __shared__ __align__(16) uint8_t ldsb[];

    const int64_t N = a.tg.N, C = a.C, NP = (N + LB_RS - 1) / LB_RS * LB_RS;
    const int ntile = (int)((C + CT - 1) / CT);
    int tile, split;
    lb_map(blk, ntile, nsplit, &tile, &split);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int64_t cw = (int64_t)tile * CT + 16 * w;
    const uint16_t* Xp = (const uint16_t*)a.ws.xp;
    const uint8_t* Yp = (const uint8_t*)a.ws.yp;

    // theta = hi + mid + lo, three BF16 B operands per k-step
    bf16x8 th[3][KS];
    {
        floatx8 v[KS];
        lb_load_theta<KS>(a, xsrc, nullptr, 0, cw + l16, g, v);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) lb_split_theta(v[ks], th[0][ks], th[1][ks], th[2][ks]);
    }
    const int64_t r_begin = (int64_t)split * rows_per_split;
    int64_t r_end = r_begin + rows_per_split;
    if (r_end > NP) r_end = NP;
    const int nsub = r_begin < r_end ? (int)((r_end - r_begin) / LB_RS) : 0;

    // copy k of a wave's J for sub-tile sidx (the last one past the end)
    auto copy_k = [&](int sidx, int k, uint8_t* __restrict__ base) {
        if (sidx >= nsub) sidx = nsub - 1;
        const int64_t r0 = r_begin + (int64_t)sidx * LB_RS;
        int ln = lane;
        asm volatile("" : "+v"(ln));
        if (k == JW) {
            __builtin_amdgcn_global_load_lds((const void*)(Yp + r0 + 4 * (ln & 7)), (lds_void_t*)(base + XB), 4, 0, 0);
            return;
        }
        int i = w + P::NW * k;
        if (i >= XI) i = XI - 1;          // a repeated copy keeps the count equal over the waves
        lb_copy_x_block<KS>((const char*)(Xp + r0 * DP), base, i, ln);
    };
    uint32_t xoff[2][2];
    lb_xfrag_offsets<KS>(l16, g, xoff);
    auto xfrag = [&](const uint8_t* xb, const uint32_t* o2, int ks) {
        return *(const bf16x8*)(xb + o2[ks & 1] + 128 * (ks >> 1));
    };
    // Log-likelihood terms of one half, y s - softplus(s), for the lane's rows 0..3
    // (those at or past `left` skipped: the data's end), in slices like the
    // gradient's residuals; a lane's four terms are added in FP32 before the FP64
    // sum (a rounding of about 1e-7 of a few terms, far below what the accept test
    // resolves).
    double lp = 0.0;
    float ex[4], lg[4], t4 = 0.f;
    auto term_slice = [&](int st, int n, const floatx4& sv, uint32_t yw, int left) {
        const int first = n > 4 ? 1 : 0, span = n > 4 ? n - 3 : 1;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            // KS = 16: theta leaves no registers for values between steps
            auto at = [&](int k) { const int t = first + v * span / 4 + (KS > 12 ? 0 : k); return (t < n ? t : n - 1) == st; };
            if (at(0)) ex[v] = softplus_exp(sv[v]);
            if (at(1)) lg[v] = softplus_log(ex[v]);
            if (at(2)) {
                const float t = fmaf((float)((yw >> (8 * v)) & 0xffu), sv[v], -softplus_sum(sv[v], ex[v], lg[v]));
                const float tm = v < left ? t : 0.f;
                t4 = v == 0 ? tm : t4 + tm;
            }
        }
        if (st == n - 1) lp += (double)t4;
    };
    constexpr int PD = KS == 1 || KS > 12 ? 2 : 4;         // fragments read ahead of the MFMAs (KS = 16: theta fills the registers)
    floatx4 sprev = {0.f, 0.f, 0.f, 0.f};                  // S of the previous half, its labels and rows left
    uint32_t yprev = 0u;
    int lprev = 0;
    // One sub-tile, and the copies of the one SUBS later; reads and copies through
    // restrict pointers as in the gradient.
    auto step = [&](int sidx, uint8_t* __restrict__ xw, const uint8_t* __restrict__ xr) {
        const uint8_t* xb = xr + (sidx % NB) * BUF;
        const int64_t rest = N - (r_begin + (int64_t)sidx * LB_RS);
        const uint2 yl = *(const uint2*)(xb + XB + 8 * g);
        const int left = (int)(rest < LB_RS ? rest : LB_RS) - 8 * g;
        uint32_t o1[2] = {xoff[0][0], xoff[0][1]}, o2[2] = {xoff[1][0], xoff[1][1]};
        auto frag = [&](int st) { return st < KS ? xfrag(xb, o1, st) : xfrag(xb, o2, st - KS); };
        asm volatile("" : "+v"(o1[0]), "+v"(o1[1]));
        bf16x8 fr[PD];
#pragma unroll
        for (int st = 0; st < PD; ++st) {
            if (st == KS) asm volatile("" : "+v"(o2[0]), "+v"(o2[1]));
            fr[st] = frag(st);
        }
        floatx4 sh[2];
#pragma unroll
        for (int st = 0; st < 2 * KS; ++st) {
            const int h = st / KS, ks = st % KS;
            const bf16x8 f = fr[st % PD];
#pragma unroll
            for (int term = 2; term >= 0; --term) {
                const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
                sh[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, th[term][ks], ks == 0 && term == 2 ? zero : sh[h], 0, 0,
                                                                0);
            }
            if (st + PD < 2 * KS) {
                if (st + PD == KS) asm volatile("" : "+v"(o2[0]), "+v"(o2[1]));
                fr[st % PD] = frag(st + PD);
            }
            if (h == 0) term_slice(ks, KS, sprev, yprev, lprev);
            else term_slice(ks, KS, sh[0], yl.x, left);
            const int k = (st * J + KS - 1) / KS;
            if (k < J && (k * KS) / J == st) copy_k(sidx + SUBS, k, xw + ((sidx + SUBS) % NB) * BUF);
            if (J > KS && st == 0) copy_k(sidx + SUBS, 1, xw + ((sidx + SUBS) % NB) * BUF);
            if (st & 1) __builtin_amdgcn_sched_barrier(0);
        }
        sprev = sh[1];
        yprev = yl.y;
        lprev = left - 4;
    };
    if (nsub > 0) {
#pragma unroll
        for (int u = 0; u < SUBS; ++u)
#pragma unroll
            for (int k = 0; k < J; ++k) copy_k(u, k, ldsb + u * BUF);
    }
    for (int sidx = 0; sidx < nsub; ++sidx) {
        if (sidx % SUBS == 0) {
            wait_vmcnt<0>();               // the only copies outstanding are this stage's
            lds_barrier();
        }
        step(sidx, ldsb, ldsb);
    }
    wait_vmcnt<0>();                       // no copy may land in LDS after the end
#pragma unroll
    for (int st = 0; st < 3; ++st) term_slice(st, 3, sprev, yprev, lprev);
    // lanes holding chain l16: l16, l16 + 16, + 32, + 48
    lp += __shfl_xor(lp, 16, 64);
    lp += __shfl_xor(lp, 32, 64);
    const int64_t c = cw + l16;
    if (g == 0 && c < C) a.ws.part_lp[(int64_t)split * C + c] = lp;
}

// lpq[c] = sum over splits (fixed order) of the log-probability partials
__device__ __forceinline__ void lr16_lp_sum_body(const PlainArgs& a, int nsplit, int blk) {
    const int64_t c = (int64_t)blk * blockDim.x + threadIdx.x;
    if (c >= a.C) return;
    double l = 0.0;
    for (int s = 0; s < nsplit; ++s) l += a.ws.part_lp[(int64_t)s * a.C + c];
    a.ws.lpq[c] = l;
}

template <int KS>
__global__ __launch_bounds__(64 * LbGrad<KS>::NW) void k_lr16_grad_pipe(PlainArgs a, const float* __restrict__ xsrc,
                                                        const float* __restrict__ psrc, int drift,
                                                        int64_t rows_per_split, int nsplit) {
    lr16_grad_body<KS>(a, xsrc, psrc, drift, rows_per_split, nsplit, blockIdx.x);
}

template <int KS>
__global__ __launch_bounds__(64 * LbLogp<KS>::NW) void k_lr16_logp_pipe(PlainArgs a, const float* __restrict__ xsrc,
                                                        int64_t rows_per_split, int nsplit) {
    lr16_logp_body<KS>(a, xsrc, rows_per_split, nsplit, blockIdx.x);
}

__global__ __launch_bounds__(256) void k_lr16_lp_sum(PlainArgs a, int nsplit) { lr16_lp_sum_body(a, nsplit, blockIdx.x); }

// ---------------------------------------------------------------------------
// Few chains: the kernels above give a wave 16 or 32 chains and all rows of its
// split, so a launch has ceil(C / 256) (ceil(C / 128)) tiles x at most 8 splits
// of workgroups -- 8 on 256 CUs at 200 chains, and each walks its rows alone, at
// the rate one CU pulls X and X^T.  Here a workgroup of 8 waves owns 16 CS
// chains and one split, and its waves share the work of a row: in a stage of NS
// sub-tiles the waves form S and the residuals of 16-row halves (wave w those of
// chain tile w % CS); the packed residuals go through LDS; after a barrier wave
// w accumulates dim tiles w, w + 8, .. of G^T over the stage's sub-tiles in
// their order.  Every output sees the MFMAs it sees above, in the same order
// (the split count is the same too): the partials are bitwise the same.
//
// X alone is copied global -> LDS (contiguous rows; the 64-byte pieces of X^T
// would take a cache line each), NBUF - 1 stages ahead, and read there by rows
// for S and transposed (ds_read_b64_tr_b16) for G^T; 16-byte slots are swizzled
// by f(row) = 2 (row & 3) + ((row >> 3) & 1), distinct over the 8 rows of a row
// phase and even-distinct over the 4 of a transposed one.
// ---------------------------------------------------------------------------
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

template <int KS, int CS>
struct LbFew {
    static constexpr int NW = 8;
    static constexpr int DP = 32 * KS, RB = 2 * DP;                      // dims and bytes of a row
    static constexpr int NS = KS <= 2 ? 8 : (KS <= 6 ? 4 : 2);           // sub-tiles per stage
    static constexpr int XB = NS * LB_RS * RB;                           // bytes of a stage
    static constexpr int BUF = XB + 256;                                 // and its labels
    static constexpr int RES = NS * CS * 1024;                           // bytes of a stage's residuals
    static constexpr int NBUF = 4 * BUF + RES <= 160 * 1024 ? 4 : (3 * BUF + RES <= 160 * 1024 ? 3 : 2);
    static constexpr int XI = XB / 1024;                                 // 1 KB copy blocks of a stage
    static constexpr int J = XI / NW + 1;                                // copies per wave, labels included
    static constexpr int NH = 2 * NS;                                    // 16-row halves of a stage
    static constexpr int NT = 2 * KS, TPW = (NT + NW - 1) / NW;          // dim tiles, per wave
    static_assert(XI % NW == 0, "copies must split evenly over the waves");
};
__device__ __forceinline__ int lb_few_swz(int row, int slots) {
    return (((row & 3) << 1) | ((row >> 3) & 1)) & (slots - 1 < 7 ? slots - 1 : 7);
}
// Copy of the stage at xsrc (labels ysrc) into buf.  Only the first `rows` rows
// belong to the split: later ones repeat the first and are never used.
template <int KS, int CS>
__device__ __forceinline__ void lb_few_copy(const char* xsrc, const uint8_t* ysrc, int rows, uint8_t* __restrict__ buf,
                                            int w, int lane) {
    using P = LbFew<KS, CS>;
    constexpr int SR = 4 * KS;
    int ln = lane;
    asm volatile("" : "+v"(ln));
#pragma unroll
    for (int k = 0; k < P::J - 1; ++k) {
        const int i = w + P::NW * k, q = i * 64 + ln;
        const int row = q / SR, c = (q % SR) ^ lb_few_swz(row, SR);
        const uint32_t off = (uint32_t)((row < rows ? row : 0) * P::RB + 16 * c);
        __builtin_amdgcn_global_load_lds((const void*)(xsrc + off), (lds_void_t*)(buf + i * 1024), 16, 0, 0);
    }
    __builtin_amdgcn_global_load_lds((const void*)(ysrc + (4 * ln < rows ? 4 * ln : 0)), (lds_void_t*)(buf + P::XB), 4,
                                     0, 0);
}

// Four dims d0 .. d0 + 3 (d0 < D) of a row of D >= 4 floats by one 16-byte load at
// whatever alignment, moved back inside the row where it would run past its end
// (lb_row4), and the dims it was asked for out of it, zeros past D (lb_pick4).
struct __attribute__((packed, aligned(4))) f32x4u { floatx4 v; };
__device__ __forceinline__ floatx4 lb_row4(const float* __restrict__ row, int d0, int D) {
    return ((const f32x4u*)(row + (d0 + 4 <= D ? d0 : D - 4)))->v;
}
__device__ __forceinline__ floatx4 lb_pick4(floatx4 v, int d0, int D) {
    const int sh = d0 + 4 <= D ? 0 : d0 + 4 - D;
    floatx4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float e = v[j];
#pragma unroll
        for (int k = 1; j + k < 4; ++k) e = sh == k ? v[j + k] : e;
        r[j] = d0 + j < D ? e : 0.f;
    }
    return r;
}
// theta (drifted when drift) of chains c0 .. c0 + NC - 1, loaded once by the
// workgroup: unit u = 512 k + thread is dims 4 (u % (8 KS)) of chain u / (8 KS).
// (Every wave loading the rows for itself had cost a third of the launch at D =
// 150, where rows are read by single floats.)
template <int KS, int NC>
struct LbTheta {
    static constexpr int NU = (NC * 8 * KS + 511) / 512;
    floatx4 v[NU];
    __device__ __forceinline__ void load(const PlainArgs& a, const float* __restrict__ x, const float* __restrict__ p,
                                         int drift, int64_t c0) {
        const int D = (int)a.tg.D;
        floatx4 pv[NU];
        float eps[NU];
        if (D >= 4) {
#pragma unroll
            for (int k = 0; k < NU; ++k) {
                const int64_t cc = c0 + chain(k) < a.C ? c0 + chain(k) : 0;
                const int d0 = dim(k) < D ? dim(k) : 0;
                v[k] = lb_row4(x + cc * D, d0, D);
                if (drift) {
                    pv[k] = lb_row4(p + cc * D, d0, D);
                    eps[k] = (float)a.ws.eps[cc];
                }
            }
        } else {
            asm volatile("" ::: "memory");        // keeps the two kinds of loads apart
#pragma unroll
            for (int k = 0; k < NU; ++k) {
                const int64_t cc = c0 + chain(k) < a.C ? c0 + chain(k) : 0;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    // as lb_row4 would deliver them: d0 = 0, moved back by 4 - D
                    const int d = j - (4 - D) > 0 ? j - (4 - D) : 0;
                    v[k][j] = x[cc * D + d];
                    if (drift) pv[k][j] = p[cc * D + d];
                }
                if (drift) eps[k] = (float)a.ws.eps[cc];
            }
        }
#pragma unroll
        for (int k = 0; k < NU; ++k) {
            const bool ok = c0 + chain(k) < a.C;
            const int d0 = dim(k);
            v[k] = lb_pick4(v[k], d0, D);
            if (drift) {
                pv[k] = lb_pick4(pv[k], d0, D);
#pragma unroll
                for (int j = 0; j < 4; ++j) v[k][j] = fmaf(eps[k], pv[k][j], v[k][j]);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) v[k][j] = ok && d0 + j < D ? v[k][j] : 0.f;
        }
    }
    // the chain and first dim of this thread's unit k (chain NC or more: none)
    __device__ __forceinline__ int chain(int k) const { return (512 * k + (int)threadIdx.x) / (8 * KS); }
    __device__ __forceinline__ int dim(int k) const { return 4 * ((512 * k + (int)threadIdx.x) % (8 * KS)); }
};

template <int KS, int CS>
__global__ __launch_bounds__(512) void k_lr16_grad_few(PlainArgs a, const float* __restrict__ xsrc,
                                                       const float* __restrict__ psrc, int drift,
                                                       int64_t rows_per_split, int nsplit) {
    using P = LbFew<KS, CS>;
    constexpr int RB = P::RB, NS = P::NS, XB = P::XB, BUF = P::BUF, NBUF = P::NBUF, J = P::J, NH = P::NH, NT = P::NT, TPW = P::TPW,
                  NW = P::NW, NG = NW / CS, HW = (NH + NG - 1) / NG;
    extern __shared__ __align__(16) uint8_t ldsb[];
    // NBUF stages of X, then the residuals [NS][CS][64 lanes][16 bytes]
    const int64_t D = a.tg.D, C = a.C, NP = (a.tg.N + LB_RS - 1) / LB_RS * LB_RS;
    const int ntile = (int)((C + 16 * CS - 1) / (16 * CS));
    int tile, split;
    lb_map(blockIdx.x, ntile, nsplit, &tile, &split);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int64_t cw = (int64_t)tile * (16 * CS);
    const int wcs = w % CS, wg = w / CS;                  // chain tile and half group of S

    const int64_t r_begin = (int64_t)split * rows_per_split;
    int64_t r_end = r_begin + rows_per_split;
    if (r_end > NP) r_end = NP;
    const int nsub = r_begin < r_end ? (int)((r_end - r_begin) / LB_RS) : 0;
    const int nst = (nsub + NS - 1) / NS;
    const char* xs = (const char*)a.ws.xp + r_begin * RB;
    const uint8_t* ys = (const uint8_t*)a.ws.yp + r_begin;
    auto copy_in = [&](int t, uint8_t* __restrict__ dst) {
        const int left = (nsub - NS * t) * LB_RS;
        lb_few_copy<KS, CS>(xs + (int64_t)t * XB, ys + t * (NS * LB_RS), left < NS * LB_RS ? left : NS * LB_RS, dst, w, lane);
    };
    // theta of the workgroup's chains through the last stage buffer (free until the
    // first stage has passed its barrier) as B operands
    bf16x8 thb[KS];
    auto prologue = [&](uint8_t* __restrict__ tb, uint8_t* __restrict__ dst) {
        constexpr int TS = RB + 16;                       // bytes of a chain's row there
        LbTheta<KS, 16 * CS> th;
        th.load(a, xsrc, psrc, drift, cw);
#pragma unroll
        for (int t = 0; t < NBUF - 1; ++t)
            if (t < nst) copy_in(t, dst + t * BUF);
#pragma unroll
        for (int k = 0; k < th.NU; ++k)
            if (th.chain(k) < 16 * CS) *(uint2*)(tb + th.chain(k) * TS + 2 * th.dim(k)) = pack4_bf16(th.v[k]);
        lds_barrier();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) thb[ks] = *(const bf16x8*)(tb + (16 * wcs + l16) * TS + 64 * ks + 16 * g);
    };
    prologue(ldsb + (NBUF - 1) * BUF, ldsb);
    floatx4 gacc[CS][TPW];
#pragma unroll
    for (int cs = 0; cs < CS; ++cs)
#pragma unroll
        for (int j = 0; j < TPW; ++j) gacc[cs][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    // offsets in a sub-tile: row fragments of half mt (even / odd k-step), the transposed
    // blocks of the wave's dim tiles
    uint32_t xo[2][2], to[TPW];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        const int row = 8 * (l16 >> 2) + 4 * mt + (l16 & 3), f = lb_few_swz(row, 4 * KS);
#pragma unroll
        for (int e = 0; e < 2; ++e) xo[mt][e] = (uint32_t)(row * RB + 16 * ((g + 4 * e) ^ f));
    }
    {
        const int row = 8 * g + (l16 >> 2), f = lb_few_swz(row, 4 * KS);
#pragma unroll
        for (int j = 0; j < TPW; ++j) {
            const int nt = w + NW * j < NT ? w + NW * j : NT - 1;
            to[j] = (uint32_t)(row * RB + 16 * ((2 * nt + ((l16 & 3) >> 1)) ^ f) + 8 * (l16 & 1));
        }
    }
    // one stage; the copy target, the buffer read and the residuals are distinct, which
    // the restrict qualifiers tell the compiler: the LDS reads wait for no copy in flight
    auto stage = [&](int t, uint8_t* __restrict__ dst, const uint8_t* __restrict__ xb, uint8_t* __restrict__ rbuf) {
        // stage t complete: at most the copies of the stages after it outstanding
        if (NBUF >= 4 && t + 2 < nst) wait_vmcnt<2 * J>();
        else if (NBUF >= 3 && t + 1 < nst) wait_vmcnt<J>();
        else wait_vmcnt<0>();
        lds_barrier();
        if (t + NBUF - 1 < nst) copy_in(t + NBUF - 1, dst);
        const int ns = nsub - NS * t < NS ? nsub - NS * t : NS;
#pragma unroll
        for (int u = 0; u < HW; ++u) {
            const int h = wg + NG * u;                    // uniform over the wave
            if (h < 2 * ns) {
                const uint8_t* xh = xb + (h >> 1) * (LB_RS * RB);
                const uint32_t o0 = (h & 1) ? xo[1][0] : xo[0][0], o1 = (h & 1) ? xo[1][1] : xo[0][1];
                bf16x8 xa[KS];
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) xa[ks] = *(const bf16x8*)(xh + ((ks & 1) ? o1 : o0) + 128 * (ks >> 1));
                floatx4 sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
                    sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[ks], thb[ks], sacc, 0, 0, 0);
                // every fragment read first (one LDS latency), then the chain of MFMAs
                __builtin_amdgcn_sched_group_barrier(0x100, KS, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, KS, 0);
                // labels of the lane's rows 8 g + 4 mt .. + 3
                const uint32_t yw = *(const uint32_t*)(xb + XB + LB_RS * (h >> 1) + 8 * g + 4 * (h & 1));
                floatx4 r;
#pragma unroll
                for (int v = 0; v < 4; ++v) r[v] = (float)((yw >> (8 * v)) & 0xffu) - sigmoid_hw(sacc[v]);
                *(uint2*)(rbuf + ((((h >> 1) * CS + wcs) * 64 + lane) * 16 + 8 * (h & 1))) = pack4_bf16(r);
            }
        }
        lds_barrier();
        // a wave's tiles past NT repeat the last one (not stored)
        auto gsub = [&](int s) {
            bf16x8 ra[CS], bx[TPW];
#pragma unroll
            for (int cs = 0; cs < CS; ++cs) ra[cs] = *(const bf16x8*)(rbuf + ((s * CS + cs) * 64 + lane) * 16);
#pragma unroll
            for (int j = 0; j < TPW; ++j) {
                const uint8_t* p = xb + s * (LB_RS * RB) + to[j];
                const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
                const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * RB));
                bx[j] = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
            }
#pragma unroll
            for (int j = 0; j < TPW; ++j)
#pragma unroll
                for (int cs = 0; cs < CS; ++cs)
                    gacc[cs][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ra[cs], bx[j], gacc[cs][j], 0, 0, 0);
        };
        if (ns == NS) {
#pragma unroll
            for (int s = 0; s < NS; ++s) gsub(s);
        } else {
            for (int s = 0; s < ns; ++s) gsub(s);
        }
    };
    for (int t = 0; t < nst; ++t)
        stage(t, ldsb + ((t + NBUF - 1) % NBUF) * BUF, ldsb + (t % NBUF) * BUF, ldsb + NBUF * BUF);
#pragma unroll
    for (int cs = 0; cs < CS; ++cs)
#pragma unroll
        for (int j = 0; j < TPW; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t c = cw + 16 * cs + 4 * g + v;
                const int64_t d = 16 * (w + NW * j) + l16;
                if (c < C && d < D) a.ws.part_g[((int64_t)split * C + c) * D + d] = gacc[cs][j][v];
            }
}

// The accurate log-probability for few chains, likewise: a workgroup owns 16
// chains and one split, the waves form the logits and the FP32 sums of 4 rows'
// terms of the stage's halves, and wave 0 adds those in FP64 in the row order of
// the kernel above (bitwise the same partials).
template <int KS>
__global__ __launch_bounds__(512) void k_lr16_logp_few(PlainArgs a, const float* __restrict__ xsrc,
                                                       int64_t rows_per_split, int nsplit) {
    using P = LbFew<KS, 1>;
    constexpr int RB = P::RB, NS = P::NS, XB = P::XB, BUF = P::BUF, NBUF = P::NBUF, J = P::J, NH = P::NH, NW = P::NW,
                  HW = (NH + NW - 1) / NW;
    extern __shared__ __align__(16) uint8_t ldsb[];
    // NBUF stages of X, then the terms [2][NH][64]
    const int64_t N = a.tg.N, C = a.C, NP = (N + LB_RS - 1) / LB_RS * LB_RS;
    const int ntile = (int)((C + 15) / 16);
    int tile, split;
    lb_map(blockIdx.x, ntile, nsplit, &tile, &split);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int64_t c = (int64_t)tile * 16 + l16;
    const int64_t r_begin = (int64_t)split * rows_per_split;
    int64_t r_end = r_begin + rows_per_split;
    if (r_end > NP) r_end = NP;
    const int nsub = r_begin < r_end ? (int)((r_end - r_begin) / LB_RS) : 0;
    const int nst = (nsub + NS - 1) / NS;
    const char* xs = (const char*)a.ws.xp + r_begin * RB;
    const uint8_t* ys = (const uint8_t*)a.ws.yp + r_begin;
    auto copy_in = [&](int t, uint8_t* __restrict__ dst) {
        const int left = (nsub - NS * t) * LB_RS;
        lb_few_copy<KS, 1>(xs + (int64_t)t * XB, ys + t * (NS * LB_RS), left < NS * LB_RS ? left : NS * LB_RS, dst, w, lane);
    };
    bf16x8 th[3][KS];
    auto prologue = [&](uint8_t* __restrict__ tb, uint8_t* __restrict__ dst) {
        constexpr int TS = 2 * RB + 16;                   // FP32 theta through the last stage buffer
        LbTheta<KS, 16> tv;
        tv.load(a, xsrc, nullptr, 0, (int64_t)tile * 16);
#pragma unroll
        for (int t = 0; t < NBUF - 1; ++t)
            if (t < nst) copy_in(t, dst + t * BUF);
#pragma unroll
        for (int k = 0; k < tv.NU; ++k)
            if (tv.chain(k) < 16) *(floatx4*)(tb + tv.chain(k) * TS + 4 * tv.dim(k)) = tv.v[k];
        lds_barrier();
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const float* r = (const float*)(tb + l16 * TS) + 32 * ks + 8 * g;
            const floatx4 u0 = *(const floatx4*)r, u1 = *(const floatx4*)(r + 4);
            lb_split_theta(floatx8{u0[0], u0[1], u0[2], u0[3], u1[0], u1[1], u1[2], u1[3]}, th[0][ks], th[1][ks],
                           th[2][ks]);
        }
    };
    prologue(ldsb + (NBUF - 1) * BUF, ldsb);
    uint32_t xo[2][2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt) {
        const int row = 8 * (l16 >> 2) + 4 * mt + (l16 & 3), f = lb_few_swz(row, 4 * KS);
#pragma unroll
        for (int e = 0; e < 2; ++e) xo[mt][e] = (uint32_t)(row * RB + 16 * ((g + 4 * e) ^ f));
    }
    double lp = 0.0;
    auto stage = [&](int t, uint8_t* __restrict__ dst, const uint8_t* __restrict__ xb, float* __restrict__ tbuf) {
        if (NBUF >= 4 && t + 2 < nst) wait_vmcnt<2 * J>();
        else if (NBUF >= 3 && t + 1 < nst) wait_vmcnt<J>();
        else wait_vmcnt<0>();
        lds_barrier();
        if (t + NBUF - 1 < nst) copy_in(t + NBUF - 1, dst);
        // the sums of stage t - 1 (its terms were complete at the barrier)
        auto add = [&](int tp) {
            const int np = nsub - NS * tp < NS ? nsub - NS * tp : NS;
            for (int h = 0; h < 2 * np; ++h) lp += (double)tbuf[((tp & 1) * NH + h) * 64 + lane];
        };
        if (w == 0 && t > 0) add(t - 1);
        const int ns = nsub - NS * t < NS ? nsub - NS * t : NS;
#pragma unroll
        for (int u = 0; u < HW; ++u) {
            const int h = w + NW * u;
            if (h < 2 * ns) {
                const uint8_t* xh = xb + (h >> 1) * (LB_RS * RB);
                const uint32_t o0 = (h & 1) ? xo[1][0] : xo[0][0], o1 = (h & 1) ? xo[1][1] : xo[0][1];
                floatx4 sacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const bf16x8 ax = *(const bf16x8*)(xh + ((ks & 1) ? o1 : o0) + 128 * (ks >> 1));
#pragma unroll
                    for (int term = 2; term >= 0; --term)
                        sacc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ax, th[term][ks], sacc, 0, 0, 0);
                }
                const int64_t row0 = r_begin + (int64_t)LB_RS * (NS * t + (h >> 1)) + 8 * g + 4 * (h & 1);
                const bool whole = row0 + 4 <= N;
                const uint32_t yw = *(const uint32_t*)(xb + XB + LB_RS * (h >> 1) + 8 * g + 4 * (h & 1));
                float t4 = 0.f;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float s = sacc[v];
                    const float y = (float)((yw >> (8 * v)) & 0xffu);
                    const float tv = fmaf(y, s, -softplus_hw(s));
                    t4 += (whole || row0 + v < N) ? tv : 0.f;
                }
                tbuf[((t & 1) * NH + h) * 64 + lane] = t4;
            }
        }
        if (t + 1 == nst) {
            lds_barrier();
            if (w == 0) add(t);
        }
    };
    for (int t = 0; t < nst; ++t)
        stage(t, ldsb + ((t + NBUF - 1) % NBUF) * BUF, ldsb + (t % NBUF) * BUF, (float*)(ldsb + NBUF * BUF));
    if (w != 0) return;
    lp += __shfl_xor(lp, 16, 64);
    lp += __shfl_xor(lp, 32, 64);
    if (g == 0 && c < C) a.ws.part_lp[(int64_t)split * C + c] = lp;
}

// ---------------------------------------------------------------------------
// Several requests in one launch (the serving form): job j owns blocks
// begin[k] .. begin[k] + nblk[k] - 1 of the grid of kernel kind k; its
// arguments are copied out of the device job table into registers, and the
// body is the one-request kernel's with the job-local block index, so every
// request computes bitwise what it computes alone.
// ---------------------------------------------------------------------------
template <int KS>
__global__ __launch_bounds__(64 * LbGrad<KS>::NW) void k_lr16_grad_multi(const Lr16Job* __restrict__ jobs, int njobs) {
    int64_t lb;
    const int j = lr16_job_of(jobs, njobs, LR16_KIND_GRAD, blockIdx.x, &lb);
    if (j < 0) return;
    const PlainArgs a = jobs[j].a;
    lr16_grad_body<KS>(a, (const float*)a.ws.xq, (const float*)a.ws.pq, 1, jobs[j].rows_g, jobs[j].nsplit_g, (int)lb);
}

template <int KS>
__global__ __launch_bounds__(64 * LbLogp<KS>::NW) void k_lr16_logp_multi(const Lr16Job* __restrict__ jobs, int njobs) {
    int64_t lb;
    const int j = lr16_job_of(jobs, njobs, LR16_KIND_LOGP, blockIdx.x, &lb);
    if (j < 0) return;
    const PlainArgs a = jobs[j].a;
    lr16_logp_body<KS>(a, (const float*)a.ws.xq, jobs[j].rows_lp, jobs[j].nsplit_lp, (int)lb);
}

__global__ __launch_bounds__(256) void k_lr16_lp_sum_multi(const Lr16Job* __restrict__ jobs, int njobs) {
    int64_t lb;
    const int j = lr16_job_of(jobs, njobs, LR16_KIND_LPSUM, blockIdx.x, &lb);
    if (j < 0) return;
    const PlainArgs a = jobs[j].a;
    lr16_lp_sum_body(a, jobs[j].nsplit_lp, (int)lb);
}

// Padded copies: X [N, D] -> Xp [NP, DP] and Xt [DP, NP] (zeros outside), y -> yp
// [NP] (zeros past N); 32 x 32 tiles through LDS for the transpose.
__global__ __launch_bounds__(256) void k_pad_bf16(const uint16_t* __restrict__ X, const uint8_t* __restrict__ y,
                                                  uint16_t* __restrict__ Xp, uint16_t* __restrict__ Xt,
                                                  uint8_t* __restrict__ yp, int64_t N, int64_t D, int64_t NP,
                                                  int64_t DP) {
    __shared__ uint16_t tile[32][33];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int64_t n0 = (int64_t)blockIdx.x * 32, d0 = (int64_t)blockIdx.y * 32;
    for (int r = ty; r < 32; r += 8) {
        const int64_t n = n0 + r, d = d0 + tx;
        const uint16_t v = (n < N && d < D) ? X[n * D + d] : (uint16_t)0;
        tile[r][tx] = v;
        Xp[n * DP + d] = v;
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) Xt[(d0 + r) * NP + n0 + tx] = tile[tx][r];
    if (blockIdx.y == 0 && threadIdx.x < 32) {
        const int64_t n = n0 + threadIdx.x;
        yp[n] = n < N ? y[n] : (uint8_t)0;
    }
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
// 32-dim k-steps of the padded dims for D dims (0 beyond 512)
static int lb_ks(int64_t D) {
    const int64_t k = (D + 31) / 32;
    for (int v : {1, 2, 4, 6, 8, 12, 16})
        if (k <= v) return v;
    return 0;
}

bool bf16_grad_supported(const TargetDev& tg) { return tg.kind == HMC_TGT_LOGREG && tg.x_bf16 && lb_ks(tg.D) > 0; }

size_t lb_pad_bytes(int64_t N, int64_t D, int64_t* np, int64_t* dp) {
    const int64_t NP = (N + LB_RS - 1) / LB_RS * LB_RS, DP = 32 * (int64_t)lb_ks(D);
    if (np) *np = NP;
    if (dp) *dp = DP;
    return (size_t)NP * (size_t)DP * 2;
}

static int lb_grad_ct(int64_t D) { return lb_ks(D) <= 8 ? LbGrad<8>::CT : LbGrad<16>::CT; }
static int lb_logp_ct(int64_t D) { return lb_ks(D) <= 8 ? LbLogp<8>::CT : LbLogp<16>::CT; }

// row splits: a power of two (so that blocks map to XCDs by split) filling the
// 256 CUs once, at most 8, at least 4 sub-tiles each
static int lb_nsplit_for(int ntile, int64_t N) {
    int s = 1;
    while (s < 8 && ntile * 2 * s <= 256 && (N + 2 * s - 1) / (2 * s) >= 4 * LB_RS) s *= 2;
    return s;
}
int lb_grad_nsplit(int64_t N, int64_t C, int64_t D) {
    const int ct = lb_grad_ct(D);
    return lb_nsplit_for((int)((C + ct - 1) / ct), N);
}
int lb_grad_nsplit_t(const PlainArgs& a) {
    return a.tune.lr16_nsplit > 0 ? a.tune.lr16_nsplit : lb_grad_nsplit(a.tg.N, a.C, a.tg.D);
}
int lb_logp_nsplit(int64_t N, int64_t C, int64_t D) {
    const int ct = lb_logp_ct(D);
    return lb_nsplit_for((int)((C + ct - 1) / ct), N);
}

static int64_t rows_for(int64_t N, int nsplit) {
    const int64_t r = (N + nsplit - 1) / nsplit;
    return (r + LB_RS - 1) / LB_RS * LB_RS;
}

hipError_t launch_pad_bf16(const PlainArgs& a, hipStream_t s) {
    int64_t NP = 0, DP = 0;
    (void)lb_pad_bytes(a.tg.N, a.tg.D, &NP, &DP);
    const dim3 grid((unsigned)(NP / 32), (unsigned)(DP / 32));
    hipLaunchKernelGGL(k_pad_bf16, grid, dim3(256), 0, s, (const uint16_t*)a.tg.X, a.tg.y, (uint16_t*)a.ws.xp,
                       (uint16_t*)a.ws.xt, (uint8_t*)a.ws.yp, a.tg.N, a.tg.D, NP, DP);
    return hipGetLastError();
}

template <int KS, int CS>
static hipError_t lb_few_launch(const PlainArgs& a, const float* x, const float* p, int drift, int nsplit,
                                int64_t rows, hipStream_t s) {
    using P = LbFew<KS, CS>;
    constexpr int lds = P::NBUF * P::BUF + P::RES;
    static_assert((P::NBUF - 1) * P::BUF + 16 * CS * (P::RB + 16) <= lds, "theta's staging");
    static_assert(lds <= 160 * 1024, "LDS");
    const int64_t ntile = (a.C + 16 * CS - 1) / (16 * CS);
    if (lds > 65536)
        (void)hipFuncSetAttribute((const void*)k_lr16_grad_few<KS, CS>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    hipLaunchKernelGGL((k_lr16_grad_few<KS, CS>), dim3((unsigned)(ntile * nsplit)), dim3(512), lds, s, a, x, p, drift,
                       rows, nsplit);
    return hipGetLastError();
}

// Chain tiles per workgroup of the few-chain kernel, 0: the many-chain kernel.  As few
// chains per workgroup as lets its workgroups (one per CU) run in one round, or up to
// D = 256 in one and a half: a round of 64 chains takes half the time of the 256-chain
// kernel's, which any number of chains up to a full round takes (beyond D = 256, two
// thirds of the 128-chain one's).  Per gradient and its partial sum: 20011 x 150, 200
// chains 140 -> 32 us; 30000 x 250, 1000 chains 255 -> 76, 2000 chains 260 -> 115, 3000
// chains 265 -> 214; 30000 x 512, 2048 chains 274 -> 195.  Past the line: 50000 x 256,
// 4000 chains 350 in two rounds against 304; 30000 x 512, 3000 chains 342 against 293.
static int lb_few_cs(int ks, int64_t C, int nsplit) {
    auto blocks = [&](int cs) { return (C + 16 * cs - 1) / (16 * cs) * nsplit; };
    if (blocks(1) <= 256) return 1;
    if (blocks(2) <= 256) return 2;
    return blocks(4) <= (ks <= 8 ? 384 : 256) ? 4 : 0;
}

template <int KS>
static hipError_t lb_grad_k(const PlainArgs& a, const float* x, const float* p, int drift, hipStream_t s) {
    using P = LbGrad<KS>;
    const int ntile = (int)((a.C + P::CT - 1) / P::CT);
    const int nsplit = lb_grad_nsplit_t(a);
    const int64_t NP = (a.tg.N + LB_RS - 1) / LB_RS * LB_RS;
    const int64_t rows = rows_for(NP, nsplit);
    switch (lb_few_cs(KS, a.C, nsplit)) {
    case 1: return lb_few_launch<KS, 1>(a, x, p, drift, nsplit, rows, s);
    case 2: return lb_few_launch<KS, 2>(a, x, p, drift, nsplit, rows, s);
    case 4: return lb_few_launch<KS, 4>(a, x, p, drift, nsplit, rows, s);
    }
    const size_t lds = (size_t)P::LDS;
    if (lds > 65536)
        (void)hipFuncSetAttribute((const void*)k_lr16_grad_pipe<KS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds);
    hipLaunchKernelGGL(k_lr16_grad_pipe<KS>, dim3((unsigned)(ntile * nsplit)), dim3(64 * P::NW), lds, s, a, x, p,
                       drift, rows, nsplit);
    return hipGetLastError();
}

template <int KS>
static hipError_t lb_logp_k(const PlainArgs& a, const float* x, hipStream_t s) {
    using P = LbLogp<KS>;
    const int ntile = (int)((a.C + P::CT - 1) / P::CT);
    const int nsplit = lb_logp_nsplit(a.tg.N, a.C, a.tg.D);
    const int64_t NP = (a.tg.N + LB_RS - 1) / LB_RS * LB_RS;
    // Up to two rounds of 16-chain workgroups (four where the three terms of theta are
    // few) against the kernel below, whole transitions less the gradients: 20011 x
    // 150, 200 chains 134 -> 47 us; 30000 x 250, 1000 chains (504 workgroups) 209 -> 161,
    // 2000 chains (1000) 214 -> 301; 40000 x 60, 1500 chains (752) 177 -> 101.
    if ((a.C + 15) / 16 * nsplit <= (KS <= 2 ? 1024 : 512)) {
        using F = LbFew<KS, 1>;
        constexpr int flds = F::NBUF * F::BUF + 2 * F::NH * 64 * 4;
        static_assert((F::NBUF - 1) * F::BUF + 16 * (2 * F::RB + 16) <= flds, "theta's staging");
        static_assert(flds <= 160 * 1024, "LDS");
        if (flds > 65536)
            (void)hipFuncSetAttribute((const void*)k_lr16_logp_few<KS>, hipFuncAttributeMaxDynamicSharedMemorySize, flds);
        hipLaunchKernelGGL(k_lr16_logp_few<KS>, dim3((unsigned)((a.C + 15) / 16 * nsplit)), dim3(512), flds, s, a, x,
                           rows_for(NP, nsplit), nsplit);
        hipLaunchKernelGGL(k_lr16_lp_sum, dim3((unsigned)((a.C + 255) / 256)), dim3(256), 0, s, a, nsplit);
        return hipGetLastError();
    }
    const size_t lds = (size_t)P::LDS;
    if (lds > 65536)
        (void)hipFuncSetAttribute((const void*)k_lr16_logp_pipe<KS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                  (int)lds);
    hipLaunchKernelGGL(k_lr16_logp_pipe<KS>, dim3((unsigned)(ntile * nsplit)), dim3(64 * P::NW), lds, s, a, x,
                       rows_for(NP, nsplit), nsplit);
    hipLaunchKernelGGL(k_lr16_lp_sum, dim3((unsigned)((a.C + 255) / 256)), dim3(256), 0, s, a, nsplit);
    return hipGetLastError();
}

int lr16_batch_class(const PlainArgs& a) {
    if (a.tg.kind != HMC_TGT_LOGREG || !a.bf16_grad || a.f64) return -1;
    const int ks = lb_ks(a.tg.D);
    return ks > 0 ? ks : -1;
}

int64_t lr16_alone_cost(const PlainArgs& a, int64_t* subs) {
    const int ns = lb_grad_nsplit_t(a);
    *subs = rows_for((a.tg.N + LB_RS - 1) / LB_RS * LB_RS, ns) / LB_RS;
    const int cs = lb_few_cs(lb_ks(a.tg.D), a.C, ns);
    if (cs == 0) return 1024;
    const int64_t blocks = (a.C + 16 * cs - 1) / (16 * cs) * ns;
    return cs == 1 ? blocks : (cs == 2 ? 3 * blocks / 2 : 5 * blocks / 2);
}

void lr16_job_shape(const PlainArgs& a, Lr16Job* j) {
    const int64_t NP = (a.tg.N + LB_RS - 1) / LB_RS * LB_RS;
    j->nsplit_g = lb_grad_nsplit_t(a);
    j->nsplit_lp = lb_logp_nsplit(a.tg.N, a.C, a.tg.D);
    j->rows_g = rows_for(NP, j->nsplit_g);
    j->rows_lp = rows_for(NP, j->nsplit_lp);
    const int64_t ctg = lb_grad_ct(a.tg.D), ctl = lb_logp_ct(a.tg.D);
    j->nblk[LR16_KIND_GRAD] = (a.C + ctg - 1) / ctg * j->nsplit_g;
    j->nblk[LR16_KIND_LOGP] = (a.C + ctl - 1) / ctl * j->nsplit_lp;
    j->nblk[LR16_KIND_LPSUM] = (a.C + 255) / 256;
}

template <int KS>
static hipError_t lb_multi_k(int kind, const Lr16Job* jobs, int njobs, int64_t blocks, hipStream_t s) {
    const dim3 grid((unsigned)blocks);
    if (kind == LR16_KIND_GRAD) {
        const size_t lds = (size_t)LbGrad<KS>::LDS;
        if (lds > 65536)
            (void)hipFuncSetAttribute((const void*)k_lr16_grad_multi<KS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)lds);
        hipLaunchKernelGGL(k_lr16_grad_multi<KS>, grid, dim3(64 * LbGrad<KS>::NW), lds, s, jobs, njobs);
    } else if (kind == LR16_KIND_LOGP) {
        const size_t lds = (size_t)LbLogp<KS>::LDS;
        if (lds > 65536)
            (void)hipFuncSetAttribute((const void*)k_lr16_logp_multi<KS>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)lds);
        hipLaunchKernelGGL(k_lr16_logp_multi<KS>, grid, dim3(64 * LbLogp<KS>::NW), lds, s, jobs, njobs);
    } else {
        hipLaunchKernelGGL(k_lr16_lp_sum_multi, grid, dim3(256), 0, s, jobs, njobs);
    }
    return hipGetLastError();
}

hipError_t launch_lr16_kind_multi(int kind, int64_t D, const Lr16Job* jobs_dev, int njobs, int64_t blocks,
                                  hipStream_t s) {
    if (blocks <= 0) return hipSuccess;
    switch (lb_ks(D)) {
    case 1: return lb_multi_k<1>(kind, jobs_dev, njobs, blocks, s);
    case 2: return lb_multi_k<2>(kind, jobs_dev, njobs, blocks, s);
    case 4: return lb_multi_k<4>(kind, jobs_dev, njobs, blocks, s);
    case 6: return lb_multi_k<6>(kind, jobs_dev, njobs, blocks, s);
    case 8: return lb_multi_k<8>(kind, jobs_dev, njobs, blocks, s);
    case 12: return lb_multi_k<12>(kind, jobs_dev, njobs, blocks, s);
    case 16: return lb_multi_k<16>(kind, jobs_dev, njobs, blocks, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_lr16_grad(const PlainArgs& a, const float* x, const float* p, int drift, hipStream_t s) {
    switch (lb_ks(a.tg.D)) {
    case 1: return lb_grad_k<1>(a, x, p, drift, s);
    case 2: return lb_grad_k<2>(a, x, p, drift, s);
    case 4: return lb_grad_k<4>(a, x, p, drift, s);
    case 6: return lb_grad_k<6>(a, x, p, drift, s);
    case 8: return lb_grad_k<8>(a, x, p, drift, s);
    case 12: return lb_grad_k<12>(a, x, p, drift, s);
    case 16: return lb_grad_k<16>(a, x, p, drift, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_lr16_logp(const PlainArgs& a, const float* x, hipStream_t s) {
    switch (lb_ks(a.tg.D)) {
    case 1: return lb_logp_k<1>(a, x, s);
    case 2: return lb_logp_k<2>(a, x, s);
    case 4: return lb_logp_k<4>(a, x, s);
    case 6: return lb_logp_k<6>(a, x, s);
    case 8: return lb_logp_k<8>(a, x, s);
    case 12: return lb_logp_k<12>(a, x, s);
    case 16: return lb_logp_k<16>(a, x, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace hmc
