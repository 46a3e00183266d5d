// k_logreg_f32.hip -- full-precision gradient of Bayesian logistic regression
// (FP32 gradients, X stored FP32 or BF16) for the plain form, on BF16 matrix
// instructions with exact operand splits:
//     S = X theta               (M = rows, N = chains, K = dims)
//     G = X^T R,  R = y - sigmoid(S)   (M = dims, N = chains, K = rows)
// An FP32 number is the exact sum of three BF16 numbers (its mantissa cut into
// 8 + 8 + 8 bits), and a BF16 x BF16 product is exact in FP32, so with FP32
// accumulation
//     X in BF16: 3 products   x (t_h + t_m + t_l)        -- every product formed
//     X in FP32: 8 products   of the 3 x 3; the one left out is below 2^-30
//                             of the leading one (a third term cut off is below
//                             2^-15 of its number)
// give the FP32 result with fewer roundings than v_mfma_f32_16x16x4f32, which
// rounds its accumulator after every 4 terms where v_mfma_f32_16x16x32_bf16
// rounds after 32 (six products, leaving out those below 2^-23, had twice the
// error of FP32 MFMA at D = 25).  One 16x16x32 BF16 MFMA takes 16 cycles of a
// SIMD and the eight FP32 MFMAs of the same block 256, so the split costs 48
// (128 for FP32 X) against 256.
//
// Against the FP32-MFMA kernel before it, a twentieth of a transition of 20 leapfrogs
// with its log-probability, and the gradient's error against 64 bits (2-norm, one
// step; before and after): 100000 x 256, BF16 X, 2048 chains 2613 -> 618 us, 9.8e-7 -> 5.8e-7;
// 20000 x 400, BF16 X, 2000 chains 1400 -> 317 us, 1.5e-6 -> 4.6e-7; 5000 x 300,
// FP32 X, 700 chains 325 -> 84 us, 1.4e-6 -> 4.0e-7; 10000 x 25, FP32 X, 1024
// chains 84 -> 28.9 us, 3.1e-7 -> 1.4e-7.  At 100000 x 256 the MFMAs take 0.28
// ms; the rest is the residuals' vector work (14 instructions and two
// transcendentals each) and the waits of two waves per SIMD, which theta's
// three terms and G (160 registers) allow.  At D <= 64 the residuals bound it.
//
// Work decomposition: a workgroup of 4 waves owns 64 chains (16 per wave) and
// one split of the rows.  A stage of 32 rows is read from global memory into
// registers one stage ahead, split into BF16 planes and written to LDS
// row-major; the first
// contraction reads rows (ds_read_b128), the second reads the same tile
// transposed (ds_read_b64_tr_b16), so X needs no second copy.  16-byte slots
// of a row are XOR-swizzled by f(row) = 2 (row & 3) + ((row >> 2) & 1): the 8
// rows of a b128 phase hit 8 distinct slots, and so do the 4 rows x 2 slots of
// a transposed phase.
//
// Lane layouts (v_mfma_f32_16x16x32_bf16): A[i][k] at lane i + 16 (k / 8),
// element k % 8; B[k][j] at lane j + 16 (k / 8); D[i][j] in VGPR i % 4 of lane
// j + 16 (i / 4).  A lane (chain l16, group g) gets S of rows 16 h + 4 g + v of
// half h, which are the K elements 4 h + v of its group in the second
// contraction: the residuals become the B operand in place.
#include "hmc_internal.hpp"

namespace hmc {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

constexpr int LS_NW = 4;            // waves per workgroup
constexpr int LS_RS = 32;           // rows per sub-tile

// The BF16 terms of an FP32 value by truncation, as the upper halves of three
// words.  Inf and NaN give NaN terms.
__device__ __forceinline__ void split3(float x, uint32_t& h, uint32_t& m, uint32_t& l) {
    h = __float_as_uint(x) & 0xffff0000u;
    const float r1 = x - __uint_as_float(h);
    m = __float_as_uint(r1) & 0xffff0000u;
    l = __float_as_uint(r1 - __uint_as_float(m));
}
// The same for a chain's position.  An infinite one (a trajectory that diverged)
// enters as the largest BF16 number: times an entry of X it gives an infinite logit,
// or one whose sigmoid is 0 or 1 as well, and times the zeros that stand for rows past
// a split's end and for the smaller terms of X it gives zero and no NaN, so that the
// other coordinates' gradients stay as finite as in FP32.  NaN stays in the smaller terms.
__device__ __forceinline__ void split3_pos(float x, uint32_t& h, uint32_t& m, uint32_t& l) {
    const uint32_t b = __float_as_uint(x);
    h = min(b & 0x7fff0000u, 0x7f7f0000u) | (b & 0x80000000u);
    const float r1 = (b & 0x7fffffffu) == 0x7f800000u ? 0.f : x - __uint_as_float(h);
    m = __float_as_uint(r1) & 0xffff0000u;
    l = __float_as_uint(r1 - __uint_as_float(m));
}
// the upper halves of a (low 16 bits of the result) and b (high 16 bits)
__device__ __forceinline__ uint32_t pack_hi(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// two floats to BF16, rounded to nearest even, a in the low half (v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    const floatx2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// e^-|s| on the hardware exp2 (1 ulp).  ACC: corrected to first order for the
// rounding of its argument (relative |s| 7e-8) and of log2 e (one-sided, |s| 1.3e-8),
// which the rows of a log-probability or of a narrow gradient add up: 100000 x 5,
// 500 chains, the log-probability off by 1.7e-4 without, 2.0e-5 with it (6.5e-5 with
// expf).  A Newton step on the reciprocal below changed nothing.
template <bool ACC>
__device__ __forceinline__ float exp_neg_abs(float s) {
    const float c = -1.4426950408889634f, as = fabsf(s);       // -log2 e, rounded; off by -1.93e-8
    const float t = c * as, e = __builtin_amdgcn_exp2f(t);
    if constexpr (!ACC) return e;
    const float d = fmaf(-1.92596303e-8f, as, fmaf(c, as, -t));
    return fmaf(0.69314718055994531f * e, t > -200.f ? d : 0.f, e);    // s infinite: d = NaN, e = 0
}
// sigmoid(z) from e = e^-|z|: 1 / (1 + e) for z >= 0, e / (1 + e) below
__device__ __forceinline__ float sigmoid_from(float z, float e) {
    const float r = __builtin_amdgcn_rcpf(1.0f + e);
    return z >= 0.f ? r : e * r;
}

__device__ __forceinline__ int ls_swz(int row) { return ((row & 3) << 1) | ((row >> 2) & 1); }

// waves per SIMD that the registers (theta's three terms and G) allow
constexpr int ls_wps(int ks) { return ks <= 8 ? 2 : 1; }

template <int XT, int KS>
struct LsShape {
    static constexpr int RB = (64 * KS + 127) / 128 * 128;   // bytes of a row in LDS
    static constexpr int PLANE = LS_RS * RB;                    // one term of a stage
    static constexpr int YB = 4 * LS_RS;                        // labels of a stage, as words
    static constexpr int BUF = XT * PLANE + YB;
    // two stages in LDS (one barrier per stage) where two workgroups still fit a
    // CU's 160 KB, else one stage and two barriers
    static constexpr int NB = 2 * BUF <= 80 * 1024 ? 2 : 1;
    static constexpr int LDS = NB * BUF;
};

// The part of one stage of X held by a thread, in units of 8 columns of a row
// (one 16-byte slot of an LDS plane): unit u = k 256 + thread is slot u % ns of
// row u / ns, ns = ceil(D / 8).  The global loads are 16 bytes wide at whatever
// alignment the row has; the last slot of a row may read into the next row, and
// those columns are masked when the unit is stored.  Only the last unit of X
// itself is read element by element.  Offsets do not change from stage to stage.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
struct __attribute__((packed, aligned(2))) raw16 { u32x4 v; };

template <int XT, int KS>
struct LsStage {
    using P = LsShape<XT, KS>;
    static constexpr int NV = (LS_RS * 4 * KS + 64 * LS_NW - 1) / (64 * LS_NW);   // units per thread (padded width)
    static constexpr int WV = XT == 1 ? 4 : 8;               // words per unit
    uint32_t raw[NV * WV];
    uint32_t goff[NV];                                       // element offset from the stage's first element
    uint32_t loff[NV];                                       // LDS byte offset, row << 20 (up to 255: past the stage for narrow X)
    int nv_last;                                             // valid columns of a row's last slot
    int nel_row;                                             // D

    __device__ __forceinline__ void init(int D) {
        const int ns = (D + 7) >> 3;
        nv_last = D - 8 * (ns - 1);
        nel_row = D;
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int u = k * 64 * LS_NW + (int)threadIdx.x;
            const int row = u / ns, slot = u - row * ns;
            goff[k] = (uint32_t)(row * D + 8 * slot);
            loff[k] = (uint32_t)(row * P::RB + 16 * (slot ^ ls_swz(row))) | (uint32_t)row << 20 |
                      (slot == ns - 1 ? 0x80000000u : 0u);
        }
    }
    __device__ __forceinline__ int row(int k) const { return (int)(loff[k] >> 20) & 0x7ff; }
    // Stage of nrow rows at element e0 of X (end elements).  inner: the whole
    // stage and the 7 elements after it lie inside X.
    __device__ __forceinline__ void fetch(const void* X, int64_t e0, int nrow, int64_t end) {
        constexpr int W = XT == 1 ? 2 : 4;                   // bytes of an element
        const char* base = (const char*)X + e0 * W;
        if (nrow == LS_RS && e0 + (int64_t)LS_RS * nel_row + 7 <= end) {
#pragma unroll
            for (int k = 0; k < NV; ++k)
                if (row(k) < LS_RS) load_unit(k, base + W * goff[k]);
        } else {
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                if (row(k) >= nrow) continue;
                const int64_t e = e0 + goff[k];
                if (e + 8 <= end) {
                    load_unit(k, base + W * goff[k]);
                } else if constexpr (XT == 1) {
                    const uint16_t* p = (const uint16_t*)X + e;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const uint32_t lo = e + 2 * j < end ? p[2 * j] : 0u;
                        const uint32_t hi = e + 2 * j + 1 < end ? p[2 * j + 1] : 0u;
                        raw[4 * k + j] = lo | hi << 16;
                    }
                } else {
                    const uint32_t* p = (const uint32_t*)X + e;
#pragma unroll
                    for (int j = 0; j < 8; ++j) raw[8 * k + j] = e + j < end ? p[j] : 0u;
                }
            }
        }
    }
    __device__ __forceinline__ void load_unit(int k, const char* p) {
        const u32x4 v = ((const raw16*)p)->v;
        raw[WV * k] = v.x; raw[WV * k + 1] = v.y; raw[WV * k + 2] = v.z; raw[WV * k + 3] = v.w;
        if constexpr (XT == 3) {
            const u32x4 u = ((const raw16*)(p + 16))->v;
            raw[WV * k + 4] = u.x; raw[WV * k + 5] = u.y; raw[WV * k + 6] = u.z; raw[WV * k + 7] = u.w;
        }
    }
    // rows nrow .. LS_RS - 1 and the columns past a row's end are written as zero
    __device__ __forceinline__ void store(uint8_t* buf, int nrow) const {
        const bool whole = nrow == LS_RS && nv_last == 8;
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int r = row(k);
            if (r >= LS_RS) continue;                        // units past the stage (D below the padded width)
            uint8_t* o = buf + (loff[k] & 0xfffffu);
            uint32_t v[WV];
#pragma unroll
            for (int j = 0; j < WV; ++j) v[j] = raw[WV * k + j];
            if (!whole) {
                const int nv = r >= nrow ? 0 : ((loff[k] & 0x80000000u) ? nv_last : 8);
                if (nv < 8) {
#pragma unroll
                    for (int j = 0; j < WV; ++j) {
                        if constexpr (XT == 1) v[j] = nv >= 2 * j + 2 ? v[j] : (nv == 2 * j + 1 ? v[j] & 0xffffu : 0u);
                        else v[j] = j < nv ? v[j] : 0u;
                    }
                }
            }
            if constexpr (XT == 1) {
                *(uint4*)o = make_uint4(v[0], v[1], v[2], v[3]);
            } else {
                uint32_t h[8], m[8], l[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) split3(__uint_as_float(v[j]), h[j], m[j], l[j]);
                *(uint4*)o = make_uint4(pack_hi(h[0], h[1]), pack_hi(h[2], h[3]), pack_hi(h[4], h[5]),
                                        pack_hi(h[6], h[7]));
                *(uint4*)(o + P::PLANE) = make_uint4(pack_hi(m[0], m[1]), pack_hi(m[2], m[3]), pack_hi(m[4], m[5]),
                                                     pack_hi(m[6], m[7]));
                *(uint4*)(o + 2 * P::PLANE) = make_uint4(pack_hi(l[0], l[1]), pack_hi(l[2], l[3]),
                                                         pack_hi(l[4], l[5]), pack_hi(l[6], l[7]));
            }
        }
    }
};

// LOGP: the log-likelihood of every chain as well (the bootstrap, the last
// step of a trajectory and the NUTS leaves).  ACC: the corrected exponential.
template <int XT, int KS, bool LOGP, bool ACC>
__global__ __launch_bounds__(64 * LS_NW, ls_wps(KS)) void k_lr32_step(
    PlainArgs a, const float* __restrict__ xsrc, const float* __restrict__ psrc, int drift, int ntile, int nsplit,
    int64_t rows_per_split) {
    using P = LsShape<XT, KS>;
    constexpr int NT = 2 * KS, RB = P::RB, PLANE = P::PLANE, BUF = P::BUF, NB = P::NB;
    extern __shared__ __align__(16) uint8_t lds[];
    const int64_t N = a.tg.N, C = a.C;
    const int D = (int)a.tg.D;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    // blocks b and b + 8 share an XCD: with a multiple of 8 splits all tiles of a split run on one XCD's L2
    int tile, split;
    if ((nsplit & 7) == 0) {
        const int b = (int)blockIdx.x >> 3;
        split = ((int)blockIdx.x & 7) + 8 * (b / ntile);
        tile = b % ntile;
    } else {
        split = (int)blockIdx.x / ntile;
        tile = (int)blockIdx.x % ntile;
    }
    const int64_t c0 = (int64_t)tile * (16 * LS_NW) + 16 * w;
    const int64_t c = c0 + l16;
    const bool wave_on = c0 < C;             // uniform over the wave
    const bool cv = c < C;

    const int64_t r_begin = (int64_t)split * rows_per_split;
    int64_t r_end = r_begin + rows_per_split;
    if (r_end > N) r_end = N;
    const int nst = r_begin < r_end ? (int)((r_end - r_begin + LS_RS - 1) / LS_RS) : 0;
    auto stage_rows = [&](int st) -> int {
        const int64_t left = r_end - r_begin - (int64_t)st * LS_RS;
        return (int)(left < LS_RS ? left : LS_RS);
    };

    LsStage<XT, KS> stg;
    stg.init(D);
    // the label of row threadIdx.x of a stage (the converting store waits for it, not the load)
    uint32_t ylab = 0u;
    auto fetch = [&](int st) {
        stg.fetch(a.tg.X, (r_begin + (int64_t)st * LS_RS) * D, stage_rows(st), N * D);
        if ((int)threadIdx.x < LS_RS) {
            const int64_t r = r_begin + (int64_t)st * LS_RS + threadIdx.x;
            ylab = a.tg.y[r < r_end ? r : r_end - 1];
        }
    };
    auto put = [&](int st) {
        uint8_t* b = lds + (NB == 2 ? (st & 1) * BUF : 0);
        stg.store(b, stage_rows(st));
        if ((int)threadIdx.x < LS_RS) ((uint32_t*)(b + XT * PLANE))[threadIdx.x] = ylab;
    };
    if (nst > 0) fetch(0);

    // the slots past a row's last one stay zero in every plane
    {
        const int ns = (D + 7) >> 3, pad = 4 * KS - ns;
        for (int i = threadIdx.x; i < NB * XT * LS_RS * pad; i += 64 * LS_NW) {
            const int pr = i / pad, slot = ns + i - pr * pad;    // pr = (buffer, plane, row)
            const int b = pr / (XT * LS_RS), pl = (pr / LS_RS) % XT, row = pr % LS_RS;
            *(uint4*)(lds + b * BUF + pl * PLANE + row * RB + 16 * (slot ^ ls_swz(row))) = make_uint4(0u, 0u, 0u, 0u);
        }
    }

    // theta (drifted) of chain c as B operands, three terms: dims 32 ks + 8 g .. + 7
    bf16x8 th[3][KS];
    {
        const double* sc = a.ws.scale;
        const double eps = cv ? a.ws.eps[c] : 0.0;
        const float* xr = xsrc + (cv ? c : 0) * D;
        const float* pr = (drift ? psrc : xsrc) + (cv ? c : 0) * D;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            float xv[8], pv[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int d = 32 * ks + 8 * g + e, dd = d < D ? d : 0;
                xv[e] = xr[dd];
                pv[e] = pr[dd];
            }
            uint32_t h[8], m[8], l[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int d = 32 * ks + 8 * g + e;
                float t = xv[e];
                if (drift) t = fmaf(sc ? (float)(eps * sc[d < D ? d : 0]) : (float)eps, pv[e], t);
                split3_pos(cv && d < D ? t : 0.f, h[e], m[e], l[e]);
            }
            auto packed = [](const uint32_t (&v)[8]) {
                return __builtin_bit_cast(bf16x8, make_uint4(pack_hi(v[0], v[1]), pack_hi(v[2], v[3]),
                                                             pack_hi(v[4], v[5]), pack_hi(v[6], v[7])));
            };
            th[0][ks] = packed(h);
            th[1][ks] = packed(m);
            th[2][ks] = packed(l);
        }
    }

    // fragment offsets: rows of the first contraction (even / odd k-step; half 1 is
    // 16 rows on), transposed blocks of the second (dim tile nt by nt % 4)
    uint32_t xo[2], to[4];
    {
        const int row = l16, f = ls_swz(row);
#pragma unroll
        for (int e = 0; e < 2; ++e) xo[e] = (uint32_t)(row * RB + 16 * ((g + 4 * e) ^ f));
        const int tr = 4 * g + (l16 >> 2), ft = ls_swz(tr);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            to[k] = (uint32_t)(tr * RB + 16 * ((2 * k + ((l16 & 3) >> 1)) ^ ft) + 8 * (l16 & 1));
    }

    // How G's products are added up.  One after the other into G (X in FP32: 8 a
    // stage), the small ones are rounded at G's size, and those of a truncated split,
    // all of their residual's sign, to one side: at 100000 x 2, FP32 X, 500 chains a
    // gradient was off by 1.0e-6 (2-norm; FP32 MFMA 2.3e-7), at 100000 x 130, 4000
    // chains by 1.9e-6 (5.7e-7).  So the residuals are split by rounding, the partials
    // summed by eights, and G rounds once a stage: now 6.7e-8 and 1.2e-7.  Up to 128
    // dims the products besides the leading one have accumulators of their own (no
    // slower, but for 33 to 64 dims of FP32 X, where they would cost a wave: 98.5 ->
    // 103.5 us a step at 20000 x 60, 2048 chains); elsewhere a stage's products meet in
    // a sum that starts at zero (20000 x 150, FP32 X, 1000 chains 115 -> 117 us; beyond
    // 256 dims fewer spills: 512 dims 458 -> 433, BF16 X 315 -> 212).  BF16 X, whose
    // three products lose less, goes without at 129 to 256 dims (256 dims 199 -> 206):
    // 3.7e-7 at 100000 x 130.
    constexpr bool GC = KS <= 4 && !(XT == 3 && KS == 2), GS = !GC && (XT == 3 || KS > 8);
    floatx4 gacc[NT], gcor[GC ? NT : 1];
#pragma unroll
    for (int n = 0; n < NT; ++n) gacc[n] = gcor[GC ? n : 0] = floatx4{0.f, 0.f, 0.f, 0.f};
    double lp = 0.0;

    if (nst > 0) {
        put(0);
        if (nst > 1) fetch(1);
    }
    for (int st = 0; st < nst; ++st) {
        __syncthreads();
        if (NB == 2 && st + 1 < nst) {
            put(st + 1);
            if (st + 2 < nst) fetch(st + 2);
        }
        const uint8_t* buf = lds + (NB == 2 ? (st & 1) * BUF : 0);
        if (wave_on) {
            // S of the 32 rows: leading products and corrections in accumulators of their own
            floatx4 sh[2], sl[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                sh[h] = floatx4{0.f, 0.f, 0.f, 0.f};
                sl[h] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
            // Operand fragments are read a step ahead where the registers allow; the
            // scheduling barriers keep the reads there (the scheduler, short of
            // registers, gathers them in front of their own MFMAs), and the wave in its
            // G part goes before the SIMD's other one.  100000 x 256, 2048 chains: 549 ->
            // 523 us a gradient with its finish; 30000 x 128, 4096 chains 202 -> 198.
            // Elsewhere the second set of fragments spills or waves leave (400 dims 201
            // -> 220) or nothing changes (20 dims 106, X in FP32 at 128 dims 221 -> 222).
            constexpr int RD = XT == 1 && KS >= 4 && KS <= 8 && !LOGP ? 2 : 1;
            auto read_x = [&](int ks, bf16x8 (&xa)[2][XT]) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int t = 0; t < XT; ++t)
                        xa[h][t] = *(const bf16x8*)(buf + xo[ks & 1] + 128 * (ks >> 1) + h * 16 * RB + t * PLANE);
            };
            auto read_t = [&](int n0, bf16x8 (&xt)[2][XT]) {
#pragma unroll
                for (int n = 0; n < 2; ++n)
#pragma unroll
                    for (int t = 0; t < XT; ++t) {
                        const uint8_t* p = buf + to[(n0 + n) & 3] + 128 * ((n0 + n) >> 2) + t * PLANE;
                        const s16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p);
                        const s16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 16 * RB));
                        xt[n][t] = __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7);
                    }
            };
            bf16x8 xf[RD][2][XT];
            if (RD == 2) read_x(0, xf[0]);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                if (RD == 1) read_x(ks, xf[0]);
                else if (ks + 1 < KS) read_x(ks + 1, xf[(ks + 1) % RD]);
                const bf16x8(&xa)[2][XT] = xf[ks % RD];
#define LS_MFMA(A, B, ACC) ACC = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, B, ACC, 0, 0, 0)
#pragma unroll
                for (int i = 0; i < (XT == 1 ? 2 : 7); ++i) {
                    // corrections, smallest first: (X term, theta term)
                    constexpr int XI[7] = {2, 1, 2, 0, 1, 1, 0}, TI[7] = {1, 2, 0, 2, 1, 0, 1};
                    const int xi = XT == 1 ? 0 : XI[i], ti = XT == 1 ? 2 - i : TI[i];
#pragma unroll
                    for (int h = 0; h < 2; ++h) LS_MFMA(xa[h][xi], th[ti][ks], sl[h]);
                    if (i == 0)
#pragma unroll
                        for (int h = 0; h < 2; ++h) LS_MFMA(xa[h][0], th[0][ks], sh[h]);
                }
                if (RD == 2) __builtin_amdgcn_sched_barrier(0);
            }
            if (RD == 2) read_t(0, xf[0]);
            const uint32_t* yl = (const uint32_t*)(buf + XT * PLANE) + 4 * g;
            // residuals y - sigmoid(s) = y ? sigmoid(-s) : -sigmoid(s), split into three BF16
            // terms by rounding; rows past the split are zero in X and add nothing to G
            float rf[8];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint4 yw = *(const uint4*)(yl + 16 * h);
                const uint32_t yv[4] = {yw.x, yw.y, yw.z, yw.w};
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float s = sh[h][v] + sl[h][v];
                    const float z = yv[v] ? -s : s;
                    const float e = exp_neg_abs<ACC>(s);
                    const float sg = sigmoid_from(z, e);
                    const float r = yv[v] ? sg : -sg;
                    rf[4 * h + v] = r;
                    if constexpr (LOGP) {
                        const int64_t row = r_begin + (int64_t)st * LS_RS + 16 * h + 4 * g + v;
                        if (row < r_end) lp -= (double)(fmaxf(z, 0.f) + log1pf(e));
                    }
                }
            }
            bf16x8 rb[3];
            uint32_t rw[3][4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float a0 = rf[2 * j], a1 = rf[2 * j + 1];
#pragma unroll
                for (int t = 0; t < 3; ++t) {
                    rw[t][j] = pack_bf16(a0, a1);
                    a0 -= __uint_as_float(rw[t][j] << 16);
                    a1 -= __uint_as_float(rw[t][j] & 0xffff0000u);
                }
            }
#pragma unroll
            for (int t = 0; t < 3; ++t)
                rb[t] = __builtin_bit_cast(bf16x8, make_uint4(rw[t][0], rw[t][1], rw[t][2], rw[t][3]));
            // G += X^T R, two dim tiles at a time
            if (RD == 2) __builtin_amdgcn_s_setprio(1);
#pragma unroll
            for (int n0 = 0; n0 < NT; n0 += 2) {
                if (RD == 1) read_t(n0, xf[0]);
                else if (n0 + 2 < NT) read_t(n0 + 2, xf[(n0 / 2 + 1) % RD]);
                const bf16x8(&xt)[2][XT] = xf[(n0 / 2) % RD];
                floatx4 gs[2];
                if (GS)
#pragma unroll
                    for (int n = 0; n < 2; ++n) gs[n] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < (XT == 1 ? 3 : 8); ++i) {
                    constexpr int XI[8] = {2, 1, 2, 0, 1, 1, 0, 0}, TI[8] = {1, 2, 0, 2, 1, 0, 1, 0};
                    const int xi = XT == 1 ? 0 : XI[i], ti = XT == 1 ? 2 - i : TI[i];
#pragma unroll
                    for (int n = 0; n < 2; ++n) {
                        if (GS) LS_MFMA(xt[n][xi], rb[ti], gs[n]);
                        else if (GC && xi + ti > 0) LS_MFMA(xt[n][xi], rb[ti], gcor[GC ? n0 + n : 0]);
                        else LS_MFMA(xt[n][xi], rb[ti], gacc[n0 + n]);
                    }
                }
                if (GS)
#pragma unroll
                    for (int n = 0; n < 2; ++n) gacc[n0 + n] += gs[n];
                if (RD == 2) __builtin_amdgcn_sched_barrier(0);
            }
#undef LS_MFMA
            if (RD == 2) __builtin_amdgcn_s_setprio(0);
        }
        if (NB == 1 && st + 1 < nst) {
            __syncthreads();
            put(st + 1);
            if (st + 2 < nst) fetch(st + 2);
        }
    }

    // the partial of this split: lane (l16, g) holds G[c][16 n + 4 g + v]
    if constexpr (LOGP) {
        lp += __shfl_xor(lp, 16, 64);
        lp += __shfl_xor(lp, 32, 64);
    }
    if (!cv) return;
    float* pg = a.ws.part_g + ((int64_t)split * C + c) * D;
    const bool v4 = (D & 3) == 0;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
        if (GC) gacc[n] += gcor[GC ? n : 0];
        const int d = 16 * n + 4 * g;
        if (v4) {
            if (d < D) *(floatx4*)(pg + d) = gacc[n];
        } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (d + v < D) pg[d + v] = gacc[n][v];
        }
    }
    if (LOGP && g == 0) a.ws.part_lp[(int64_t)split * C + c] = lp;
}

// ---------------------------------------------------------------------------
// Launcher
// ---------------------------------------------------------------------------
template <int XT, int KS, bool LOGP, bool ACC>
static hipError_t ls_launch(const PlainArgs& a, const float* x, const float* p, int drift, int nsplit, int64_t rows,
                            hipStream_t s) {
    using P = LsShape<XT, KS>;
    const int ntile = (int)((a.C + 16 * LS_NW - 1) / (16 * LS_NW));
    auto kern = k_lr32_step<XT, KS, LOGP, ACC>;
    if (P::LDS > 65536)
        (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, P::LDS);
    hipLaunchKernelGGL(kern, dim3((unsigned)((int64_t)ntile * nsplit)), dim3(64 * LS_NW), P::LDS, s, a, x, p, drift,
                       ntile, nsplit, rows);
    return hipGetLastError();
}

template <int XT>
static hipError_t ls_ks(const PlainArgs& a, const float* x, const float* p, int drift, int want_logp, int nsplit,
                        int64_t rows, hipStream_t s) {
    const int ks = (int)((a.tg.D + 31) / 32);
    // Gradients of up to 16 dims take the corrected exponential too.  Near the mode,
    // where the rows' terms cancel, what is left of the link's error beside FP32 MFMA's
    // whole error (100000 rows, FP32 X, 500 chains, without and with): 2 dims 1.18,
    // 0.32; 8 dims 0.55, 0.30; 16 dims 0.38, 0.37; 32 dims 0.40, 0.48.  It costs 50000 x
    // 8 (2048 chains) 136 -> 150 us a step and would cost 10000 x 25 28.5 -> 29.5.
    if (!want_logp && a.tg.D <= 16) return ls_launch<XT, 1, false, true>(a, x, p, drift, nsplit, rows, s);
#define LS_KS(K) \
    if (ks <= K) return want_logp ? ls_launch<XT, K, true, true>(a, x, p, drift, nsplit, rows, s) \
                              : ls_launch<XT, K, false, false>(a, x, p, drift, nsplit, rows, s);
    LS_KS(1) LS_KS(2) LS_KS(3) LS_KS(4) LS_KS(5) LS_KS(6) LS_KS(7) LS_KS(8) LS_KS(10) LS_KS(12) LS_KS(14) LS_KS(16)
#undef LS_KS
    return hipErrorInvalidValue;
}

// Row splits of a launch, at most the 64 (a quarter of the CUs at 64 chains or
// fewer) whose partials the workspace holds: two workgroups of 64 chains per CU (one
// beyond D = 256) as long as a split keeps two sub-tiles, then up to the waves that
// the registers let a SIMD hold (4 at D <= 64) while a split keeps 256 rows, below
// which the partials that k_logreg_finish adds cost more than the waves give
// (10000 x 25, 1024 chains: 28.6 us per step at 32 splits, 30.8 at 64; 6931 x 12,
// 3691 chains: 47.7 us at 16 splits, 52.7 at 8).
int lr32_nsplit(const PlainArgs& a) {
    const int64_t cap = logreg_nsplit_cap(a.tg.N, a.C);
    if (a.tune.lr_nsplit > 0) return (int)(a.tune.lr_nsplit < cap ? a.tune.lr_nsplit : cap);
    const int ks = (int)((a.tg.D + 31) / 32);
    const int occ = ks <= 2 ? 4 : ks == 3 ? 3 : ks <= 8 ? 2 : 1;
    const int64_t tiles = (a.C + 63) / 64;
    int64_t few = 256 * (occ < 2 ? 1 : 2) / tiles, want = 256 * occ / tiles;
    if (few > a.tg.N / 64) few = a.tg.N / 64;
    if (want > a.tg.N / 256) want = a.tg.N / 256;
    if (want < few) want = few;
    if (want > 8) want = want / 8 * 8;           // a split's tiles on one XCD
    if (want > cap) want = cap;
    return (int)(want < 1 ? 1 : want);
}

// rows per split: a multiple of the sub-tile
int64_t lr32_rows(int64_t N, int64_t nsplit) {
    const int64_t r = (N + nsplit - 1) / nsplit;
    return (r + LS_RS - 1) / LS_RS * LS_RS;
}

hipError_t launch_lr32_grad(const PlainArgs& a, const float* x, const float* p, int drift, int want_logp,
                            int nsplit, int64_t rows, hipStream_t s) {
    return a.tg.x_bf16 ? ls_ks<1>(a, x, p, drift, want_logp, nsplit, rows, s)
                       : ls_ks<3>(a, x, p, drift, want_logp, nsplit, rows, s);
}

}  // namespace hmc
