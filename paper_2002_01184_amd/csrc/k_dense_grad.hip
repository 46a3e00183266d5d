// k_dense_grad.hip -- gradient of the dense Gaussian, g = -P x, at a state that
// is already drifted, with the kick and the next drift: the plain form's
// leapfrog step beyond D = 128, the bootstrap gradient and the NUTS leaves at
// every D.
//
// A launch takes (x, p) to g = -P x, p += kick g and, when asked, x_next = x +
// eps p.  Rows of P are spread over the grid, so every workgroup reads its
// chains' whole x while others write their rows of x_next: the next position
// goes to another buffer than x, and no workgroup waits for another.
//
// A workgroup (4 waves) owns 16 NC chains and 64 rows of P, wave w the 16 rows
// of M-tile 4 blockIdx.y + w, on v_mfma_f32_16x16x4f32 (A[i][k] at lane i + 16 k,
// B[k][j] at lane j + 16 k, D[i][j] in VGPR i % 4 of lane j + 16 (i / 4)).  The
// contraction index is k = g4 KM + ks (KM = 4 ceil(D / 16); lane group g4 takes
// its own quarter of the dims) with even and odd k-steps in two accumulators:
// the operand layout and MFMA sequence of the fused dense kernel and of
// k_dense_step, so all forms give bitwise the same gradient.  P and x go
// through LDS 16 k-steps at a time (four 16-column pieces of every row, loaded
// 16 bytes a lane into registers two chunks ahead; a CU's LDS holds three
// workgroups of one chain tile or two of two), each lane reading the operands of
// 4 k-steps with one ds_read_b128 (row stride 84 floats: 8 consecutive rows hit
// distinct bank quads).
//
// The kernel it replaces gave each workgroup 16 chains and all of P, read from
// global memory 4 bytes a lane at a stride of a row: 48.9 us per step at D = 300,
// 1000 chains (63 workgroups); this one 12.5 us (floor 1.2 us of MFMA, a
// launch 3 to 4 us).
#include "hmc_internal.hpp"

namespace hmc {

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int DG_KC = 16;                   // k-steps per chunk
constexpr int DG_PS = DG_KC + 4;            // floats of a 16-column piece in LDS
constexpr int DG_RS = 4 * DG_PS + 4;        // floats of a row (its four pieces)

struct __attribute__((packed, aligned(4))) f32x4u { floatx4 v; };   // 16 bytes at any float

// DIRECT (D <= 32): a wave reads its own operands from global memory, at most two
// 16-byte pieces a row, without LDS and barriers; the workgroup has a wave per 16
// rows.  D = 8, 14318 chains 5.7 -> 4.5 us (an empty launch takes
// about as long).
template <int NC, bool DIRECT>
__global__ __launch_bounds__(256) void k_dense_grad(PlainArgs a, const float* __restrict__ x, float* __restrict__ xnext,
                                                    float* __restrict__ p, float* __restrict__ gd, double kick_scale) {
    constexpr int CT = 16 * NC;                       // chains per workgroup
    constexpr int NR = 64 + CT;                       // rows staged: 64 of P, CT of x
    constexpr int NV = NR * 4 * (DG_KC / 4) / 256;    // 16-byte loads per thread and chunk
    __shared__ __attribute__((aligned(16))) float lds[2][DIRECT ? 1 : NR * DG_RS];
    const int D = (int)a.tg.D;
    const int ntiles = (D + 15) / 16, KM = 4 * ntiles, nch = (KM + DG_KC - 1) / DG_KC;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i16 = lane & 15, g4 = lane >> 4;
    const int64_t c0 = (int64_t)blockIdx.x * CT;
    const int mt = 4 * (int)blockIdx.y + w;
    const float* P = (const float*)a.tg.prec;
    // columns col .. col + 3 of a row of D floats, zeros past its end
    auto load4 = [&](const float* row, int col) {
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
        if (col + 4 <= D) v = ((const f32x4u*)(row + col))->v;
        else
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (col + j < D) v[j] = row[col + j];
        return v;
    };

    // unit u of a chunk: row u / 16 (P rows, then chains), piece and 4-column group of the rest
    floatx4 raw0[NV], raw1[NV];
    auto fetch = [&](int ch, floatx4 (&raw)[NV]) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int u = k * 256 + (int)threadIdx.x, r = u >> 4, pc = (u >> 2) & 3, q = u & 3;
            const int ks = DG_KC * ch + 4 * q, col = pc * KM + ks;
            const bool isp = r < 64;
            const int64_t row = isp ? (int64_t)blockIdx.y * 64 + r : c0 + (r - 64);
            const float* src = (isp ? P : x) + row * D + col;
            floatx4 v = {0.f, 0.f, 0.f, 0.f};
            if (ks < KM && row < (isp ? (int64_t)D : a.C)) {
                if (col + 4 <= D) v = ((const f32x4u*)src)->v;
                else
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (col + j < D) v[j] = src[j];
            }
            raw[k] = v;
        }
    };
    auto put = [&](int ch, const floatx4 (&raw)[NV]) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const int u = k * 256 + (int)threadIdx.x, r = u >> 4, pc = (u >> 2) & 3, q = u & 3;
            *(floatx4*)(&lds[ch & 1][r * DG_RS + pc * DG_PS + 4 * q]) = raw[k];
        }
    };
    floatx4 da[DIRECT ? 2 : 1], db[DIRECT ? 2 : 1][NC];
    if constexpr (DIRECT) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const floatx4 zero = {0.f, 0.f, 0.f, 0.f};
            const int r = 16 * mt + i16, col = g4 * KM + 4 * q;
            const bool on = 4 * q < KM;
            da[q] = on && r < D ? load4(P + (int64_t)r * D, col) : zero;
#pragma unroll
            for (int n = 0; n < NC; ++n) {
                const int64_t c = c0 + 16 * n + i16;
                db[q][n] = on && c < a.C ? load4(x + c * D, col) : zero;
            }
        }
    } else {
        fetch(0, raw0);
        if (nch > 1) fetch(1, raw1);
    }

    // this lane's 4 dims of its chains
    const int d0 = 16 * mt + 4 * g4;
    float pv[NC][4], xv[NC][4];
    double ec[NC], bt[NC];
#pragma unroll
    for (int n = 0; n < NC; ++n) {
        const int64_t c = c0 + 16 * n + i16;
        const bool ok = c < a.C;
        ec[n] = ok ? a.ws.eps[c] : 0.0;
        bt[n] = ok && a.ws.beta ? a.ws.beta[c] : 1.0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const bool in = ok && d0 + v < D;
            pv[n][v] = p && in ? p[c * D + d0 + v] : 0.f;
            xv[n][v] = xnext && in ? x[c * D + d0 + v] : 0.f;
        }
    }

    floatx4 acc[NC][2];
#pragma unroll
    for (int n = 0; n < NC; ++n) acc[n][0] = acc[n][1] = floatx4{0.f, 0.f, 0.f, 0.f};
    if constexpr (DIRECT) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (4 * q < KM)
#pragma unroll
                for (int n = 0; n < NC; ++n)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc[n][j & 1] =
                            __builtin_amdgcn_mfma_f32_16x16x4f32(da[q][j], db[q][n][j], acc[n][j & 1], 0, 0, 0);
    } else {
        put(0, raw0);
        if (nch > 2) fetch(2, raw0);
        // one chunk; nx holds chunk ch + 1 and takes chunk ch + 3
        auto chunk = [&](int ch, floatx4 (&nx)[NV]) {
            __syncthreads();
            if (ch + 1 < nch) {
                put(ch + 1, nx);
                if (ch + 3 < nch) fetch(ch + 3, nx);
            }
            if (mt < ntiles) {
                const float* pa = &lds[ch & 1][(16 * w + i16) * DG_RS + g4 * DG_PS];
                const float* xb = &lds[ch & 1][(64 + i16) * DG_RS + g4 * DG_PS];
                auto four = [&](int q) {
                    const floatx4 av = *(const floatx4*)(pa + 4 * q);
#pragma unroll
                    for (int n = 0; n < NC; ++n) {
                        const floatx4 bv = *(const floatx4*)(xb + 16 * n * DG_RS + 4 * q);
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            acc[n][j & 1] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[j], bv[j], acc[n][j & 1], 0, 0, 0);
                    }
                };
                const int left = KM - DG_KC * ch;
                if (left >= DG_KC) {
#pragma unroll
                    for (int q = 0; q < DG_KC / 4; ++q) four(q);
                } else {
                    for (int q = 0; q < left / 4; ++q) four(q);
                }
            }
        };
        for (int ch = 0; ch < nch; ch += 2) {
            chunk(ch, raw1);
            if (ch + 1 < nch) chunk(ch + 1, raw0);
        }
    }
    if (mt >= ntiles) return;
    const double* sc = a.ws.scale;
#pragma unroll
    for (int n = 0; n < NC; ++n) {
        const int64_t c = c0 + 16 * n + i16;
        if (c >= a.C) continue;
        const float keps = (float)(kick_scale * ec[n] * bt[n]);
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int d = d0 + v;
            if (d >= D) continue;
            const int64_t i = c * D + d;
            const float gv = -(acc[n][0][v] + acc[n][1][v]);
            if (p) {
                const float kd = sc ? (float)(kick_scale * ec[n] * bt[n] * sc[d]) : keps;
                const float pn = fmaf(kd, gv, pv[n][v]);
                p[i] = pn;
                if (xnext) xnext[i] = fmaf(sc ? (float)(ec[n] * sc[d]) : (float)ec[n], pn, xv[n][v]);
            }
            if (gd) gd[i] = gv;
        }
    }
}

hipError_t launch_dense_grad(const PlainArgs& a, const float* x, float* xnext, float* p, float* gd, double kick_scale,
                             hipStream_t s) {
    const unsigned rows = (unsigned)((a.tg.D + 63) / 64);
    // Two chain tiles per workgroup (every A operand feeds two MFMAs, P is read
    // half as often) once one tile each would take more than one round: three of
    // those workgroups fit a CU's LDS.  One against two tiles, whole steps of ten
    // leapfrogs: D = 300, 3000 chains (940 workgroups) 279, 254 us; D = 512, 1900
    // chains (952) 336, 298; below the line D = 300, 2000 chains (625) 215, 231; D =
    // 150, 4000 chains (750) 182, 194.
    const int64_t tiles = (a.C + 15) / 16;
    if (a.tg.D <= 32)
        hipLaunchKernelGGL((k_dense_grad<1, true>), dim3((unsigned)tiles), dim3(a.tg.D <= 16 ? 64 : 128), 0, s, a, x,
                           xnext, p, gd, kick_scale);
    else if (tiles * rows > 768)
        hipLaunchKernelGGL((k_dense_grad<2, false>), dim3((unsigned)((tiles + 1) / 2), rows), dim3(256), 0, s, a, x, xnext, p,
                           gd, kick_scale);
    else
        hipLaunchKernelGGL((k_dense_grad<1, false>), dim3((unsigned)tiles, rows), dim3(256), 0, s, a, x, xnext, p, gd,
                           kick_scale);
    return hipGetLastError();
}

}  // namespace hmc
