// First-order backward of float32 rows over blocks with linear states: the
// method of fm_linear.hip (see there) with every operand in full.
//
// Every pass is out_t = sum_r (alpha_r + X_r.Z_t) Y_r with 1 / G_r inside X and
// alpha, so that no operand stands under a shared scale (fm_pairs.h: bf16
// triples, six MFMAs a product; rows taken apart while they are staged):
//   dv:   X = u q~,  Y = dO,  Z = k^,  alpha = u
//   dk^:  X = u dO,  Y = q~,  Z = v,   alpha = -u delta
//   dq~:  X = v,     Y = k^,  Z = dO,  alpha = -delta_t,  times u_t     u = 1 / G
// The D x D state sum_r Y_r X_r^T of the rows outside a block is summed in
// float32, taken apart like a row and contracted with Z.
//
// A workgroup walks up to N / 64 steps, whose staging (loads, taking apart) is
// longer than their MFMAs: bound by that chain with few heads, by its number
// of workgroups with many.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

#include "fm_internal.h"
#include "fm_pairs.h"
#include "fm_pairs_rows.h"

namespace fm {
namespace lin32 {

using namespace pr;

enum Pass { DV = 1, DQ = 2, DK = 3 };

struct Args {
    const float *q, *k, *v, *dout;
    const Row32 *info;
    float *dq, *dk, *dv;
    int N, BH;
    float tau;
};

template <int D_, bool CAUSAL_>
struct Cfg {
    static constexpr int D = D_;
    static constexpr bool CAUSAL = CAUSAL_;
    static constexpr int NW = 8, NTH = 512, QB = 256, BK = 64;
    static constexpr int KS = D / 16, CT = D < 32 ? 1 : D / 32;
    static constexpr int LPT = D / 8, TPP = NTH / LPT, NP = (BK + TPP - 1) / TPP;
    static constexpr int RS = row_stride<D>(), VS = tr_stride<D>();
    // X planes are read by rows and transposed over 32 columns: at D = 16 the
    // transposed reads run 8 halves past the row, into the next one
    static constexpr int XH = BK * RS + 16, YH = BK * VS;
    static constexpr int NT = CT * CT;                 // 32 x 32 tiles of the state
    static constexpr int TPW = NT > NW ? NT / NW : 1;  // per wave
    static constexpr int NTW = NT < NW ? NT : NW;      // waves with tiles of their own
    static constexpr int GW = NW / NTW;                // waves sharing a tile, by K steps
    static constexpr int STEPS = BK / 16;
    static constexpr int TILE = 2 * (3 * XH + 3 * YH) + 4 * BK;
    static constexpr int SP = 32 * CT * RS;            // a plane of the state
    static constexpr int RED = 4 * NW * TPW * 32 * 33; // the waves' partial tiles
    static constexpr int SUMS = 4 * TPP * D;           // the threads' alpha Y sums
    static constexpr int max2(int a, int b) { return a > b ? a : b; }
    static constexpr int SMEM = max2(max2(TILE, RED), max2(2 * 3 * SP, SUMS));
    static_assert(SMEM <= 158 * 1024 && TILE % 16 == 0, "LDS");
};

template <typename C, int PASS>
__device__ __forceinline__ void block(unsigned char *smem, float *ssum, const Args &a, int head, int qb)
{
    constexpr int D = C::D, KS = C::KS, CT = C::CT, RS = C::RS, VS = C::VS;
    const int N = a.N;
    _Float16 *const xp = (_Float16 *)smem, *const yp = xp + 3 * C::XH;
    float *const rowA = (float *)(yp + 3 * C::YH);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    const size_t hb = (size_t)head * N * D;
    const float *const xrow = (PASS == DV ? a.q : PASS == DQ ? a.v : a.dout) + hb;
    const float *const yrow = (PASS == DV ? a.dout : PASS == DQ ? a.k : a.q) + hb;
    const float *const zrow = (PASS == DV ? a.k : PASS == DQ ? a.dout : a.v) + hb;
    const Row32 *const info = a.info + (size_t)head * N;
    const int q0 = qb * C::QB + 32 * wave, col = q0 + r32;
    const bool cok = col < N;
    constexpr bool BEFORE = PASS == DQ;   // columns see rows r <= t (else r >= t)
    const int nt = (N + C::BK - 1) / C::BK;
    // steps [p0, p1) hold the block's own rows (pairs), [s0, s1) the rest
    constexpr int PB = C::QB / C::BK;
    const int p0 = C::CAUSAL ? qb * PB : 0, p1 = C::CAUSAL ? min(nt, (qb + 1) * PB) : 0;
    const int s0 = !C::CAUSAL ? 0 : BEFORE ? 0 : p1, s1 = !C::CAUSAL ? nt : BEFORE ? p0 : nt;

    const Row32 cw = info[cok ? col : 0];
    // staging
    const int sc = tid % C::LPT, st0 = tid / C::LPT;
    RawRow<float, 8> xr[C::NP], yr[C::NP];
    Row32 ri[C::NP];
    auto load = [&](int t) {
#pragma unroll
        for (int p = 0; p < C::NP; ++p) {
            const unsigned n = (unsigned)min(t * C::BK + st0 + C::TPP * p, N - 1);
            const unsigned off = n * (unsigned)D + 8u * sc;
            xr[p].load(xrow + off, true);
            yr[p].load(yrow + off, true);
            ri[p] = info[n];
        }
    };
    float ysum[8];
    // writes the loaded step t to LDS (rows past the end weigh nothing); sum:
    // the step enters the state
    auto stage = [&](int t, bool sum) {
#pragma unroll
        for (int p = 0; p < C::NP; ++p) {
            const int row = st0 + C::TPP * p;
            if (C::BK % C::TPP != 0 && row >= C::BK) continue;
            const bool in = t * C::BK + row < N;
            const float u = in ? ri[p].u : 0.f;
            const float al = PASS == DV ? u : PASS == DQ ? (in ? 1.0f : 0.f) : -u * ri[p].delta;
            float x[8], y[8];
            h8 w[3];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                x[i] = xr[p].get(i);
                y[i] = yr[p].get(i);
                if constexpr (PASS == DV) x[i] = (x[i] - ri[p].mq) * ri[p].rq * u;
                else if constexpr (PASS == DQ) y[i] = in ? (y[i] - ri[p].mk) * ri[p].rk : 0.f;
                else {
                    x[i] *= u;
                    y[i] = (y[i] - ri[p].mq) * ri[p].rq;
                }
                if (PASS != DQ && !in) y[i] = 0.f;
            }
            split3(x, w);
#pragma unroll
            for (int i = 0; i < 3; ++i) *(h8 *)(xp + i * C::XH + row * RS + 8 * sc) = w[i];
            split3(y, w);
#pragma unroll
            for (int i = 0; i < 3; ++i) *(h8 *)(yp + i * C::YH + row * VS + 8 * sc) = w[i];
            if (PASS != DQ && sc == 0) rowA[row] = in ? al : 0.f;
            if (sum) {
#pragma unroll
                for (int i = 0; i < 8; ++i) ysum[i] = fmaf(in ? al : 0.f, y[i], ysum[i]);
            }
        }
    };

    f16v acc[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[c] = f16v{};

    // ---- the state over the rows outside the block ------------------------
    if (s0 < s1) {
        f16v sh[C::TPW];
#pragma unroll
        for (int i = 0; i < C::TPW; ++i) sh[i] = f16v{};
#pragma unroll
        for (int i = 0; i < 8; ++i) ysum[i] = 0.f;
        const int tile0 = (wave % C::NTW) * C::TPW, part = wave / C::NTW;
        load(s0);
        for (int t = s0; t < s1; ++t) {
            __syncthreads();
            stage(t, true);
            if (t + 1 < s1) load(t + 1);
            __syncthreads();
            if (C::GW > C::STEPS && part >= C::STEPS) continue;
#pragma unroll
            for (int i = 0; i < C::TPW; ++i) {
                const int yc = (tile0 + i) / CT, xc = (tile0 + i) % CT;
                f16v lo = f16v{}, hi = f16v{};   // as mma33
#pragma unroll
                for (int e0 = 0; e0 < C::STEPS; e0 += C::GW) {
                    const int e = e0 + part;
                    h8 y[3], x[3];
#pragma unroll
                    for (int j = 0; j < 3; ++j) {
                        y[j] = ld_tr<VS>(yp + j * C::YH, 16 * e, 32 * yc);
                        x[j] = ld_tr<RS>(xp + j * C::XH, 16 * e, 32 * xc);
                    }
#pragma unroll
                    for (int o = 2; o > 0; --o)
#pragma unroll
                        for (int j = 0; j <= o; ++j) lo = mma_b(y[j], x[o - j], lo);
                    hi = mma_b(y[0], x[0], hi);
                }
                sh[i] += hi + lo;
            }
        }
        // the threads' sums of alpha Y: [token lane][channel]
        float *const su = (float *)smem;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8; ++i) su[st0 * D + 8 * sc + i] = ysum[i];
        __syncthreads();
        if (tid < D) {
            const float *p = su + tid;
            float s[4] = {0.f, 0.f, 0.f, 0.f};
            for (int i = 0; i < C::TPP; i += 4)
#pragma unroll
                for (int j = 0; j < 4; ++j) s[j] += p[(size_t)(i + j) * D];
            ssum[tid] = (s[0] + s[1]) + (s[2] + s[3]);
        }
        __syncthreads();
        // partial tiles -> sums -> planes [y][x]
        float *const red = (float *)smem;
#pragma unroll
        for (int i = 0; i < C::TPW; ++i)
#pragma unroll
            for (int j = 0; j < 16; ++j)
                red[((wave * C::TPW + i) * 32 + 8 * (j / 4) + 4 * h + j % 4) * 33 + r32] = sh[i][j];
        __syncthreads();
        constexpr int SE = 32 * CT * 32 * CT, EPT = SE / C::NTH;
        static_assert(SE % C::NTH == 0, "state elements per thread");
        float sv[EPT];
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            const int e = tid + C::NTH * i, y = e / (32 * CT), x = e % (32 * CT);
            const int tl = (y / 32) * CT + x / 32;
            float s = 0.f;
            for (int w = 0; w < C::GW; ++w)
                s += red[(((tl / C::TPW + w * C::NTW) * C::TPW + tl % C::TPW) * 32 + y % 32) * 33 + x % 32];
            sv[i] = y < D && x < D ? s : 0.f;
        }
        __syncthreads();
        uint16_t *const st = (uint16_t *)smem;
#pragma unroll
        for (int i = 0; i < EPT; ++i) {
            const int e = tid + C::NTH * i, y = e / (32 * CT), x = e % (32 * CT);
            if (x < D) {
                float s = sv[i];
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    const bf16_t b = f32_to_bf16(s);
                    st[j * C::SP + y * RS + x] = b;
                    s -= bf16_to_f32(b);
                }
            }
        }
        __syncthreads();
    }

    // own columns Z as B operands (after the state: their registers are its own)
    h8 z[KS][3];
    {
        float x[D / 2];
        load_cols<float, D>(zrow, col, N, x);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if constexpr (PASS == DV) {
#pragma unroll
                for (int i = 0; i < 8; ++i) x[8 * ks + i] = cok ? (x[8 * ks + i] - cw.mk) * cw.rk : 0.f;
            }
            split3(x + 8 * ks, z[ks]);
        }
    }

    if (s0 < s1) {
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const f16v f = dot33<KS>((const _Float16 *)smem + (32 * c + r32) * RS + 8 * h, C::SP, z);
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int d = 32 * c + 8 * (j / 4) + 4 * h + j % 4;
                const float ys = D % 32 == 0 || d < D ? ssum[d < D ? d : 0] : 0.f;
                acc[c][j] = PASS == DQ ? fmaf(-cw.delta, ys, f[j]) : f[j] + ys;
            }
        }
    }

    // ---- the block's own rows, pair by pair -------------------------------
    // (at D = 128 Z and the output leave no registers for rows on their way)
    constexpr bool AHEAD = D < 128;
    if (AHEAD && p0 < p1) load(p0);
    for (int t = p0; t < p1; ++t) {
        if constexpr (!AHEAD) load(t);
        __syncthreads();
        stage(t, false);
        if (AHEAD && t + 1 < p1) load(t + 1);
        __syncthreads();
#pragma unroll 1
        for (int j = 0; j < C::BK / 32; ++j) {
            const int kb = t * C::BK + 32 * j;
            if (kb >= N || (BEFORE ? kb > q0 : kb < q0)) continue;
            const f16v s = dot33<KS>(xp + (32 * j + r32) * RS + 8 * h, C::XH, z);
            float w[16];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                float4 A = make_float4(-cw.delta, -cw.delta, -cw.delta, -cw.delta);
                if constexpr (PASS != DQ) A = *(const float4 *)(rowA + 32 * j + 8 * b + 4 * h);
#pragma unroll
                for (int i = 0; i < 4; ++i) w[4 * b + i] = s[4 * b + i] + ((const float *)&A)[i];
            }
            if (kb == q0 || kb + 32 > N) {
                asm volatile("");
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int row = kb + 8 * (i / 4) + 4 * h + i % 4;
                    if (row >= N || (BEFORE ? row > col : row < col)) w[i] = 0.f;
                }
            }
            h8 w3[2][3];
#pragma unroll
            for (int e = 0; e < 2; ++e) split3(w + 8 * e, w3[e]);
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                h8 y[3][2];
#pragma unroll
                for (int i = 0; i < 3; ++i)
#pragma unroll
                    for (int e = 0; e < 2; ++e) y[i][e] = ld_tr<VS>(yp + i * C::YH, 32 * j + 16 * e, 32 * c);
                acc[c] += mma33(y, w3);
            }
        }
    }

    if constexpr (PASS == DQ) {
        const float f = a.tau * cw.u;
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[c][i] *= f;
    }
    const size_t at = hb + (size_t)(cok ? col : 0) * D;
    if constexpr (PASS != DV) standardise_back<float, D>((PASS == DQ ? a.q : a.k) + at, acc);
    if (cok) store_col<float, D>((PASS == DQ ? a.dq : PASS == DK ? a.dk : a.dv) + at, acc);
}

template <typename C>
__global__ __launch_bounds__(C::NTH, 2) void bwd_kernel(Args a, int nqb)
{
    __shared__ alignas(16) unsigned char smem[C::SMEM];
    __shared__ float ssum[C::D];
    const int head = blockIdx.x % a.BH, rest = blockIdx.x / a.BH, pass = rest % 3, i = rest / 3;
    // the blocks with the most rows first
    if (pass == 0) block<C, DQ>(smem, ssum, a, head, nqb - 1 - i);
    else if (pass == 1) block<C, DK>(smem, ssum, a, head, i);
    else block<C, DV>(smem, ssum, a, head, i);
}

template <int D, bool CAUSAL>
hipError_t run_bwd(const float *q, const float *k, const float *v, const float *o, const float *dout,
                   const float *g, float *dq, float *dk, float *dv, int BH, int N, float qs, void *ws,
                   hipStream_t st)
{
    typedef Cfg<D, CAUSAL> C;
    const long long rows = (long long)BH * N, pb = (rows * (D / 8) + 255) / 256;
    const int nqb = (N + C::QB - 1) / C::QB;
    if (!grid_fits(pb, 256) || !grid_fits(3LL * BH * nqb, C::NTH)) return hipErrorInvalidConfiguration;
    Row32 *info = (Row32 *)ws;
    hipLaunchKernelGGL((bwd32_prep_kernel<D>), dim3((unsigned)pb), dim3(256), 0, st, q, k, o, dout, g, info,
                       rows, qs);
    const Args a{q, k, v, dout, info, dq, dk, dv, N, BH, qs};
    hipLaunchKernelGGL((bwd_kernel<C>), dim3((unsigned)(3LL * BH * nqb)), dim3(C::NTH), 0, st, a, nqb);
    return hipGetLastError();
}

}  // namespace lin32

hipError_t linear_bwd32(const void *q, const void *k, const void *v, const void *o, const void *dout,
                        const float *g, void *dq, void *dk, void *dv, int BH, int N, int D, int causal,
                        float qs, void *ws, hipStream_t st)
{
#define GO2(DD, CA)                                                                                \
    lin32::run_bwd<DD, CA>((const float *)q, (const float *)k, (const float *)v, (const float *)o, \
                           (const float *)dout, g, (float *)dq, (float *)dk, (float *)dv, BH, N, qs, ws, st)
#define GO(DD) return causal ? GO2(DD, true) : GO2(DD, false)
    switch (D) {
    case 16: GO(16);
    case 32: GO(32);
    case 64: GO(64);
    case 128: GO(128);
    }
#undef GO
#undef GO2
    return hipErrorInvalidValue;
}

}  // namespace fm
