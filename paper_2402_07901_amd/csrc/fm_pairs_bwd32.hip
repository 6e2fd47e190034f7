// Pair backward without shared scales (p = 2; all calls but bf16 rows at D = 64,
// see pairs_grade32): the gradient of fm_pairs_bwd.hip (see there for the
// formulas and the three roles) with every operand in full.
//
// Nothing is known about the range of v, dO and 1 / G, and a causal row or a
// column may never meet the largest value of its tile, so no operand stands
// under a shared scale: q~, k^, v, dO and the weights are bf16 triples
// (fm_pairs.h), six MFMAs a product (bf16 rows of v and dO as they are, one or
// three MFMAs), and 1 / G enters the weights in float32.
// bwd32_prep leaves six floats per row; a step stages the raw rows and takes
// them apart on the way into LDS (the same bytes from memory as two fp16
// planes, and no planes to write).  Bound by vector issue beside the MFMAs once
// the chip is full (float32 rows: 11 other instructions an MFMA, taking floats apart for the
// most part; MFMAs busy 32%), by a workgroup's walk down its rows before that;
// the table at the end holds the paces.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

#include "fm_internal.h"
#include "fm_pairs.h"
#include "fm_pairs_rows.h"

namespace fm {
namespace pr {
namespace f32 {

enum Role { ROLE_Q = 0, ROLE_K = 1, ROLE_V = 2 };

template <typename T_, int D_, bool CAUSAL_, int NWQ_, int NWK_, int BK_>
struct Cfg {
    typedef T_ T;
    static constexpr bool F32 = sizeof(T) == 4;
    static constexpr int RP = F32 ? 3 : 1;   // parts of a row of v or dO
    static constexpr int D = D_, NWQ = NWQ_, NWK = NWK_, BK = BK_;
    static constexpr bool CAUSAL = CAUSAL_;
    static constexpr int NTH = 64 * NWQ * NWK, QB = 32 * NWQ;
    static constexpr int KS = D / 16, CT = D < 32 ? 1 : D / 32;
    static constexpr int LPT = D / 8, TPP = NTH / LPT, NP = (BK + TPP - 1) / TPP;
    static constexpr int RS = row_stride<D>(), VS = tr_stride<D>();
    static constexpr int XH = BK * RS, AH = BK * VS, PH = XH > AH ? XH : AH;
    // x (scores; also contracted by roles Q and K) and the staged values, three
    // planes each, and two floats per row
    static constexpr int TILE = 2 * (3 * XH + RP * PH) + 8 * BK;
    // waves per SIMD: at D = 128, float32 rows, a wave's own columns take 192
    // registers, so its workgroup of four is alone on the CU
    static constexpr int WPS = D >= 128 && F32 ? 1 : 2;
    // two steps' tiles in turn where LDS has room beside the other workgroups
    // of the CU: one barrier a step instead of two
    static constexpr int ROOM = 160 * 1024 * NWQ * NWK / (4 * WPS) - 256;
    // bf16 rows at D = 128: the own columns' last part waits in LDS
    static constexpr bool OLDS = D >= 128 && !F32;
    static constexpr int OB = OLDS ? 2 * QB * RS : 0;
    static constexpr bool DB = 2 * TILE + OB <= ROOM;
    static constexpr int RED_BYTES = NWK > 1 ? 4 * NWQ * NWK * 32 * 32 * CT : 0;
    static constexpr int LOOP_BYTES = (DB ? 2 : 1) * TILE + OB;
    static constexpr int SMEM = LOOP_BYTES > RED_BYTES ? LOOP_BYTES : RED_BYTES;
    static_assert(BK % (32 * NWK) == 0 && NWQ * NWK <= 4 * WPS, "shape");
    static_assert(SMEM <= 160 * 1024 - 256 && TILE % 16 == 0, "LDS");
};

struct Args {
    const void *q, *k, *v, *dout;
    const Row32 *info;
    void *dq, *dk, *dv;
    int N, BH;
    float tau;
};

template <typename C, int ROLE>
__device__ __forceinline__ void block(unsigned char *smem, const Args &a, int head, int qb)
{
    typedef typename C::T T;
    constexpr int D = C::D, KS = C::KS, CT = C::CT, RS = C::RS, VS = C::VS, RP = C::RP;
    const int N = a.N;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    const int wq = wave / C::NWK, wk = wave % C::NWK;
    const size_t hb = (size_t)head * N * D;
    // own columns and staged rows
    const T *const own = (const T *)(ROLE == ROLE_Q ? a.q : a.k) + hb, *const stg = (const T *)(ROLE == ROLE_Q ? a.k : a.q) + hb;
    const T *const ownv = (const T *)(ROLE == ROLE_Q ? a.dout : a.v) + hb, *const stgv = (const T *)(ROLE == ROLE_Q ? a.v : a.dout) + hb;
    const Row32 *const info = a.info + (size_t)head * N;
    const int q0 = qb * C::QB + 32 * wq, col = q0 + r32;
    const bool cok = col < N;
    const int rbeg = C::CAUSAL && ROLE != ROLE_Q ? qb * C::QB : 0;
    const int rend = C::CAUSAL && ROLE == ROLE_Q ? min(N, (qb + 1) * C::QB) : N;
    const int t0 = rbeg / C::BK, t1 = (rend + C::BK - 1) / C::BK;

    // staging: this thread's 8 channels and first row
    const int sc = tid % C::LPT, st0 = tid / C::LPT;
    RawRow<T, 8> xr[C::NP], vr[C::NP];
    float mx[C::NP], rx[C::NP], ru[C::NP], rd[C::NP];
    auto load_tile = [&](int t) {
#pragma unroll
        for (int p = 0; p < C::NP; ++p) {
            // rows past the end repeat the last one: masked (role Q) or given weight 0
            const unsigned n = (unsigned)min(t * C::BK + st0 + C::TPP * p, N - 1);
            const unsigned off = n * (unsigned)D + 8u * sc;
            xr[p].load(stg + off, true);
            vr[p].load(stgv + off, true);
            const Row32 w = info[n];
            mx[p] = ROLE == ROLE_Q ? w.mk : w.mq;
            rx[p] = ROLE == ROLE_Q ? w.rk : w.rq;
            ru[p] = w.u;
            rd[p] = w.delta;
        }
    };
    load_tile(t0);

    // own columns as B operands: x and (roles Q, K) dO or v
    constexpr int OP = C::OLDS ? 2 : 3;
    _Float16 *const olw = (_Float16 *)(smem + (C::DB ? 2 : 1) * C::TILE) + (32 * wq + r32) * RS + 8 * h;
    h8 ox[KS][OP], ov[ROLE != ROLE_V ? KS : 1][RP];
    const Row32 cw = info[cok ? col : 0];
    {
        float x[D / 2];
        load_cols<T, D>(own, col, N, x);
        const float m = ROLE == ROLE_Q ? cw.mq : cw.mk, r = ROLE == ROLE_Q ? cw.rq : cw.rk;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
            for (int i = 0; i < 8; ++i) x[8 * ks + i] = cok ? (x[8 * ks + i] - m) * r : 0.f;
            h8 w[3];
            split3(x + 8 * ks, w);
#pragma unroll
            for (int i = 0; i < OP; ++i) ox[ks][i] = w[i];
            if (C::OLDS && wk == 0) *(h8 *)(olw + 16 * ks) = w[2];
        }
        if constexpr (ROLE != ROLE_V) {
            load_cols<T, D>(ownv, col, N, x);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                h8 w[3];
                split3(x + 8 * ks, w);
#pragma unroll
                for (int i = 0; i < RP; ++i) ov[ks][i] = w[i];   // (a bf16 row is its own first part)
            }
        }
    }

    f16v acc[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[c] = f16v{};

    // One 32-row tile j of the staged step against the wave's columns; masked:
    // some of its pairs lie beyond the diagonal or the last row.
    auto tile = [&](const _Float16 *xp, int j, int kb, bool masked) {
        const _Float16 *const vp = xp + 3 * C::XH;
        const float *const rowU = (const float *)(vp + RP * C::PH), *const rowD = rowU + C::BK;
        f16v s = f16v{};
        if constexpr (C::OLDS) {
            const _Float16 *const q = xp + (32 * j + r32) * RS + 8 * h;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const h8 a0 = ld8(q + 16 * ks), a1 = ld8(q + C::XH + 16 * ks), a2 = ld8(q + 2 * C::XH + 16 * ks);
                s = mma_b(a2, ox[ks][0], s);
                s = mma_b(a1, ox[ks][1], s);
                s = mma_b(a0, ld8(olw + 16 * ks), s);
                s = mma_b(a1, ox[ks][0], s);
                s = mma_b(a0, ox[ks][1], s);
                s = mma_b(a0, ox[ks][0], s);
            }
        } else {
            s = dot33<KS, C::F32>(xp + (32 * j + r32) * RS + 8 * h, C::XH, ox);
        }
        f16v d = f16v{};
        if constexpr (ROLE != ROLE_V && RP == 3) d = dot33<KS>(vp + (32 * j + r32) * RS + 8 * h, C::PH, ov);
        else if constexpr (ROLE != ROLE_V) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                d = mma_b(ld8(vp + (32 * j + r32) * RS + 8 * h + 16 * ks), ov[ks][0], d);
        }
        float w[16];
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            float4 U, E;
            if constexpr (ROLE != ROLE_Q) U = *(const float4 *)(rowU + 32 * j + 8 * b + 4 * h);
            if constexpr (ROLE == ROLE_K) E = *(const float4 *)(rowD + 32 * j + 8 * b + 4 * h);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int e = 4 * b + i;
                if constexpr (ROLE == ROLE_Q) w[e] = (1.0f + s[e]) * (d[e] - cw.delta);
                else if constexpr (ROLE == ROLE_K)
                    w[e] = (1.0f + s[e]) * fmaf(d[e], ((const float *)&U)[i], -((const float *)&E)[i]);
                else w[e] = fmaf(s[e], s[e] + 2.0f, 2.0f) * ((const float *)&U)[i];   // U: u / 2
            }
        }
        if (masked) {
            asm volatile("");   // a branch, not a compare and select per element of every tile
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int row = kb + 8 * (i / 4) + 4 * h + i % 4;
                if (ROLE == ROLE_Q ? row >= N || (C::CAUSAL && row > col) : row < col) w[i] = 0.f;
            }
        }
        h8 w3[2][3];
#pragma unroll
        for (int e = 0; e < 2; ++e) split3(w + 8 * e, w3[e]);
        constexpr int AS = ROLE == ROLE_V ? VS : RS, PL = ROLE == ROLE_V ? C::PH : C::XH;
        const _Float16 *const ap = ROLE == ROLE_V ? vp : xp;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            constexpr int AP = ROLE == ROLE_V ? RP : 3;
            h8 x[AP][2];
#pragma unroll
            for (int i = 0; i < AP; ++i)
#pragma unroll
                for (int e = 0; e < 2; ++e) x[i][e] = ld_tr<AS>(ap + i * PL, 32 * j + 16 * e, 32 * c);
            if constexpr (C::F32) {
                acc[c] += mma33(x, w3);
            } else {   // one chain, smallest first: bf16 shows no more
#pragma unroll
                for (int o = 2; o >= 0; --o)
#pragma unroll
                    for (int i = 0; i < AP && i <= o; ++i)
#pragma unroll
                        for (int e = 0; e < 2; ++e) acc[c] = mma_b(x[i][e], w3[e][o - i], acc[c]);
            }
        }
    };

    // writes the loaded step t to a buffer
    auto stage = [&](_Float16 *xp, int t) {
        _Float16 *const vp = xp + 3 * C::XH;
        float *const rowU = (float *)(vp + RP * C::PH), *const rowD = rowU + C::BK;
        constexpr int VST = ROLE == ROLE_V ? VS : RS;
#pragma unroll
        for (int p = 0; p < C::NP; ++p) {
            const int row = st0 + C::TPP * p;
            if (C::BK % C::TPP != 0 && row >= C::BK) continue;
            float x[8];
            h8 y[3];
#pragma unroll
            for (int i = 0; i < 8; ++i) x[i] = (xr[p].get(i) - mx[p]) * rx[p];
            split3(x, y);
#pragma unroll
            for (int i = 0; i < 3; ++i) *(h8 *)(xp + i * C::XH + row * RS + 8 * sc) = y[i];
            if constexpr (RP == 1) {
                *(uint4 *)(vp + row * VST + 8 * sc) = *(uint4 *)vr[p].w;
            } else {
#pragma unroll
                for (int i = 0; i < 8; ++i) x[i] = vr[p].get(i);
                split3(x, y);
#pragma unroll
                for (int i = 0; i < 3; ++i) *(h8 *)(vp + i * C::PH + row * VST + 8 * sc) = y[i];
            }
            if (ROLE != ROLE_Q && sc == 0) {
                const bool in = t * C::BK + row < N;
                rowU[row] = in ? (ROLE == ROLE_V ? 0.5f * ru[p] : ru[p]) : 0.f;
                if constexpr (ROLE == ROLE_K) rowD[row] = in ? ru[p] * rd[p] : 0.f;
            }
        }
    };
    auto compute = [&](const _Float16 *buf, int t) {
#pragma unroll 1
        for (int j = wk; j < C::BK / 32; j += C::NWK) {
            const int kb = t * C::BK + 32 * j;
            if (kb >= N || (C::CAUSAL && ROLE == ROLE_Q && kb > q0 + 31)) break;
            if (C::CAUSAL && ROLE != ROLE_Q && kb + 31 < q0) continue;
            tile(buf, j, kb, ROLE == ROLE_Q ? (C::CAUSAL && kb + 31 > q0) || kb + 32 > N
                                            : C::CAUSAL && kb < q0 + 31);
        }
    };

    if constexpr (C::DB) {
        constexpr int BUF = C::TILE / 2;
        if (t0 < t1) stage((_Float16 *)smem, t0);
        if (t0 + 1 < t1) load_tile(t0 + 1);
        __syncthreads();
        for (int t = t0; t < t1; ++t) {
            compute((const _Float16 *)smem + ((t - t0) & 1) * BUF, t);
            if (t + 1 < t1) {
                stage((_Float16 *)smem + ((t + 1 - t0) & 1) * BUF, t + 1);
                if (t + 2 < t1) load_tile(t + 2);
            }
            __syncthreads();
        }
    } else {
        for (int t = t0; t < t1; ++t) {
            __syncthreads();
            stage((_Float16 *)smem, t);
            if (t + 1 < t1) load_tile(t + 1);
            __syncthreads();
            compute((const _Float16 *)smem, t);
        }
    }
    // partial sums of the waves that shared the columns
    if constexpr (C::NWK > 1) {
        float *red = (float *)smem;
        constexpr int W = 32 * 32 * CT;
        __syncthreads();
        if (wk > 0) {
            float *mine = red + wave * W;
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    mine[32 * (32 * c + 8 * (i / 4) + 4 * h + i % 4) + r32] = acc[c][i];
        }
        __syncthreads();
        if (wk > 0) return;
#pragma unroll
        for (int w = 1; w < C::NWK; ++w) {
            const float *part = red + (wave + w) * W;
#pragma unroll
            for (int c = 0; c < CT; ++c)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    acc[c][i] += part[32 * (32 * c + 8 * (i / 4) + 4 * h + i % 4) + r32];
        }
    }

    if constexpr (ROLE == ROLE_Q) {
        const float f = a.tau * cw.u;
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[c][i] *= f;
    }
    const size_t at = hb + (size_t)(cok ? col : 0) * D;
    if constexpr (ROLE != ROLE_V) standardise_back<T, D>((const T *)(ROLE == ROLE_Q ? a.q : a.k) + at, acc);
    if (cok) store_col<T, D>((T *)(ROLE == ROLE_Q ? a.dq : ROLE == ROLE_K ? a.dk : a.dv) + at, acc);
}

// Block order: heads in groups of hgrp; within a group the columns with the
// most rows first (role Q: the last queries; K, V: the first keys), the three
// roles of a column block side by side.
template <typename C>
__global__ __launch_bounds__(C::NTH, C::WPS) void bwd32_kernel(Args a, int nqb, int hgrp)
{
    __shared__ alignas(16) unsigned char smem[C::SMEM];
    const int b = blockIdx.x, per = 3 * hgrp * nqb, grp = b / per, r = b - grp * per;
    const int gs = min(hgrp, a.BH - grp * hgrp);
    const int head = grp * hgrp + r % gs, rest = r / gs, role = rest % 3, i = rest / 3;
    if (role == 0) block<C, ROLE_Q>(smem, a, head, nqb - 1 - i);
    else if (role == 1) block<C, ROLE_K>(smem, a, head, i);
    else block<C, ROLE_V>(smem, a, head, i);
}

template <typename C>
hipError_t launch(const void *q, const void *k, const void *v, const void *o, const void *dout,
                  const float *g, void *dq, void *dk, void *dv, int BH, int N, float qs, void *ws,
                  hipStream_t st)
{
    const long long rows = (long long)BH * N, pb = (rows * (C::D / 8) + 255) / 256;
    const int nqb = (N + C::QB - 1) / C::QB, hgrp = BH < 32 ? BH : 32;
    if (!grid_fits(pb, 256) || !grid_fits(3LL * BH * nqb, C::NTH)) return hipErrorInvalidConfiguration;
    Row32 *info = (Row32 *)ws;
    typedef typename C::T T;
    hipLaunchKernelGGL((bwd32_prep_kernel<T, C::D>), dim3((unsigned)pb), dim3(256), 0, st, (const T *)q,
                       (const T *)k, (const T *)o, (const T *)dout, g, info, rows, qs);
    const Args a{q, k, v, dout, info, dq, dk, dv, N, BH, qs};
    hipLaunchKernelGGL((bwd32_kernel<C>), dim3((unsigned)(3LL * BH * nqb)), dim3(C::NTH), 0, st, a, nqb, hgrp);
    return hipGetLastError();
}

// The workgroup shapes and their measured paces, as in the forward's tables:
// t = t0 + |(a N, b pairs)|_2 us for the whole call, fitted to 1 to 96 heads of
// 130 to 32768 tokens (the choice is within 1% of the best one on average, 21%
// at most).  Float32 rows, 8 heads of 2048 tokens, causal: D = 32 74 us (fp16 pairs under
// shared scales 64, the moment kernels 155), D = 64 121 (592).
constexpr Shape B16[] = {{32, 6.5f, 3.4f, 3.7f}, {32, 6.5f, 6.7f, 2.5f}, {256, 7.9f, 41.4f, 1.85f}};
constexpr Shape B32[] = {{32, 14.3f, 5.3f, 6.f}, {64, 14.3f, 11.5f, 3.6f}, {256, 9.9f, 52.4f, 1.92f}};
constexpr Shape B64[] = {{64, 15.7f, 15.1f, 9.2f}, {128, 13.7f, 42.6f, 6.1f}, {256, 11.3f, 70.4f, 3.97f}};
constexpr Shape B128[] = {{128, 22.7f, 110.f, 13.5f}};
// bf16 rows, fitted likewise (against 280 sizes the choice takes 1.00 to 1.03
// times the best one's time on average, 1.34 at most; H64, whose calls have fewer
// than 128 tokens, by estimate).  8 heads of 4096 tokens, causal, D = 128: 593 us
// (fp16 pairs under shared scales about 410, the moment kernels 5290); with rows
// of v and dO 2^20 larger than the others dk was off by 6e-2 there, 3e-3 here.
constexpr Shape H16[] = {{32, 6.35f, 2.8f, 2.7f}, {32, 6.3f, 4.8f, 2.2f}, {256, 8.2f, 32.f, 1.24f}};
constexpr Shape H32[] = {{32, 9.f, 3.6f, 5.2f}, {64, 8.75f, 11.f, 2.8f}, {256, 6.1f, 35.f, 1.63f}};
constexpr Shape H64[] = {{64, 15.7f, 15.1f, 8.f}, {128, 13.7f, 38.f, 5.f}, {256, 11.3f, 60.f, 3.4f}};
constexpr Shape H128[] = {{128, 15.4f, 72.5f, 9.7f}, {256, 13.8f, 129.f, 5.24f}};

template <typename T, int D, bool CAUSAL>
hipError_t launch_shape(const void *q, const void *k, const void *v, const void *o, const void *dout,
                        const float *g, void *dq, void *dk, void *dv, int BH, int N, float qs, int shape,
                        void *ws, hipStream_t st)
{
#define L(S, ...)                                                                                  \
    do {                                                                                           \
        typedef Cfg<T, D, CAUSAL, __VA_ARGS__> C;                                                  \
        static_assert(C::QB == (S).qb, "table");                                                   \
        return launch<C>(q, k, v, o, dout, g, dq, dk, dv, BH, N, qs, ws, st);                      \
    } while (0)
    constexpr bool F32 = sizeof(T) == 4;
    if constexpr (D == 16) {
        if (shape == 0) L(B16[0], 1, 8, 256);
        if (shape == 1) L(B16[1], 1, 4, 128);
        if (shape == 2) L(B16[2], 8, 1, 64);
    } else if constexpr (D == 32) {
        if (shape == 0) L(B32[0], 1, 8, 256);
        if (shape == 1) L(B32[1], 2, 4, 128);
        if (shape == 2) L(B32[2], 8, 1, 64);
    } else if constexpr (D == 64) {
        if (shape == 0) L(B64[0], 2, 4, 128);
        if (shape == 1) L(B64[1], 4, 2, 64);
        if (shape == 2) L(B64[2], 8, 1, 64);
    } else if constexpr (F32) {
        if (shape == 0) L(B128[0], 4, 1, 32);
    } else {
        if (shape == 0) L(H128[0], 4, 2, 64);
        if (shape == 1) L(H128[1], 8, 1, 32);
    }
#undef L
    return hipErrorInvalidValue;
}

}  // namespace f32
}  // namespace pr

int pairs_bwd32_pick(int BH, int N, int D, int causal, int is_bf16, const pr::Moments &m)
{
    using namespace pr;
    using namespace pr::f32;
    switch (D) {
    case 16: return pick(is_bf16 ? H16 : B16, 3, m, BH, N, causal, 3);
    case 32: return pick(is_bf16 ? H32 : B32, 3, m, BH, N, causal, 3);
    case 64: return pick(is_bf16 ? H64 : B64, 3, m, BH, N, causal, 3);
    case 128: return is_bf16 ? pick(H128, 2, m, BH, N, causal, 3) : pick(B128, 1, m, BH, N, causal, 3);
    }
    return -1;
}

hipError_t pairs_bwd32(const void *q, const void *k, const void *v, const void *o, const void *dout,
                       const float *g, void *dq, void *dk, void *dv, int BH, int N, int D, int causal,
                       int is_bf16, float qs, int shape, void *ws, hipStream_t st)
{
#define GO3(T, DD, CA)                                                                             \
    pr::f32::launch_shape<T, DD, CA>(q, k, v, o, dout, g, dq, dk, dv, BH, N, qs, shape, ws, st)
#define GO2(T, DD) (causal ? GO3(T, DD, true) : GO3(T, DD, false))
#define GO(DD) return is_bf16 ? GO2(bf16_t, DD) : GO2(float, DD)
    switch (D) {
    case 16: GO(16);
    case 32: GO(32);
    case 64: GO(64);
    case 128: GO(128);
    }
#undef GO
#undef GO2
#undef GO3
    return hipErrorInvalidValue;
}

}  // namespace fm
