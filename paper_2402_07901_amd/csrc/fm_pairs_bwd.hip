// Pair backward of fp16 operands (see fm_pairs.h; p = 2, bf16 rows of D = 64,
// causal or at least 128 tokens; the others:
// fm_pairs_bwd32.hip): the custom gradient of Sec. 2.5 (only
// O and G saved) over explicit (query, key) pairs.  With q~ = tau q^,
// u = 1 / G, delta_i = dO_i.O_i and t = 1 + q~_i.k^_n = f_2'(tau s),
//   dv_n  = sum_i f_2 u_i dO_i,               f_2 = (t^2 + 1) / 2,
//   dq~_i = sum_n T_in k^_n,  dk^_n = sum_i T_in q~_i,
//   T_in  = t u_i (dO_i.v_n - delta_i)
// (Sec. 2.3, Eq. "bound"), then the standardisation backward (Eqs. 6-7) of the
// finished rows.  bwd_prep writes q~, k^, v and dO as fp16 planes
// and four words per row; bwd_kernel holds three kinds of workgroups
// in one launch, each with 32 columns per wave in registers and the other side
// staged in steps of BK rows: role Q (columns queries, out dq), role K (columns
// keys, out dk) and role V (columns keys, out dv).  No atomics: every output
// row has one owner, results repeat bit for bit.
//
// Scales.  1/G falls from about 1 to 1/(tens of N) along a causal sequence, so
// a row's power of two goes to the contraction's A operand and its pairs fill
// the fp16 range.  Role K: with G_i = 2^k / rho (1/2 < rho <= 1) and
// 2^h > |dO_i.v_n|, |delta_i| for the workgroup's keys n, the pairs carry
// rho t (dO_i.v_n - delta_i) 2^-h and row i's A operand 2^(h - k - M) <= 1, M
// the largest h - k of the rows read; role V: dO_i / G_i 2^-M; role Q: 1/G_i
// stays out of the sum.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "fm_internal.h"
#include "fm_pairs.h"
#include "fm_pairs_rows.h"

namespace fm {
namespace pr {

enum Role { ROLE_Q = 0, ROLE_K = 1, ROLE_V = 2 };

template <typename T_, int D_, bool CAUSAL_, int NQ_, int NWQ_, int NWK_, int BK_>
struct BwdCfg {
    typedef T_ T;
    static constexpr int D = D_, NQ = NQ_, NWQ = NWQ_, NWK = NWK_, BK = BK_;
    static constexpr bool CAUSAL = CAUSAL_;
    static constexpr int NTH = 64 * NWQ * NWK;
    static constexpr int QB = 32 * NQ * NWQ;
    static constexpr int KS = D / 16, CT = D < 32 ? 1 : D / 32;
    static constexpr int LPT = D / 8, TPP = NTH / LPT, NP = (BK + TPP - 1) / TPP;
    static constexpr int RS = row_stride<D>(), VS = tr_stride<D>();
    static constexpr int XH = BK * RS, AH = BK * VS;
    // planes of a step: x (scores), val (dO.v), and the contraction's A
    // operand where it is not x itself (role K: scaled q~; role V: scaled dO u)
    static constexpr int TILE_Q = 2 * 2 * XH;
    static constexpr int TILE_K = 2 * (2 * XH + AH) + 8 * BK;
    static constexpr int TILE = TILE_K;   // role V: fewer planes
    // two steps' tiles in turn where LDS has room beside the other workgroups
    // of the CU (eight waves in all): one barrier a step instead of two
    static constexpr bool DB = 2 * TILE <= 160 * 1024 * NWQ * NWK / 8 - 256;
    static constexpr int NB = DB ? 2 : 1;
    static constexpr int LOOP_BYTES = NB * TILE;
    static constexpr int RED_BYTES = NWK > 1 ? 4 * NWQ * NWK * 32 * 32 * CT : 0;
    static constexpr int SMEM = LOOP_BYTES > RED_BYTES ? LOOP_BYTES : RED_BYTES;
    static_assert(BK % (32 * NWK) == 0 && (NWK == 1 || NQ == 1) && TILE_K >= TILE_Q, "shape");
};

struct BwdArgs {
    const void *q, *k;
    const float *g;
    const _Float16 *planes;
    const RowInfoH *info;
    void *dq, *dk, *dv;
    int N, BH;
    float qs;   // tau
};

template <typename C, int ROLE>
__device__ __forceinline__ void bwd_block(unsigned char *smem, int *sred, const BwdArgs &a, int head,
                                          int qb)
{
    typedef typename C::T T;
    constexpr int D = C::D, NQ = C::NQ, KS = C::KS, CT = C::CT, RS = C::RS, VS = C::VS;
    const int N = a.N;
    // a step's planes (a buffer of them), in halves from its start: x, the
    // staged values (roles Q, K), the contraction's A operand (K, V), and
    // role K's row factors
    constexpr int OV = C::XH, OA = ROLE == ROLE_V ? OV : OV + C::XH, OB = OA + C::AH;
    static_assert(C::TILE % 16 == 0, "alignment");

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    const int wq = wave / C::NWK, wk = wave % C::NWK;
    const size_t hb = (size_t)head * N * D, np = (size_t)a.BH * N * D;
    // own columns and staged rows
    const _Float16 *const qpl = a.planes + hb, *const kpl = a.planes + np + hb;
    const _Float16 *const own = ROLE == ROLE_Q ? qpl : kpl, *const stg = ROLE == ROLE_Q ? kpl : qpl;
    const RowInfoH *const info = a.info + (size_t)head * N;
    // fp16 planes of v, dO and dO rho
    const _Float16 *const hpl = a.planes + (ROLE == ROLE_Q ? 2 : ROLE == ROLE_K ? 3 : 4) * np + hb;
    const float *const g = a.g + (size_t)head * N;
    const int q0 = qb * C::QB + 32 * NQ * wq;
    const int rbeg = C::CAUSAL && ROLE != ROLE_Q ? qb * C::QB : 0;
    const int rend = C::CAUSAL && ROLE == ROLE_Q ? min(N, (qb + 1) * C::QB) : N;
    const int t0 = rbeg / C::BK, t1 = (rend + C::BK - 1) / C::BK;

    // staging: this thread's 8 channels and first row
    const int sc = tid % C::LPT, st0 = tid / C::LPT;
    RawRow<bf16_t, 8> xr[C::NP], hr[C::NP];   // fp16 words
    RowInfoH ri[C::NP];
    // rows past the end repeat the last one: masked (role Q) or given weight 0
    auto load_tile = [&](int t) {
#pragma unroll
        for (int p = 0; p < C::NP; ++p) {
            const unsigned n = (unsigned)min(t * C::BK + st0 + C::TPP * p, N - 1);
            const unsigned off = n * (unsigned)D + 8u * sc;
            xr[p].load((const bf16_t *)stg + off, true);
            hr[p].load((const bf16_t *)hpl + off, true);
            ri[p] = info[n];
        }
    };
    load_tile(t0);

    // Q: the largest exponent of the staged v; V: of dO / G; K: of the own v
    // (MO), then of h - k
    constexpr int LD = D == 16 ? 4 : D == 32 ? 5 : D == 64 ? 6 : 7;
    if (tid < 2) sred[tid] = NO_EXP;
    __syncthreads();
    int MO = 0;
    if constexpr (ROLE == ROLE_K) {
        const int n = qb * C::QB + tid;
        if (tid < C::QB && n < N && info[n].e_v > NO_EXP) atomicMax(&sred[1], (int)info[n].e_v);
        __syncthreads();
        MO = sred[1] == NO_EXP ? 0 : sred[1];
    }
    // h - e of a row of dO
    auto row_h = [&](const RowInfoH &x) { return max(LD + MO, exp_above(fabsf(x.delta)) - 10); };
    {
        int m = NO_EXP;
        for (int n = rbeg + tid; n < rend; n += C::NTH) {
            const RowInfoH x = info[n];
            if constexpr (ROLE == ROLE_Q) {
                m = max(m, (int)x.e_v);
            } else if (x.e_do != NO_EXP) {
                m = max(m, ROLE == ROLE_K ? x.eg + row_h(x) : x.eg);
            }
        }
        if (m > NO_EXP) atomicMax(&sred[0], m);
    }
    __syncthreads();
    const int M = sred[0] == NO_EXP ? 0 : sred[0];
    // role Q: T = t (dP - delta) with |dP| < D 2^24 (values below 2^14 and 2^10)
    constexpr int X = -10 - 2 * LD;

    // own columns as B operands: x, and (roles Q, K) dO or v scaled
    h8 oh[NQ][KS];
    h8 vo[ROLE != ROLE_V ? NQ : 1][KS];
    float dcol[NQ];
    int ecol[NQ];
#pragma unroll
    for (int t = 0; t < NQ; ++t) {
        const int n = q0 + 32 * t + r32;
        const bool ok = n < N;
        const size_t off = (size_t)(ok ? n : 0) * D + 8 * h;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const h8 x = *(const h8 *)(own + off + 16 * ks);
            oh[t][ks] = ok ? x : h8{};
        }
        if constexpr (ROLE != ROLE_V) {
            const RowInfoH w = info[ok ? n : 0];
            const _Float16 *const pl = a.planes + (ROLE == ROLE_Q ? 3 : 2) * np + hb;
            const _Float16 s = ROLE == ROLE_Q ? (_Float16)1.0f : half2i((w.e_v == NO_EXP ? 0 : w.e_v) - MO);
            ecol[t] = ROLE == ROLE_Q ? (w.e_do == NO_EXP ? 0 : w.e_do) : MO;
            dcol[t] = ROLE == ROLE_Q ? w.delta * exp2i(14 - M) * exp2i(X) : 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) vo[t][ks] = *(const h8 *)(pl + off + 16 * ks) * s;
        }
    }

    f16v acc[NQ][CT];
#pragma unroll
    for (int t = 0; t < NQ; ++t)
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            acc[t][c] = f16v{};
        }

    // One 32-row tile j of the staged step against the wave's columns; masked:
    // some of its pairs lie beyond the diagonal.
    auto tile = [&](const _Float16 *xhi, int j, int kb, bool masked) {
        const _Float16 *const vhi = xhi + OV, *const ahi = xhi + OA;
        const float *const rowB = (const float *)(xhi + OB), *const rowD = rowB + C::BK;
        f16v s[NQ], d[ROLE != ROLE_V ? NQ : 1];
#pragma unroll
        for (int u = 0; u < NQ; ++u)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                s[u][i] = 1.0f;   // 1 + tau s
                if constexpr (ROLE != ROLE_V) d[u][i] = 0.0f;
            }
        const _Float16 *xp = xhi + (32 * j + r32) * RS + 8 * h;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const h8 x = ld8(xp + 16 * ks);
#pragma unroll
            for (int u = 0; u < NQ; ++u) s[u] = mma(x, oh[u][ks], s[u]);
        }
        if constexpr (ROLE != ROLE_V) {
            const _Float16 *vp = vhi + (32 * j + r32) * RS + 8 * h;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const h8 x = ld8(vp + 16 * ks);
#pragma unroll
                for (int u = 0; u < NQ; ++u) d[u] = mma(x, vo[u][ks], d[u]);
            }
        }
        h8 th[NQ][2], lo;
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
            const int col = q0 + 32 * u + r32, last = C::CAUSAL ? min(col, N - 1) : N - 1;
            float w[16];
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                float4 B, E;
                if constexpr (ROLE == ROLE_K) {
                    B = *(const float4 *)(rowB + 32 * j + 8 * b + 4 * h);
                    E = *(const float4 *)(rowD + 32 * j + 8 * b + 4 * h);
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float st = s[u][4 * b + i];
                    if constexpr (ROLE == ROLE_V) w[4 * b + i] = fmaf(st, st, 1.0f);
                    else if constexpr (ROLE == ROLE_Q)
                        w[4 * b + i] = st * fmaf(d[u][4 * b + i], exp2i(X), -dcol[u]);
                    else
                        w[4 * b + i] = st * fmaf(d[u][4 * b + i], ((const float *)&B)[i], -((const float *)&E)[i]);
                }
            }
            if (masked) {
                asm volatile("");   // a branch, not a compare and select per element of every tile
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int row = kb + 8 * (i / 4) + 4 * h + i % 4;
                    if (ROLE == ROLE_Q ? row > last : row < col) w[i] = 0.f;
                }
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) split8<false>(w + 8 * e, th[u][e], lo);
        }
        constexpr int AS = ROLE == ROLE_Q ? RS : VS;
        const _Float16 *const ap = ROLE == ROLE_Q ? xhi : ahi;
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                const h8 x = ld_tr<AS>(ap, 32 * j + 16 * e, 32 * c);
#pragma unroll
                for (int u = 0; u < NQ; ++u) acc[u][c] = mma(x, th[u][e], acc[u][c]);
            }
    };

    // writes the loaded step t to a buffer
    auto stage = [&](_Float16 *xhi, int t) {
        _Float16 *const vhi = xhi + OV, *const ahi = xhi + OA;
        float *const rowB = (float *)(xhi + OB), *const rowD = rowB + C::BK;
#pragma unroll
        for (int p = 0; p < C::NP; ++p) {
            const int row = st0 + C::TPP * p;
            const bool ok = C::BK % C::TPP == 0 || row < C::BK;
            const int n = t * C::BK + row;
            const bool in = n < N && n >= rbeg;   // the others weigh nothing
            const h8 x0 = __builtin_bit_cast(h8, *(uint4 *)xr[p].w);
            if (ok) *(h8 *)(xhi + row * RS + 8 * sc) = x0;
            const h8 z = __builtin_bit_cast(h8, *(uint4 *)hr[p].w);
            if constexpr (ROLE == ROLE_Q) {
                if (ok) *(h8 *)(vhi + row * RS + 8 * sc) = z * half2i(4 + ri[p].e_v - M);
            } else if constexpr (ROLE == ROLE_V) {
                if (ok) *(h8 *)(ahi + row * VS + 8 * sc) = z * (in ? half2i(4 + ri[p].eg - M) : (_Float16)0.0f);
            } else {
                const int hm = row_h(ri[p]), y = in ? min(max(ri[p].eg + hm - M, -40), 0) : -40;
                if (ok) {
                    *(h8 *)(vhi + row * RS + 8 * sc) = z;
                    *(h8 *)(ahi + row * VS + 8 * sc) = x0 * half2i(11 + y);
                    if (sc == 0) {
                        // the scales of dO.v (values below 2^10) and delta in T
                        const float B = in ? ri[p].rho * exp2i(MO - 8 - LD - hm) : 0.f;
                        rowB[row] = B;
                        rowD[row] = in ? ri[p].rho * exp2i(2 - LD - hm) * ri[p].delta : 0.f;
                    }
                }
            }
        }
    };
    auto compute = [&](const _Float16 *buf, int t) {
#pragma unroll 1
        for (int j = wk; j < C::BK / 32; j += C::NWK) {
            const int kb = t * C::BK + 32 * j;
            if (kb >= N || (C::CAUSAL && ROLE == ROLE_Q && kb > q0 + 32 * NQ - 1)) break;
            if (C::CAUSAL && ROLE != ROLE_Q && kb + 31 < q0) continue;
            tile(buf, j, kb, ROLE == ROLE_Q ? (C::CAUSAL && kb + 31 > q0) || kb + 32 > N
                                       : C::CAUSAL && kb < q0 + 32 * NQ - 1);
        }
    };

    if constexpr (C::DB) {
        constexpr int BH2 = C::TILE / 2;
        if (t0 < t1) stage((_Float16 *)smem, t0);
        if (t0 + 1 < t1) load_tile(t0 + 1);
        __syncthreads();
        for (int t = t0; t < t1; ++t) {
            _Float16 *const buf = (_Float16 *)smem + ((t - t0) & 1) * BH2;
            compute(buf, t);
            if (t + 1 < t1) {
                stage((_Float16 *)smem + ((t + 1 - t0) & 1) * BH2, t + 1);
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
                    mine[32 * (32 * c + 8 * (i / 4) + 4 * h + i % 4) + r32] = acc[0][c][i];
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
                    acc[0][c][i] += part[32 * (32 * c + 8 * (i / 4) + 4 * h + i % 4) + r32];
        }
    }

    const float tau = a.qs;
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        const int n = q0 + 32 * u + r32;
        const bool ok = n < N;
        T *const out = (T *)(ROLE == ROLE_Q ? a.dq : ROLE == ROLE_K ? a.dk : a.dv) + hb + (size_t)(ok ? n : 0) * D;
        // out of the scales (in two factors: each a normal number)
        float f0, f1;
        if constexpr (ROLE == ROLE_V) {
            f0 = 0.5f * exp2i(-14);
            f1 = exp2i(M);
        } else if constexpr (ROLE == ROLE_K) {
            f0 = exp2i(LD - 23);
            f1 = exp2i(M);
        } else {
            f0 = tau / g[ok ? n : 0] * exp2i(-X - 24);
            f1 = exp2i(ecol[u]) * exp2i(M);
        }
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[u][c][i] = acc[u][c][i] * f0 * f1;
        if constexpr (ROLE != ROLE_V)
            standardise_back<T, D>((const T *)(ROLE == ROLE_Q ? a.q : a.k) + hb + (size_t)(ok ? n : 0) * D, acc[u]);
        if (ok) store_col<T, D>(out, acc[u]);
    }
}

// Block order: heads in groups of hgrp; within a group the columns with the
// most rows first (role Q: the last queries; K, V: the first keys), the three
// roles of a column block side by side.
template <typename C>
__global__ __launch_bounds__(C::NTH, 2) void bwd_kernel(BwdArgs a, int nqb, int hgrp)
{
    __shared__ alignas(16) unsigned char smem[C::SMEM];
    __shared__ int sred[2];
    const int b = blockIdx.x, per = 3 * hgrp * nqb, grp = b / per, r = b - grp * per;
    const int gs = min(hgrp, a.BH - grp * hgrp);
    const int head = grp * hgrp + r % gs, rest = r / gs, role = rest % 3, i = rest / 3;
    if (role == 0) bwd_block<C, ROLE_Q>(smem, sred, a, head, nqb - 1 - i);
    else if (role == 1) bwd_block<C, ROLE_K>(smem, sred, a, head, i);
    else bwd_block<C, ROLE_V>(smem, sred, a, head, i);
}

template <typename C>
hipError_t launch_bwd(const void *q, const void *k, const void *v, const void *o, const void *dout,
                      const float *g, void *dq, void *dk, void *dv, int BH, int N, float qs,
                      void *ws, hipStream_t st)
{
    typedef typename C::T T;
    const long long rows = (long long)BH * N, pb = (rows * (C::D / 8) + 255) / 256;
    const int nqb = (N + C::QB - 1) / C::QB, hgrp = BH < 32 ? BH : 32;
    if (!grid_fits(pb, 256) || !grid_fits(3LL * BH * nqb, C::NTH)) return hipErrorInvalidConfiguration;
    _Float16 *planes = (_Float16 *)ws;
    RowInfoH *info = (RowInfoH *)(planes + 5 * (size_t)rows * C::D);
    hipLaunchKernelGGL((bwd_prep_kernel<T, C::D>), dim3((unsigned)pb), dim3(256), 0, st,
                       (const T *)q, (const T *)k, (const T *)v, (const T *)o, (const T *)dout, g,
                       planes, info, rows, qs);
    const BwdArgs a{q, k, g, planes, info, dq, dk, dv, N, BH, qs};
    hipLaunchKernelGGL((bwd_kernel<C>), dim3((unsigned)(3LL * BH * nqb)), dim3(C::NTH), 0, st, a, nqb, hgrp);
    return hipGetLastError();
}

// The workgroup shapes and their measured paces, as in the forward's tables:
// t = t0 + |(a N, b pairs)|_2 us for the whole call, fitted to 1 to 96 heads
// of 33 to 4096 tokens.  Against every shape and the moment kernels at 507
// sizes, up to 200000 tokens, the choice takes 1.00 to 1.03 times the best one's
// time on average, and at most 1.36 on the wrong side of the line.
constexpr Shape BH64[] = {{64, 13.5f, 10.f, 2.15f}, {128, 13.5f, 14.f, 1.5f}, {256, 13.f, 23.f, 1.22f},
                          {256, 15.f, 36.f, 1.1f}};

Moments moments_bwd(int D, int causal, bool grade32)
{
    if (!grade32 && causal) return {12.f, 0.f, 113.f, 3.6f};
    if (!grade32) return {40.f, .5f, 68.f, 3.25f};
    switch (D) {
    case 16: return causal ? Moments{36.f, .27f, 5.7f, 2.f} : Moments{37.5f, .4f, 6.3f, 1.21f};
    case 32: return causal ? Moments{72.f, .2f, 9.f, 6.15f} : Moments{71.f, 1.05f, 5.7f, 3.9f};
    case 64: return causal ? Moments{103.f, 2.f, 34.f, 29.6f} : Moments{101.f, 5.9f, 15.4f, 18.7f};
    default: return causal ? Moments{130.f, 0.f, 236.f, 162.f} : Moments{150.f, 0.f, 175.f, 168.f};
    }
}

template <bool CAUSAL>
hipError_t launch_bwd_shape(const void *q, const void *k, const void *v, const void *o,
                            const void *dout, const float *g, void *dq, void *dk, void *dv, int BH,
                            int N, float qs, int shape, void *ws, hipStream_t st)
{
#define L(S, ...)                                                                                  \
    do {                                                                                           \
        typedef BwdCfg<bf16_t, 64, CAUSAL, __VA_ARGS__> C;                                         \
        static_assert(C::QB == (S).qb, "table");                                                   \
        return launch_bwd<C>(q, k, v, o, dout, g, dq, dk, dv, BH, N, qs, ws, st);                  \
    } while (0)
    if (shape == 0) L(BH64[0], 1, 2, 4, 128);
    if (shape == 1) L(BH64[1], 1, 4, 2, 128);
    if (shape == 2) L(BH64[2], 1, 8, 1, 64);
    if (shape == 3) L(BH64[3], 2, 4, 1, 32);
#undef L
    return hipErrorInvalidValue;
}

}  // namespace pr

int pairs_bwd_plan(int BH, int N, int D, int p, int causal, int is_bf16, size_t ws_bytes)
{
    using namespace pr;
    if (p != 2) return -1;
    const bool grade32 = pairs_grade32(N, D, causal, is_bf16);
    const size_t rows = (size_t)BH * N;
    const size_t per_row = grade32 ? (size_t)ROW32_BYTES : 10 * (size_t)D + sizeof(RowInfoH);
    if (ws_bytes < rows * per_row) return -1;
    const Moments m = moments_bwd(D, causal, grade32);
    if (grade32) return pairs_bwd32_pick(BH, N, D, causal, is_bf16, m);
    return pick(BH64, 4, m, BH, N, causal, 3);
}

hipError_t pairs_bwd(const void *q, const void *k, const void *v, const void *o, const void *dout,
                     const float *g, void *dq, void *dk, void *dv, int BH, int N, int D, int causal,
                     int is_bf16, float qs, int shape, void *ws, hipStream_t st)
{
    if (pairs_grade32(N, D, causal, is_bf16))
        return pairs_bwd32(q, k, v, o, dout, g, dq, dk, dv, BH, N, D, causal, is_bf16, qs, shape, ws, st);
    return causal ? pr::launch_bwd_shape<true>(q, k, v, o, dout, g, dq, dk, dv, BH, N, qs, shape, ws, st)
                  : pr::launch_bwd_shape<false>(q, k, v, o, dout, g, dq, dk, dv, BH, N, qs, shape, ws, st);
}

}  // namespace fm
