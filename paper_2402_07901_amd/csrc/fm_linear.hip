// First order (p = 1, f = 1 + tau s) over blocks: forward and backward as
// linear attention.
//
// Every pass is out_t = sum_r (alpha_r + X_r.Z_t) Y_r over the rows r that
// column t sees (Sec. 2.4 at p = 1; Sec. 2.5's gradient with f' = 1):
//   forward: X = k^,   Y = v,   Z = q~,  alpha = 1          (and the row sums G)
//   dv:      X = u q~, Y = dO,  Z = k^,  alpha = u          u = 1 / G
//   dk^:     X = dO,   Y = q~,  Z = v,   alpha = -delta     each row times u
//   dq~:     X = v,    Y = k^,  Z = dO,  alpha = -delta_t   times u_t
// A workgroup takes 256 columns t.  Rows wholly before (after) its block, or
// every row without the mask, only enter the D x D state sum_r Y_r X_r^T and
// sum_r alpha_r Y_r, which each workgroup sums for itself: a 64-row step is a
// few MFMAs per wave, less than its staging, so no state leaves the chip and
// one launch does a pass.  The block's own rows go through 32 x 32 pair tiles.
//
// No operand stands under a shared scale, since a row may never meet the
// largest one of its block: bf16 rows (v, dO) are their own bf16 plane, float32
// rows and what is computed in float32 (k^, q~, the weights, the state) are bf16
// triples (fm_pairs.h).  Rows are taken apart while they are staged.
//
// That work grows as N^2 / 256 per head and takes over from the scans with
// state prefixes (fm_f32_mfma.hip) where heads x tokens fill the chip and N
// is not too long (the table at the end).  Bound by staging: with few heads by
// the chain of up to N / 64 steps, with many by its vector work.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

#include "fm_internal.h"
#include "fm_pairs.h"
#include "fm_pairs_rows.h"

namespace fm {
namespace lin {

using namespace pr;

enum Pass { FWD = 0, DV = 1, DQ = 2, DK = 3 };

struct Args {
    const void *q, *k, *v, *dout;
    const Row32 *info;        // backward
    void *out, *dk, *dv;      // out: O or dq
    float *gout;
    int N, BH;
    float tau;
};

template <typename T_, int D_, bool CAUSAL_>
struct Cfg {
    typedef T_ T;
    static constexpr bool F32 = sizeof(T) == 4;
    static constexpr int RP = F32 ? 3 : 1;             // parts of a row of v or dO
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
    static constexpr int max2(int a, int b) { return a > b ? a : b; }
    static constexpr int PLANES = max2(3 * XH + RP * YH, RP * XH + 3 * YH);
    static constexpr int TILE = 2 * PLANES + 8 * BK;
    static constexpr int SP = 32 * CT * RS;            // a plane of the state
    static constexpr int RED = 4 * NW * TPW * 32 * 33; // the waves' partial tiles
    static constexpr int SUMS = 4 * 2 * TPP * D;       // the threads' alpha Y (and X) sums
    static constexpr int SMEM = max2(max2(TILE, RED), max2(2 * 3 * SP, SUMS));
    static_assert(SMEM <= 158 * 1024 && (2 * PLANES) % 16 == 0, "LDS");
    // bf16 rows, D <= 64: at most 128 registers in the backward, two workgroups a CU
    static constexpr int BWD_WAVES = D <= 64 && !F32 ? 4 : 2;
};

// Rows x columns: the staged one's PA parts read by rows from their planes.  SEP:
// the leading products summed apart (as mma33), else one chain.
template <int KS, int PA, int PB, bool SEP>
__device__ __forceinline__ f16v dot_parts(const _Float16 *p, int plane, const h8 (&o)[KS][PB])
{
    f16v y = f16v{}, z = f16v{};
    constexpr int TOP = PA + PB - 2 < 2 ? PA + PB - 2 : 2;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        h8 x[PA];
#pragma unroll
        for (int i = 0; i < PA; ++i) x[i] = ld8(p + i * plane + 16 * ks);
#pragma unroll
        for (int s = TOP; s >= 0; --s)
#pragma unroll
            for (int i = 0; i < PA; ++i) {
                if (s - i < 0 || s - i >= PB) continue;
                if (SEP && s == 0) z = mma_b(x[0], o[ks][0], z);
                else y = mma_b(x[i], o[ks][s - i], y);
            }
    }
    return SEP && TOP ? y + z : SEP ? z : y;
}

template <typename C, int PASS>
__device__ __forceinline__ void block(unsigned char *smem, float *ssum, const Args &a, int head, int qb)
{
    typedef typename C::T T;
    constexpr bool F32 = C::F32;
    // parts of X, Y, Z
    constexpr int XP = PASS == FWD || PASS == DV ? 3 : C::RP, ZP = XP, YP = PASS == FWD || PASS == DV ? C::RP : 3;
    constexpr int D = C::D, KS = C::KS, CT = C::CT, RS = C::RS, VS = C::VS;
    const int N = a.N;
    _Float16 *const xp = (_Float16 *)smem, *const yp = xp + XP * C::XH;
    float *const rowA = (float *)(smem + 2 * C::PLANES), *const rowU = rowA + C::BK;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    const size_t hb = (size_t)head * N * D;
    const T *const xrow = (const T *)(PASS == FWD ? a.k : PASS == DV ? a.q : PASS == DQ ? a.v : a.dout) + hb;
    const T *const yrow = (const T *)(PASS == FWD ? a.v : PASS == DV ? a.dout : PASS == DQ ? a.k : a.q) + hb;
    const T *const zrow = (const T *)(PASS == FWD ? a.q : PASS == DV ? a.k : PASS == DQ ? a.dout : a.v) + hb;
    const Row32 *const info = PASS == FWD ? nullptr : a.info + (size_t)head * N;
    const int q0 = qb * C::QB + 32 * wave, col = q0 + r32;
    const bool cok = col < N;
    constexpr bool BEFORE = PASS == FWD || PASS == DQ;   // columns see rows r <= t (else r >= t)
    const int nt = (N + C::BK - 1) / C::BK;
    // steps [p0, p1) hold the block's own rows (pairs), [s0, s1) the rest
    constexpr int PB = C::QB / C::BK;
    const int p0 = C::CAUSAL ? qb * PB : 0, p1 = C::CAUSAL ? min(nt, (qb + 1) * PB) : 0;
    const int s0 = !C::CAUSAL ? 0 : BEFORE ? 0 : p1, s1 = !C::CAUSAL ? nt : BEFORE ? p0 : nt;

    Row32 cw = {};
    if constexpr (PASS != FWD) cw = info[cok ? col : 0];
    // staging
    const int sc = tid % C::LPT, st0 = tid / C::LPT;
    RawRow<T, 8> xr[C::NP], yr[C::NP];
    Row32 ri[C::NP];
    auto load = [&](int t) {
#pragma unroll
        for (int p = 0; p < C::NP; ++p) {
            const unsigned n = (unsigned)min(t * C::BK + st0 + C::TPP * p, N - 1);
            const unsigned off = n * (unsigned)D + 8u * sc;
            xr[p].load(xrow + off, true);
            yr[p].load(yrow + off, true);
            if constexpr (PASS != FWD) ri[p] = info[n];
        }
    };
    float ysum[8], xsum[8];
    // writes the loaded step t to LDS (rows past the end weigh nothing); sum:
    // the step enters the state
    auto stage = [&](int t, bool sum) {
#pragma unroll
        for (int p = 0; p < C::NP; ++p) {
            const int row = st0 + C::TPP * p;
            const bool ok = C::BK % C::TPP == 0 || row < C::BK;
            const bool in = ok && t * C::BK + row < N;
            const float u = PASS == FWD ? 1.0f : ri[p].u;
            // alpha, with the row factor where the state takes it with Y
            const float al = !in ? 0.f : PASS == FWD || PASS == DQ ? 1.0f : PASS == DV ? u : sum ? -ri[p].delta : -u * ri[p].delta;
            float x[8], y[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                x[i] = xr[p].get(i);
                y[i] = yr[p].get(i);
                if constexpr (PASS == DV) x[i] = in ? (x[i] - ri[p].mq) * ri[p].rq * u : 0.f;
                if constexpr (PASS == DQ) y[i] = (y[i] - ri[p].mk) * ri[p].rk;
                if constexpr (PASS == DK) y[i] = (y[i] - ri[p].mq) * ri[p].rq * (sum ? u : 1.0f);
                y[i] = in ? y[i] : 0.f;
            }
            if constexpr (PASS == FWD) standardise_group<D>(x, in);
            if (!ok) continue;
            if constexpr (XP == 3) {
                h8 w[3];
                split3(x, w);
#pragma unroll
                for (int i = 0; i < 3; ++i) *(h8 *)(xp + i * C::XH + row * RS + 8 * sc) = w[i];
            } else {
                *(uint4 *)(xp + row * RS + 8 * sc) = *(uint4 *)xr[p].w;
            }
            if constexpr (YP == 3) {
                h8 w[3];
                split3(y, w);
#pragma unroll
                for (int i = 0; i < 3; ++i) *(h8 *)(yp + i * C::YH + row * VS + 8 * sc) = w[i];
            } else {
                *(uint4 *)(yp + row * VS + 8 * sc) = in ? *(uint4 *)yr[p].w : make_uint4(0u, 0u, 0u, 0u);
            }
            if ((PASS == DV || PASS == DK) && sc == 0) {
                rowA[row] = al;
                if constexpr (PASS == DK) rowU[row] = in ? u : 0.f;
            }
            if (sum) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    ysum[i] = fmaf(al, y[i], ysum[i]);
                    if constexpr (PASS == FWD) xsum[i] += x[i];
                }
            }
        }
    };

    f16v acc[CT];
#pragma unroll
    for (int c = 0; c < CT; ++c) acc[c] = f16v{};
    float rs = 0.f;

    // ---- the state over the rows outside the block ------------------------
    if (s0 < s1) {
        // float32 rows: a step's products on their own and one rounded add (the
        // matrix pipe's chained sums are cut toward zero); bf16 rows: the chains
        // themselves (the adds cost 398 -> 433 us on 64 heads of 3001 tokens for no
        // bit that bf16 shows)
        f16v sh[C::TPW], sl[C::TPW];
#pragma unroll
        for (int i = 0; i < C::TPW; ++i) sh[i] = sl[i] = f16v{};
#pragma unroll
        for (int i = 0; i < 8; ++i) ysum[i] = xsum[i] = 0.f;
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
                f16v lo = F32 ? f16v{} : sl[i], hi = F32 ? f16v{} : sh[i];   // as mma33
#pragma unroll
                for (int e0 = 0; e0 < C::STEPS; e0 += C::GW) {
                    const int e = e0 + part;
                    h8 y[YP], x[XP];
#pragma unroll
                    for (int j = 0; j < YP; ++j) y[j] = ld_tr<VS>(yp + j * C::YH, 16 * e, 32 * yc);
#pragma unroll
                    for (int j = 0; j < XP; ++j) x[j] = ld_tr<RS>(xp + j * C::XH, 16 * e, 32 * xc);
#pragma unroll
                    for (int o = 2; o > 0; --o)
#pragma unroll
                        for (int j = 0; j < YP; ++j)
                            if (o - j >= 0 && o - j < XP) lo = mma_b(y[j], x[o - j], lo);
                    hi = mma_b(y[0], x[0], hi);
                }
                if constexpr (F32) {
                    sh[i] += hi + lo;
                } else {
                    sh[i] = hi;
                    sl[i] = lo;
                }
            }
        }
        // the threads' sums of alpha Y: [token lane][channel]
        float *const su = (float *)smem;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            su[st0 * D + 8 * sc + i] = ysum[i];
            if constexpr (PASS == FWD) su[(C::TPP + st0) * D + 8 * sc + i] = xsum[i];
        }
        __syncthreads();
        if (tid < (PASS == FWD ? 2 : 1) * D) {
            const float *p = su + (tid / D) * C::TPP * D + tid % D;
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
                red[((wave * C::TPW + i) * 32 + 8 * (j / 4) + 4 * h + j % 4) * 33 + r32] = sh[i][j] + sl[i][j];
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
    h8 z[KS][ZP];
    {
        float x[D / 2];
        load_cols<T, D>(zrow, col, N, x);
        if constexpr (PASS == FWD) standardise_cols<D>(x, cok, a.tau);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if constexpr (PASS == DV) {
#pragma unroll
                for (int i = 0; i < 8; ++i) x[8 * ks + i] = cok ? (x[8 * ks + i] - cw.mk) * cw.rk : 0.f;
            }
            if constexpr (PASS == FWD) {
                // half a column's q~ . sum k^ on each half lane (their sums are added)
                if (s0 < s1) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) rs = fmaf(x[8 * ks + i], ssum[D + 16 * ks + 8 * h + i], rs);
                }
            }
            h8 w[3];
            split3(x + 8 * ks, w);
#pragma unroll
            for (int i = 0; i < ZP; ++i) z[ks][i] = w[i];   // (a bf16 row is its own first part)
        }
    }

    if (s0 < s1) {
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            const f16v f = dot_parts<KS, 3, ZP, true>((const _Float16 *)smem + (32 * c + r32) * RS + 8 * h, C::SP, z);
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int d = 32 * c + 8 * (j / 4) + 4 * h + j % 4;
                const float ys = D % 32 == 0 || d < D ? ssum[d < D ? d : 0] : 0.f;
                acc[c][j] = PASS == DQ ? fmaf(-cw.delta, ys, f[j]) : f[j] + ys;
            }
        }
    }

    // ---- the block's own rows, pair by pair -------------------------------
    // (where Z and the output leave no registers for rows on their way: no prefetch)
    constexpr bool AHEAD = D < (F32 || PASS == FWD ? 128 : 64);
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
            const f16v s = dot_parts<KS, XP, ZP, F32>(xp + (32 * j + r32) * RS + 8 * h, C::XH, z);
            float w[16], x[PASS == FWD ? 16 : 1];   // x: the scores of visible pairs
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                float4 A, U;
                if constexpr (PASS == DV || PASS == DK) A = *(const float4 *)(rowA + 32 * j + 8 * b + 4 * h);
                if constexpr (PASS == DK) U = *(const float4 *)(rowU + 32 * j + 8 * b + 4 * h);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int e = 4 * b + i;
                    if constexpr (PASS == FWD) w[e] = (x[e] = s[e]) + 1.0f;
                    else if constexpr (PASS == DQ) w[e] = s[e] - cw.delta;
                    else if constexpr (PASS == DV) w[e] = s[e] + ((const float *)&A)[i];
                    else w[e] = fmaf(s[e], ((const float *)&U)[i], ((const float *)&A)[i]);
                }
            }
            if (kb == q0 || kb + 32 > N) {
                asm volatile("");
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int row = kb + 8 * (i / 4) + 4 * h + i % 4;
                    if (row >= N || (BEFORE ? row > col : row < col)) {
                        w[i] = 0.f;
                        if constexpr (PASS == FWD) x[i] = 0.f;
                    }
                }
            }
            h8 w3[2][3];
#pragma unroll
            for (int e = 0; e < 2; ++e) split3(w + 8 * e, w3[e]);
            if constexpr (PASS == FWD) {
                // the scores' sum; G counts its keys exactly
#pragma unroll
                for (int d = 8; d; d /= 2)
#pragma unroll
                    for (int i = 0; i < d; ++i) x[i] += x[i + d];
                rs += x[0];
            }
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                h8 y[YP][2];
#pragma unroll
                for (int i = 0; i < YP; ++i)
#pragma unroll
                    for (int e = 0; e < 2; ++e) y[i][e] = ld_tr<VS>(yp + i * C::YH, 32 * j + 16 * e, 32 * c);
                if constexpr (F32) {
                    acc[c] += mma33(y, w3);
                } else {
                    f16v z2 = acc[c];
#pragma unroll
                    for (int o = 2; o >= 0; --o)
#pragma unroll
                        for (int i = 0; i < YP; ++i)
                            if (o - i >= 0)
#pragma unroll
                                for (int e = 0; e < 2; ++e) z2 = mma_b(y[i][e], w3[e][o - i], z2);
                    acc[c] = z2;
                }
            }
        }
    }

    if constexpr (PASS == FWD) {
        const float G = half_sum(rs) + (float)(C::CAUSAL ? col + 1 : N);
        if (cok && a.gout && h == 0) a.gout[(size_t)head * N + col] = G;
        const float f = 1.0f / G;
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[c][i] *= f;
    }
    if constexpr (PASS == DQ) {
        const float f = a.tau * cw.u;
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[c][i] *= f;
    }
    const size_t at = hb + (size_t)(cok ? col : 0) * D;
    if constexpr (PASS == DQ || PASS == DK) standardise_back<T, D>((const T *)(PASS == DQ ? a.q : a.k) + at, acc);
    if (cok) store_col<T, D>((T *)(PASS == DK ? a.dk : PASS == DV ? a.dv : a.out) + at, acc);
}

template <typename C>
__global__ __launch_bounds__(C::NTH, 2) void fwd_kernel(Args a, int nqb)
{
    __shared__ alignas(16) unsigned char smem[C::SMEM];
    __shared__ float ssum[2 * C::D];
    // the blocks with the most rows first
    block<C, FWD>(smem, ssum, a, blockIdx.x % a.BH, nqb - 1 - blockIdx.x / a.BH);
}

template <typename C>
__global__ __launch_bounds__(C::NTH, C::BWD_WAVES) void bwd_kernel(Args a, int nqb)
{
    __shared__ alignas(16) unsigned char smem[C::SMEM];
    __shared__ float ssum[2 * C::D];
    const int head = blockIdx.x % a.BH, rest = blockIdx.x / a.BH, pass = rest % 3, i = rest / 3;
    if (pass == 0) block<C, DQ>(smem, ssum, a, head, nqb - 1 - i);
    else if (pass == 1) block<C, DK>(smem, ssum, a, head, i);
    else block<C, DV>(smem, ssum, a, head, i);
}

template <int D, bool CAUSAL>
hipError_t run_fwd(const void *q, const void *k, const void *v, void *out, float *g, int BH, int N,
                   float qs, hipStream_t st)
{
    typedef Cfg<bf16_t, D, CAUSAL> C;
    const int nqb = (N + C::QB - 1) / C::QB;
    if (!grid_fits((long long)BH * nqb, C::NTH)) return hipErrorInvalidConfiguration;
    const Args a{q, k, v, nullptr, nullptr, out, nullptr, nullptr, g, N, BH, qs};
    hipLaunchKernelGGL((fwd_kernel<C>), dim3((unsigned)(BH * nqb)), dim3(C::NTH), 0, st, a, nqb);
    return hipGetLastError();
}

template <typename T, int D, bool CAUSAL>
hipError_t run_bwd(const void *q, const void *k, const void *v, const void *o, const void *dout,
                   const float *g, void *dq, void *dk, void *dv, int BH, int N, float qs, void *ws,
                   hipStream_t st)
{
    typedef Cfg<T, D, CAUSAL> C;
    const long long rows = (long long)BH * N, pb = (rows * (D / 8) + 255) / 256;
    const int nqb = (N + C::QB - 1) / C::QB;
    if (!grid_fits(pb, 256) || !grid_fits(3LL * BH * nqb, C::NTH)) return hipErrorInvalidConfiguration;
    Row32 *info = (Row32 *)ws;
    hipLaunchKernelGGL((bwd32_prep_kernel<T, D>), dim3((unsigned)pb), dim3(256), 0, st, (const T *)q,
                       (const T *)k, (const T *)o, (const T *)dout, g, info, rows, qs);
    const Args a{q, k, v, dout, info, dq, dk, dv, nullptr, N, BH, qs};
    hipLaunchKernelGGL((bwd_kernel<C>), dim3((unsigned)(3LL * BH * nqb)), dim3(C::NTH), 0, st, a, nqb);
    return hipGetLastError();
}

// First-order calls that run here: scores with |tau s| <= 1 (tau D <= 1), so
// that no weight is negative and G rarely comes close to cancelling; the scans
// keep the others, and the float32 forward.
//
// Paces, us: a workgroup takes w + a N rows / 1000 (half the rows under the
// causal mask, on average), 256 run at once; the scans take s + o heads N /
// 1000.  Fitted to 1 to 64 heads of 256 to 8192 tokens; the choice takes 1.00 to
// 1.02 times the better one's time on average (1.6 at most: few long heads that
// stay with the scans).  Measured, scans -> here, causal, tau = 1/D:
// bf16 D = 64, 64 heads of 4096 308 -> 180 forward, 1329 -> 451 backward; 8 of 4096
// 63 -> 68 (stays) and 246 -> 80; 64 of 256 21 -> 15 and 92 -> 20; 1 of 8192 25 ->
// 119 (stays).  D = 128, 64 of 2048 390 -> 152 and 1943 -> 414.  Float32 backward:
// 8 of 2048, D = 32 71 -> 41; 64 of 2048, D = 64 676 -> 283; D = 128 1974 -> 702.
struct Pace {
    float w, a, s, o;
};
constexpr Pace FP[] = {{}, {2.2f, 8.7f, 12.f, .5f}, {5.7f, 12.1f, 11.f, 1.3f}, {13.f, 36.7f, 15.f, 4.f}};
// backward: bf16 rows, float32 rows
constexpr Pace BP[] = {{4.6f, 5.3f, 37.f, 1.f}, {5.f, 6.1f, 38.f, 2.2f}, {9.3f, 11.f, 38.f, 4.8f}, {15.f, 36.8f, 50.f, 14.5f}};
constexpr Pace BF[] = {{5.8f, 7.8f, 37.f, 1.f}, {7.5f, 10.4f, 38.f, 2.2f}, {12.2f, 18.3f, 38.f, 4.8f}, {21.3f, 56.f, 50.f, 14.5f}};

}  // namespace lin

bool linear_plan(int BH, int N, int D, int p, int causal, int is_bf16, float qs, int backward, size_t ws_bytes)
{
    using namespace lin;
    // (at D = 16 the forward's scans are the faster ones at every size)
    if (p != 1 || qs * (float)D > 1.0f || (!backward && (!is_bf16 || D == 16))) return false;
    const size_t rows = (size_t)BH * N;
    if (!grid_fits((backward ? 3LL : 1LL) * BH * ((N + 255LL) / 256), 512)) return false;
    if (backward && ws_bytes < rows * ROW32_BYTES) return false;
    const Pace &x = (!backward ? FP : is_bf16 ? BP : BF)[D == 16 ? 0 : D == 32 ? 1 : D == 64 ? 2 : 3];
    const double n = 1e-3 * N, blocks = (double)BH * ((N + 255) / 256) * (backward ? 3 : 1) / 256;
    const double t = 5 + std::hypot(x.w + x.a * n, blocks * (x.w + x.a * n * (causal ? .5 : 1)));
    return t < 0.9 * (x.s + x.o * BH * n);
}

hipError_t linear_fwd(const void *q, const void *k, const void *v, void *out, float *g, int BH,
                      int N, int D, int causal, float qs, hipStream_t st)
{
#define GO(DD)                                                                                     \
    return causal ? lin::run_fwd<DD, true>(q, k, v, out, g, BH, N, qs, st)                 \
                  : lin::run_fwd<DD, false>(q, k, v, out, g, BH, N, qs, st)
    switch (D) {
    case 32: GO(32);
    case 64: GO(64);
    case 128: GO(128);
    }
#undef GO
    return hipErrorInvalidValue;
}

hipError_t linear_bwd(const void *q, const void *k, const void *v, const void *o, const void *dout,
                      const float *g, void *dq, void *dk, void *dv, int BH, int N, int D, int causal,
                      int is_bf16, float qs, void *ws, hipStream_t st)
{
#define GO3(T, DD, CA) lin::run_bwd<T, DD, CA>(q, k, v, o, dout, g, dq, dk, dv, BH, N, qs, ws, st)
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
