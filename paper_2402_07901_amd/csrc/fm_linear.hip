// First order (p = 1, f = 1 + tau s) over blocks: forward and backward of bf16
// rows as linear attention, float32-grade operands (fm_pairs.h).  The backward
// of float32 rows: fm_linear32.hip.
//
// Every pass is out_t = sum_r (alpha + X_r.Z_t) Y_r over the rows r that
// column t sees (Sec. 2.4 at p = 1; Sec. 2.5's gradient with f' = 1):
//   forward: X = k^, Y = v,  Z = q~,  alpha = 1 (and the row sums G)
//   dv:      X = q~, Y = u,  Z = k^,  alpha = 1           u_i = dO_i / G_i
//   dq~:     X = v,  Y = k^, Z = dO,  alpha = -delta_t    times 1 / G_t
//   dk^:     X = u,  Y = q~, Z = v,   alpha = -c_r        c_i = dO_i.O_i / G_i
// A workgroup takes 256 columns t.  Rows wholly before (after) its block, or
// every row without the mask, only enter the D x D state sum_r Y_r X_r^T and
// sum_r alpha_r Y_r, which each workgroup sums for itself: a 64-row step is a
// few MFMAs per wave, less than its staging, so no state leaves the chip and
// one launch does a pass.  The block's own rows go through 32 x 32 pair tiles.
// That work grows as N^2 / 256 per head and takes over from the scans with
// state prefixes (fm_f32_mfma.hip) where heads x tokens fill the chip and N
// is not too long (the table at the end).
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
    const float *g;
    const _Float16 *planes;   // q~ / sc hi, lo, k^ hi, lo (backward)
    const RowInfo *info;
    void *out, *dk, *dv;      // out: O or dq
    float *gout;
    int N, BH;
    float qs, qn, sc;         // tau = qn sc, sc a power of two
};

template <typename T_, int D_, bool CAUSAL_>
struct Cfg {
    typedef T_ T;
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
    static constexpr int GW = NT < NW ? NW / NT : 1;   // waves sharing a tile, by K steps
    static constexpr int STEPS = BK / 16;
    static constexpr bool ZLDS = D >= 128;             // Z's lo part in LDS
    static constexpr int TILE = 2 * (2 * XH + 2 * YH) + 4 * BK;
    static constexpr int SP = 32 * CT * RS;            // a plane of the state
    static constexpr int RED = 4 * NW * TPW * 32 * 33; // the waves' partial tiles
    static constexpr int SUMS = 4 * 2 * TPP * D;       // the threads' alpha Y (and X) sums
    static constexpr int BODY0 = TILE > RED ? TILE : RED;
    static constexpr int BODY1 = 4 * SP > SUMS ? 4 * SP : SUMS;
    static constexpr int BODY = (BODY0 > BODY1 ? BODY0 : BODY1) + 15 & ~15;
    static constexpr int SMEM = BODY + (ZLDS ? 2 * QB * RS : 0);
    static_assert(SMEM <= 158 * 1024, "LDS");
    // D <= 64: at most 128 registers in the backward, two workgroups a CU
    static constexpr int BWD_WAVES = D <= 64 ? 4 : 2;
};

template <typename C, int PASS>
__device__ __forceinline__ void block(unsigned char *smem, int *sred, float *ssum, const Args &a,
                                      int head, int qb)
{
    typedef typename C::T T;
    constexpr int D = C::D, KS = C::KS, CT = C::CT, RS = C::RS, VS = C::VS;
    // operands with a lo part: bf16 rows need none
    constexpr bool XSPL = PASS != DQ, YSPL = PASS != FWD, ZSPL = PASS == FWD || PASS == DV;
    constexpr bool UNIT = PASS == FWD || PASS == DV;   // alpha = 1
    const int N = a.N;
    _Float16 *const xp = (_Float16 *)smem, *const yp = xp + 2 * C::XH;
    float *const rowD = (float *)(yp + 2 * C::YH);
    _Float16 *const zlo = (_Float16 *)(smem + C::BODY);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    const size_t hb = (size_t)head * N * D, np = (size_t)a.BH * N * D;
    const T *const qr = (const T *)a.q + hb, *const kr = (const T *)a.k + hb, *const vr = (const T *)a.v + hb;
    const T *const dor = PASS == FWD ? nullptr : (const T *)a.dout + hb;
    const _Float16 *const qpl = PASS == FWD ? nullptr : a.planes + hb;
    const _Float16 *const kpl = PASS == FWD ? nullptr : a.planes + 2 * np + hb;
    const RowInfo *const info = PASS == FWD ? nullptr : a.info + (size_t)head * N;
    const float *const g = PASS == FWD ? nullptr : a.g + (size_t)head * N;
    const int q0 = qb * C::QB + 32 * wave, col = q0 + r32;
    const bool cok = col < N;
    constexpr bool BEFORE = PASS == FWD || PASS == DQ;   // columns see rows r <= t (else r >= t)
    const int nt = (N + C::BK - 1) / C::BK;
    // steps [p0, p1) hold the block's own rows (pairs), [s0, s1) the rest
    constexpr int PB = C::QB / C::BK;
    const int p0 = C::CAUSAL ? qb * PB : 0, p1 = C::CAUSAL ? min(nt, (qb + 1) * PB) : 0;
    const int s0 = !C::CAUSAL ? 0 : BEFORE ? 0 : p1, s1 = !C::CAUSAL ? nt : BEFORE ? p0 : nt;
    const int rbeg = C::CAUSAL && !BEFORE ? qb * C::QB : 0, rend = C::CAUSAL && BEFORE ? min(N, (qb + 1) * C::QB) : N;

    constexpr int LD = D == 16 ? 4 : D == 32 ? 5 : D == 64 ? 6 : 7;
    // exponents: M of the staged v (DQ) or dO / G (DV, DK); MO of v (DK); MC of c (DK)
    int M = 0, MO = 0, MC = NO_EXP;
    if constexpr (PASS != FWD) {
        if (tid < 3) sred[tid] = NO_EXP;
        __syncthreads();
        int m = NO_EXP, mo = NO_EXP, mc = NO_EXP;
        for (int n = tid; n < N; n += C::NTH) {
            const RowInfo x = info[n];
            mo = max(mo, (int)x.e_v);
            if (n < rbeg || n >= rend) continue;
            if constexpr (PASS == DQ) {
                m = max(m, (int)x.e_v);
            } else if (x.e_do != NO_EXP && 1.0f / fabsf(g[n]) <= 3.4028235e38f) {
                // (G may be zero at tau D = 1, where q^ = -k^ in the first row:
                // such a row has no finite gradient, and no part in the scale of
                // the rows that other columns see)
                m = max(m, x.e_do - g_exp(g[n]));
                if (PASS == DK) mc = max(mc, exp_above(fabsf(x.delta / g[n])));
            }
        }
        if (m > NO_EXP) atomicMax(&sred[0], m);
        if (PASS == DK && mo > NO_EXP) atomicMax(&sred[1], mo);
        if (PASS == DK && mc > NO_EXP) atomicMax(&sred[2], mc);
        __syncthreads();
        M = sred[0] == NO_EXP ? 0 : sred[0];
        MO = PASS == DK && sred[1] != NO_EXP ? sred[1] : 0;
        MC = PASS == DK ? sred[2] : NO_EXP;
    }

    // own columns Z as B operands
    h8 zh[KS], zl[ZSPL && !C::ZLDS ? KS : 1];
    _Float16 *const zlw = zlo + (32 * wave + r32) * RS + 8 * h;
    float acol = 0.f, cw = 1.0f;   // DQ: delta in the scale of X.Z; the weights' scale (DQ, DK)
    int ecol = 0;
    {
        float z[D / 2];
        if constexpr (PASS == FWD) {
            load_cols<T, D>(qr, col, N, z);
            standardise_cols<D>(z, cok, a.qn);
        } else if constexpr (PASS != DV) {
            load_cols<T, D>(PASS == DQ ? dor : vr, col, N, z);
            const RowInfo w = info[cok ? col : 0];
            ecol = PASS == DQ ? (w.e_do == NO_EXP ? 0 : w.e_do) : MO;
            const float s = exp2i(10 - ecol);
#pragma unroll
            for (int i = 0; i < D / 2; ++i) z[i] *= s;
            int H = LD + 24;
            if constexpr (PASS == DQ) {
                acol = (cok ? w.delta : 0.f) * s * exp2i(14 - M);
                H = max(H, exp_above(fabsf(acol)));
            } else if (MC != NO_EXP) {
                H = max(H, MC + 24 - M - MO);
            }
            cw = exp2i(14 - H);
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            h8 lo = h8{};
            if constexpr (PASS == DV) {
                const size_t off = (size_t)(cok ? col : 0) * D + 8 * h + 16 * ks;
                zh[ks] = *(const h8 *)(kpl + off);
                lo = *(const h8 *)(kpl + np + off);
            } else {
                split8<ZSPL>(z + 8 * ks, zh[ks], lo);
            }
            if constexpr (ZSPL) {
                if constexpr (C::ZLDS) *(h8 *)(zlw + 16 * ks) = lo;
                else zl[ks] = lo;
            }
        }
    }
    auto zlo_of = [&](int ks) -> h8 {
        if constexpr (C::ZLDS) return ld8(zlw + 16 * ks);
        else return zl[ks];
    };

    // staging
    const int sc = tid % C::LPT, st0 = tid / C::LPT;
    RawRow<T, 8> r0[C::NP], r1[PASS == FWD ? C::NP : 1];
    RawRow<bf16_t, 8> ph[PASS == FWD ? 1 : C::NP], pl[PASS == FWD ? 1 : C::NP];   // fp16 words
    RowInfo ri[C::NP];
    float gr[C::NP];
    auto load = [&](int t) {
#pragma unroll
        for (int p = 0; p < C::NP; ++p) {
            const unsigned n = (unsigned)min(t * C::BK + st0 + C::TPP * p, N - 1);
            const unsigned off = n * (unsigned)D + 8u * sc;
            r0[p].load((PASS == FWD || PASS == DQ ? vr : dor) + off, true);
            if constexpr (PASS == FWD) {
                r1[p].load(kr + off, true);
            } else {
                const _Float16 *const b = PASS == DQ ? kpl : qpl;
                ph[p].load((const bf16_t *)b + off, true);
                pl[p].load((const bf16_t *)b + np + off, true);
                if constexpr (PASS != DQ) {
                    ri[p] = info[n];
                    gr[p] = g[n];
                }
            }
        }
    };
    float vmax = 0.f, vscale = 1.0f;
    float ysum[8], xsum[8];
    // writes the loaded step t to LDS; rows outside weigh nothing; SUM: the
    // step enters the state
    auto stage = [&](int t, bool sum) {
#pragma unroll
        for (int p = 0; p < C::NP; ++p) {
            const int row = st0 + C::TPP * p, n = t * C::BK + row;
            const bool ok = C::BK % C::TPP == 0 || row < C::BK;
            const bool in = ok && n < N;
            float x[8], y[8];
            h8 xh, xl, yh, yl;
            float al = in ? 1.0f : 0.f;
            if constexpr (PASS == FWD) {
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    y[i] = r0[p].get(i);
                    vmax = fmaxf(vmax, fabsf(y[i]));
                    y[i] = in ? y[i] * vscale : 0.f;
                    x[i] = r1[p].get(i);
                }
                standardise_group<D>(x, in);
                split8<true>(x, xh, xl);
                split8<false>(y, yh, yl);
            } else {
                const h8 ah = __builtin_bit_cast(h8, *(uint4 *)ph[p].w), bl = __builtin_bit_cast(h8, *(uint4 *)pl[p].w);
                const float f = !in ? 0.f : PASS == DQ ? exp2i(14 - M) : exp2i(14 - M) / gr[p];
                float z[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) z[i] = in ? r0[p].get(i) * f : 0.f;
                h8 zh8, zl8;
                split8<PASS != DQ>(z, zh8, zl8);
                if constexpr (PASS == DV) {
                    xh = ah; xl = bl; yh = zh8; yl = zl8;
#pragma unroll
                    for (int i = 0; i < 8; ++i) y[i] = z[i];
                } else {
                    xh = zh8; xl = zl8;
                    const h8 zero = h8{};
                    yh = in ? ah : zero;
                    yl = in ? bl : zero;
#pragma unroll
                    for (int i = 0; i < 8; ++i) y[i] = (float)yh[i] + (float)yl[i];
                }
                if constexpr (PASS == DK) {
                    al = in ? -(ri[p].delta * f * exp2i(10 - MO)) : 0.f;
                    if (ok && sc == 0) rowD[row] = al;
                }
            }
            if (ok) {
                *(h8 *)(xp + row * RS + 8 * sc) = xh;
                if constexpr (XSPL) *(h8 *)(xp + C::XH + row * RS + 8 * sc) = xl;
                *(h8 *)(yp + row * VS + 8 * sc) = yh;
                if constexpr (YSPL) *(h8 *)(yp + C::YH + row * VS + 8 * sc) = yl;
                if (sum) {
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        ysum[i] = fmaf(al, y[i], ysum[i]);
                        if constexpr (PASS == FWD) xsum[i] += x[i];
                    }
                }
            }
        }
    };

    f16v acc[CT];
    float rs = 0.f;
    if constexpr (PASS == FWD) {
        // value scale of the head: the first step read, with headroom (below; a
        // step of zeros, e.g. a padded prefix, takes the largest scale there is,
        // which any later value outgrows)
        load(p0 < s0 ? p0 : s0);
#pragma unroll
        for (int p = 0; p < C::NP; ++p)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float y = fabsf(r0[p].get(i));
                if (y <= 3.4028235e38f) vmax = fmaxf(vmax, y);
            }
        if (tid == 0) sred[0] = 0;
        __syncthreads();
        atomicMax(&sred[0], __float_as_int(vmax));
        __syncthreads();
        vscale = pow2_scale(__int_as_float(sred[0]), 7);
        vmax = 0.f;
    }
    for (int attempt = 0;; ++attempt) {
#pragma unroll
        for (int c = 0; c < CT; ++c) acc[c] = f16v{};
        rs = 0.f;

        // ---- the state over the rows outside the block -------------------
        if (s0 < s1) {
            f16v sh[C::TPW], sl[C::TPW];
#pragma unroll
            for (int i = 0; i < C::TPW; ++i) sh[i] = sl[i] = f16v{};
#pragma unroll
            for (int i = 0; i < 8; ++i) ysum[i] = xsum[i] = 0.f;
            const int tile0 = (wave % (C::NT < C::NW ? C::NT : C::NW)) * C::TPW, part = wave / (C::NT < C::NW ? C::NT : C::NW);
            load(s0);
            for (int t = s0; t < s1; ++t) {
                __syncthreads();
                stage(t, true);
                if (t + 1 < s1) load(t + 1);
                __syncthreads();
#pragma unroll
                for (int i = 0; i < C::TPW; ++i) {
                    const int yc = (tile0 + i) / CT, xc = (tile0 + i) % CT;
#pragma unroll
                    for (int e0 = 0; e0 < C::STEPS; e0 += C::GW) {
                        const int e = e0 + part;
                        if (C::STEPS % C::GW != 0 && e >= C::STEPS) break;
                        const h8 ya = ld_tr<VS>(yp, 16 * e, 32 * yc), xb = ld_tr<RS>(xp, 16 * e, 32 * xc);
                        sh[i] = mma(ya, xb, sh[i]);
                        if constexpr (XSPL) sl[i] = mma(ya, ld_tr<RS>(xp + C::XH, 16 * e, 32 * xc), sl[i]);
                        if constexpr (YSPL) sl[i] = mma(ld_tr<VS>(yp + C::YH, 16 * e, 32 * yc), xb, sl[i]);
                    }
                }
            }
            // the threads' sums of alpha Y (and X): [token lane][channel]
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
            if (tid == 0) sred[1] = 0;
            __syncthreads();
            // partial tiles -> sums -> fp16 planes [y][x] below 2^14
            float *const red = (float *)smem;
#pragma unroll
            for (int i = 0; i < C::TPW; ++i)
#pragma unroll
                for (int j = 0; j < 16; ++j)
                    red[((wave * C::TPW + i) * 32 + 8 * (j / 4) + 4 * h + j % 4) * 33 + r32] = sh[i][j] + sl[i][j];
            __syncthreads();
            constexpr int SE = 32 * CT * 32 * CT, EPT = (SE + C::NTH - 1) / C::NTH;
            float sv[EPT], sm = 0.f;
#pragma unroll
            for (int i = 0; i < EPT; ++i) {
                const int e = tid + C::NTH * i, y = e / (32 * CT), x = e % (32 * CT);
                const int tl = (y / 32) * CT + x / 32;
                float s = 0.f;
                for (int w = 0; w < C::GW; ++w)
                    s += red[(((tl / C::TPW + w * (C::NT < C::NW ? C::NT : C::NW)) * C::TPW + tl % C::TPW) * 32 + y % 32) * 33 + x % 32];
                sv[i] = y < D && x < D ? s : 0.f;
                const float m = fabsf(sv[i]);
                if (m <= 3.4028235e38f) sm = fmaxf(sm, m);
            }
            atomicMax(&sred[1], __float_as_int(sm));
            __syncthreads();
            const float ss = pow2_scale(__int_as_float(sred[1]), 14), is = 1.0f / ss;
            _Float16 *const st = (_Float16 *)smem;
#pragma unroll
            for (int i = 0; i < EPT; ++i) {
                const int e = tid + C::NTH * i, y = e / (32 * CT), x = e % (32 * CT);
                if (x < D) {
                    const _Float16 hi = (_Float16)(sv[i] * ss);
                    st[y * RS + x] = hi;
                    st[C::SP + y * RS + x] = (_Float16)rest(sv[i] * ss, hi);
                }
            }
            __syncthreads();
            float dot = 0.f;
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                f16v P = f16v{}, Q = f16v{};
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const h8 A = ld8(st + (32 * c + r32) * RS + 16 * ks + 8 * h);
                    const h8 B = ld8(st + C::SP + (32 * c + r32) * RS + 16 * ks + 8 * h);
                    P = mma(A, zh[ks], P);
                    Q = mma(B, zh[ks], Q);
                    if constexpr (ZSPL) Q = mma(A, zlo_of(ks), Q);
                }
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const int d = 32 * c + 8 * (j / 4) + 4 * h + j % 4;
                    const float ys = D % 32 == 0 || d < D ? ssum[d < D ? d : 0] : 0.f;
                    const float f = (P[j] + Q[j]) * is;
                    acc[c][j] = UNIT ? fmaf(f, a.sc, ys) : PASS == DQ ? fmaf(-acol, ys, f) * cw : (f + ys) * cw;
                }
            }
            if constexpr (PASS == FWD) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const h8 lo = zlo_of(ks);
#pragma unroll
                    for (int i = 0; i < 8; ++i)
                        dot = fmaf((float)zh[ks][i] + (float)lo[i], ssum[D + 16 * ks + 8 * h + i], dot);
                }
                // half the count on each half lane (their sums are added)
                rs = fmaf(dot, a.sc, 0.5f * (float)min(N - s0 * C::BK, (s1 - s0) * C::BK));
            }
        }

        // ---- the block's own rows, pair by pair ---------------------------
        if (p0 < p1) load(p0);
        for (int t = p0; t < p1; ++t) {
            __syncthreads();
            stage(t, false);
            if (t + 1 < p1) load(t + 1);
            __syncthreads();
#pragma unroll 1
            for (int j = 0; j < C::BK / 32; ++j) {
                const int kb = t * C::BK + 32 * j;
                if (kb >= N || (BEFORE ? kb > q0 : kb < q0)) continue;
                f16v s;
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    float4 dd = make_float4(0.f, 0.f, 0.f, 0.f);
                    if constexpr (PASS == DK) dd = *(const float4 *)(rowD + 32 * j + 8 * b + 4 * h);
#pragma unroll
                    for (int i = 0; i < 4; ++i) s[4 * b + i] = PASS == DK ? ((const float *)&dd)[i] : PASS == DQ ? -acol : 0.f;
                }
                const _Float16 *const xr = xp + (32 * j + r32) * RS + 8 * h;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const h8 A = ld8(xr + 16 * ks);
                    if constexpr (ZSPL) s = mma(A, zlo_of(ks), s);
                    if constexpr (XSPL) s = mma(ld8(xr + C::XH + 16 * ks), zh[ks], s);
                    s = mma(A, zh[ks], s);
                }
                float w[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) w[i] = UNIT ? fmaf(s[i], a.sc, 1.0f) : s[i] * cw;
                if (kb == q0 || kb + 32 > N) {
                    asm volatile("");
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int row = kb + 8 * (i / 4) + 4 * h + i % 4;
                        if (row >= N || (BEFORE ? row > col : row < col)) w[i] = 0.f;
                    }
                }
                h8 wh[2], wl[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) split8<true>(w + 8 * e, wh[e], wl[e]);
                if constexpr (PASS == FWD) {
#pragma unroll
                    for (int d = 8; d; d /= 2)
#pragma unroll
                        for (int i = 0; i < d; ++i) w[i] += w[i + d];
                    rs += w[0];
                }
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    const h8 A0 = ld_tr<VS>(yp, 32 * j, 32 * c), A1 = ld_tr<VS>(yp, 32 * j + 16, 32 * c);
                    f16v z = acc[c];
                    z = mma(A0, wl[0], z);
                    z = mma(A1, wl[1], z);
                    if constexpr (YSPL) {
                        z = mma(ld_tr<VS>(yp + C::YH, 32 * j, 32 * c), wh[0], z);
                        z = mma(ld_tr<VS>(yp + C::YH, 32 * j + 16, 32 * c), wh[1], z);
                    }
                    z = mma(A0, wh[0], z);
                    z = mma(A1, wh[1], z);
                    acc[c] = z;
                }
            }
        }
        if constexpr (PASS != FWD) break;
        if (attempt || !__syncthreads_or(vmax * vscale > 65504.0f)) break;
        // a value outgrew the first step's scale: the largest finite one of
        // the rows read
        const float m = largest_finite<T, D>(vr, sc, st0, C::TPP, rend);
        if (tid == 0) sred[0] = 0;
        __syncthreads();
        atomicMax(&sred[0], __float_as_int(m));
        __syncthreads();
        vscale = pow2_scale(__int_as_float(sred[0]), 14);
    }

    // out of the scales
    float f0 = 1.0f, f1 = 1.0f;
    if constexpr (PASS == FWD) {
        const float G = half_sum(rs);
        if (cok && a.gout && h == 0) a.gout[(size_t)head * N + col] = G;
        f0 = 1.0f / G;
        f1 = 1.0f / vscale;
    } else if constexpr (PASS == DV) {
        f0 = exp2i(M - 14);
    } else if constexpr (PASS == DQ) {
        f0 = a.qs / g[cok ? col : 0] / cw;
        f1 = exp2i(ecol - 10) * exp2i(M - 14);
    } else {
        f0 = a.sc / cw * exp2i(M - 14);
        f1 = exp2i(MO - 10);
    }
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[c][i] = acc[c][i] * f0 * f1;
    if constexpr (PASS == DQ || PASS == DK) standardise_back<T, D>((PASS == DQ ? qr : kr) + (size_t)(cok ? col : 0) * D, acc);
    if (cok) store_col<T, D>((T *)(PASS == DK ? a.dk : PASS == DV ? a.dv : a.out) + hb + (size_t)col * D, acc);
}

template <typename C>
__global__ __launch_bounds__(C::NTH, 2) void fwd_kernel(Args a, int nqb)
{
    __shared__ alignas(16) unsigned char smem[C::SMEM];
    __shared__ int sred[3];
    __shared__ float ssum[2 * C::D];
    // the blocks with the most rows first
    block<C, FWD>(smem, sred, ssum, a, blockIdx.x % a.BH, nqb - 1 - blockIdx.x / a.BH);
}

template <typename C>
__global__ __launch_bounds__(C::NTH, C::BWD_WAVES) void bwd_kernel(Args a, int nqb)
{
    __shared__ alignas(16) unsigned char smem[C::SMEM];
    __shared__ int sred[3];
    __shared__ float ssum[2 * C::D];
    const int head = blockIdx.x % a.BH, rest = blockIdx.x / a.BH, pass = rest % 3, i = rest / 3;
    if (pass == 0) block<C, DQ>(smem, sred, ssum, a, head, nqb - 1 - i);
    else if (pass == 1) block<C, DK>(smem, sred, ssum, a, head, i);
    else block<C, DV>(smem, sred, ssum, a, head, i);
}

// tau = qn sc with sc a power of two and 1 <= qn < 2: q~'s planes hold q^ qn,
// whose lo parts a small tau would push below fp16's range.
float scale_of(float qs)
{
    int e = 0;
    frexpf(qs, &e);
    return ldexpf(1.0f, e - 1);
}

template <typename T, int D, bool CAUSAL>
hipError_t run_fwd(const void *q, const void *k, const void *v, void *out, float *g, int BH, int N,
                   float qs, hipStream_t st)
{
    typedef Cfg<T, D, CAUSAL> C;
    const int nqb = (N + C::QB - 1) / C::QB;
    if (!grid_fits((long long)BH * nqb, C::NTH)) return hipErrorInvalidConfiguration;
    const float sc = scale_of(qs);
    const Args a{q, k, v, nullptr, nullptr, nullptr, nullptr, out, nullptr, nullptr, g, N, BH, qs, qs / sc, sc};
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
    const float sc = scale_of(qs);
    _Float16 *planes = (_Float16 *)ws;
    RowInfo *info = (RowInfo *)(planes + 4 * (size_t)rows * D);
    hipLaunchKernelGGL((bwd_prep_kernel<T, D, true>), dim3((unsigned)pb), dim3(256), 0, st,
                       (const T *)q, (const T *)k, (const T *)v, (const T *)o, (const T *)dout, g,
                       planes, (void *)info, rows, qs / sc);
    const Args a{q, k, v, dout, g, planes, info, dq, dk, dv, nullptr, N, BH, qs, qs / sc, sc};
    hipLaunchKernelGGL((bwd_kernel<C>), dim3((unsigned)(3LL * BH * nqb)), dim3(C::NTH), 0, st, a, nqb);
    return hipGetLastError();
}

// First-order calls that run here: scores with |tau s| <= 1 (tau D <= 1), so
// that no weight is negative and G rarely comes close to cancelling, which
// would show the bf16 rows' 22-bit operands (at tau = 1 the error of O was ten
// times the float32 scans', whose 24 bits those calls keep).  Float32 rows: the
// backward only (a float32 forward's G would go from 3.2e-8 to 4.6e-8).
//
// Paces, us: a workgroup takes w + a N rows / 1000 (half the rows under the
// causal mask, on average), 256 run at once; the scans take s + o heads N /
// 1000.  Measured, scans -> here (D = 64, causal, tau = 1/64): 64 heads of 3001
// tokens bf16 226 -> 118 forward, 976 -> 313 backward; 8 of 3001 51 -> 49 and
// 197 -> 73; 64 of 256 21 -> 17 and 91 -> 29; 1 of 8192 26 -> 103 (stays).
// Float32 backward, causal: 8 heads of 2048, D = 32 71 -> 42; 64 of 2048, D = 64
// 677 -> 276; D = 128 1974 -> 683.
struct Pace {
    float w, a, s, o;
};
constexpr Pace FP[] = {{}, {13.f, 10.6f, 12.f, .5f}, {13.f, 11.5f, 11.f, 1.1f}, {50.f, 33.f, 15.f, 2.9f}};
// backward: bf16 rows, float32 rows
constexpr Pace BP[] = {{13.f, 8.f, 37.f, 1.f}, {15.f, 11.f, 38.f, 2.2f}, {18.f, 14.f, 38.f, 4.8f}, {31.f, 39.f, 50.f, 14.5f}};
constexpr Pace BF[] = {{5.6f, 7.8f, 37.f, 1.f}, {7.4f, 10.5f, 38.f, 2.2f}, {12.3f, 17.9f, 38.f, 4.8f}, {21.4f, 55.5f, 50.f, 14.5f}};

}  // namespace lin

bool linear_plan(int BH, int N, int D, int p, int causal, int is_bf16, float qs, int backward, size_t ws_bytes)
{
    using namespace lin;
    // (at D = 16 the forward's scans are the faster ones at every size)
    if (p != 1 || qs * (float)D > 1.0f || (!backward && (!is_bf16 || D == 16))) return false;
    const size_t rows = (size_t)BH * N;
    if (!grid_fits((backward ? 3LL : 1LL) * BH * ((N + 255LL) / 256), 512)) return false;
    if (backward && ws_bytes < rows * (is_bf16 ? 8 * (size_t)D + sizeof(RowInfo) : ROW32_BYTES)) return false;
    const Pace &x = (!backward ? FP : is_bf16 ? BP : BF)[D == 16 ? 0 : D == 32 ? 1 : D == 64 ? 2 : 3];
    const double n = 1e-3 * N, blocks = (double)BH * ((N + 255) / 256) * (backward ? 3 : 1) / 256;
    const double t = 5 + std::hypot(x.w + x.a * n, blocks * (x.w + x.a * n * (causal ? .5 : 1)));
    return t < 0.9 * (x.s + x.o * BH * n);
}

hipError_t linear_fwd(const void *q, const void *k, const void *v, void *out, float *g, int BH,
                      int N, int D, int causal, float qs, hipStream_t st)
{
#define GO(DD)                                                                                     \
    return causal ? lin::run_fwd<bf16_t, DD, true>(q, k, v, out, g, BH, N, qs, st)                 \
                  : lin::run_fwd<bf16_t, DD, false>(q, k, v, out, g, BH, N, qs, st)
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
    if (!is_bf16) return linear_bwd32(q, k, v, o, dout, g, dq, dk, dv, BH, N, D, causal, qs, ws, st);
#define GO2(DD, CA) lin::run_bwd<bf16_t, DD, CA>(q, k, v, o, dout, g, dq, dk, dv, BH, N, qs, ws, st)
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
