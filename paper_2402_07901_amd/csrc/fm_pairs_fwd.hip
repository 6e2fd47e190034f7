// Pair forward (see fm_pairs.h): O_i = sum_n w_in v_n / sum_n w_in with the
// weights formed 32 keys x 32 queries at a time, one launch and no workspace
// (the shape with KP: k^ once as an fp16 plane in the workspace, a launch before).
//
// A workgroup of NWQ x NWK waves takes NWQ 32-query columns tiles (NQ per
// wave); NWK waves share a query tile and split the keys.  Per step it stages
// BK keys (standardised on the way, Sec. 2.2) and their values in LDS, the
// next step's rows already on their way into registers.
//
// Value scale.  At D = 64 bf16 values go to fp16 under a power-of-two scale per
// 8-column group (the float32-grade calls hold values as bf16 parts and need
// none).  It is taken from the first staged tile with 8 binary digits of headroom; each
// thread keeps the largest magnitude that it stages, and only if that
// overflowed the headroom (a later token more than 2^8 times the first tile's
// largest) the workgroup finds the true maximum and runs its keys again.  A
// group that is zero over the whole first tile (a padded or zeroed prefix)
// says nothing about the later values: its scale is the largest there is, which
// any value outgrows.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fm_internal.h"
#include "fm_pairs.h"

namespace fm {
namespace pr {

template <typename T_, int D_, bool CAUSAL_, bool SPL_, bool KP_, int NQ_, int NWQ_, int NWK_, int BK_>
struct FwdCfg {
    typedef T_ T;
    static constexpr int D = D_, NQ = NQ_, NWQ = NWQ_, NWK = NWK_, BK = BK_;
    static constexpr bool CAUSAL = CAUSAL_, SPL = SPL_, KP = KP_;
    // SPL: the weights as bf16 triples; float32 values in three bf16 parts, bf16
    // values as they are.  A float32 tile's contribution is summed on its own,
    // the small products first, and added with a rounded float32 add (the matrix
    // pipe's own chained sums round toward zero).
    static constexpr bool F32 = sizeof(T) == 4;
    static constexpr int VP = F32 ? 3 : 1;
    static constexpr float QKS = SPL ? 256.0f : 1.0f;      // of q^ and of k^
    static constexpr int NTH = 64 * NWQ * NWK;
    static constexpr int QB = 32 * NQ * NWQ;              // queries per workgroup
    static constexpr int KS = D / 16;                     // contraction steps of a score
    static constexpr int CT = D < 32 ? 1 : D / 32;        // 32-column value tiles
    static constexpr int LPT = D / 8;                     // staging lanes per token
    static constexpr int TPP = NTH / LPT;                 // tokens per staging pass
    static constexpr int NP = (BK + TPP - 1) / TPP;       // passes
    static constexpr int RS = row_stride<D>(), VS = tr_stride<D>();
    static constexpr int KH = BK * RS, VH = BK * VS;      // halves per plane
    static constexpr int TILE_BYTES = 2 * ((SPL ? 2 : 1) * KH + VP * VH);
    // the waves' partial numerators meet in LDS when they split the keys
    static constexpr int RED_BYTES = NWK > 1 ? 4 * NWQ * NWK * 32 * (32 * CT + 1) : 0;
    // at D = 128 the queries' lo parts wait in LDS: the registers go to the
    // prefetch
    static constexpr bool QLDS = SPL && D >= 128;
    static constexpr int LOOP_BYTES = TILE_BYTES + (QLDS ? 2 * QB * RS : 0);
    static constexpr int SMEM = LOOP_BYTES > RED_BYTES ? LOOP_BYTES : RED_BYTES;
    static_assert(BK % (32 * NWK) == 0 && D % 16 == 0 && (NWK == 1 || NQ == 1) && !(KP && SPL), "shape");
    static_assert(SMEM <= 160 * 1024 - 256, "LDS");
    // waves per SIMD: four waves that fill a CU's LDS are alone on it
    static constexpr int WPS = NTH <= 256 && SMEM > 80 * 1024 ? 1 : 2;
};

template <typename C>
__global__ __launch_bounds__(C::NTH, C::WPS) void fwd_kernel(
    const typename C::T *__restrict__ q, const typename C::T *__restrict__ k,
    const typename C::T *__restrict__ v, const _Float16 *__restrict__ khat,
    typename C::T *__restrict__ out, float *__restrict__ g, int N, int BH, int nqb, int hgrp, float qs, float sc2)
{
    typedef typename C::T T;
    constexpr int D = C::D, NQ = C::NQ, KS = C::KS, CT = C::CT, LPT = C::LPT, RS = C::RS, VS = C::VS;
    constexpr bool SPL = C::SPL, F32 = C::F32;
    __shared__ alignas(16) unsigned char smem[C::SMEM];
    __shared__ unsigned int smax[LPT];
    __shared__ float sscale[LPT];
    _Float16 *const khi = (_Float16 *)smem, *const klo = khi + C::KH;
    _Float16 *const vhi = khi + (SPL ? 2 : 1) * C::KH;
    _Float16 *const qlo = (_Float16 *)(smem + C::TILE_BYTES);

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r32 = lane & 31, h = lane >> 5;
    const int wq = wave / C::NWK, wk = wave % C::NWK;

    // Block order: heads in groups of hgrp (a multiple of 8 where there are
    // as many, so that a head's blocks share an XCD's L2), within a group the
    // blocks with the most keys first.
    int head, qb;
    {
        const int b = blockIdx.x, per = hgrp * nqb, grp = b / per, r = b - grp * per;
        const int gs = min(hgrp, BH - grp * hgrp);
        head = grp * hgrp + r % gs;
        qb = nqb - 1 - r / gs;
    }
    const size_t hb = (size_t)head * N * D;
    q += hb;
    k += hb;
    v += hb;
    khat += hb;
    out += hb;
    const int q0 = qb * C::QB + 32 * NQ * wq;      // this wave's first query
    const int kend = C::CAUSAL ? min(N, (qb + 1) * C::QB) : N;
    const int nt = (kend + C::BK - 1) / C::BK;

    // the wave's queries, standardised, as B operands
    h8 qh[NQ][KS], ql[NQ][SPL && !C::QLDS ? KS : 1];
    _Float16 *const qlw = qlo + (32 * NQ * wq + r32) * RS + 8 * h;
#pragma unroll
    for (int t = 0; t < NQ; ++t) {
        float x[D / 2];
        const int n = q0 + 32 * t + r32;
        load_cols<T, D>(q, n, N, x);
        standardise_cols<D>(x, n < N, qs * C::QKS);
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            h8 lo;
            split8<SPL>(x + 8 * ks, qh[t][ks], lo);
            if constexpr (C::QLDS) {
                if (wk == 0) *(h8 *)(qlw + 32 * t * RS + 16 * ks) = lo;
            } else {
                ql[t][SPL ? ks : 0] = lo;
            }
        }
    }

    // staging: this thread's 8 channels and first token
    const int sc = tid % LPT, st0 = tid / LPT;
    RawRow<T, 8> kr[C::KP ? 1 : C::NP], vr[C::NP];
    RawRow<bf16_t, 8> kph[C::KP ? C::NP : 1];   // fp16 words
    auto load_tile = [&](int t) {
#pragma unroll
        for (int p = 0; p < C::NP; ++p) {
            // rows past the end repeat the last one: their weights are masked
            const unsigned n = (unsigned)min(t * C::BK + st0 + C::TPP * p, N - 1);
            const unsigned off = n * (unsigned)D + 8u * sc;
            if constexpr (C::KP) {
                kph[p].load((const bf16_t *)khat + off, true);
            } else {
                kr[p].load(k + off, true);
            }
            vr[p].load(v + off, true);
        }
    };
    float vmax = 0.f;
    auto raw_max = [&]() {
#pragma unroll
        for (int p = 0; p < C::NP; ++p)
#pragma unroll
            for (int i = 0; i < 8; ++i) vmax = fmaxf(vmax, fabsf(vr[p].get(i)));
    };
    // per column group: the scale that puts the largest m below 2^top
    auto set_scale = [&](float m, int top) {
        if (tid < LPT) smax[tid] = 0u;
        __syncthreads();
        atomicMax(&smax[sc], __float_as_uint(m));
        __syncthreads();
        const float s = pow2_scale(__uint_as_float(smax[sc]), top);
        if (tid < LPT) sscale[tid] = s;
        return s;
    };

    load_tile(0);
    float vscale = 1.0f;
    if constexpr (!SPL) {
        raw_max();
        vscale = set_scale(vmax <= 3e38f ? vmax : 0.f, 7);
    }

    f16v acc[NQ][CT];
    float rs[NQ];
    // One 32-key tile j of the staged step against the wave's queries; masked:
    // some of its pairs lie beyond the diagonal or the last key.
    auto tile = [&](int j, int kb, bool masked) {
        f16v s[NQ];
#pragma unroll
        for (int u = 0; u < NQ; ++u)
#pragma unroll
            for (int i = 0; i < 16; ++i) s[u][i] = SPL ? 0.0f : 1.0f;
        const _Float16 *kp = khi + (32 * j + r32) * RS + 8 * h;
        // the products with a lo part first, while the sum is small (at
        // D = 128 side by side with the main ones: fewer live operands)
        if constexpr (SPL && D < 128) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                const h8 a = ld8(kp + 16 * ks), b = ld8(kp + C::KH + 16 * ks);
#pragma unroll
                for (int u = 0; u < NQ; ++u) {
                    if constexpr (F32) s[u] = mma(b, ql[u][C::QLDS ? 0 : ks], s[u]);
                    s[u] = mma(a, ql[u][C::QLDS ? 0 : ks], s[u]);
                    s[u] = mma(b, qh[u][ks], s[u]);
                }
            }
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const h8 a = ld8(kp + 16 * ks);
            if constexpr (SPL && D >= 128) {
                const h8 b = ld8(kp + C::KH + 16 * ks);
#pragma unroll
                for (int u = 0; u < NQ; ++u) {
                    const h8 lo = ld8(qlw + 32 * u * RS + 16 * ks);
                    if constexpr (F32) s[u] = mma(b, lo, s[u]);
                    s[u] = mma(a, lo, s[u]);
                    s[u] = mma(b, qh[u][ks], s[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < NQ; ++u) s[u] = mma(a, qh[u][ks], s[u]);
        }
        // weights 2 f_2 = (1 + s)^2 + 1 (the factor 2 cancels in F / G and is
        // taken out of G)
        h8 wh[SPL ? 1 : NQ][2], w3[SPL ? NQ : 1][2][3];
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
            const int qb0 = q0 + 32 * u;
            float w[16], z[F32 ? 16 : 1];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                if constexpr (F32) {
                    // 2 f_2 - 2 = s (s + 2): what G has beside its count of keys
                    const float x = s[u][i] * sc2;
                    z[i] = x * (x + 2.0f);
                    w[i] = z[i] + 2.0f;
                } else {
                    const float t = SPL ? fmaf(s[u][i], sc2, 1.0f) : s[u][i];
                    w[i] = fmaf(t, t, 1.0f);
                }
            }
            if (masked) {
                asm volatile("");   // a branch, not a compare and select per element of every tile
                const int last = C::CAUSAL ? qb0 + r32 : N - 1;
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    if (kb + 8 * (i / 4) + 4 * h + i % 4 > last) {
                        w[i] = 0.f;
                        if constexpr (F32) z[i] = 0.f;
                    }
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                h8 lo;
                if constexpr (SPL) split3(w + 8 * e, w3[u][e]);
                else split8<false>(w + 8 * e, wh[u][e], lo);
            }
            if constexpr (SPL) {
                float *const y = F32 ? z : w;
#pragma unroll
                for (int d = 8; d; d /= 2)
#pragma unroll
                    for (int i = 0; i < d; ++i) y[i] += y[i + d];
                rs[u] += y[0];
            } else {
                // the sum of the rounded weights, as the numerator takes them
                const h2 one = {(_Float16)1.0f, (_Float16)1.0f};
#pragma unroll
                for (int i = 0; i < 16; i += 2)
                    rs[u] = __builtin_amdgcn_fdot2(h2{wh[u][i / 8][i % 8], wh[u][i / 8][i % 8 + 1]},
                                                   one, rs[u], false);
            }
        }
        if constexpr (SPL) {
#pragma unroll
            for (int c = 0; c < CT; ++c) {
                h8 a[C::VP][2];
#pragma unroll
                for (int i = 0; i < C::VP; ++i)
#pragma unroll
                    for (int e = 0; e < 2; ++e) a[i][e] = ld_tr<VS>(vhi + i * C::VH, 32 * j + 16 * e, 32 * c);
#pragma unroll
                for (int u = 0; u < NQ; ++u) {
                    if constexpr (F32) {
                        acc[u][c] += mma33(a, w3[u]);
                    } else {
#pragma unroll
                        for (int o = 2; o >= 0; --o)
#pragma unroll
                            for (int e = 0; e < 2; ++e) acc[u][c] = mma_b(a[0][e], w3[u][e][o], acc[u][c]);
                    }
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int c = 0; c < CT; ++c) {
                    const h8 a = ld_tr<VS>(vhi, 32 * j + 16 * e, 32 * c);
#pragma unroll
                    for (int u = 0; u < NQ; ++u) acc[u][c] = mma(a, wh[u][e], acc[u][c]);
                }
        }
    };

    for (int attempt = 0;; ++attempt) {
#pragma unroll
        for (int t = 0; t < NQ; ++t) {
            rs[t] = 0.f;
#pragma unroll
            for (int c = 0; c < CT; ++c) acc[t][c] = f16v{};
        }
        for (int t = 0; t < nt; ++t) {
            __syncthreads();
#pragma unroll
            for (int p = 0; p < C::NP; ++p) {
                const int row = st0 + C::TPP * p;
                float y[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    y[i] = vr[p].get(i);
                    if constexpr (!SPL) {
                        vmax = fmaxf(vmax, fabsf(y[i]));
                        y[i] *= vscale;
                    }
                }
                h8 hi, lo;
                const bool ok = C::BK % C::TPP == 0 || row < C::BK;
                if constexpr (SPL && !F32) {
                    if (ok) *(uint4 *)(vhi + row * VS + 8 * sc) = *(uint4 *)vr[p].w;
                } else if constexpr (SPL) {
                    h8 y3[3];
                    split3(y, y3);
#pragma unroll
                    for (int i = 0; i < 3; ++i)
                        if (ok) *(h8 *)(vhi + i * C::VH + row * VS + 8 * sc) = y3[i];
                } else {
                    split8<false>(y, hi, lo);
                    if (ok) *(h8 *)(vhi + row * VS + 8 * sc) = hi;
                }
                if constexpr (C::KP) {
                    if (ok) *(uint4 *)(khi + row * RS + 8 * sc) = *(uint4 *)kph[p].w;
                } else {
                    float x[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) x[i] = kr[p].get(i);
                    standardise_group<D>(x, true, C::QKS);
                    split8<SPL>(x, hi, lo);
                    if (ok) {
                        *(h8 *)(khi + row * RS + 8 * sc) = hi;
                        if constexpr (SPL) *(h8 *)(klo + row * RS + 8 * sc) = lo;
                    }
                }
            }
            if (t + 1 < nt) load_tile(t + 1);
            __syncthreads();
#pragma unroll 1
            for (int j = wk; j < C::BK / 32; j += C::NWK) {
                const int kb = t * C::BK + 32 * j;
                if (kb >= N || (C::CAUSAL && kb > q0 + 32 * NQ - 1)) break;
                tile(j, kb, (C::CAUSAL && kb + 31 > q0) || kb + 32 > N);
            }
        }
        if (SPL || attempt || !__syncthreads_or(vmax * vscale > 65504.0f)) break;
        vscale = set_scale(largest_finite<T, D>(v, sc, st0, C::TPP, kend), 14);
        load_tile(0);
    }

    auto keys_of = [&](int n) { return C::CAUSAL ? n + 1 : N; };
    // O = F / G.  Where waves split the keys their partial sums meet in LDS
    // first, [wave][column][query], and each wave finishes a share of the
    // columns.
    if constexpr (C::NWK == 1) {
#pragma unroll
        for (int u = 0; u < NQ; ++u) {
            const int n = q0 + 32 * u + r32;
            const float G = half_sum(rs[u]) + (F32 ? 2.0f * (float)keys_of(n) : 0.f);
            if (n < N) {
                if (g && h == 0) g[(size_t)head * N + n] = 0.5f * G;
                const float r = 1.0f / G;
#pragma unroll
                for (int c = 0; c < CT; ++c)
#pragma unroll
                    for (int b = 0; b < 4; ++b) {
                        const int d = 32 * c + 8 * b + 4 * h;
                        if (D % 32 == 0 || d < D) {
                            const float f = SPL ? r : r / sscale[d / 8];
                            T *o = out + (size_t)n * D + d;
                            if constexpr (sizeof(T) == 2) {
                                *(uint2 *)o = make_uint2(
                                    mx::pack_bf16x2(acc[u][c][4 * b] * f, acc[u][c][4 * b + 1] * f),
                                    mx::pack_bf16x2(acc[u][c][4 * b + 2] * f, acc[u][c][4 * b + 3] * f));
                            } else {
                                *(float4 *)o = make_float4(acc[u][c][4 * b] * f, acc[u][c][4 * b + 1] * f,
                                                           acc[u][c][4 * b + 2] * f, acc[u][c][4 * b + 3] * f);
                            }
                        }
                    }
            }
        }
    } else {
        constexpr int W = 32 * CT + 1;   // columns and the row sum, 32 floats each
        float *red = (float *)smem;
        __syncthreads();
        float *mine = red + wave * 32 * W;
        const float G0 = half_sum(rs[0]);
        if (h == 0) mine[32 * 32 * CT + r32] = G0;
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int i = 0; i < 16; ++i)
                mine[32 * (32 * c + 8 * (i / 4) + 4 * h + i % 4) + r32] = acc[0][c][i];
        __syncthreads();
        const float *part = red + wq * C::NWK * 32 * W;
        float G = 0.f;
#pragma unroll
        for (int w = 0; w < C::NWK; ++w) G += part[w * 32 * W + 32 * 32 * CT + r32];
        const int n = q0 + r32;
        if constexpr (F32) G += 2.0f * (float)keys_of(n);
        if (n < N) {
            if (g && h == 0 && wk == 0) g[(size_t)head * N + n] = 0.5f * G;
            const float r = 1.0f / G;
            // columns of this wave and half wave, 4 at a time
#pragma unroll
            for (int d = 4 * (2 * wk + h); d < D; d += 8 * C::NWK) {
                const float f = SPL ? r : r / sscale[d / 8];
                float x[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    x[i] = 0.f;
#pragma unroll
                    for (int w = 0; w < C::NWK; ++w) x[i] += part[w * 32 * W + 32 * (d + i) + r32];
                    x[i] *= f;
                }
                T *o = out + (size_t)n * D + d;
                if constexpr (sizeof(T) == 2)
                    *(uint2 *)o = make_uint2(mx::pack_bf16x2(x[0], x[1]), mx::pack_bf16x2(x[2], x[3]));
                else *(float4 *)o = make_float4(x[0], x[1], x[2], x[3]);
            }
        }
    }
}

// k^ in fp16 for the kernel that reads each key from many workgroups: one
// thread per 8 channels.
template <typename T, int D>
__global__ __launch_bounds__(256) void khat_kernel(const T *__restrict__ k, _Float16 *__restrict__ khat,
                                                   long long rows)
{
    const long long row = ((long long)blockIdx.x * 256 + threadIdx.x) / (D / 8);
    const int c = threadIdx.x % (D / 8);
    const bool ok = row < rows;
    RawRow<T, 8> raw;
    raw.load(k + (size_t)(ok ? row : 0) * D + 8 * c, ok);
    float x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = raw.get(i);
    standardise_group<D>(x, ok);
    h8 hi, lo;
    split8<false>(x, hi, lo);
    if (ok) *(h8 *)(khat + (size_t)row * D + 8 * c) = hi;
}

// The workgroup shapes (queries per wave / 32, query columns, key columns of
// waves, keys per step; KP: k^ from khat_kernel) and what each measured on an
// MI355X: t = t0 + |(a N, b pairs)|_2 us, a (ns per key) one workgroup's pace
// down its keys, b (ps per pair) the chip's when full, fitted to calls of 1 to
// 96 heads of 256 to 8192 tokens (D = 16, 32 and float32 rows: 33 to 100000),
// causal (pairs = heads N (N + queries per workgroup) / 2; without the mask b is
// 0.85 to 0.95 of it).  Waves that split the keys shorten a, waves that share a
// staged tile lower b.  Against every shape and the moment kernels timed at 801
// sizes, up to 100000 tokens, the choice takes 1.01 to 1.06 times the best one's
// time on average; where it is on the wrong side of the line between pairs and
// moments, at most 1.34 times (1.42 at 22 us).
// fp16 operands: bf16, D = 64
constexpr Shape SH64[] = {{32, 5.f, 7.6f, 1.13f}, {64, 4.f, 9.6f, .68f}, {128, 5.f, 13.f, .455f},
                          {128, 4.f, 20.5f, .375f}, {256, 7.f, 17.f, .31f}, {512, 6.f, 31.f, .275f}};
// float32-grade operands, bf16 rows (SS64, whose calls have fewer than 128 keys,
// by an earlier form's paces; the others against 195 sizes: 1.00 to 1.02, 1.24 at most)
constexpr Shape SS16[] = {{32, 3.7f, 2.95f, .59f}, {64, 3.85f, 4.9f, .363f}, {256, 4.7f, 13.2f, .316f}};
constexpr Shape SS32[] = {{32, 3.8f, 4.1f, .75f}, {64, 4.f, 6.05f, .505f}, {256, 4.3f, 20.8f, .38f}};
constexpr Shape SS64[] = {{64, 6.f, 15.4f, 1.14f}, {128, 6.f, 21.2f, .82f}, {256, 6.f, 36.5f, .71f}};
constexpr Shape SS128[] = {{64, 7.8f, 23.f, 2.2f}, {128, 6.3f, 36.f, 1.55f}, {256, 5.7f, 47.7f, 1.47f}};
// float32 rows (bf16 triples for the values: 1.0 to 1.5 of the time that fp16
// pairs took, whose values depended on a shared scale)
constexpr Shape SF16[] = {{32, 4.5f, 4.1f, .68f}, {64, 4.4f, 7.9f, .575f}, {256, 3.8f, 27.f, .485f}};
constexpr Shape SF32[] = {{32, 5.5f, 5.6f, 1.1f}, {64, 5.2f, 9.f, .72f}, {256, 4.4f, 31.f, .59f}};
constexpr Shape SF64[] = {{64, 7.f, 16.1f, 1.5f}, {128, 6.6f, 28.6f, 1.19f}, {256, 5.9f, 54.5f, 1.06f}};
constexpr Shape SF128[] = {{64, 9.4f, 49.f, 3.6f}, {128, 10.9f, 53.f, 2.27f}, {256, 9.3f, 97.f, 1.99f}};

Moments moments_fwd(int BH, int N, int D, int causal, bool grade32)
{
    // the causal scan cut into many segments
    if (!grade32 && causal)
        if (const int S = causal_multi_segments(BH, N)) return {40.f, 0.f, 83.f / S, 0.f};
    if (!grade32 && causal) return {12.f, 0.f, 50.f, .95f};
    if (!grade32) return {25.f, .5f, 5.5f, .87f};
    switch (D) {
    case 16: return causal ? Moments{14.f, .07f, 1.9f, .46f} : Moments{14.f, .14f, 1.9f, .31f};
    case 32: return causal ? Moments{16.f, .36f, 2.5f, 1.8f} : Moments{17.f, .55f, 2.5f, 1.21f};
    case 64: return causal ? Moments{30.f, .63f, 9.1f, 9.8f} : Moments{30.f, 2.1f, 6.f, 6.6f};
    default: return causal ? Moments{30.f, 0.f, 81.f, 50.f} : Moments{35.f, 0.f, 57.f, 53.f};
    }
}

template <typename C>
hipError_t launch_fwd(const void *q, const void *k, const void *v, void *out, float *g, int BH,
                      int N, float qs, void *ws, hipStream_t st)
{
    typedef typename C::T T;
    const int nqb = (N + C::QB - 1) / C::QB;
    const int hgrp = BH < 32 ? BH : 32;
    const long long rows = (long long)BH * N, pb = (rows * (C::D / 8) + 255) / 256;
    if (!grid_fits((long long)BH * nqb, C::NTH) || (C::KP && !grid_fits(pb, 256)))
        return hipErrorInvalidConfiguration;
    // float32-grade scores: q^ carries tau's mantissa, its power of two
    // follows the sum (a small tau would push the lo parts below fp16's range)
    int e = 0;
    if (C::SPL) frexpf(qs, &e);
    const float sc2 = C::SPL ? ldexpf(1.0f, e - 1) : 1.0f;
    _Float16 *khat = (_Float16 *)ws;
    if (C::KP)
        hipLaunchKernelGGL((khat_kernel<T, C::D>), dim3((unsigned)pb), dim3(256), 0, st, (const T *)k,
                           khat, rows);
    hipLaunchKernelGGL((fwd_kernel<C>), dim3((unsigned)((long long)BH * nqb)), dim3(C::NTH), 0, st,
                       (const T *)q, (const T *)k, (const T *)v, khat, (T *)out, g, N, BH, nqb, hgrp,
                       qs / sc2, sc2 / (C::QKS * C::QKS));
    return hipGetLastError();
}

template <typename T, int D, bool CAUSAL, bool SPL>
hipError_t launch_shape(const void *q, const void *k, const void *v, void *out, float *g, int BH,
                        int N, float qs, int shape, void *ws, hipStream_t st)
{
#define L(KP, NQ, NWQ, NWK, BK)                                                                    \
    do {                                                                                           \
        typedef FwdCfg<T, D, CAUSAL, SPL, KP, NQ, NWQ, NWK, BK> C;                              \
        static_assert(C::QB == S.qb, "table");                                                     \
        return launch_fwd<C>(q, k, v, out, g, BH, N, qs, ws, st);                                  \
    } while (0)
    constexpr bool F32 = sizeof(T) == 4;
    if constexpr (D <= 32) {
        constexpr const Shape *const X = D == 16 ? (F32 ? SF16 : SS16) : F32 ? SF32 : SS32;
        if (shape == 0) { constexpr Shape S = X[0]; L(false, 1, 1, 8, 256); }
        if (shape == 1) { constexpr Shape S = X[1]; L(false, 1, 2, 4, 128); }
        if (shape == 2) { constexpr Shape S = X[2]; L(false, 1, 8, 1, 128); }
    } else if constexpr (D == 64 && !SPL) {
        if (shape == 0) { constexpr Shape S = SH64[0]; L(false, 1, 1, 8, 256); }
        if (shape == 1) { constexpr Shape S = SH64[1]; L(false, 1, 2, 4, 128); }
        if (shape == 2) { constexpr Shape S = SH64[2]; L(false, 1, 4, 2, 128); }
        if (shape == 3) { constexpr Shape S = SH64[3]; L(false, 1, 4, 1, 64); }
        if (shape == 4) { constexpr Shape S = SH64[4]; L(true, 1, 8, 1, 128); }
        if (shape == 5) { constexpr Shape S = SH64[5]; L(false, 2, 8, 1, 128); }
    } else if constexpr (D == 64) {
        constexpr const Shape *const X = F32 ? SF64 : SS64;
        if (shape == 0) { constexpr Shape S = X[0]; L(false, 1, 2, 4, 128); }
        if (shape == 1) { constexpr Shape S = X[1]; L(false, 1, 4, 2, 64); }
        if (shape == 2) { constexpr Shape S = X[2]; L(false, 1, 8, 1, 64); }
    } else if constexpr (sizeof(T) == 2) {
        if (shape == 0) { constexpr Shape S = SS128[0]; L(false, 1, 2, 4, 128); }
        if (shape == 1) { constexpr Shape S = SS128[1]; L(false, 1, 4, 2, 64); }
        if (shape == 2) { constexpr Shape S = SS128[2]; L(false, 1, 8, 1, 64); }
    } else {
        if (shape == 0) { constexpr Shape S = SF128[0]; L(false, 1, 2, 2, 64); }
        if (shape == 1) { constexpr Shape S = SF128[1]; L(false, 1, 4, 2, 64); }
        if (shape == 2) { constexpr Shape S = SF128[2]; L(false, 1, 8, 1, 32); }
    }
#undef L
    return hipErrorInvalidValue;
}

}  // namespace pr

int pairs_fwd_plan(int BH, int N, int D, int p, int causal, int is_bf16, size_t ws_bytes)
{
    using namespace pr;
    if (p != 2) return -1;
    const bool grade32 = pairs_grade32(N, D, causal, is_bf16);
    const Moments m = moments_fwd(BH, N, D, causal, grade32);
    switch (D) {
    case 16: return pick(is_bf16 ? SS16 : SF16, 3, m, BH, N, causal, 1);
    case 32: return pick(is_bf16 ? SS32 : SF32, 3, m, BH, N, causal, 1);
    case 64:
        if (grade32) return pick(is_bf16 ? SS64 : SF64, 3, m, BH, N, causal, 1);
        // shape 4 keeps k^ in the workspace
        return pick(SH64, 6, m, BH, N, causal, 1, ws_bytes < (size_t)BH * N * 128 ? 4 : -1);
    case 128: return is_bf16 ? pick(SS128, 3, m, BH, N, causal, 1) : pick(SF128, 3, m, BH, N, causal, 1);
    }
    return -1;
}

hipError_t pairs_fwd(const void *q, const void *k, const void *v, void *out, float *g, int BH,
                     int N, int D, int causal, int is_bf16, float qs, int shape, void *ws,
                     hipStream_t st)
{
#define GO(T, DD, CA, SPL) return pr::launch_shape<T, DD, CA, SPL>(q, k, v, out, g, BH, N, qs, shape, ws, st)
#define GO2(T, DD)                                                                                 \
    do {                                                                                           \
        if (causal) GO(T, DD, true, true);                                                         \
        GO(T, DD, false, true);                                                                    \
    } while (0)
    if (is_bf16) {
        switch (D) {
        case 16: GO2(bf16_t, 16);
        case 32: GO2(bf16_t, 32);
        case 64:
            if (causal) GO(bf16_t, 64, true, false);
            if (pairs_grade32(N, D, causal, is_bf16)) GO(bf16_t, 64, false, true);
            GO(bf16_t, 64, false, false);
        case 128: GO2(bf16_t, 128);
        }
    } else {
        switch (D) {
        case 16: GO2(float, 16);
        case 32: GO2(float, 32);
        case 64: GO2(float, 64);
        case 128: GO2(float, 128);
        }
    }
#undef GO2
#undef GO
    return hipErrorInvalidValue;
}

}  // namespace fm
