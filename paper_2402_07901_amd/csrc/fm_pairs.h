// Shared pieces of the pair kernels (fm_pairs_fwd.hip, fm_pairs_bwd.hip,
// fm_pairs_bwd32.hip):
// Fastmax evaluated over explicit (query, key) pairs, 32 x 32 at a time in
// registers, for sequences short enough that a pair costs less than its share
// of the moments (Sec. 2.4's factorisation pays once N exceeds about D^2; the
// rules at each launcher state the measured lines).  The weights
// f_p(q^.k^) never leave the registers.
//
// v_mfma_f32_32x32x16_f16 lane layout (lane = 32h + r): A holds row r, K
// indices 8h..8h+7; B holds column r, the same K indices; accumulator element
// i holds column r, row 8(i/4) + 4h + i%4.  Scores are formed as
// S^T = K^ Q^T (rows keys, columns queries), so the weights of a 32-key tile
// are, element for element, the B operands of two 16-key contraction steps
// once the keys of a step are numbered K index 8h + r <-> key
// 8(r/4) + 4h + r%4: nothing moves between lanes.  The A operand of that
// contraction (16 keys of a value column) is read from the row-major tile by
// ds_read_b64_tr_b16, which hands lane i of 16 the column i of a 4 x 16 block.
//
// float32-grade operands.  The standardised q^ and k^ and the weights, whose
// range is known, are held as two fp16 numbers hi + lo, a product takes three
// MFMAs (hi hi, lo hi, hi lo); the forward multiplies q^ and k^ by 2^8 each,
// which keeps lo out of fp16's subnormals (24 bits, not 22; the scores' 2^16
// goes into the factor that they are read with).  Values have no known
// range: fp16 numbers under a shared scale lose what lies far below the
// scale's largest value, even if a row or column never meets that value.
// float32 values are held as three bf16 numbers, which take a float32 apart
// into 8 + 8 + 8 bits: every bit of every exponent, no scale; the weights meet
// them in the same form and a product takes six MFMAs (the other three of nine
// are 2^-26 of it and less).  bf16 values are one such plane: three MFMAs.
//
// fp16 operands (bf16 rows, D = 64, causal or at least 128 tokens): one plane
// each, the values under a power-of-two scale per 8-column group.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "fm_common.h"
#include "fm_internal.h"
#include "fm_f32_mfma.h"
#include "fm_mfma.h"

namespace fm {
namespace pr {

using m32::RawRow;
using mx::cat;
using mx::h2;
using mx::h4;
using mx::h8;
using mx::ld8;
using mx::static_for;
typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef short s4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f16v mma(h8 a, h8 b, f16v c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// Operands that hold bf16 numbers (words of the same h8).
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ f16v mma_b(h8 a, h8 b, f16v c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(b8, a), __builtin_bit_cast(b8, b), c, 0, 0, 0);
}

// Two floats to two halves, round to nearest even.
__device__ __forceinline__ h2 cvt2(float a, float b)
{
    return __builtin_convertvector((f2{a, b}), h2);
}

// x - (float)h
__device__ __forceinline__ float rest(float x, _Float16 h) { return fmaf((float)h, -1.0f, x); }

// Row strides (halves) of the staged tiles.  Rows read 16 bytes per lane,
// one row per lane (scores): D + 8, which puts 16 consecutive rows on 16
// distinct groups of four banks.  Rows read through the transposing load
// (values): a stride of 16 banks modulo 32, so that the four rows of a block
// fall on distinct banks.
template <int D> constexpr int row_stride() { return D + 8; }
template <int D> constexpr int tr_stride() { return D <= 32 ? 32 : D + 32; }

// The A operand of a 16-key contraction step: keys key0 + {0..15} (numbered
// as above) of columns col0..col0+31 of a row-major tile of row stride S.
template <int S>
__device__ __forceinline__ h8 ld_tr(const _Float16 *tile, int key0, int col0)
{
    typedef s4v __attribute__((address_space(3))) *lp;
    const int lane = threadIdx.x & 63, h = lane >> 5, g = (lane >> 4) & 1, j = (lane >> 2) & 3, c = lane & 3;
    const _Float16 *p = tile + (key0 + 4 * h + j) * S + col0 + 16 * g + 4 * c;
    const s4v a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)p);
    const s4v b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lp)(p + 8 * S));
    return cat(__builtin_bit_cast(h4, a), __builtin_bit_cast(h4, b));
}

// Sum over an aligned group of L = 2, 4, 8 or 16 lanes, in every lane, with
// DPP moves.
template <int L>
__device__ __forceinline__ float group_sum(float x)
{
    static_assert(L == 2 || L == 4 || L == 8 || L == 16, "lanes per token");
    x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, true));
    if constexpr (L >= 4)
        x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xF, 0xF, true));
    if constexpr (L >= 8)
        x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xF, 0xF, true));
    if constexpr (L >= 16)
        x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x140, 0xF, 0xF, true));
    return x;
}

// Sum of a lane's and its partner's (lane ^ 32) values, in both.
__device__ __forceinline__ float half_sum(float x)
{
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Eight floats as fp16 hi and (SPL) lo parts.
template <bool SPL>
__device__ __forceinline__ void split8(const float *x, h8 &hi, h8 &lo)
{
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
        const h2 a = cvt2(x[i], x[i + 1]);
        hi[i] = a[0];
        hi[i + 1] = a[1];
        if constexpr (SPL) {
            const h2 b = cvt2(rest(x[i], a[0]), rest(x[i + 1], a[1]));
            lo[i] = b[0];
            lo[i + 1] = b[1];
        }
    }
}

// Eight floats as three bf16 parts, each the rest of the ones before it rounded
// to nearest: they add up to the float, and a part is at most 2^-9 of the one
// before it.
typedef __bf16 b2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split3(const float *x, h8 (&p)[3])
{
    uint4 w[3];
    uint32_t *const o[3] = {(uint32_t *)&w[0], (uint32_t *)&w[1], (uint32_t *)&w[2]};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float a = x[2 * i], b = x[2 * i + 1];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const uint32_t u = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2{a, b}), b2));
            o[j][i] = u;
            if (j < 2) {
                a -= __uint_as_float(u << 16);
                b -= __uint_as_float(u & 0xffff0000u);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < 3; ++j) p[j] = __builtin_bit_cast(h8, w[j]);
}

// The products of two such operands over 32 rows (two K steps e).  The matrix
// pipe cuts its sums toward zero: the leading products, 16 bits each, are summed
// on their own, where little is cut, the others (2^-8 of them and less) apart,
// and the two meet in a rounded add.
__device__ __forceinline__ f16v mma33(const h8 (&a)[3][2], const h8 (&b)[2][3])
{
    f16v y = f16v{}, z = f16v{};
#pragma unroll
    for (int o = 2; o >= 0; --o)
#pragma unroll
        for (int i = 0; i <= o; ++i)
#pragma unroll
            for (int e = 0; e < 2; ++e) (o ? y : z) = mma_b(a[i][e], b[e][o - i], o ? y : z);
    return y + z;
}

// Rows x columns of two triples, the staged one read by rows from its planes.
// SEP: the leading products apart, as mma33; else one chain.
template <int KS, bool SEP = true>
__device__ __forceinline__ f16v dot33(const _Float16 *p, int plane, const h8 (&o)[KS][3])
{
    f16v y = f16v{}, z = f16v{};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const h8 a0 = ld8(p + 16 * ks), a1 = ld8(p + plane + 16 * ks), a2 = ld8(p + 2 * plane + 16 * ks);
        y = mma_b(a2, o[ks][0], y);
        y = mma_b(a1, o[ks][1], y);
        y = mma_b(a0, o[ks][2], y);
        y = mma_b(a1, o[ks][0], y);
        y = mma_b(a0, o[ks][1], y);
        if constexpr (SEP) z = mma_b(a0, o[ks][0], z);
        else y = mma_b(a0, o[ks][0], y);
    }
    if constexpr (SEP) return y + z;
    return y;
}

// 1 / sqrt(v): the hardware's approximation (1 ulp) with one Newton step, so
// that a row's scale is no larger an error than its elements' rounding.
__device__ __forceinline__ float rsqrt1(float v)
{
    const float r = __builtin_amdgcn_rsqf(v);
    return fmaf(0.5f * r, fmaf(-v * r, r, 1.0f), r);
}

// Standardises the 8 channels a lane holds of a token (Sec. 2.2, Eqs. 6-7:
// population std, no epsilon; the token's D/8 lanes are an aligned group) in
// place, times scale.  Every lane of the wave takes part.
template <int D>
__device__ __forceinline__ void standardise_group(float (&x)[8], bool valid, float scale = 1.0f)
{
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) s += x[i];
    const float mu = group_sum<D / 8>(s) * (1.0f / D);
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        x[i] -= mu;
        v = fmaf(x[i], x[i], v);
    }
    const float r = valid ? rsqrt1(group_sum<D / 8>(v) * (1.0f / D)) * scale : 0.0f;
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] *= r;
}

// The B operands of a row-major matrix whose rows are this wave's 32 columns
// (queries or keys): lane (r, h) loads channels 16 ks + 8h .. + 7 of row r.
template <typename T, int D>
__device__ __forceinline__ void load_cols(const T *rows, int n, int N, float (&x)[D / 2])
{
    const int h = (threadIdx.x >> 5) & 1;
    const bool valid = n < N;
    RawRow<T, 8> raw[D / 16];
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks)
        raw[ks].load(rows + (size_t)(valid ? n : 0) * D + 16 * ks + 8 * h, valid);
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks)
#pragma unroll
        for (int i = 0; i < 8; ++i) x[8 * ks + i] = raw[ks].get(i);
}

// Standardises such rows (the two half lanes of a column hold its channels)
// and scales them.
template <int D>
__device__ __forceinline__ void standardise_cols(float (&x)[D / 2], bool valid, float scale)
{
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < D / 2; ++i) s += x[i];
    const float mu = half_sum(s) * (1.0f / D);
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < D / 2; ++i) {
        x[i] -= mu;
        v = fmaf(x[i], x[i], v);
    }
    const float r = valid ? rsqrt1(half_sum(v) * (1.0f / D)) * scale : 0.0f;
#pragma unroll
    for (int i = 0; i < D / 2; ++i) x[i] *= r;
}

// A column's D values as a wave holds them: tile c, element i is channel
// 32 c + 8 (i / 4) + 4 h + i % 4, both halves of the wave together all D.
// The standardisation backward in place: dx = (dx^ - mean dx^ - x^ mean(dx^ x^))
// / sigma (Eqs. 6-7), x the raw row.
template <typename T, int D, int CT>
__device__ __forceinline__ void standardise_back(const T *__restrict__ xrow, f16v (&acc)[CT])
{
    const int h = (threadIdx.x >> 5) & 1;
    float x[CT][16], sum = 0.f;
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int dd = 32 * c + 8 * b + 4 * h;
            const bool in = D % 32 == 0 || dd < D;
            RawRow<T, 4> raw;
            raw.load(xrow + (in ? dd : 0), in);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x[c][4 * b + i] = raw.get(i);
                sum += x[c][4 * b + i];
            }
        }
    const float mu = half_sum(sum) * (1.0f / D);
    float var = 0.f, m1 = 0.f, m2 = 0.f;
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            if (D % 32 == 0 || 32 * c + 8 * (i / 4) + 4 * h < D) {
                x[c][i] -= mu;
                var = fmaf(x[c][i], x[c][i], var);
                m1 += acc[c][i];
                m2 = fmaf(acc[c][i], x[c][i], m2);
            }
        }
    const float r = rsqrt1(half_sum(var) * (1.0f / D));
    m1 = half_sum(m1) * (1.0f / D);
    m2 = half_sum(m2) * (1.0f / D) * r * r;
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[c][i] = (acc[c][i] - m1 - x[c][i] * m2) * r;
}

// Stores such a column as a row of D channels.
template <typename T, int D, int CT>
__device__ __forceinline__ void store_col(T *__restrict__ out, const f16v (&acc)[CT])
{
    const int h = (threadIdx.x >> 5) & 1;
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int dd = 32 * c + 8 * b + 4 * h;
            if (D % 32 == 0 || dd < D) {
                if constexpr (sizeof(T) == 2)
                    *(uint2 *)(out + dd) = make_uint2(mx::pack_bf16x2(acc[c][4 * b], acc[c][4 * b + 1]),
                                                      mx::pack_bf16x2(acc[c][4 * b + 2], acc[c][4 * b + 3]));
                else
                    *(float4 *)(out + dd) =
                        make_float4(acc[c][4 * b], acc[c][4 * b + 1], acc[c][4 * b + 2], acc[c][4 * b + 3]);
            }
        }
}

// Power of two 2^(top - e), 2^e the least power of two above m (m finite,
// >= 0): values up to m scaled by it stay below 2^top.  The result and its
// inverse are normal numbers; for m = 0 it is the largest, 2^126.
__device__ __forceinline__ float pow2_scale(float m, int top)
{
    int e = (int)(__float_as_uint(m) >> 23) - 126;   // m < 2^e
    int x = top - e + 127;
    x = x < 1 ? 1 : (x > 253 ? 253 : x);
    return __uint_as_float((uint32_t)x << 23);
}

// The largest finite magnitude of 8 channels (the c-th group) of rows n0, n0 +
// step, .. below end: a value scale's second attempt.
template <typename T, int D>
__device__ __forceinline__ float largest_finite(const T *__restrict__ rows, int c, int n0, int step, int end)
{
    float m = 0.f;
    for (int n = n0; n < end; n += step) {
        RawRow<T, 8> x;
        x.load(rows + (size_t)n * D + 8 * c, true);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float y = fabsf(x.get(i));
            if (y <= 3.4028235e38f) m = fmaxf(m, y);
        }
    }
    return m;
}

// A workgroup shape: queries (keys) per workgroup and its paces, and the
// moment kernels' t = t0 + h heads + max(a N, b heads N) us (a and b in ns per
// token).
struct Shape {
    int qb;
    float t0, a, b;
};
struct Moments {
    float t0, h, a, b;
};

// The fastest shape whose grid fits the dispatch limits (kinds workgroups of at
// most 512 threads per block of queries), or -1 where the moment kernels are
// faster (by 3% at least: near the line the rule stays with them) or no shape
// fits.  skip: a shape left out.
inline int pick(const Shape *s, int n, const Moments &m, int BH, int N, int causal, int kinds, int skip = -1)
{
    const double tok = (double)N;
    const double mtok = std::max(tok, 128.0);   // their chunk
    double best = 0.97 * (m.t0 + m.h * BH + 1e-3 * std::max(m.a * mtok, m.b * mtok * BH));
    int shape = -1;
    for (int i = 0; i < n; ++i) {
        if (i == skip || !grid_fits((long long)kinds * BH * ((N - 1) / s[i].qb + 1), 512)) continue;
        const double pairs = causal ? 0.5 * BH * tok * (tok + s[i].qb) : 0.95 * BH * tok * tok;
        const double t = s[i].t0 + std::hypot(1e-3 * s[i].a * tok, 1e-6 * s[i].b * pairs);
        if (t < best) {
            best = t;
            shape = i;
        }
    }
    return shape;
}

}  // namespace pr

// float32-grade operands, as the float32 moment kernels have, wherever the
// fp16 ones do not serve a call: they take bf16 at D = 64, without the mask
// from 128 keys up (with fewer, rounding the operands shows in G).
inline bool pairs_grade32(int N, int D, int causal, int is_bf16)
{
    return !(is_bf16 && D == 64 && (causal || N >= 128));
}

}  // namespace fm
