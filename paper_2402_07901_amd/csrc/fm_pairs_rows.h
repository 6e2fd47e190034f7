// What the backwards prepare per row.  fp16 operands (fm_pairs_bwd.hip): the
// planes of q~, k^, v and dO, delta = dO.O, and the powers of two of dO, v and
// dO / G.  The others: at the end.
#pragma once

#include <type_traits>

#include "fm_internal.h"
#include "fm_pairs.h"

namespace fm {
namespace pr {

// Exponents of zero and non-finite rows: they take no part in a maximum.
constexpr int NO_EXP = -1000;

// Least e with m < 2^e for finite m > 0.
__device__ __forceinline__ int exp_above(float m)
{
    const int x = (int)(__float_as_uint(m) >> 23);
    return m > 0.f && x < 255 ? x - 126 : NO_EXP;
}

__device__ __forceinline__ float exp2i(int n)
{
    n = n < -126 ? -126 : (n > 127 ? 127 : n);
    return __uint_as_float((uint32_t)(n + 127) << 23);
}

__device__ __forceinline__ int g_exp(float G) { return (int)((__float_as_uint(G) >> 23) & 255) - 127; }

template <int L>
__device__ __forceinline__ float group_max(float x)
{
    auto mv = [](float y, auto ctl) {
        return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(y), decltype(ctl)::value, 0xF, 0xF, true));
    };
    x = fmaxf(x, mv(x, std::integral_constant<int, 0xB1>{}));
    if constexpr (L >= 4) x = fmaxf(x, mv(x, std::integral_constant<int, 0x4E>{}));
    if constexpr (L >= 8) x = fmaxf(x, mv(x, std::integral_constant<int, 0x141>{}));
    if constexpr (L >= 16) x = fmaxf(x, mv(x, std::integral_constant<int, 0x140>{}));
    return x;
}

// The per-row words of the fp16 calls, which keep v, dO and dO rho as fp16
// planes, each row scaled by a power of two to below 2^10, so that a step
// stages them with one packed multiply per pair: delta in dO's scale, rho, and
// the exponents of dO, v and dO / G.
struct RowInfoH {
    float delta, rho;
    short e_do, e_v;
    int eg;
};
static_assert(sizeof(RowInfoH) == 16, "bytes per row");

// 2^n as a half, flushed to zero below its range (n at most 15).
__device__ __forceinline__ _Float16 half2i(int n) { return n < -24 ? (_Float16)0.0f : (_Float16)exp2i(n); }

// One thread per 8 channels of a row of the whole call.
template <typename T, int D>
__global__ __launch_bounds__(256) void bwd_prep_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ v,
    const T *__restrict__ o, const T *__restrict__ dout, const float *__restrict__ g,
    _Float16 *__restrict__ planes, RowInfoH *__restrict__ info, long long rows, float tau)
{
    constexpr int L = D / 8;
    const long long row = ((long long)blockIdx.x * 256 + threadIdx.x) / L;
    const int c = threadIdx.x % L;
    const bool ok = row < rows;
    const size_t off = (size_t)(ok ? row : 0) * D + 8 * c, np = (size_t)rows * D;
    RawRow<T, 8> rq, rk, rv, ro, rd;
    rq.load(q + off, ok);
    rk.load(k + off, ok);
    rv.load(v + off, ok);
    ro.load(o + off, ok);
    rd.load(dout + off, ok);
    float x[8];
    h8 hi, lo;
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = rq.get(i);
    standardise_group<D>(x, ok);
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] *= tau;
    split8<false>(x, hi, lo);
    if (ok) *(h8 *)(planes + off) = hi;
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = rk.get(i);
    standardise_group<D>(x, ok);
    split8<false>(x, hi, lo);
    if (ok) *(h8 *)(planes + np + off) = hi;
    float d = 0.f, md = 0.f, mv = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        d = fmaf(rd.get(i), ro.get(i), d);
        md = fmaxf(md, fabsf(rd.get(i)));
        mv = fmaxf(mv, fabsf(rv.get(i)));
    }
    d = group_sum<L>(d);
    md = group_max<L>(md);
    mv = group_max<L>(mv);
    const int ed = exp_above(md), ev = exp_above(mv);
    const int e = ed == NO_EXP ? 0 : ed;
    const float G = g[ok ? row : 0];
    const int kx = g_exp(G);
    const float rho = exp2i(kx) / G, fd = exp2i(10 - e), fv = exp2i(10 - (ev == NO_EXP ? 0 : ev));
    float y[8], z[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        x[i] = rv.get(i) * fv;
        y[i] = rd.get(i) * fd;
        z[i] = y[i] * rho;
    }
    if (ok) {
        split8<false>(x, hi, lo);
        *(h8 *)(planes + 2 * np + off) = hi;
        split8<false>(y, hi, lo);
        *(h8 *)(planes + 3 * np + off) = hi;
        split8<false>(z, hi, lo);
        *(h8 *)(planes + 4 * np + off) = hi;
        if (c == 0)
            info[row] = RowInfoH{d * fd, rho, (short)ed, (short)ev, ed == NO_EXP ? NO_EXP : ed - kx};
    }
}

// What the backwards without shared scales (fm_pairs_bwd32.hip, fm_linear.hip)
// keep per row: q~ = (q - mq) rq (tau in rq), k^ = (k - mk) rk, delta = dO.O,
// u = 1 / G.
struct Row32 {
    float mq, rq, mk, rk, delta, u;
};
static_assert(sizeof(Row32) == ROW32_BYTES, "bytes per row");

// Mean and 1 / std (Sec. 2.2, Eqs. 6-7) of the row whose 8 channels a lane holds.
template <typename T, int D>
__device__ __forceinline__ float2 row_stats(const RawRow<T, 8> &raw)
{
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) s += raw.get(i);
    const float mu = group_sum<D / 8>(s) * (1.0f / D);
    float v = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float x = raw.get(i) - mu;
        v = fmaf(x, x, v);
    }
    return make_float2(mu, rsqrt1(group_sum<D / 8>(v) * (1.0f / D)));
}

// One thread per 8 channels of a row of the whole call.
template <typename T, int D>
__global__ __launch_bounds__(256) void bwd32_prep_kernel(
    const T *__restrict__ q, const T *__restrict__ k, const T *__restrict__ o,
    const T *__restrict__ dout, const float *__restrict__ g, Row32 *__restrict__ info,
    long long rows, float tau)
{
    constexpr int L = D / 8;
    const long long row = ((long long)blockIdx.x * 256 + threadIdx.x) / L;
    const int c = threadIdx.x % L;
    const bool ok = row < rows;
    const size_t off = (size_t)(ok ? row : 0) * D + 8 * c;
    RawRow<T, 8> rq, rk, ro, rd;
    rq.load(q + off, ok);
    rk.load(k + off, ok);
    ro.load(o + off, ok);
    rd.load(dout + off, ok);
    float d = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) d = fmaf(rd.get(i), ro.get(i), d);
    d = group_sum<L>(d);
    const float2 a = row_stats<T, D>(rq), b = row_stats<T, D>(rk);
    if (ok && c == 0) info[row] = Row32{a.x, a.y * tau, b.x, b.y, d, 1.0f / g[row]};
}

}  // namespace pr
}  // namespace fm
