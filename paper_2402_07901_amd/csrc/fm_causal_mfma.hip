// Causal Fastmax forward on CDNA4 MFMA, head dimension 64, p = 2, bf16 I/O:
// the launches around the scan of fm_causal_scan.h (its header describes the
// scan), and the standardisation of q and k that precedes it.
#include <hip/hip_runtime.h>

#include <limits.h>

#include <algorithm>
#include <atomic>

#include "fm_causal_scan.h"
#include "fm_common.h"
#include "fm_internal.h"
#include "fm_mfma.h"

namespace fm {
namespace mfma_causal {

using namespace mx;

__global__ __launch_bounds__(NTH, 2) void fwd_causal_kernel(const _Float16 *__restrict__ q,
                                                            const _Float16 *__restrict__ k,
                                                            const bf16_t *__restrict__ v,
                                                            bf16_t *__restrict__ out,
                                                            float *__restrict__ g, int N, int BH,
                                                            SegArgs sa)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    Smem &sm = *reinterpret_cast<Smem *>(smem_raw);
    scan_block<false>(sm, q, k, v, out, g, nullptr, N, BH, blockIdx.x, BH * NSL, sa);
}

// The build (MULTI = 1) and the scan (2) of a sequence cut into many segments.
template <int MULTI>
__global__ __launch_bounds__(NTH, 2) void multi_kernel(const bf16_t *__restrict__ q,
                                                       const _Float16 *__restrict__ k,
                                                       const bf16_t *__restrict__ v,
                                                       bf16_t *__restrict__ out,
                                                       float *__restrict__ g, int N, int BH,
                                                       SegArgs sa)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    Smem &sm = *reinterpret_cast<Smem *>(smem_raw);
    scan_block<false, MULTI>(sm, (const _Float16 *)q, k, v, out, g, nullptr, N, BH, blockIdx.x,
                             BH * NSL, sa);
}

// Summaries of segments 1 .. nseg - 1 as left by the build (each its
// predecessor's sums) -> prefixes, in place: one thread per 4-byte word (two
// state halves, or one float), summed in float32.
__global__ __launch_bounds__(256) void seg_prefix_kernel(unsigned char *__restrict__ sums, int nseg,
                                                         int cseg)
{
    const size_t w = (size_t)blockIdx.x * 256 + threadIdx.x;
    constexpr size_t WA = SUM_AST / 4, WY = WA + SUM_Y3 / 4, WM = WY + SUM_MISC / 4;
    if (w >= WM) return;
    uint32_t *p = (uint32_t *)(sums + (size_t)blockIdx.y * nseg * SUM_BYTES) + w;
    constexpr size_t ST = SUM_BYTES / 4;
    constexpr int BT = 8;
    // the scaled copy of y2 follows y2 (its own word is rewritten from it)
    const bool half = w < WA, y2 = w >= WY && w < WY + D, y2s = w >= WY + D && w < WY + 2 * D;
    if (y2s) return;
    float r0 = 0.f, r1 = 0.f;
    for (int s0 = 1; s0 < nseg; s0 += BT) {
        uint32_t x[BT];
#pragma unroll
        for (int i = 0; i < BT; ++i) x[i] = s0 + i < nseg ? p[(size_t)(s0 + i) * ST] : 0u;
#pragma unroll
        for (int i = 0; i < BT; ++i) {
            if (s0 + i >= nseg) break;
            if (half) {
                const h2 a = __builtin_bit_cast(h2, x[i]);
                r0 += (float)a[0];
                r1 += (float)a[1];
                const h2 o = {(_Float16)r0, (_Float16)r1};
                p[(size_t)(s0 + i) * ST] = __builtin_bit_cast(uint32_t, o);
            } else {
                r0 += __uint_as_float(x[i]);
                p[(size_t)(s0 + i) * ST] = __float_as_uint(r0);
                if (y2) {
                    const int gexp = max(0, pow2_exponent(64.0f * (float)((s0 + i) * cseg * C)));
                    p[(size_t)(s0 + i) * ST + D] = __float_as_uint(ldexpf(2.0f, -gexp) * r0);
                }
            }
        }
    }
}

// k^ in fp16 and the largest |v| of 32 tokens per 16-column slice.
__global__ __launch_bounds__(256) void khat_vmax_kernel(const bf16_t *__restrict__ k,
                                                        const bf16_t *__restrict__ v,
                                                        _Float16 *__restrict__ kh,
                                                        float *__restrict__ vmax, int N, int nvb)
{
    __shared__ unsigned int m[NSL];
    const int head = blockIdx.x / nvb, blk = blockIdx.x - head * nvb;
    const int n = 32 * blk + (threadIdx.x >> 3), cg = threadIdx.x & 7;
    const size_t off = ((size_t)head * N + n) * D + 8 * cg;
    const bool valid = n < N;
    if (threadIdx.x < NSL) m[threadIdx.x] = 0u;
    float xk[8] = {}, xv[8] = {};
    if (valid) {
        bf16x8_to_f32(*(const uint4 *)(k + off), xk);
        bf16x8_to_f32(*(const uint4 *)(v + off), xv);
    }
    const h8 hk = standardise8(xk, valid);
    if (valid) *(h8 *)(kh + off) = hk;
    float mv = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) mv = fmaxf(mv, fabsf(xv[i]));
    __syncthreads();
    atomicMax(&m[cg >> 1], __float_as_uint(mv));
    __syncthreads();
    if (threadIdx.x < NSL) vmax[(size_t)blockIdx.x * NSL + threadIdx.x] = __uint_as_float(m[threadIdx.x]);
}

// q^, k^ (Sec. 2.2, Eqs. 6-7) in fp16 for the scan: an octet of lanes per row,
// 32 rows per workgroup.  q^ is multiplied by the score scale qs, so every
// later step sees the scaled score qs q^.k^.
__global__ __launch_bounds__(256) void standardise_qk(const bf16_t *__restrict__ q,
                                                      const bf16_t *__restrict__ k,
                                                      _Float16 *__restrict__ qh,
                                                      _Float16 *__restrict__ kh, size_t rows,
                                                      float qs, unsigned int *__restrict__ flags,
                                                      int nflags)
{
    // the segment flags of the scan that follows start lowered
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < nflags; i += 256) flags[i] = 0u;
    const size_t r = (size_t)blockIdx.x * 32 + (threadIdx.x >> 3);
    const int cg = threadIdx.x & 7;
    const bool valid = r < rows;
    float xq[8] = {}, xk[8] = {};
    if (valid) {
        bf16x8_to_f32(*(const uint4 *)(q + r * D + 8 * cg), xq);
        bf16x8_to_f32(*(const uint4 *)(k + r * D + 8 * cg), xk);
    }
    const h8 hq = standardise8(xq, valid, qs), hk = standardise8(xk, valid);
    if (valid) {
        *(h8 *)(qh + r * D + 8 * cg) = hq;
        *(h8 *)(kh + r * D + 8 * cg) = hk;
    }
}

}  // namespace mfma_causal

namespace {

size_t a256(size_t x) { return (x + 255) & ~(size_t)255; }

// The launches fill this many CUs (one scan workgroup per CU): an MI355X.
constexpr long TARGET_CUS = 256;

std::atomic<int> scan_segment_mode{0};

}  // namespace

int set_scan_segment_mode(int mode)
{
    return scan_segment_mode.exchange(mode);
}

// Auto: split when two segments per item take fewer rounds of half-length
// workgroups than one workgroup per item takes rounds (384 items on 256 CUs:
// 3 half rounds instead of 2 full ones; 256 items: no split).
ScanSplit causal_scan_split(int items, int nch, bool auto_split)
{
    const int mode = scan_segment_mode.load();
    if (nch < 2 || mode == 1 || (mode == 0 && !auto_split)) return ScanSplit{0, 0, 1};
    bool split = true;
    if (mode == 0) {
        const long r1 = (items + TARGET_CUS - 1) / TARGET_CUS;
        const long r2 = (2L * items + TARGET_CUS - 1) / TARGET_CUS;
        split = r2 < 2 * r1;
    }
    if (!split) return ScanSplit{0, 0, 1};
    return ScanSplit{1, nch / 2, mode == 3 ? 0 : 1};
}

size_t causal_scan_seg_workspace(int items, int nch)
{
    if (nch < 2) return 0;
    return a256((size_t)items * mfma_causal::SUM_BYTES) + a256((size_t)items * 4);
}

size_t mfma_causal_fwd_workspace(int BH, int N)
{
    const size_t rows = (size_t)BH * N;
    const int nch = (N + mfma_causal::C - 1) / mfma_causal::C;
    return 2 * a256(rows * mx::D * 2) + causal_scan_seg_workspace(BH * mfma_causal::NSL, nch);
}

// Segments of the many-segment scan: as many as fill the CUs once, limited by
// the summaries' room beside k^ in the workspace and to eight chunks at least;
// fewer than three are not worth the build (a chunk's build takes about half
// its scan's time).  Its grids are a little larger than the plain scan's (heads
// end in blocks of their own): a call that only the latter fit stays with it.  Measured, us per forward, S segments against one or two:
// B1 H8 N65536 (S = 8) 3340 -> 712; B1 H16 N32768 (4) 1650 -> 708;
// B1 H21 N32768 (3) 1650 -> 947.
int causal_multi_segments(int BH, int N)
{
    using namespace mfma_causal;
    const size_t rows = (size_t)BH * N;
    const int nch = (N + C - 1) / C;
    const long items = (long)BH * NSL;
    const size_t have = mfma_causal_fwd_workspace(BH, N);
    const size_t used = a256(rows * mx::D * 2) + a256((size_t)BH * ((N + 31) / 32) * NSL * 4);
    long S = TARGET_CUS / items;
    if (have <= used) return 0;
    S = std::min(S, (long)((have - used) / ((size_t)items * SUM_BYTES)));
    S = std::min(S, (long)(nch / 8));
    if (S < 3) return 0;
    const int cseg = ((nch + (int)S - 1) / (int)S + 1) & ~1;
    S = (nch + cseg - 1) / cseg;
    if (S < 3 || !grid_fits((long long)BH * ((N + 31) / 32), 256) || !grid_fits(items * S, NTH)) return 0;
    return (int)S;
}

size_t mfma_causal_smem_bytes() { return sizeof(mfma_causal::Smem); }

bool mfma_causal_fwd_grids_fit(int BH, int N)
{
    using namespace mfma_causal;
    const size_t rows = (size_t)BH * N;
    const int items = BH * NSL;
    const ScanSplit plan = causal_scan_split(items, (N + C - 1) / C, true);
    return grid_fits((long long)((rows + 31) / 32), 256) &&
           grid_fits((long long)items * (1 + plan.split), NTH);
}

namespace {

hipError_t multi_fwd(const void *q, const void *k, const void *v, void *out, float *g, int BH,
                     int N, float qs, int S, void *ws, hipStream_t st)
{
    using namespace mfma_causal;
    const size_t rows = (size_t)BH * N;
    const int items = BH * NSL, nch = (N + C - 1) / C, nvb = (N + 31) / 32;
    const int cseg = ((nch + S - 1) / S + 1) & ~1;
    unsigned char *p = (unsigned char *)ws;
    _Float16 *kh = (_Float16 *)p;
    p += a256(rows * D * 2);
    float *vmax = (float *)p;
    p += a256((size_t)BH * nvb * NSL * 4);
    const SegArgs sa{p, nullptr, 0, 0, 0, S, cseg, nvb, vmax, qs};
    hipLaunchKernelGGL(khat_vmax_kernel, dim3((unsigned)(BH * nvb)), dim3(256), 0, st,
                       (const bf16_t *)k, (const bf16_t *)v, kh, vmax, N, nvb);
    const int smem = (int)sizeof(Smem);
    hipError_t e = hipFuncSetAttribute((const void *)multi_kernel<1>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e == hipSuccess)
        e = hipFuncSetAttribute((const void *)multi_kernel<2>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(multi_kernel<1>, dim3(items * (S - 1)), dim3(NTH), smem, st, (const bf16_t *)q,
                       (const _Float16 *)kh, (const bf16_t *)v, (bf16_t *)out, g, N, BH, sa);
    hipLaunchKernelGGL(seg_prefix_kernel,
                       dim3((unsigned)(((SUM_AST + SUM_Y3 + SUM_MISC) / 4 + 255) / 256), (unsigned)items),
                       dim3(256), 0, st, sa.sum, S, cseg);
    hipLaunchKernelGGL(multi_kernel<2>, dim3(items * S), dim3(NTH), smem, st, (const bf16_t *)q,
                       (const _Float16 *)kh, (const bf16_t *)v, (bf16_t *)out, g, N, BH, sa);
    return hipGetLastError();
}

}  // namespace

hipError_t mfma_causal_fwd(const void *q, const void *k, const void *v, void *out, float *g,
                           int BH, int N, float qs, void *ws, hipStream_t st)
{
    using namespace mfma_causal;
    static_assert(sizeof(Smem) <= 160 * 1024, "LDS budget");
    static_assert(NHT == 2 * C, "one helper thread per (token pair, v half)");
    const size_t rows = (size_t)BH * N;
    const int items = BH * NSL, nch = (N + C - 1) / C;
    const ScanSplit plan = causal_scan_split(items, nch, true);
    if (!mfma_causal_fwd_grids_fit(BH, N)) return hipErrorInvalidConfiguration;
    if (const int S = causal_multi_segments(BH, N))
        return multi_fwd(q, k, v, out, g, BH, N, qs, S, ws, st);
    unsigned char *p = (unsigned char *)ws;
    _Float16 *qh = (_Float16 *)p;
    p += a256(rows * D * 2);
    _Float16 *kh = (_Float16 *)p;
    p += a256(rows * D * 2);
    SegArgs sa{nullptr, nullptr, plan.split, plan.csplit, plan.wait, 0, 0, 0, nullptr, 1.0f};
    if (plan.split) {
        sa.sum = p;
        sa.flags = (unsigned int *)(p + a256((size_t)items * SUM_BYTES));
    }
    hipLaunchKernelGGL(standardise_qk, dim3((unsigned)((rows + 31) / 32)), dim3(256), 0, st,
                       (const bf16_t *)q, (const bf16_t *)k, qh, kh, rows, qs, sa.flags,
                       plan.split ? items : 0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t smem = sizeof(Smem);
    e = hipFuncSetAttribute((const void *)fwd_causal_kernel,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(fwd_causal_kernel, dim3(items * (1 + plan.split)), dim3(NTH), smem, st,
                       (const _Float16 *)qh, (const _Float16 *)kh, (const bf16_t *)v,
                       (bf16_t *)out, g, N, BH, sa);
    return hipGetLastError();
}

}  // namespace fm
