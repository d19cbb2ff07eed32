// rsos_moments.hpp -- gfx950 kernels of the height-distribution moments.
//
// The skewness S_h and kurtosis Q_h of the heights (Eqs. (13)-(15)) are
// ratios of sample averages of the central moments Phi_2..Phi_4 of each
// surface's height distribution.  These kernels compute, for one state, the
// exact power sums about an integer reference, from which the host forms
// the central moments.
#pragma once

#include "rsos_kernels.hpp"

namespace rsosk {

// ---------------------------------------------------------------------------
// Power sums of the height distribution (the moments of Eqs. (13)-(15)):
// C_k = sum over sites of (h - R)^k, k = 1..4, with R = floor(S1 / L^2) of
// the current state, exact.  |h - R| never exceeds the largest height H,
// and the library keeps L^2 H^2 < 2^63, so C_1 and C_2 fit int64 and C_3,
// C_4 fit int128.  Four sites with |h - R| < 2^7 at a time are summed in 32
// bits (24-bit products: x^4 < 2^28) and added to int64 once; otherwise a
// thread sums the sites with |h - R| < 2^11 in int64 (terms below 2^44, at
// most 2^16 sites per thread) and the rare others in int128.  Workgroup
// totals go to part[4 * blockIdx.x + k], and power_sums_final adds them into
// out[0..3] and puts the record behind them, so that one copy brings both.
// One read of the lattice, bound by it: 8192 consecutive sites of a workgroup
// in flight at a time.  A call (us): L = 4096 57 -> 33 (two synchronous
// copies were 20 of them), L = 16384 216 -> 202, with 16-bit storage 152 ->
// 118.  (With each thread's loads a grid apart L = 16384 took 240: eight
// streams 8 MiB apart.)  With 16-bit storage R is also
// the reference the residues are decoded against (floor(S1 / L^2) of the
// same time), so h - R = int16(r - R mod 2^16).
// ---------------------------------------------------------------------------
typedef __int128 i128;

__device__ __forceinline__ i128 shfl_xor_i128(i128 v, int m)
{
    const unsigned long long lo = (unsigned long long)v, hi = (unsigned long long)((unsigned __int128)v >> 64);
    const unsigned long long l2 = __shfl_xor(lo, m, 64), h2 = __shfl_xor(hi, m, 64);
    return (i128)(((unsigned __int128)h2 << 64) | l2);
}

// Sum over the workgroup; result valid in thread 0.
template <int NT>
__device__ __forceinline__ void block_reduce_i128x4(i128 v[4])
{
    __shared__ i128 red[4][NT / 64];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v[k] += shfl_xor_i128(v[k], off);
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    if (l == 0)
        for (int k = 0; k < 4; ++k) red[k][w] = v[k];
    __syncthreads();
    if (threadIdx.x == 0)
        for (int k = 0; k < 4; ++k)
            for (int i = 1; i < NT / 64; ++i) v[k] += red[k][i];
}

struct PowerAcc {
    long long a[4] = {0, 0, 0, 0};
    i128 b[4] = {0, 0, 0, 0};
    __device__ __forceinline__ void add(int x)
    {
        if (x >= -2048 && x < 2048) {
            const int x2 = x * x;
            a[0] += x;
            a[1] += x2;
            a[2] += (long long)x2 * x;
            a[3] += (long long)x2 * x2;
        } else {
            const i128 X = x, X2 = X * X;
            b[0] += X;
            b[1] += X2;
            b[2] += X2 * X;
            b[3] += X2 * X2;
        }
    }
    // four sites
    __device__ __forceinline__ void add4(int x, int y, int z, int w)
    {
        const int hi = max(max(x, y), max(z, w)), lo = min(min(x, y), min(z, w));
        if (hi < 128 && lo > -128) {
            const int x2 = __mul24(x, x), y2 = __mul24(y, y), z2 = __mul24(z, z), w2 = __mul24(w, w);
            a[0] += x + y + z + w;
            a[1] += x2 + y2 + z2 + w2;
            a[2] += __mul24(x2, x) + __mul24(y2, y) + __mul24(z2, z) + __mul24(w2, w);
            a[3] += __mul24(x2, x2) + __mul24(y2, y2) + __mul24(z2, z2) + __mul24(w2, w2);
        } else {
            add(x);
            add(y);
            add(z);
            add(w);
        }
    }
};

// S = int32_t: heights; S = uint16_t: residues.  n % 8 == 0, 16-byte
// aligned buffer; rec points to the current log record (S1 first).
template <typename S>
__global__ __launch_bounds__(256) void power_sums_partial(const S *__restrict__ h, long long n,
                                                          const long long *__restrict__ rec,
                                                          long long *__restrict__ part)
{
    const long long R = rec[0] / n;
    PowerAcc acc;
    constexpr int CPC = 16 / sizeof(S);
    const long long nch = n / CPC;
    const int Rl = (int)R;  // |h - R| fits int32: the wrapping difference is exact
    constexpr int kUnroll = sizeof(S) == 4 ? 8 : 4;  // 8192 sites of a workgroup at a time
    auto take = [&](const v4u &v) {
        if constexpr (sizeof(S) == 4) {
            acc.add4((int)(v.x - (uint32_t)Rl), (int)(v.y - (uint32_t)Rl), (int)(v.z - (uint32_t)Rl), (int)(v.w - (uint32_t)Rl));
        } else {
            const uint32_t r0 = (uint32_t)R & 0xFFFFu;
            auto lo = [&](uint32_t w) { return (int)(int16_t)(uint16_t)(w - r0); };
            acc.add4(lo(v.x), lo(v.x >> 16), lo(v.y), lo(v.y >> 16));
            acc.add4(lo(v.z), lo(v.z >> 16), lo(v.w), lo(v.w >> 16));
        }
    };
    const gv4u *src = (const gv4u *)h;
    // each workgroup's loads in flight are of consecutive chunks
    long long c = (long long)blockIdx.x * (256 * kUnroll) + threadIdx.x;
    for (; c + (kUnroll - 1) * 256 < nch; c += (long long)gridDim.x * (256 * kUnroll)) {
        v4u v[kUnroll];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) v[u] = src[c + u * 256];
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) take(v[u]);
    }
    for (; c < nch; c += 256) {
        const v4u v = src[c];
        take(v);
    }
    // sums of a wave: 64-bit DPP additions where no partial sum can leave 64
    // bits, else 128-bit shuffles
    bool small = true;
#pragma unroll
    for (int k = 0; k < 4; ++k) small = small && acc.b[k] == 0 && acc.a[k] < (1ll << 56) && acc.a[k] > -(1ll << 56);
    __shared__ i128 red[4][4];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    i128 v[4];
    if (__all(small)) {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = (i128)wave_sum63_64(acc.a[k]);
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = (i128)acc.a[k] + acc.b[k];
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) v[k] += shfl_xor_i128(v[k], off);
        }
    }
    if (l == 63)
        for (int k = 0; k < 4; ++k) red[k][w] = v[k];
    __syncthreads();
    if (threadIdx.x < 4) {
        const int k = threadIdx.x;
        reinterpret_cast<i128 *>(part)[4 * blockIdx.x + k] = red[k][0] + red[k][1] + red[k][2] + red[k][3];
    }
}

__global__ __launch_bounds__(256) void power_sums_final(const long long *__restrict__ part, int nparts,
                                                        const long long *__restrict__ rec, long long *__restrict__ out)
{
    i128 v[4] = {0, 0, 0, 0};
    const i128 *p = reinterpret_cast<const i128 *>(part);
    for (int i = threadIdx.x; i < nparts; i += 256)
        for (int k = 0; k < 4; ++k) v[k] += p[4 * i + k];
    block_reduce_i128x4<256>(v);
    if (threadIdx.x == 0) {
        i128 *o = reinterpret_cast<i128 *>(out);
        for (int k = 0; k < 4; ++k) o[k] = v[k];
        out[8] = rec[0];
    }
}

}  // namespace rsosk
