// Device side of the exact squared width (Sec. I height reconstruction,
// Eq. (Wdef)) inside the persistent batch kernel, and workgroup scans and sums shared
// with the per-lattice width and spectrum kernels.
//
// h(x,y) = H0 + G(y) + P_y(x), with G(y) = sum_{k<y} sigma_y(0,k) and
// P_y(x) = sum_{l<x} sigma_x(l,y).  One workgroup measures a lattice of up to 8192
// sites per side: a wavefront takes a run of rows, as many rows at a time as fit
// side by side in its lanes with a word per lane; a lane sums its word through a
// 256-entry table of 8-site chunks, a prefix scan over the row's lanes gives every
// word's first height, and the row's rotation and its G relative to the run enter
// in closed form.  Lanes keep their own sums until the run ends; the runs are then
// joined.
#pragma once

#include "okpz_internal.h"

namespace okpz {
namespace core {

// Table of 8-site chunks.  For a byte c (bit i = site i, sigma_i = +1 when
// set) and the partial heights q_0 = 0, q_{i+1} = q_i + sigma_i, entry c holds
// s2 = sum_{i<8} q_i^2 in bits 0..7, s1 = sum_{i<8} q_i in bits 8..15 and
// d = q_8 in bits 16..23 (s1 and d as signed bytes).  A chunk whose first site
// sits at height B then adds 8 B + s1 to the sum of heights and
// 8 B^2 + 2 B s1 + s2 to the sum of squares.  Built by the whole workgroup;
// the caller synchronises before use.
__device__ __forceinline__ void width_lut_build(uint32_t *lut)
{
    for (int c = threadIdx.x; c < 256; c += blockDim.x) {
        int32_t q = 0, s1 = 0, s2 = 0;
        for (int i = 0; i < 8; ++i) {
            s1 += q;
            s2 += q * q;
            q += ((c >> i) & 1) ? 1 : -1;
        }
        lut[c] = (uint32_t)s2 | ((uint32_t)(s1 & 0xff) << 8) | ((uint32_t)(q & 0xff) << 16);
    }
}

// Sums of h - H0 and its square over rows [y_lo, y_hi) of lattice view v, by the whole
// workgroup, in thread 0's s1 and s2 (sides up to 8192: |h - H0| <= 2^14, so the sum of
// squares over 2^26 sites stays below 2^54).  lut: the chunk table; part: LDS, five words
// per wavefront.  Starts and ends with a barrier.
//
// What bounds it: the latency of one workgroup's passes.  1024 x 1024: two rows per
// pass, 32 passes per wavefront; a reduction over the lanes for every row and a
// second pass over the rows' sums took about three times as long, a fifth of a
// finite-size-scaling ensemble with a sample every ten to twenty sweeps.
__device__ __forceinline__ void width_workgroup(const LatticeView &v, const uint32_t *lut, int64_t *part,
                                                int y_lo, int y_hi, int64_t &s1, int64_t &s2)
{
    const int tid = threadIdx.x, lane = tid & 63, nwave = blockDim.x >> 6;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int xs0 = (v.Lx - v.ox) % v.Lx;  // stored column of physical column 0
    const int wq = xs0 >> 5;
    const uint32_t bq = (uint32_t)(xs0 & 31);
    // 2^ls lanes per row
    const int ls = v.W >= 64 ? 6 : v.W <= 1 ? 0 : 32 - __builtin_clz(v.W - 1);
    const int R = 64 >> ls, sub = lane >> ls, c = lane & ((1 << ls) - 1);
    const int rpw = (y_hi - y_lo + nwave - 1) / nwave;
    const int ya = min(y_hi, y_lo + wave * rpw), yb = min(y_hi, ya + rpw);
    int32_t g0 = 0;  // the wave's share of G(y_lo)
    for (int y = tid; y < y_lo; y += (int)blockDim.x)
        g0 += ((v.planes[(size_t)v.Ly * v.W + (size_t)y * v.W + wq] >> bq) & 1u) ? 1 : -1;
    __syncthreads();  // the table

    int64_t A = 0, B = 0;
    int32_t g = 0;  // G of the pass's first row relative to the run's
    for (int y0 = ya; y0 < yb; y0 += R) {
        const int y = min(y0 + sub, yb - 1);
        const bool live = y0 + sub < yb;
        const uint32_t *row = v.planes + (size_t)y * v.W;
        const bool up = live && ((row[(size_t)v.Ly * v.W + wq] >> bq) & 1u);
        int64_t a1 = 0, a2 = 0;
        int32_t carry = 0, q0 = 0, sites = 0;
        for (int base = 0; base < v.W; base += 64) {  // one pass unless the row is longer than 64 words
            const int k = base + c;
            const bool has = live && k < v.W;
            const uint32_t word = has ? row[k] : 0u;
            int32_t h = 0, t1 = 0, t2 = 0;  // height relative to the word's first site; sums
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t e = lut[(word >> (8 * j)) & 255u];
                const int32_t u = 8 * h + (int32_t)(int8_t)(e >> 8);
                t1 += u;
                t2 += __mul24(h, u + (int32_t)(int8_t)(e >> 8)) + (int32_t)(e & 0xffu);
                h += (int32_t)(int8_t)(e >> 16);
            }
            if (!has) h = t1 = t2 = 0;
            int32_t incl = h;  // over the lanes of the row
            for (int o = 1; o < (1 << ls); o <<= 1) {
                const int32_t t = __shfl_up(incl, o, 64);
                if (c >= o) incl += t;
            }
            const int32_t b = carry + incl - h;  // Q at the word's first site
            const int32_t n = has ? 32 : 0;
            a1 += n * b + t1;
            a2 += (int64_t)b * (n * b + 2 * t1) + t2;
            sites += n;
            if (wq >= base && wq < base + 64) {  // Q(xs0), from the lane holding its word
                const uint32_t below = word & ((1u << bq) - 1u);
                q0 = __shfl(b + 2 * (int32_t)__popc(below) - (int32_t)bq, (sub << ls) + wq - base, 64);
            }
            carry += __shfl(incl, (sub << ls) + (1 << ls) - 1, 64);
        }
        // the rows' column-0 steps, one bit per row in its first lane
        const uint64_t ups = __ballot(up && c == 0);
        const uint64_t lower = ups & ((uint64_t(1) << (sub << ls)) - 1);
        const int64_t k = g + 2 * (int)__popcll(lower) - sub - q0;
        A += a1 + sites * k;
        B += a2 + 2 * k * a1 + sites * k * k;
        g += 2 * (int)__popcll(ups) - min(R, yb - y0);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        A += __shfl_down(A, o, 64);
        B += __shfl_down(B, o, 64);
        g0 += __shfl_down(g0, o, 64);
    }
    if (lane == 0) {
        part[4 * wave] = g;
        part[4 * wave + 1] = A;
        part[4 * wave + 2] = B;
        part[4 * wave + 3] = (int64_t)(yb - ya) * v.Lx;
        part[4 * nwave + wave] = g0;
    }
    __syncthreads();
    if (tid == 0) {
        int64_t G = 0;
        for (int w = 0; w < nwave; ++w) G += part[4 * nwave + w];
        s1 = s2 = 0;
        for (int w = 0; w < nwave; ++w) {
            const int64_t *r = part + 4 * w;
            s1 += r[1] + r[3] * G;
            s2 += r[2] + 2 * G * r[1] + r[3] * G * G;
            G += r[0];
        }
    }
    __syncthreads();
}

// Exclusive prefix sum of v over the workgroup in thread order; *total gets
// the workgroup's sum.  lds: 16 entries.  Ends with a barrier.
__device__ __forceinline__ int64_t block_exclusive_scan(int64_t v, int64_t *lds, int64_t *total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwave = blockDim.x >> 6;
    int64_t incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int64_t t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) lds[wave] = incl;
    __syncthreads();
    int64_t off = 0, tot = 0;
    for (int w = 0; w < nwave; ++w) {
        const int64_t s = lds[w];
        if (w < wave) off += s;
        tot += s;
    }
    __syncthreads();
    *total = tot;
    return off + incl - v;
}

// Sum of a 128-bit value over the workgroup, returned in every thread.
// lds: 32 entries.  Ends with a barrier.
__device__ __forceinline__ __int128 block_sum_i128(__int128 v, int64_t *lds)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwave = blockDim.x >> 6;
    uint64_t lo = (uint64_t)v, hi = (uint64_t)((unsigned __int128)v >> 64);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint64_t alo = __shfl_down(lo, o, 64), ahi = __shfl_down(hi, o, 64);
        const unsigned __int128 s = (((unsigned __int128)hi << 64) | lo) +
                                    (((unsigned __int128)ahi << 64) | alo);
        lo = (uint64_t)s;
        hi = (uint64_t)(s >> 64);
    }
    if (lane == 0) {
        lds[2 * wave] = (int64_t)lo;
        lds[2 * wave + 1] = (int64_t)hi;
    }
    __syncthreads();
    unsigned __int128 t = 0;
    for (int w = 0; w < nwave; ++w)
        t += ((unsigned __int128)(uint64_t)lds[2 * w + 1] << 64) | (uint64_t)lds[2 * w];
    __syncthreads();
    return (__int128)t;
}

}  // namespace core
}  // namespace okpz
