// Exact squared width of one lattice (Sec. I height reconstruction,
// Eq. (Wdef)) on gfx950.
//
// h(x,y) = H0 + G(y) + P_y(x).  A wavefront takes a run of rows and reads each
// row's sigma_x words once, in stored order, four words per lane and pass.  A
// lane sums its 128 sites through a table of 10- and 11-site chunks, a
// wavefront prefix scan of the lanes' height changes gives every lane's first
// height, and the row's rotation and its G relative to the run's first row
// enter in closed form.  Nothing is reduced across lanes until the run ends.  The
// runs of a workgroup are then joined, each workgroup writes a record
//   {delta, A, B}: sum of its rows' sigma_y(0,y), sum and sum of squares of its
//   heights relative to its first row's column 0,
// and one workgroup joins the records: n sites at offset G add n G + A and
// n G^2 + 2 G A + B.
//
// What bounds it: vector instructions and table reads (about 120 VALU and 22 LDS
// cycles per 64 words of a wavefront), near the N/8 bytes of the sigma_x plane.
// 65536^2: 136 us for 537 MB, 3.9 TB/s (178 us with four 8-site lookups per word and
// a reduction over the lanes per row); a call on 256^2 with its five words written
// to host memory by the kernel 21 us (about 57 us with two small copies).
#include "width.h"
#include "width_core.h"

namespace okpz {
namespace {

constexpr int kRowThreads = 256;
constexpr int kWaves = kRowThreads / 64;
constexpr int kTotalThreads = 256;
constexpr int kPassWords = 256;  // words of a row per pass of a wavefront

// Chunk tables: entry c of the 11-site table (2048 entries) and of the 10-site
// table after it (1024).  For the partial heights q_0 = 0, q_{i+1} = q_i + sigma_i:
// sum of q_i^2 in bits 0..12, sum of q_i plus kBias in bits 13..23 and the height
// change in bits 24..31 (signed), so that adding entries adds the first two and
// keeps the running height, for up to twelve chunks and less than 128 sites.
constexpr int kBias = 55;
struct alignas(16) ChunkTable {
    uint32_t e[2048 + 1024];
};
constexpr ChunkTable make_chunks()
{
    ChunkTable t{};
    for (int k = 0; k < 2; ++k) {
        const int n = k ? 10 : 11;
        for (int c = 0; c < (1 << n); ++c) {
            int q = 0, s1 = 0, s2 = 0;
            for (int i = 0; i < n; ++i) {
                s1 += q;
                s2 += q * q;
                q += ((c >> i) & 1) ? 1 : -1;
            }
            t.e[2048 * k + c] = (uint32_t)s2 | ((uint32_t)(s1 + kBias) << 13) | ((uint32_t)(q & 0xff) << 24);
        }
    }
    return t;
}
__device__ const ChunkTable kChunks = make_chunks();

// Sums over the sites of up to four words, heights relative to the first site:
// s1 = sum q, s2 = sum q^2, d = the height change.
struct LaneSums {
    int32_t s1, s2, d;
};

template <bool kFull>
__device__ __forceinline__ LaneSums lane_sums(const uint32_t w[4], int nw, const uint32_t *tab)
{
    uint32_t acc = 0;
    int32_t d = 0;
    // over the 11-site and the 10-site chunks, B the height of a chunk's first site:
    // sum B, sum B^2, and sum B (s1 + bias) over both
    int32_t b11 = 0, b10 = 0, bb11 = 0, bb10 = 0, bs = 0;
    auto chunk = [&](uint32_t byte_off, int32_t &sb, int32_t &sbb) {
        const uint32_t e = *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(tab) + byte_off);
        const int32_t B = (int32_t)acc >> 24;
        sb += B;
        sbb += __mul24(B, B);
        bs += __mul24(B, (int32_t)((e >> 13) & 0x7ffu));
        acc += e;
        d = B + ((int32_t)e >> 24);
    };
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        if (kFull || t < nw) {
            chunk((w[t] << 2) & 0x1ffcu, b11, bb11);
            chunk((w[t] >> 9) & 0x1ffcu, b11, bb11);
            chunk(8192u + ((w[t] >> 20) & 0xffcu), b10, bb10);
        }
    }
    LaneSums r;
    r.s1 = 11 * b11 + 10 * b10 + (int32_t)((acc >> 13) & 0x7ffu) - 3 * kBias * nw;
    r.s2 = 11 * bb11 + 10 * bb10 + 2 * (bs - kBias * (b11 + b10)) + (int32_t)(acc & 0x1fffu);
    r.d = d;
    return r;
}

// Inclusive prefix sum over the wavefront.
__device__ __forceinline__ int32_t wave_scan(int32_t x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr 1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // lane 15 of a row to the next one
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // lane 31 to the upper half
    return x;
}

// Record of a run of rows: {delta, A, B}, heights relative to the run's first.
struct Run {
    int64_t delta, A;
    unsigned __int128 B;
    int64_t sites;
};
// The run `b` after the run `a`.
__device__ __forceinline__ void join(Run &a, const Run &b)
{
    const int64_t G = a.delta;
    a.B += b.B + (unsigned __int128)(2 * (__int128)G * b.A + (__int128)b.sites * G * G);
    a.A += b.A + b.sites * G;
    a.sites += b.sites;
    a.delta += b.delta;
}

// rpw: rows per wavefront.  rec: 4 words per workgroup.
__global__ __launch_bounds__(kRowThreads) void width_kernel(LatticeView v, int rpw, int64_t *rec)
{
    __shared__ uint32_t tab[2048 + 1024];
    __shared__ int64_t part[kWaves][5];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    for (int i = tid; i < (2048 + 1024) / 4; i += kRowThreads)
        reinterpret_cast<uint4 *>(tab)[i] = reinterpret_cast<const uint4 *>(kChunks.e)[i];

    const int xs0 = (v.Lx - v.ox) % v.Lx;  // stored column of physical column 0
    const int wq = xs0 >> 5;
    const uint32_t bq = (uint32_t)(xs0 & 31);
    const bool vec = (v.W & 3) == 0;  // rows are 16-byte aligned
    const int ya = min(v.Ly, (blockIdx.x * kWaves + wave) * rpw), yb = min(v.Ly, ya + rpw);

    auto load = [&](int y, int base, uint32_t w[4]) {
        const uint32_t *row = v.planes + (size_t)y * v.W;
        const int k0 = base + lane * 4;
        if (vec) {
            uint4 q = uint4{0, 0, 0, 0};
            if (k0 < v.W) q = *reinterpret_cast<const uint4 *>(row + k0);
            w[0] = q.x; w[1] = q.y; w[2] = q.z; w[3] = q.w;
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t) w[t] = k0 + t < v.W ? row[k0 + t] : 0u;
        }
    };
    __syncthreads();  // the table

    Run run{0, 0, 0, 0};  // this lane's share; delta and sites are the wavefront's
    int32_t g = 0;        // G(y) relative to the run's first row
    uint64_t bits = 0;    // sigma_y at physical column 0 of the next 64 rows
    for (int y = ya; y < yb; ++y) {
        if (((y - ya) & 63) == 0) {
            const uint32_t *col = v.planes + ((size_t)v.Ly + y) * v.W + wq;
            bits = __ballot(y + lane < yb && ((col[(size_t)min(lane, yb - 1 - y) * v.W] >> bq) & 1u));
        }
        int64_t a1 = 0, a2 = 0;
        int32_t carry = 0, q0 = 0, sites = 0;
        auto pass = [&](int base, const uint32_t w[4]) {
            const int nw = max(0, min(4, v.W - base - lane * 4));
            const LaneSums s = base + kPassWords <= v.W ? lane_sums<true>(w, 4, tab) : lane_sums<false>(w, nw, tab);
            const int32_t incl = wave_scan(s.d);
            const int32_t b = carry + incl - s.d;  // height of the lane's first site
            const int32_t nb = 32 * nw * b;        // |b| <= 2^20, nw <= 4
            a1 += nb + s.s1;
            a2 += (int64_t)b * (nb + 2 * s.s1) + s.s2;
            sites += 32 * nw;
            if (wq >= base && wq < base + kPassWords) {
                // Q(xs0), the stored-order height at physical column 0
                const int tq = wq & 3, lq = (wq - base) >> 2;
                int32_t Bq = b;
                uint32_t word = w[0];
#pragma unroll
                for (int t = 1; t < 4; ++t) {
                    if (t <= tq) {
                        Bq += 2 * (int32_t)__popc(w[t - 1]) - 32;
                        word = w[t];
                    }
                }
                const uint32_t below = word & ((1u << bq) - 1u);
                q0 = __builtin_amdgcn_readlane(Bq + 2 * (int32_t)__popc(below) - (int32_t)bq, lq);
            }
            carry += __builtin_amdgcn_readlane(incl, 63);
        };
        // two passes' words in flight at once
        for (int base = 0; base < v.W; base += 2 * kPassWords) {
            uint32_t w0[4], w1[4];
            load(y, base, w0);
            load(y, base + kPassWords, w1);
            pass(base, w0);
            if (base + kPassWords < v.W) pass(base + kPassWords, w1);
        }
        // heights of the row relative to the run: Q + k with k = G - Q(xs0) (the
        // row's slopes sum to zero, so the rotation drops out)
        const int64_t k = g - q0;
        run.A += a1 + sites * k;
        run.B += (unsigned __int128)(uint64_t)(a2 + 2 * k * a1 + sites * k * k);
        g += (bits & 1) ? 1 : -1;
        bits >>= 1;
    }
    // over the lanes, then over the workgroup's runs
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        run.A += __shfl_down(run.A, o, 64);
        const uint64_t lo = __shfl_down((uint64_t)run.B, o, 64), hi = __shfl_down((uint64_t)(run.B >> 64), o, 64);
        run.B += ((unsigned __int128)hi << 64) | lo;
    }
    if (lane == 0) {
        part[wave][0] = g;
        part[wave][1] = run.A;
        part[wave][2] = (int64_t)(uint64_t)run.B;
        part[wave][3] = (int64_t)(uint64_t)(run.B >> 64);
        part[wave][4] = (int64_t)(yb - ya) * v.Lx;
    }
    __syncthreads();
    if (tid == 0) {
        Run r{0, 0, 0, 0};
        for (int i = 0; i < kWaves; ++i) {
            const Run s{part[i][0], part[i][1],
                        ((unsigned __int128)(uint64_t)part[i][3] << 64) | (uint64_t)part[i][2], part[i][4]};
            join(r, s);
        }
        int64_t *o = rec + 4 * (size_t)blockIdx.x;
        o[0] = r.delta;
        o[1] = r.A;
        o[2] = (int64_t)(uint64_t)r.B;
        o[3] = (int64_t)(uint64_t)(r.B >> 64);
    }
}

// The nrec records of rpg rows each (the last may have fewer), joined: out[0..3] =
// S1' lo, hi, S2' lo, hi (128-bit two's complement halves of the sums of h - H0
// and its square), out[4] = H0, and with t >= 0, out[-1] = t.  A launch of its own:
// the last workgroup of width_kernel joining them instead needs a release per
// workgroup, about 30 ns each one after the other (8192 rows: 70 us).
__global__ __launch_bounds__(kTotalThreads) void width_total_kernel(const int64_t *rec, int nrec, int rpg, int Lx,
                                                                    int Ly, const int64_t *h0, int64_t *out,
                                                                    int64_t t)
{
    __shared__ int64_t lds[32];
    const int tid = threadIdx.x;
    const int per = (nrec + kTotalThreads - 1) / kTotalThreads;
    const int b0 = min(nrec, tid * per), b1 = min(nrec, b0 + per);
    int64_t delta = 0;
    for (int b = b0; b < b1; ++b) delta += rec[4 * (size_t)b];
    int64_t unused;
    int64_t G = core::block_exclusive_scan(delta, lds, &unused);
    __int128 s1 = 0, s2 = 0;
    for (int b = b0; b < b1; ++b) {
        const int64_t *r = rec + 4 * (size_t)b;
        const int64_t sites = (int64_t)min(rpg, Ly - b * rpg) * Lx;
        s1 += (__int128)sites * G + r[1];
        s2 += (__int128)sites * G * G + 2 * (__int128)G * r[1] +
              (__int128)(((unsigned __int128)(uint64_t)r[3] << 64) | (uint64_t)r[2]);
        G += r[0];
    }
    const __int128 S1 = core::block_sum_i128(s1, lds);
    const __int128 S2 = core::block_sum_i128(s2, lds);
    if (tid == 0) {
        out[0] = (int64_t)(uint64_t)S1;
        out[1] = (int64_t)(uint64_t)((unsigned __int128)S1 >> 64);
        out[2] = (int64_t)(uint64_t)S2;
        out[3] = (int64_t)(uint64_t)((unsigned __int128)S2 >> 64);
        out[4] = *h0;
        if (t >= 0) out[-1] = t;
    }
}

// Rows per wavefront: enough workgroups to fill the device (eight per CU), then
// longer runs, so that a workgroup's copy of the table and its record are shared by
// more rows.
int rows_per_wave(int64_t Ly) { return (int)((Ly + kWaves * 2048 - 1) / (kWaves * 2048)); }

}  // namespace

// The spectrum's rows (psd.h: 3 Ly words at most); the width's records (four words per
// kWaves rows at most) use their place.
size_t width_scratch_words(int64_t Ly) { return 3 * (size_t)Ly + 4 * (size_t)((Ly + 255) / 256) + 4; }

hipError_t launch_width(const LatticeView &v, int64_t *rows, const int64_t *h0, int64_t *out, int64_t t,
                        hipStream_t st)
{
    const int rpw = rows_per_wave(v.Ly);
    const int nwg = (v.Ly + kWaves * rpw - 1) / (kWaves * rpw);
    hipLaunchKernelGGL(width_kernel, dim3(nwg), dim3(kRowThreads), 0, st, v, rpw, rows);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(width_total_kernel, dim3(1), dim3(kTotalThreads), 0, st, rows, nwg, kWaves * rpw, v.Lx, v.Ly,
                       h0, out, t);
    return hipGetLastError();
}

}  // namespace okpz
