// Power spectrum density of the surface along the lattice axes (Sec. III,
// Eqs. (PSD) and (hF)) on gfx950.
//
// For k = (2 pi n / Lx, 0) the transform of Eq. (hF) only sees the column
// sums of the heights, and for k = (0, 2 pi n / Ly) only the row sums:
//   h(k) = (Lx Ly)^{-1/2} sum_x e^{i k x} (X(x) - <X>),  X(x) = sum_y h(x,y).
// With h(x,y) = H0 + G(y) + P_y(x) (Sec. I reconstruction), up to constants
// that drop out of every n > 0,
//   X(x) = sum_{l<x} (2 c(l) - Ly),  c(l) = number of rows with sigma_x(l,y) = +1,
//   Y(y) = Lx G(y) + sum_x P_y(x).
// Both are linear in the sigma_x bits, so one pass over that plane (N/8 bytes)
// gives the column counts and the row sums, exactly, in integers.  Each profile,
// minus its mean, goes through a radix-2 decimation-in-frequency FFT in fp64; its
// stages are done three or four at a time in registers: first the stages that
// span more than an LDS tile, then the rest of each tile in LDS.  The output stays
// in bit-reversed order and the squares are written from there.  A side that is not
// a power of two goes through Bluestein's chirp-z form (Bluestein 1970): with
// c_j = exp(-i pi j^2 / n), X_k = c_k sum_j (x_j c_j) conj(c_{k-j}), a convolution
// done with power-of-two transforms of length M >= 2n - 1 (forward stages, a
// pointwise product in bit-reversed order, and the forward stages undone in reverse
// order, which returns natural order); |c_k| = 1 drops out of the spectrum.  The two
// axes share every launch where the scratch holds both.
//
// What bounds it: the pass over the plane from 32768^2 on (65536^2: 537 MB in 128 us,
// 4.2 TB/s, bound by the latency of a wavefront's row sums; a row pass of the width
// kernels and a column pass took 178 + 98 us and their sums 31), below that the chain of
// four to six launches: 8160 x 4064, both sides through Bluestein, 60 us per call (330 us
// with one launch per stage of 27 us tiles and serial sums over up to 254 parts).
#include "psd.h"
#include "width_core.h"

namespace okpz {
namespace {

constexpr int kFftThreads = 512;
constexpr int kWideThreads = 256;
constexpr int kTile = 4096;               // complex fp64 values per LDS tile
constexpr int kTileLog = 12;
constexpr int kWideLog = 4;               // stages of one pass over the whole transform

// carry-save adder on 32 bit positions at once: a + b + c = 2 h + l
__device__ __forceinline__ void csa(uint32_t &h, uint32_t &l, uint32_t a, uint32_t b, uint32_t c)
{
    h = __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);  // majority
    l = __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

// Sum over the wavefront, valid in lane 63.
__device__ __forceinline__ int32_t wave_sum63(int32_t x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr 1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast 15, 31
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

// One pass over the sigma_x plane.  Workgroup (strip, chunk) takes 256 word columns
// and p.R rows, a wavefront p.R / kPlaneWaves of them, a lane four words of a row.
// Columns: eight rows at a time go through a carry-save adder tree whose carry
// out is counted in byte lanes; partial[chunk * Lx + stored column] gets the sigma_x =
// +1 bonds of the chunk.  Rows, with E the strip's end: rowpart[strip * Ly + y] =
// {sum of sigma(c) (E - 1 - c), d + 65536 q} with d the strip's sum of sigma and q its
// part before the stored column xs0 of physical column 0 (|d|, |q| <= 8192).
// A bit's weight within its word is read off five masked popcounts.
// kVec: W is a multiple of four (16-byte loads, every lane has four words or none).
// kTall (PsdPlan::tall): rowsum[y] and rowsum[2 Ly + y], zero before, get the strips' sums of
// P to the row's end and of q instead, by atomic additions of eight rows at a time (16 bytes
// per strip and row beside the 1024 read), and a wavefront adds its column counters up every
// kMaxWaveRows rows.  2^18 x 2^18: 1.92 ms per call (2.61 ms with one row's additions at a
// time, at four waves per SIMD; 2.15 ms with parts of 64 MiB).
// The next eight rows are in flight while eight are counted (sixteen left two waves per
// SIMD for registers, three hide more).
template <bool kVec, bool kTall>
__global__ __launch_bounds__(kPlaneThreads, kVec && !kTall ? 4 : 3) void plane_kernel(LatticeView v, int32_t R, int32_t *partial,
                                                                            int2 *rowpart, int64_t *rowsum)
{
    // counts of a lane's 128 columns, column j of lane l at 65 j + l: neither the
    // lanes' sums nor the ordered read meet in a bank
    __shared__ uint32_t cols[128 * 65];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    for (int i = threadIdx.x; i < 128 * 65; i += kPlaneThreads) cols[i] = 0;
    const int strip = blockIdx.x, k0 = strip * kStripWords + 4 * lane;
    const int nw = max(0, min(4, v.W - k0));
    const int E = min(v.Lx, (strip + 1) * kStripCols);
    const int xs0 = (v.Lx - v.ox) % v.Lx;
    const int before = xs0 - strip * kStripCols;  // columns of the strip before xs0
    uint32_t mask[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int n = before - 128 * lane - 32 * t;
        mask[t] = n <= 0 ? 0u : n >= 32 ? ~0u : (1u << n) - 1u;
    }
    const bool split = before > 0 && before < kStripCols;
    int nbefore = 0;  // columns of this lane before xs0
#pragma unroll
    for (int t = 0; t < 4; ++t) nbefore += t < nw ? __popc(mask[t]) : 0;

    const int rw = R / kPlaneWaves;
    const int y_lo = min(v.Ly, (int)blockIdx.y * R + wave * rw), y_hi = min(v.Ly, y_lo + rw);
    int ya = y_lo, yb = kTall ? min(y_hi, y_lo + kMaxWaveRows) : y_hi;
    uint32_t ones[4], twos[4], fours[4], acc[4][8];
    auto clear = [&] {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            ones[t] = twos[t] = fours[t] = 0u;
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[t][j] = 0u;
        }
    };
    clear();
    // (rows and words beyond the ends are read from inside, and zeroed before use)
    const uint32_t *word0 = v.planes + (kVec ? min(k0, v.W - 4) : 0);
    auto load = [&](int y0, uint32_t w[kGroupRows][4]) {
#pragma unroll
        for (int i = 0; i < kGroupRows; ++i) {
            const uint32_t *p = word0 + (size_t)min(y0 + i, yb - 1) * v.W;
            if (kVec) {
                const uint4 q = *reinterpret_cast<const uint4 *>(p);
                w[i][0] = q.x; w[i][1] = q.y; w[i][2] = q.z; w[i][3] = q.w;
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t) w[i][t] = p[min(k0 + t, v.W - 1)];
            }
        }
    };
    auto count = [&](int y0, uint32_t w[kGroupRows][4]) {
        if (y0 + kGroupRows > yb) {
#pragma unroll
            for (int i = 0; i < kGroupRows; ++i)
#pragma unroll
                for (int t = 0; t < 4; ++t) w[i][t] = y0 + i < yb ? w[i][t] : 0u;
        }
        if (!kVec) {
#pragma unroll
            for (int i = 0; i < kGroupRows; ++i)
#pragma unroll
                for (int t = 0; t < 4; ++t) w[i][t] = t < nw ? w[i][t] : 0u;
        }
        // rows
        int32_t row_r = 0, row_p = 0;
#pragma unroll
        for (int i = 0; i < kGroupRows; ++i) {
            int32_t n[4], J = 0;  // set bits per word; sum of their places within the word
#pragma unroll
            for (int t = 0; t < 4; ++t) n[t] = __popc(w[i][t]);
            auto place = [&](uint32_t m) {
                J <<= 1;
#pragma unroll
                for (int t = 0; t < 4; ++t) J += __popc(w[i][t] & m);
            };
            place(0xFFFF0000u);
            place(0xFF00FF00u);
            place(0xF0F0F0F0u);
            place(0xCCCCCCCCu);
            place(0xAAAAAAAAu);
            // sigma = 2 b - 1: sum of sigma (E - 1 - c) over the lane's words
            const int32_t d = 2 * (n[0] + n[1] + n[2] + n[3]) - 32 * nw;
            const int32_t far = 2 * (n[1] + 2 * n[2] + 3 * n[3]) - 32 * (nw * (nw - 1) / 2);  // sum of t d_t
            const int32_t r = (E - 1 - 32 * k0) * d - 32 * far - (2 * J - 496 * nw);
            int32_t pack = d;
            if (split) {
                int32_t q = -nbefore;
#pragma unroll
                for (int t = 0; t < 4; ++t) q += 2 * __popc(w[i][t] & mask[t]);
                pack += q << 16;
            } else if (before > 0) {
                pack += d << 16;
            }
            const int32_t rs = wave_sum63(!kVec || nw ? r : 0), ps = wave_sum63(!kVec || nw ? pack : 0);
            if (kTall) {  // row i's sums to lane i
                const int32_t sr = __builtin_amdgcn_readlane(rs, 63), sp = __builtin_amdgcn_readlane(ps, 63);
                row_r = lane == i ? sr : row_r;
                row_p = lane == i ? sp : row_p;
            } else if (lane == 63 && y0 + i < yb) {
                rowpart[(size_t)strip * v.Ly + y0 + i] = make_int2(rs, ps);
            }
        }
        if (kTall && lane < kGroupRows && y0 + lane < yb) {
            const int32_t ds = (int16_t)row_p;
            unsigned long long *sum = reinterpret_cast<unsigned long long *>(rowsum) + y0 + lane;
            atomicAdd(sum, (unsigned long long)(row_r + (int64_t)ds * (v.Lx - E)));
            atomicAdd(sum + 2 * (size_t)v.Ly, (unsigned long long)(int64_t)((row_p - ds) >> 16));
        }
        // columns
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            uint32_t twosA, twosB, foursA, foursB, eights;
            csa(twosA, ones[t], ones[t], w[0][t], w[1][t]);
            csa(twosB, ones[t], ones[t], w[2][t], w[3][t]);
            csa(foursA, twos[t], twos[t], twosA, twosB);
            csa(twosA, ones[t], ones[t], w[4][t], w[5][t]);
            csa(twosB, ones[t], ones[t], w[6][t], w[7][t]);
            csa(foursB, twos[t], twos[t], twosA, twosB);
            csa(eights, fours[t], fours[t], foursA, foursB);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[t][j] += (eights >> j) & 0x01010101u;
        }
    };
    auto rows = [&] {  // ya .. yb
        uint32_t w0[kGroupRows][4], w1[kGroupRows][4];
        load(ya, w0);
        for (int y = ya; y < yb; y += 2 * kGroupRows) {
            load(y + kGroupRows, w1);
            count(y, w0);
            load(y + 2 * kGroupRows, w0);
            if (y + kGroupRows < yb) count(y + kGroupRows, w1);
        }
    };
    auto add_up = [&] {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            if (t >= nw || ya >= yb) continue;
#pragma unroll
            for (int b = 0; b < 32; ++b) {
                const uint32_t n = 8 * ((acc[t][b & 7] >> (b & ~7)) & 0xffu) + 4 * ((fours[t] >> b) & 1u) +
                                   2 * ((twos[t] >> b) & 1u) + ((ones[t] >> b) & 1u);
                atomicAdd(cols + 65 * (32 * t + b) + lane, n);
            }
        }
    };
    if (kTall) {
        __syncthreads();  // cols is zero
        while (ya < yb) {
            rows();
            add_up();
            clear();
            ya = yb;
            yb = min(y_hi, ya + kMaxWaveRows);
        }
    } else {
        if (ya < yb) rows();
        __syncthreads();  // cols is zero
        add_up();
    }
    __syncthreads();
    const int c0 = strip * kStripCols;
    for (int c = threadIdx.x; c < E - c0; c += kPlaneThreads)
        partial[(size_t)blockIdx.y * v.Lx + c0 + c] = (int32_t)cols[65 * (c & 127) + (c >> 7)];
}

// The profiles as scans of integer steps d(i):
//   v(i) = scale * sum_{i'<i} d(i') + e(i),
// column profile X: d(l) = 2 c(stored column of l) - Ly, scale 1, e = 0;
// row profile Y: d(y) = 2 sigma_y-bit(0,y) - 1, scale Lx, e(y) = the row's
// sum of P.  Every v is an integer below 2^41 in magnitude, exact in fp64.
// A block of kProfThreads values keeps its own prefix of d and two sums; the first
// kernel of the transforms adds up the blocks' (Profile::offsets).
struct Profile {
    const int32_t *prefix;  // sum of d over the block's values before i
    const int64_t *extra;   // e(i), or nullptr
    const int64_t *blk;     // per block: sum of d, part of sum_i v(i)
    int64_t scale;
    int32_t n, nblk;
};
struct Profiles {
    LatticeView v;
    const int32_t *partial;
    const int2 *rowpart;
    int32_t nch;
    int32_t *prefix[2];  // per axis (x, y)
    int64_t *extra;          // at first the rows' sums of the tall plane pass, if rowpart is null
    int64_t *blk[2];
    int32_t nblk[2];
};

// rows[0, Ly) and rows[2 Ly, 3 Ly) to zero, for the tall plane pass.
__global__ __launch_bounds__(kProfThreads) void clear_rows_kernel(int64_t *rows, int32_t Ly)
{
    const int i = blockIdx.x * kProfThreads + threadIdx.x;
    if (i < Ly) rows[i] = rows[2 * (size_t)Ly + i] = 0;
}

__device__ __forceinline__ int side(const LatticeView &v, int axis) { return axis ? v.Ly : v.Lx; }

// Blocks 0 .. nblk[0) take the columns, the others the rows: the parts of the plane
// pass added up into d and e, the block's prefix of d, and its sums (sum_i v(i) =
// scale sum_j d(j) (n-1-j) + sum_j e(j)).
__global__ __launch_bounds__(kProfThreads) void profile_steps_kernel(Profiles p)
{
    __shared__ int64_t lds[32];
    const LatticeView &v = p.v;
    const int axis = (int)blockIdx.x >= p.nblk[0];
    const int b = (int)blockIdx.x - (axis ? p.nblk[0] : 0);
    const int n = side(v, axis), i = b * kProfThreads + threadIdx.x;
    int64_t d = 0, e = 0;
    if (i < n) {
        if (axis == 0) {
            int xs = i - v.ox;
            if (xs < 0) xs += v.Lx;
            int32_t c = 0;
#pragma unroll 8
            for (int ch = 0; ch < p.nch; ++ch) c += p.partial[(size_t)ch * v.Lx + xs];
            d = 2 * (int64_t)c - v.Ly;
        } else {
            // sum of P = sum of Q - Lx Q(xs0), Q the stored-order prefix
            int64_t q0 = 0;
            if (!p.rowpart) {
                e = p.extra[i];
                q0 = p.extra[2 * (size_t)v.Ly + i];
            }
            for (int s = 0; p.rowpart && s * kStripCols < v.Lx; ++s) {
                const int2 r = p.rowpart[(size_t)s * v.Ly + i];
                const int32_t ds = (int16_t)r.y;
                e += r.x + (int64_t)ds * (v.Lx - min(v.Lx, (s + 1) * kStripCols));
                q0 += (r.y - ds) >> 16;
            }
            e -= v.Lx * q0;
            const int xs0 = (v.Lx - v.ox) % v.Lx;
            const uint32_t w = v.planes[((size_t)v.Ly + i) * v.W + (xs0 >> 5)];
            d = 2 * (int64_t)((w >> (xs0 & 31)) & 1u) - 1;
            p.extra[i] = e;
        }
    }
    const int64_t scale = axis ? v.Lx : 1;
    int64_t D;
    const int64_t pre = core::block_exclusive_scan(d, lds, &D);
    if (i < n) p.prefix[axis][i] = (int32_t)pre;
    const __int128 V = core::block_sum_i128(i < n ? scale * d * (int64_t)(n - 1 - i) + e : 0, lds);
    if (threadIdx.x == 0) {
        p.blk[axis][2 * (size_t)b] = D;
        p.blk[axis][2 * (size_t)b + 1] = (int64_t)V;
    }
}

// Values of a profile for a workgroup: the blocks' offsets and the mean, worked out
// once per workgroup (a launch of its own for this cost more: at most 4096 blocks).
// off: LDS of at least nblk + 1 words; its rounding makes the mean move n = 0 only.
// All threads; ends with a barrier.
__device__ __forceinline__ void profile_offsets(const Profile &p, int64_t *off, int64_t *lds)
{
    const int per = (p.nblk + (int)blockDim.x - 1) / (int)blockDim.x;
    const int b0 = min(p.nblk, (int)threadIdx.x * per), b1 = min(p.nblk, b0 + per);
    int64_t local = 0, vs = 0;
    for (int b = b0; b < b1; ++b) {
        local += p.blk[2 * (size_t)b];
        vs += p.blk[2 * (size_t)b + 1];
    }
    int64_t unused;
    int64_t run = core::block_exclusive_scan(local, lds, &unused);
    for (int b = b0; b < b1; ++b) {
        off[b] = run;
        run += p.blk[2 * (size_t)b];
    }
    const __int128 V = core::block_sum_i128(vs, lds);
    if (threadIdx.x == 0) off[p.nblk] = __double_as_longlong((double)(int64_t)V / p.n);
    __syncthreads();
}
__device__ __forceinline__ double profile_value(const Profile &p, const int64_t *off, int i)
{
    const int64_t pre = off[i / kProfThreads] + p.prefix[i];
    const int64_t v = p.scale * pre + (p.extra ? p.extra[i] : 0);
    return (double)v - __longlong_as_double(off[p.nblk]);
}
constexpr int kMaxBlocks = (1 << 20) / kProfThreads;

// ---- transforms ------------------------------------------------------------
// One axis: the n values of a profile.  chirp: through Bluestein with the buffers A
// and B of len = M values; otherwise len = n in z.
struct Axis {
    Profile prof;
    double2 *z, *A, *B;
    double *S;
    double norm;  // 1 / (Lx Ly)
    int32_t n, len, log2len;
    bool chirp;
};
struct Axes {
    Axis ax[2];
};

__device__ __forceinline__ double2 cmul(double2 a, double2 b)
{
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// z <- (z + w) at i, (z - w) e^{-i pi r / h} at i + h: one radix-2
// decimation-in-frequency stage of span h on blocks of 2h values; tw = e^{-i pi r / h}.
__device__ __forceinline__ void dif_butterfly(double2 &a, double2 &b, double2 tw)
{
    const double2 u = a, v = b;
    a = make_double2(u.x + v.x, u.y + v.y);
    b = cmul(make_double2(u.x - v.x, u.y - v.y), tw);
}

// The stage above undone without its factor 1/2: (a, b) <- (a + t, a - t),
// t = b e^{+i pi r / h}.  All stages undone in reverse order turn the
// bit-reversed transform of x back into n x in natural order, i.e. they
// apply the unnormalised inverse DFT to a bit-reversed spectrum.
__device__ __forceinline__ void dif_butterfly_undo(double2 &a, double2 &b, double2 tw)
{
    const double2 t = cmul(b, make_double2(tw.x, -tw.y));
    const double2 u = a;
    a = make_double2(u.x + t.x, u.y + t.y);
    b = make_double2(u.x - t.x, u.y - t.y);
}

// e^{-i pi r / h}, h = 1 / inv a power of two (the product is exact).
__device__ __forceinline__ double2 twiddle(int r, double inv)
{
    double s, c;
    sincospi(-(double)r * inv, &s, &c);
    return make_double2(c, s);
}

// kLog stages in registers on the 2^kLog values x[m] at i + m step of a block of
// 2^kLog step values; tw(r, l) = e^{-i pi r / h}, h = 2^l step.  A stage's twiddle
// depends on m modulo its half only.
template <int kLog, bool kUndo, class Tw>
__device__ __forceinline__ void stages(double2 *x, int i, int step, Tw tw)
{
#pragma unroll
    for (int q = 0; q < kLog; ++q) {
        const int st = kUndo ? kLog - 1 - q : q;
        const int half = (1 << kLog) >> (st + 1);
#pragma unroll
        for (int m = 0; m < half; ++m) {
            const double2 w = tw(i + m * step, kLog - 1 - st);
#pragma unroll
            for (int g = 0; g < (1 << kLog); g += 2 * half) {
                if (kUndo)
                    dif_butterfly_undo(x[g + m], x[g + m + half], w);
                else
                    dif_butterfly(x[g + m], x[g + m + half], w);
            }
        }
    }
}

// c_j = exp(-i pi j^2 / n), the phase reduced exactly: j^2 mod 2n.
__device__ __forceinline__ double2 chirp(int64_t j, int32_t n)
{
    const int64_t k = (j * j) % (2 * (int64_t)n);
    double s, c;
    sincospi(-(double)k / n, &s, &c);
    return make_double2(c, s);
}

// The Bluestein operands at j: A = x_j c_j, then zeros; B = conj(c_m) at m and
// M - m for m < n, zeros between.
__device__ __forceinline__ double2 chirped(const Axis &a, const int64_t *off, int j)
{
    if (j >= a.n) return make_double2(0.0, 0.0);
    const double x = profile_value(a.prof, off, j);
    const double2 c = chirp(j, a.n);
    return make_double2(x * c.x, x * c.y);
}
__device__ __forceinline__ double2 chirp_filter(const Axis &a, int j)
{
    const int m = j < a.n ? j : (j > a.len - a.n ? a.len - j : -1);
    if (m < 0) return make_double2(0.0, 0.0);
    const double2 c = chirp(m, a.n);
    return make_double2(c.x, -c.y);
}

// S(k) = |Z(k)|^2 / (Lx Ly); S(0) = 0 exactly (the mean is subtracted by definition).
__device__ __forceinline__ void put_spectrum(const Axis &a, uint32_t k, double2 v, double norm)
{
    if (k <= (uint32_t)(a.n >> 1)) a.S[k] = k == 0 ? 0.0 : (v.x * v.x + v.y * v.y) * norm;
}

// A pass of kLog stages over whole transforms, blocks of L values (L = len for the
// first forward and the last undone pass): thread i of a transform takes the values at
// i0 + i + m L / 2^kLog.  The first forward pass makes its operands (off: the
// profile's offsets), the last undone one writes the spectrum.
template <int kLog, bool kUndo>
__device__ __forceinline__ void wide_pass(const Axis &a, const int64_t *off, int which, int t, int32_t L)
{
    const int step = L >> kLog;
    const int i = t & (step - 1);
    const size_t base = (size_t)(t - i) << kLog;  // block's first value
    double2 *buf = a.chirp ? (which ? a.B : a.A) : a.z;
    double2 x[1 << kLog];
    const bool make = !kUndo && L == a.len;
#pragma unroll
    for (int m = 0; m < (1 << kLog); ++m) {
        const size_t j = base + i + (size_t)m * step;
        if (!make)
            x[m] = buf[j];
        else if (!a.chirp)
            x[m] = make_double2(profile_value(a.prof, off, (int)j), 0.0);
        else
            x[m] = which ? chirp_filter(a, (int)j) : chirped(a, off, (int)j);
    }
    const double unit = 1.0 / step;
    stages<kLog, kUndo>(x, i, step, [&](int r, int l) { return twiddle(r, unit / (1 << l)); });
    const bool last = kUndo && L == a.len;
    const double inv = 1.0 / a.len;
#pragma unroll
    for (int m = 0; m < (1 << kLog); ++m) {
        const size_t j = base + i + (size_t)m * step;
        if (last)
            put_spectrum(a, (uint32_t)j, make_double2(x[m].x * inv, x[m].y * inv), a.norm);
        else
            buf[j] = x[m];
    }
}

// blockIdx.y: axis, blockIdx.z: operand of a chirped axis.  Pass number `pass`
// (counted from the whole transform down) of each axis that has one.
template <bool kUndo>
__global__ __launch_bounds__(kWideThreads) void fft_wide_kernel(Axes axes, int pass)
{
    const Axis &a = axes.ax[blockIdx.y];
    if (blockIdx.z && (!a.chirp || kUndo)) return;
    if (kUndo && !a.chirp) return;
    const int left = a.log2len - kTileLog - pass * kWideLog;  // wide stages from this pass on
    if (left <= 0) return;
    const int log = left < kWideLog ? left : kWideLog;
    const int32_t L = a.len >> (pass * kWideLog);
    if ((int)blockIdx.x * kWideThreads >= (a.len >> log)) return;  // whole workgroups
    const int t = blockIdx.x * kWideThreads + threadIdx.x;
    __shared__ int64_t off[kUndo ? 1 : kMaxBlocks + 1], lds[32];
    if (!kUndo && pass == 0 && blockIdx.z == 0) profile_offsets(a.prof, off, lds);
    switch (log) {
    case 1: wide_pass<1, kUndo>(a, off, blockIdx.z, t, L); break;
    case 2: wide_pass<2, kUndo>(a, off, blockIdx.z, t, L); break;
    case 3: wide_pass<3, kUndo>(a, off, blockIdx.z, t, L); break;
    default: wide_pass<4, kUndo>(a, off, blockIdx.z, t, L); break;
    }
}

// value i of a tile, one value of padding per eight: eight consecutive values per
// lane, and values a power of two apart, spread over the banks
__device__ __forceinline__ int slot(int i) { return i + (i >> 3); }

// The stages of a tile of T = 2^logT values in LDS, up to three at a time.  tw[j] =
// e^{-2 pi i j / T}, j < T / 2, so e^{-i pi r / h} = tw[r T / (2 h)].
template <int kLog, bool kUndo>
__device__ __forceinline__ void tile_pass(double2 *tile, const double2 *tw, int logT, int logL)
{
    const int T = 1 << logT, logstep = logL - kLog;
    for (int t = threadIdx.x; t < (T >> kLog); t += kFftThreads) {
        const int i = t & ((1 << logstep) - 1);
        const int base = (t - i) << kLog;
        double2 x[1 << kLog];
#pragma unroll
        for (int m = 0; m < (1 << kLog); ++m) x[m] = tile[slot(base + i + (m << logstep))];
        stages<kLog, kUndo>(x, i, 1 << logstep, [&](int r, int l) { return tw[r << (logT - 1 - logstep - l)]; });
#pragma unroll
        for (int m = 0; m < (1 << kLog); ++m) tile[slot(base + i + (m << logstep))] = x[m];
    }
    __syncthreads();
}

template <bool kUndo>
__device__ __forceinline__ void tile_stages(double2 *tile, const double2 *tw, int logT)
{
    const int rest = logT % 3;
    if (!kUndo) {
        int logL = logT;
        for (; logL >= 3; logL -= 3) tile_pass<3, false>(tile, tw, logT, logL);
        if (rest == 2) tile_pass<2, false>(tile, tw, logT, 2);
        if (rest == 1) tile_pass<1, false>(tile, tw, logT, 1);
    } else {
        if (rest == 2) tile_pass<2, true>(tile, tw, logT, 2);
        if (rest == 1) tile_pass<1, true>(tile, tw, logT, 1);
        for (int logL = rest + 3; logL <= logT; logL += 3) tile_pass<3, true>(tile, tw, logT, logL);
    }
}

// One tile (blockIdx.x) of axis blockIdx.y.  A plain axis: the remaining forward
// stages and the spectrum.  A chirped one: the remaining stages of both operands, their
// product, and the product's first undone stages (all of them, and the spectrum,
// if the transform is one tile).
__global__ __launch_bounds__(kFftThreads) void fft_tile_kernel(Axes axes)
{
    __shared__ double2 tile[kTile + kTile / 8], tw[kTile / 2];
    __shared__ int64_t off[kTile / kProfThreads + 1], lds[32];
    const Axis &a = axes.ax[blockIdx.y];
    const int logT = a.log2len < kTileLog ? a.log2len : kTileLog, T = 1 << logT;
    if ((int)blockIdx.x >= (a.len >> logT)) return;
    for (int j = threadIdx.x; j < (T >> 1); j += kFftThreads) tw[j] = twiddle(j, 2.0 / T);
    const size_t base = (size_t)blockIdx.x << logT;
    const bool whole = a.log2len <= kTileLog;  // no wide pass made the operands
    if (whole) profile_offsets(a.prof, off, lds);
    if (!a.chirp) {
        for (int i = threadIdx.x; i < T; i += kFftThreads) 
            tile[slot(i)] = whole ? make_double2(profile_value(a.prof, off, i), 0.0) : a.z[base + i];
        __syncthreads();
        tile_stages<false>(tile, tw, logT);
        for (int i = threadIdx.x; i < T; i += kFftThreads)
            put_spectrum(a, __brev((uint32_t)(base + i)) >> (32 - a.log2len), tile[slot(i)], a.norm);
        return;
    }
    constexpr int kEach = kTile / kFftThreads;
    double2 first[kEach];
    for (int i = threadIdx.x; i < T; i += kFftThreads) tile[slot(i)] = whole ? chirped(a, off, i) : a.A[base + i];
    __syncthreads();
    tile_stages<false>(tile, tw, logT);
#pragma unroll
    for (int e = 0; e < kEach; ++e) {
        const int i = threadIdx.x + e * kFftThreads;
        if (i < T) first[e] = tile[slot(i)];
    }
    __syncthreads();
    for (int i = threadIdx.x; i < T; i += kFftThreads) tile[slot(i)] = whole ? chirp_filter(a, i) : a.B[base + i];
    __syncthreads();
    tile_stages<false>(tile, tw, logT);
#pragma unroll
    for (int e = 0; e < kEach; ++e) {
        const int i = threadIdx.x + e * kFftThreads;
        if (i < T) tile[slot(i)] = cmul(first[e], tile[slot(i)]);
    }
    __syncthreads();
    tile_stages<true>(tile, tw, logT);
    const double inv = 1.0 / a.len;
    for (int i = threadIdx.x; i < T; i += kFftThreads) {
        const double2 x = tile[slot(i)];
        if (whole)
            put_spectrum(a, (uint32_t)i, make_double2(x.x * inv, x.y * inv), a.norm);
        else
            a.A[base + i] = x;
    }
}

int log2_exact(int64_t n)
{
    int l = 0;
    while ((int64_t(1) << l) < n) ++l;
    return l;
}

// The transforms and spectra of the axes in [first, first + count).
hipError_t launch_transforms(const Axes &axes, int count, hipStream_t st)
{
    int most = 0, undo = 0, z = 1;
    int64_t tiles = 1;
    for (int i = 0; i < count; ++i) {
        const Axis &a = axes.ax[i];
        const int wide = a.log2len > kTileLog ? (a.log2len - kTileLog + kWideLog - 1) / kWideLog : 0;
        most = wide > most ? wide : most;
        if (a.chirp) {
            undo = wide > undo ? wide : undo;
            z = 2;
        }
        const int64_t t = a.log2len > kTileLog ? a.len >> kTileLog : 1;
        tiles = t > tiles ? t : tiles;
    }
    auto wide_blocks = [&](int pass) {
        int64_t b = 1;
        for (int i = 0; i < count; ++i) {
            const int left = axes.ax[i].log2len - kTileLog - pass * kWideLog;
            if (left <= 0) continue;
            const int64_t n = (axes.ax[i].len >> (left < kWideLog ? left : kWideLog)) / kWideThreads;
            b = n > b ? n : b;
        }
        return (unsigned)b;
    };
    for (int pass = 0; pass < most; ++pass)
        hipLaunchKernelGGL(fft_wide_kernel<false>, dim3(wide_blocks(pass), count, z), dim3(kWideThreads), 0, st, axes,
                           pass);
    hipLaunchKernelGGL(fft_tile_kernel, dim3((unsigned)tiles, count), dim3(kFftThreads), 0, st, axes);
    for (int pass = undo - 1; pass >= 0; --pass)
        hipLaunchKernelGGL(fft_wide_kernel<true>, dim3(wide_blocks(pass), count, 1), dim3(kWideThreads), 0, st, axes,
                           pass);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_psd(const LatticeView &v, const PsdPlan &p, int64_t *rows, void *scratch, hipStream_t st)
{
    char *base = static_cast<char *>(scratch);
    int32_t *partial = reinterpret_cast<int32_t *>(base);
    int2 *rowpart = p.tall ? nullptr : reinterpret_cast<int2 *>(base + p.off_rowpart);
    const dim3 grid((v.Lx + kStripCols - 1) / kStripCols, p.nch), threads(kPlaneThreads);
    const bool vec = (v.W & 3) == 0;
    if (p.tall) {
        hipLaunchKernelGGL(clear_rows_kernel, dim3((unsigned)blocks_of(v.Ly)), dim3(kProfThreads), 0, st, rows, v.Ly);
        if (vec)
            hipLaunchKernelGGL((plane_kernel<true, true>), grid, threads, 0, st, v, p.R, partial, rowpart, rows);
        else
            hipLaunchKernelGGL((plane_kernel<false, true>), grid, threads, 0, st, v, p.R, partial, rowpart, rows);
    } else if (vec) {
        hipLaunchKernelGGL((plane_kernel<true, false>), grid, threads, 0, st, v, p.R, partial, rowpart, rows);
    } else {
        hipLaunchKernelGGL((plane_kernel<false, false>), grid, threads, 0, st, v, p.R, partial, rowpart, rows);
    }

    Profiles pr{};
    pr.v = v;
    pr.partial = partial;
    pr.rowpart = rowpart;
    pr.nch = p.nch;
    pr.prefix[0] = reinterpret_cast<int32_t *>(base + p.off_prefix);
    pr.prefix[1] = reinterpret_cast<int32_t *>(rows + v.Ly);
    pr.extra = rows;
    pr.nblk[0] = blocks_of(v.Lx);
    pr.nblk[1] = blocks_of(v.Ly);
    pr.blk[0] = reinterpret_cast<int64_t *>(base + p.off_blk);
    pr.blk[1] = pr.blk[0] + 2 * (size_t)pr.nblk[0];
    hipLaunchKernelGGL(profile_steps_kernel, dim3((unsigned)(pr.nblk[0] + pr.nblk[1])), dim3(kProfThreads), 0, st, pr);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;

    Axes axes{};
    double2 *conv = reinterpret_cast<double2 *>(base + p.off_conv);
    double *spec = reinterpret_cast<double *>(base + p.off_spec);
    for (int i = 0; i < 2; ++i) {
        Axis &a = axes.ax[i];
        a.n = i ? v.Ly : v.Lx;
        a.chirp = !pow2(a.n);
        a.len = a.chirp ? (int32_t)conv_len(a.n) : a.n;
        a.log2len = log2_exact(a.len);
        a.prof = Profile{pr.prefix[i], i ? pr.extra : nullptr, pr.blk[i], i ? v.Lx : 1, a.n, pr.nblk[i]};
        a.z = reinterpret_cast<double2 *>(base + (i ? p.off_zy : p.off_zx));
        a.A = conv;
        a.B = conv + a.len;
        if (p.together && a.chirp) conv += 2 * (size_t)a.len;
        a.S = i ? spec + v.Lx / 2 + 1 : spec;
        a.norm = 1.0 / ((double)v.Lx * (double)v.Ly);
    }
    if (p.together) return launch_transforms(axes, 2, st);
    e = launch_transforms(axes, 1, st);
    if (e != hipSuccess) return e;
    axes.ax[0] = axes.ax[1];
    return launch_transforms(axes, 1, st);
}

}  // namespace okpz
