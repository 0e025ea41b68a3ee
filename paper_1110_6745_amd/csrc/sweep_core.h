// Device side of one Monte Carlo sweep (Sec. II, Eq. (1)) for a group of
// device-level blocks of one lattice; shared by the per-lattice sweep kernel
// and the persistent batch kernel.
//
// A workgroup owns G blocks of one sweep (G = 1 for 256 x 256 blocks, more
// for smaller blocks so that a workgroup always holds about 1024 cells):
//   1. HBM -> LDS: each block's By rows of Bx sites are cut out of the
//      periodic lattice at the sweep's random shift (one-site granularity; a
//      funnel shift of two stored words per 32 sites) and expanded to one byte
//      per site;
//   2. C*C = 64 steps in LDS: per step one cell origin per block, one site per
//      8x8 thread cell, the four-bond test on three two-bit bytes and, when
//      accepted, three byte stores;
//   3. LDS -> HBM: bytes are packed back to bits and each block is written
//      *aligned* into the other lattice copy, whose stored columns start at
//      this sweep's shift.  No two workgroups write the same word, so the
//      store needs no atomics and the shift keeps one-site granularity.
//
// LDS byte of a site holds the complemented slope bits: bit 3 = nx
// (sigma_x = -1), bit 7 = ny (sigma_y = -1), bit 0 = block border (dead) marker.
// For the site s, its left neighbour l and lower neighbour d, a local minimum
// (-1 +1; -1 +1) has s = 0, nx in l and ny in d; a local maximum has s = 0x88
// and neither; a dead site is never 0 or 0x88.  Only lanes whose s is one of the
// two read l and d, and one multiplexer and one comparison then decide.  An
// accepted move rewrites the three bytes (s ^ 0x88, l ^ 0x08, d ^ 0x80).
// Within a step no other lane reads or writes those bytes (sites attempted
// together are never nearest or diagonal neighbours: each 8x8 cell has a dead
// row and column), so plain byte stores suffice.  The two bits sit four apart so
// that the expansion is one multiplication by 1 + 2^9 + 2^18 + 2^27 per four
// sites and the packing one byte dot product.
//
// The height of site (0,0) is tracked without touching the attempt loop: the
// threads staging the row of the block that contains it count the sigma_x bonds
// of the row's prefix in the packed words, before the steps and after them (the
// row's block-border site never moves).  (One thread counting the row's bytes in
// LDS took up to 7 us of the 22 us a sweep of one 256 x 256 block needed.)
//
// What bounds it: LDS.  Per attempt of 64 cells one full byte read (4.6 cycles of
// the CU's LDS, half of it two cell rows meeting in the same banks), two reads of
// the candidates (2 x 3.2) and three byte stores (4.45 each whatever the number
// of lanes: address and data of a wave take four cycles to reach the LDS) are
// 24.4 cycles, the staging about one, of the 27.8 measured at p = 1, q = 0 on
// 32768^2 (777 us per sweep; 797 us with five bits per byte, two dependent tests
// per attempt and 28 instead of 15 VALU cycles per four staged sites).  With
// acceptance draws it is VALU issue: 254 us per sweep of 16384^2 at p = 0.95,
// q = 0.05 (324 us when every fourth step computed its draws before its site
// address instead of in the waits of the four steps before).
#pragma once

#include "okpz_internal.h"

#include <type_traits>

namespace okpz {
namespace core {

constexpr int kMaxB = 256;
constexpr int kCellsMax = (kMaxB / 8) * (kMaxB / 8);  // cells a workgroup holds
constexpr int kSteps = 64;                             // C*C with C = 8
constexpr int kMaxGroup = 64;                          // blocks per group (32 x 32)
constexpr int kPitch = 256;                            // bytes per LDS tile row
// LDS tile of a group, for every block shape: a guard row, then rows of
// kPitch bytes in bands of By rows, each band holding 256 / Bx blocks side by
// side (block g in band g / (256 / Bx), column g mod (256 / Bx)).  Site (u, v)
// of block g sits at byte kPitch + base(g) | v << 8 | u, so an attempt's three
// bytes are one address plus the offsets 256, 255 and 0 whatever the block
// size.  A full group fills the 256 x 256 sites (G Bx By = 65536).  After the
// tile: 33 origin words (32 used; the pad puts the words of consecutive blocks
// in different LDS banks) and 3 placement words per block.
__host__ __device__ inline int tile_bytes(int Bx, int By, int G)
{
    const int bpb = kPitch / Bx;
    return kPitch + ((G + bpb - 1) / bpb) * By * kPitch;
}
constexpr int kGroupLds = kPitch + 65536 + kMaxGroup * 33 * 4 + kMaxGroup * 3 * 4;

// Acceptance modes: p = 1, q = 0 (pure growth); p and q each 0 or 1;
// general p, q (per-attempt acceptance draws).  kDelayedCells added to a
// mode selects the delayed thread-cell borders of Sec. II: every cell draws
// one of its 64 sites, and a step applies the attempts on cell-bulk sites,
// then those on cell edges, then those on cell corners, with a barrier
// after each phase.  kInPlace added to a mode stores the blocks back into
// the copy they were read from (one lattice copy; the launch holds no two
// horizontally adjacent blocks).  kEagerReads added to a mode reads a site's two
// neighbour bytes together with the site for every lane: one LDS round trip less
// per step for more LDS work, which pays where a workgroup has its CU to itself.
enum Mode : int { kGrowth = 0, kFixed = 1, kDraw = 2, kDelayedCells = 4, kInPlace = 8, kEagerReads = 16 };

__device__ __forceinline__ uint32_t funnel(uint32_t hi, uint32_t lo, uint32_t sh)
{
    return __builtin_amdgcn_alignbit(hi, lo, sh);
}

// Philox4x32-10 with the three-input XORs as single bit operations.
__device__ __forceinline__ Ctr4 philox10_dev(Ctr4 c, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int i = 0; i < 10; ++i) {
        const uint64_t m0 = (uint64_t)0xD2511F53u * c.x;
        const uint64_t m1 = (uint64_t)0xCD9E8D57u * c.z;
        const uint32_t n0 = (uint32_t)__builtin_amdgcn_bitop3_b32((uint32_t)(m1 >> 32), c.y, k0, 0x96);
        const uint32_t n2 = (uint32_t)__builtin_amdgcn_bitop3_b32((uint32_t)(m0 >> 32), c.w, k1, 0x96);
        c = Ctr4{n0, (uint32_t)m1, n2, (uint32_t)m0};
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

// Rounds [r0, r1) of Philox4x32-10 on state c (the key of round i is
// (k0 + i W0, k1 + i W1)); rounds 0..9 in order give philox10_dev.
template <int r0, int r1>
__device__ __forceinline__ void philox_rounds(Ctr4 &c, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int i = r0; i < r1; ++i) {
        const uint32_t ka = k0 + (uint32_t)i * 0x9E3779B9u, kb = k1 + (uint32_t)i * 0xBB67AE85u;
        const uint64_t m0 = (uint64_t)0xD2511F53u * c.x;
        const uint64_t m1 = (uint64_t)0xCD9E8D57u * c.z;
        const uint32_t n0 = (uint32_t)__builtin_amdgcn_bitop3_b32((uint32_t)(m1 >> 32), c.y, ka, 0x96);
        const uint32_t n2 = (uint32_t)__builtin_amdgcn_bitop3_b32((uint32_t)(m0 >> 32), c.w, kb, 0x96);
        c = Ctr4{n0, (uint32_t)m1, n2, (uint32_t)m0};
    }
}

// LDS byte of a site (complemented slope bits).
constexpr uint32_t kNx = 0x08u, kNy = 0x80u, kDead = 0x01u;
constexpr uint32_t kTop = kNx | kNy;  // a local maximum's byte; a minimum's is 0

// 32 sites of a row, bits to bytes.  x and y hold the nx and ny bits reversed
// (site u in bit 31 - u).  Word m of d gets sites 4m .. 4m+3.  A byte n with
// the sites' nx in its low and ny in its high half times 1 + 2^9 + 2^18 + 2^27
// puts bit 3 - i of n at bit 3 and bit 7 - i at bit 7 of byte i, and no two
// copies of n overlap (they are 9 bits apart), so one mask leaves the bytes.
__device__ __forceinline__ void expand32(uint32_t x, uint32_t y, uint32_t d[8])
{
    const uint32_t lo = __builtin_amdgcn_bitop3_b32(x, y << 4, 0x0F0F0F0Fu, 0xE4);
    const uint32_t hi = __builtin_amdgcn_bitop3_b32(x >> 4, y, 0x0F0F0F0Fu, 0xE4);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t a = lo >> (8 * k), b = hi >> (8 * k);
        d[7 - 2 * k] = (__umul24(a & 0xffu, 0x40201u) + (a << 27)) & 0x88888888u;
        d[6 - 2 * k] = (__umul24(b & 0xffu, 0x40201u) + (b << 27)) & 0x88888888u;
    }
}

// The inverse: the nx and ny bits (site u in bit u) of 32 site bytes.  The
// weighted byte sum of four sites, 8 * (nx bits) + 128 * (ny bits), holds
// their nx in bits 3..6 and their ny in bits 7..10.
__device__ __forceinline__ void pack32(const uint32_t d[8], uint32_t &x, uint32_t &y)
{
    uint32_t q[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        uint32_t p[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            p[k] = __builtin_amdgcn_udot4(d[4 * h + k] & 0x88888888u, 0x08040201u, 0u, false);
        // four bytes, each ny << 4 | nx of four sites
        q[h] = (((p[1] << 8) | p[0]) >> 3) | (((p[3] << 8) | p[2]) << 13);
    }
    // nibbles of q[0] (sites 0..15) and q[1]: even ones are nx, odd ones ny
    auto even = [](uint32_t v) {  // nibbles 0, 2, 4, 6 to the low half
        v &= 0x0F0F0F0Fu;
        v |= v >> 4;
        return __builtin_amdgcn_perm(v, v, 0x0C0C0200u);
    };
    x = even(q[0]) | (even(q[1]) << 16);
    y = even(q[0] >> 4) | (even(q[1] >> 4) << 16);
}

__device__ __forceinline__ int ilog2(uint32_t v) { return 31 - __builtin_clz(v); }

// Blocks per group for a block size: about 1024 cells per workgroup.
__host__ __device__ inline int group_size(int Bx, int By, int nblk)
{
    const int cpb = (Bx / 8) * (By / 8);
    int g = kCellsMax / cpb;
    if (g > kMaxGroup) g = kMaxGroup;
    if (g > nblk) g = nblk;
    return g < 1 ? 1 : g;
}

// Eq. (1) for a candidate site (byte s = 0, a possible minimum, or kTop, a
// possible maximum) with its left and lower neighbours' bytes l and d: a
// minimum needs nx in l and ny in d, a maximum neither.  The multiplexer (truth
// table 0xE4: c ? a : b) takes bit 3 from l and the others from d; below bit 3
// only the dead marker can be set.
template <int kMode>
__device__ __forceinline__ bool move_allowed(uint32_t s, uint32_t l, uint32_t d)
{
    uint32_t t = __builtin_amdgcn_bitop3_b32(l, d, kNx, 0xE4);
    if (kMode != kGrowth) t ^= s;
    return t >= kTop;
}

// Set the bits of *w selected by mask to those of v and keep the others; the
// caller guarantees that nobody else writes *w meanwhile.
__device__ __forceinline__ void put_bits(uint32_t *w, uint32_t v, uint32_t mask)
{
    *w = (*w & ~mask) | (v & mask);
}

// LDS atomic XOR of one byte (a 32-bit atomic on the byte's word).
__device__ __forceinline__ void xor_byte(uint8_t *smem, uint32_t off, uint32_t v)
{
    uint32_t *w = reinterpret_cast<uint32_t *>(smem + (off & ~3u));
    atomicXor(w, v << (8 * (off & 3u)));
}

// Origin of the cell grid in step 2m + odd of a block, (y << 8) | x, from the
// block's origin word m.
__device__ __forceinline__ uint32_t origin_yx(uint32_t w, int odd) { return odd ? w >> 16 : w & 0xffffu; }

// One sweep of blocks [b0, b0 + G) of the lattice described by `a`.
//   kFixedB = 256: 256 x 256 blocks, G = 1, static geometry;
//   kFixedB = 0:   block sides 32..256 (powers of two), geometry from `a`.
// Either way the three LDS addresses of an attempt are one register plus
// offsets (the tile layout above).
// kLaneOrg (kFixedB = 0 only): the group's cells are numbered as in one
// 256 x 256 block, so that a wave spans several blocks along a whole tile
// row and each lane fetches its block's origins (the launches use it below
// 128 x 128 sites per block); otherwise the cells of a block are consecutive
// and a wave's 64 cells share a block (needs Bx By >= 4096).
// smem: at least tile_bytes(Bx, By, G) bytes; opk: G * 36 words of LDS
// (origins, then the blocks' placement when kFixedB = 0).
// kStoreThrough: with a.store_through, write the new lattice with system-scope stores,
// which go through to memory instead of staying dirty in this XCD's L2 (the persistent
// kernel's hand-over to other XCDs then has little to write back).
template <int kThreads, int kModeFull, int kFixedB, bool kStoreThrough = false, bool kLaneOrg = false>
__device__ __forceinline__ void sweep_group(SweepLaunch a, const int b0, const int G,
                                            uint8_t *__restrict__ smem, uint32_t *opk)
{
    constexpr int kMode = kModeFull & 3;
    constexpr bool kDelayed = (kModeFull & kDelayedCells) != 0;
    constexpr bool kOneCopy = (kModeFull & kInPlace) != 0;
    constexpr bool kEager = (kModeFull & kEagerReads) != 0;
    constexpr bool kDrawAccept = (kMode == kDraw);
    constexpr int kCpt = kCellsMax / kThreads;
    constexpr int kOpkStride = kFixedB ? 32 : 33;  // origin words per block (one block: no pad)
    if (kFixedB) {
        a.Bx = kFixedB;
        a.By = kFixedB;
    }
    // opaque copy of the thread index: in the persistent batch kernel this
    // keeps the compiler from hoisting thread-constant values (counters,
    // cell offsets) out of the work loop, which would pin them in registers
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int Bx = a.Bx, By = a.By;
    const int wpr = Bx >> 5;
    const int lcpb = ilog2((uint32_t)((Bx >> 3) * (By >> 3)));
    const int ncx = Bx >> 3;
    const int lwpr = ilog2((uint32_t)wpr), lby = ilog2((uint32_t)By);
    const int lbpb = 8 - ilog2((uint32_t)Bx);  // 2^lbpb blocks side by side per band
    // offset of block g's first row in the tile, after the guard row
    auto tile_base = [&](int g) -> uint32_t {
        if (kFixedB) return 0u;
        return ((uint32_t)(g >> lbpb) << (8 + lby)) | ((uint32_t)(g & ((1 << lbpb) - 1)) << (8 - lbpb));
    };

    // Block id of group member g.  Groups number the blocks of the launch:
    // all blocks in row-major order, or, for a lattice updated in place, the
    // blocks of the launch's block columns col0, col0 + col_step, ... (ncol
    // of them per block row).
    auto block_id = [&](int g) -> int {
        const int l = b0 + g;
        if (!kOneCopy) return l;
        const int bj = l / a.ncol;
        return bj * a.nbx + a.col0 + (l - bj * a.ncol) * a.col_step;
    };

    // cell origins: one counter per pair of steps and block; word m of block
    // g holds step 2m in bytes 0 (x) and 1 (y), step 2m+1 in bytes 2 and 3
    // (three bits each).
    for (int e = tid; e < G * (kSteps / 2); e += kThreads) {
        const int g = e >> 5, m = e & 31;
        const Ctr4 r = philox10_dev(Ctr4{a.s, (uint32_t)block_id(g), (uint32_t)m, kTagOrigin}, a.k0,
                                    a.k1);
        opk[(e >> 5) * kOpkStride + (e & 31)] = (r.x >> 29) | ((r.y >> 29) << 8) | ((r.z >> 29) << 16) | ((r.w >> 29) << 24);
    }

    // ---- block placement -------------------------------------------------
    // Block bid = block_id(g) starts at lattice site (sx + bi Bx, sy + bj By); that
    // column sits at stored column xs of the source copy.  Per block: xs, the
    // first row and bi (the block's word column in the destination copy).
    auto place = [&](int g, int &xs, int &y0, int &bi) {
        const int bid = block_id(g);
        bi = bid % a.nbx;
        const int bj = bid / a.nbx;
        xs = a.sx + bi * Bx - a.ox_src;
        if (xs < 0) xs += a.Lx;
        y0 = a.sy + bj * By;
    };
    int fxs = 0, fy0 = 0, fbi = 0;
    int *geo = reinterpret_cast<int *>(opk + G * kOpkStride);
    if (kFixedB) {
        place(0, fxs, fy0, fbi);
    } else {
        for (int g = tid; g < G; g += kThreads) {
            int xs, y0, bi;
            place(g, xs, y0, bi);
            geo[3 * g] = xs;
            geo[3 * g + 1] = y0;
            geo[3 * g + 2] = bi;
        }
        __syncthreads();
    }

    // ---- HBM -> LDS with periodic wrap, bits -> bytes ---------------------
    // Element e: tile row R = e >> 3 (band R >> lby, block row v = R mod By)
    // and its 32-site piece c = e & 7 (block c >> lwpr of the band, word
    // k = c mod wpr of the block row): consecutive lanes fill consecutive
    // pieces of a tile row.  A thread handles the same elements at the load and
    // at the store.
    const int nrows = kFixedB ? kFixedB : (((G + (1 << lbpb) - 1) >> lbpb) << lby);
    const size_t plane = (size_t)a.Ly * a.W;

    // H0: the height of lattice site (0,0) moves by twice the change of the
    // sigma_x count of its block row's prefix.  The thread holding a piece of
    // that row counts the piece before the steps and after them.
    const int g00 = a.blk00 - b0;
    const bool has00 = (g00 >= 0 && g00 < G);  // uniform per workgroup
    auto prefix00 = [&](int g, int v, int k, uint32_t nx) -> int {  // sigma_x = -1 bonds of the prefix in this piece
        const int n = min(32, a.u00 - 32 * k);
        if (g != g00 || v != a.v00 || n <= 0) return 0;
        return __popc(nx & (~0u >> (32 - n)));
    };
    int pre00 = 0;

    auto load_words = [&](int e, uint32_t w[4]) {
        const int c = e & 7, R = e >> 3;
        const int k = c & (wpr - 1);
        const int v = R & (By - 1);
        const int g = kFixedB ? 0 : (((R >> lby) << lbpb) | (c >> lwpr));
        if (!kFixedB && g >= G) return;  // the unused end of a last band
        const int xs = kFixedB ? fxs : geo[3 * g];
        int y = (kFixedB ? fy0 : geo[3 * g + 1]) + v;
        if (y >= a.Ly) y -= a.Ly;
        int gw = (xs >> 5) + k;
        if (gw >= a.W) gw -= a.W;
        int gw1 = gw + 1;
        if (gw1 == a.W) gw1 = 0;
        const uint32_t *r0 = a.src + (size_t)y * a.W;
        const uint32_t *r1 = r0 + plane;
        w[0] = r0[gw];
        w[1] = r0[gw1];
        w[2] = r1[gw];
        w[3] = r1[gw1];
    };
    auto stage_words = [&](int e, const uint32_t w[4]) {
        const int c = e & 7, R = e >> 3;
        const int k = c & (wpr - 1);
        const int v = R & (By - 1);
        const int g = kFixedB ? 0 : (((R >> lby) << lbpb) | (c >> lwpr));
        if (!kFixedB && g >= G) return;
        const uint32_t off = (uint32_t)((kFixedB ? fxs : geo[3 * g]) & 31);
        const uint32_t bxw = ~funnel(w[1], w[0], off);  // nx bits
        const uint32_t byw = ~funnel(w[3], w[2], off);
        if (has00) pre00 += prefix00(g, v, k, bxw);
        uint32_t d[8];
        expand32(__brev(bxw), __brev(byw), d);
        if (v == 0) {  // row v = 0 is the block border (few waves take this)
#pragma unroll
            for (int m = 0; m < 8; ++m) d[m] |= 0x01010101u * kDead;
        }
        if (k == 0) d[0] |= kDead;  // column u = 0 is the block border
        uint4 *dst = reinterpret_cast<uint4 *>(smem + kPitch + R * kPitch + 32 * c);
        dst[0] = uint4{d[0], d[1], d[2], d[3]};
        dst[1] = uint4{d[4], d[5], d[6], d[7]};
    };
    if (kFixedB) {
        // all loads of the thread's elements in flight at once
        constexpr int kEl = kFixedB ? kFixedB * 8 / kThreads : 1;
        uint32_t w[kEl][4];
#pragma unroll
        for (int i = 0; i < kEl; ++i) load_words(tid + i * kThreads, w[i]);
#pragma unroll
        for (int i = 0; i < kEl; ++i) stage_words(tid + i * kThreads, w[i]);
    } else {
        for (int e = tid; e < nrows * 8; e += kThreads) {
            uint32_t w[4] = {0, 0, 0, 0};
            load_words(e, w);
            stage_words(e, w);
        }
    }
    __syncthreads();

    // ---- the thread's cells ----------------------------------------------
    // A cell beyond the group gets zero masks and tile 0, so its site is
    // always (0,0) of block 0, a dead-border site: its attempt is a no-op.
    const uint32_t mk = ((uint32_t)(By - 1) << 8) | (uint32_t)(Bx - 1);  // (v << 8) | u
    uint32_t clo[kCpt], chi[kCpt], mkj[kCpt], cid[kCpt], bidj[kCpt];
    uint32_t gj[kCpt];
    uint32_t opreg[kCpt];
    bool any_live = false;
#pragma unroll
    for (int j = 0; j < kCpt; ++j) {
        const int q = tid + j * kThreads;
        int g, c;
        if (kLaneOrg) {
            // cell q at column q mod 32 and row q / 32 of the tile's 32 x 32
            // cells, as in one 256 x 256 block, so that a wave's 64 cells span
            // a whole tile row (all LDS banks) instead of a few neighbouring
            // blocks (fewer banks); with the origin words padded to 33 per
            // block, the blocks a wave then touches read them from different
            // banks
            const int cc = q & 31, cr = q >> 5;
            const int lcx = ilog2((uint32_t)ncx), lcy = lcpb - lcx;
            g = ((cr >> lcy) << lbpb) | (cc >> lcx);
            c = ((cr & ((1 << lcy) - 1)) << lcx) | (cc & (ncx - 1));
        } else {
            g = q >> lcpb;
            c = q & ((1 << lcpb) - 1);
        }
        const bool live = g < G;
        any_live |= live;
        cid[j] = (uint32_t)c;
        bidj[j] = (uint32_t)block_id(live ? g : 0);
        // First site of the cell, (row << 8) | column (dead cell borders: the
        // active sites start one in), as its low seven bits and its top bit per
        // byte: sums of the low part with a site and an origin stay below 256 in
        // each byte, and the top bits are added modulo 256 by an XOR.
        const uint32_t first = ((uint32_t)((c / ncx) * 8) << 8 | (uint32_t)((c % ncx) * 8)) + (kDelayed ? 0u : 0x0101u);
        clo[j] = first & 0x7F7Fu;
        mkj[j] = live ? mk : 0u;
        // the block's place in the tile, in bits that mk masks off
        chi[j] = live ? (first & 0x8080u) | tile_base(g) : 0u;
        gj[j] = live ? (uint32_t)g : 0u;
        opreg[j] = opk[(live ? g : 0) * kOpkStride + (tid & 31)];
    }
    // Candidate bytes and acceptance: a minimum moves if its draw r < Tp, a
    // maximum if r < Tq, as r <= T - 1 in 32 bits; a kind that never moves
    // (T = 0) has no candidate byte.
    const uint32_t min_byte = (kMode == kGrowth || a.Tp != 0) ? 0u : 0xFFu;
    const uint32_t max_byte = a.Tq != 0 ? kTop : 0xFFu;
    const uint32_t tp1 = (uint32_t)(a.Tp - 1), tq1 = (uint32_t)(a.Tq - 1);
    (void)min_byte;
    (void)max_byte;
    (void)tp1;
    (void)tq1;

    // Site words of 8 steps come from one Philox call per cell; the call for
    // the next 8 steps is spread over the current ones (about 1.25 rounds
    // per step), where it fills the wait for each step's LDS reads.
    uint32_t sw[kCpt][4];
#pragma unroll
    for (int j = 0; j < kCpt; ++j) {
        const Ctr4 r = philox10_dev(Ctr4{a.s, bidj[j], cid[j], kTagSite}, a.k0, a.k1);
        sw[j][0] = r.x; sw[j][1] = r.y; sw[j][2] = r.z; sw[j][3] = r.w;
    }
    // Acceptance draws of 4 steps come from one Philox call per cell, computed
    // the same way one call ahead.
    uint32_t aw[kCpt][4];
    if (kDrawAccept) {
#pragma unroll
        for (int j = 0; j < kCpt; ++j) {
            const Ctr4 r = philox10_dev(Ctr4{a.s, bidj[j], cid[j], kTagAccept}, a.k0, a.k1);
            aw[j][0] = r.x; aw[j][1] = r.y; aw[j][2] = r.z; aw[j][3] = r.w;
        }
    }

    // The 64 steps.  kUni: the 64 lanes of a wave share a block, so the
    // origin words are read across lanes into scalar registers; otherwise
    // each lane reads its block's word of the next step pair from LDS during
    // the second step of the current pair.
    auto run_steps = [&](auto uni) __attribute__((always_inline)) {
        constexpr bool kUni = decltype(uni)::value;
        uint32_t opv[kCpt];
        if (!kUni) {
#pragma unroll
            for (int j = 0; j < kCpt; ++j) opv[j] = opk[gj[j] * kOpkStride];
        }
        // steps 8 gs .. 8 gs + 7; kMore: another group follows (its Philox calls are made here)
        auto step_group = [&](int gs, auto more) __attribute__((always_inline)) {
            constexpr bool kMore = decltype(more)::value;
            Ctr4 nxt[kCpt];
#pragma unroll
            for (int j = 0; j < kCpt; ++j)
                nxt[j] = Ctr4{a.s, bidj[j], ((uint32_t)(gs + 1) << 16) | cid[j], kTagSite};
            Ctr4 nxa[kCpt];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = gs * 8 + e;
                if (kDrawAccept && (e & 3) == 0) {
#pragma unroll
                    for (int j = 0; j < kCpt; ++j)
                        nxa[j] = Ctr4{a.s, bidj[j], ((uint32_t)((k >> 2) + 1) << 16) | cid[j], kTagAccept};
                }
                // all reads of the step first: the cells' byte sets are disjoint
                uint32_t off[kCpt], sv[kCpt], lv[kCpt], dv[kCpt];
                bool on_col[kCpt], on_row[kCpt];  // delayed borders: site in the cell's left column, bottom row
#pragma unroll
                for (int j = 0; j < kCpt; ++j) {
                    if (kUni && (e & 1) == 0) opv[j] = (uint32_t)__builtin_amdgcn_readlane((int)opreg[j], k >> 1);
                    const uint32_t h16 = (e & 1) ? (sw[j][e >> 1] >> 16) : (sw[j][e >> 1] & 0xffffu);
                    uint32_t site;  // (row << 8) | column within the cell
                    if (kDelayed) {
                        // site i = floor(64 h / 2^16) of the 8 x 8 cell: column
                        // i mod 8, row i div 8
                        const uint32_t i = h16 >> 10;
                        site = (i | (i << 5)) & 0x0707u;
                        on_col[j] = (i & 7u) == 0u;
                        on_row[j] = i < 8u;
                    } else {
                        // Active site i = floor(49 h / 2^16) of the 7 x 7 (row-major),
                        // split as i = 7 q + a without a division: with 7 h = q 2^16 + r,
                        // q = floor(7 h / 2^16) = i div 7 and a = floor(7 r / 2^16) = i mod 7.
                        // One byte permute packs bits 16..23 of the two products.
                        const uint32_t Y = __umul24(h16, 7u);
                        const uint32_t X = __umul24(Y & 0xffffu, 7u);
                        site = __builtin_amdgcn_perm(Y, X, 0x0C0C0602u);
                    }
                    // plus the grid's origin and the cell's first site, row and
                    // column mod the block sides, at the block's place in the tile
                    const uint32_t o = site + origin_yx(opv[j], e & 1) + clo[j];
                    off[j] = kFixedB ? (o ^ chi[j]) : __builtin_amdgcn_bitop3_b32(o, mkj[j], chi[j], 0x6A);
                    sv[j] = smem[off[j] + kPitch];
                    if (kEager) {
                        lv[j] = smem[off[j] + kPitch - 1];
                        dv[j] = smem[off[j]];
                    }
                    // behind the site read of a pair's second step: the next
                    // pair's origin word (the last pair reads its own again)
                    if (!kUni && (e & 1) == 1) opv[j] = opk[gj[j] * kOpkStride + min((k >> 1) + 1, kSteps / 2 - 1)];
                }
                // While the reads are in flight: this step's share of the next
                // Philox calls, pinned here so that it is not sunk to its use.
                // It is filler work: at low wave priority, so that waves whose
                // step chain can go on (towards the step barrier) issue first.
                __builtin_amdgcn_s_setprio(0);
#pragma unroll
                for (int j = 0; j < kCpt; ++j) {
                    if (kMore) {
                        switch (e) {  // rounds 0,1 | 1,2 | 2,3 | 3,5 | 5,6 | 6,7 | 7,8 | 8,10
                        case 0: philox_rounds<0, 1>(nxt[j], a.k0, a.k1); break;
                        case 1: philox_rounds<1, 2>(nxt[j], a.k0, a.k1); break;
                        case 2: philox_rounds<2, 3>(nxt[j], a.k0, a.k1); break;
                        case 3: philox_rounds<3, 5>(nxt[j], a.k0, a.k1); break;
                        case 4: philox_rounds<5, 6>(nxt[j], a.k0, a.k1); break;
                        case 5: philox_rounds<6, 7>(nxt[j], a.k0, a.k1); break;
                        case 6: philox_rounds<7, 8>(nxt[j], a.k0, a.k1); break;
                        default: philox_rounds<8, 10>(nxt[j], a.k0, a.k1); break;
                        }
                        asm volatile("" : "+v"(nxt[j].x), "+v"(nxt[j].y), "+v"(nxt[j].z), "+v"(nxt[j].w));
                    }
                    if (kDrawAccept && (kMore || e < 4)) {
                        switch (e & 3) {  // the call for steps k + 4 ..
                        case 0: philox_rounds<0, 3>(nxa[j], a.k0, a.k1); break;
                        case 1: philox_rounds<3, 5>(nxa[j], a.k0, a.k1); break;
                        case 2: philox_rounds<5, 8>(nxa[j], a.k0, a.k1); break;
                        default: philox_rounds<8, 10>(nxa[j], a.k0, a.k1); break;
                        }
                        asm volatile("" : "+v"(nxa[j].x), "+v"(nxa[j].y), "+v"(nxa[j].z), "+v"(nxa[j].w));
                    }
                }
                bool up[kCpt], down[kCpt];  // the acceptance draws
                if (kDrawAccept) {
#pragma unroll
                    for (int j = 0; j < kCpt; ++j) {
                        up[j] = aw[j][e & 3] <= tp1;
                        down[j] = aw[j][e & 3] <= tq1;
                    }
                }
                __builtin_amdgcn_s_setprio(2);
                // Only a site at a local minimum (byte 0) or maximum (kTop) whose
                // draw accepts can move; only those lanes read the two neighbour
                // bytes (all lanes did, with the site, if kEager).
                auto candidate = [&](int j) -> bool {
                    if (kMode == kGrowth) return sv[j] == 0u;
                    if (kMode == kFixed) return (sv[j] == min_byte) | (sv[j] == max_byte);
                    return ((sv[j] == min_byte) & up[j]) | ((sv[j] == max_byte) & down[j]);
                };
                if (kDelayed) {
                    // Three phases.  Within one, attempted sites are never nearest
                    // neighbours.  Bulk sites are not diagonal neighbours either
                    // (as in the dead-border steps), and corners are 8 apart, so
                    // plain byte stores suffice there; an edge site and the edge
                    // site diagonally up and to the left of it (the next cell's
                    // bottom row) can share a neighbour byte, so edge flips are
                    // atomic XORs (plain stores with atomics for that pair only
                    // measured slower: 30.8 against 26.4 ms at 2^17).
                    // Every phase uses the site byte read above: a site's own byte
                    // changes only by a move at the site, at its right neighbour
                    // or at its upper neighbour.  For a bulk site those are its
                    // own cell's sites or a later-phase site of the next cell
                    // (edge); for an edge site, its own cell's or the next
                    // cell's corner; for a corner, its own cell's.  A cell
                    // attempts one site per step, so no move of an earlier
                    // phase touches the byte of a later-phase site.
                    bool cand[kCpt];
#pragma unroll
                    for (int j = 0; j < kCpt; ++j) cand[j] = candidate(j);
#pragma unroll
                    for (int ph = 0; ph < 3; ++ph) {
#pragma unroll
                        for (int j = 0; j < kCpt; ++j) {
                            const bool now = ph == 0 ? !(on_col[j] || on_row[j]) : ph == 1 ? on_col[j] != on_row[j] : on_col[j] && on_row[j];
                            if (!(cand[j] && now)) continue;
                            const bool read = !kEager || ph != 0;
                            uint32_t l0 = read ? smem[off[j] + kPitch - 1] : lv[j];
                            uint32_t d0 = read ? smem[off[j]] : dv[j];
                            // the loads zero-extend; keep the code generator from
                            // re-masking the bytes
                            asm volatile("" : "+v"(l0), "+v"(d0));
                            if (!move_allowed<kMode>(sv[j], l0, d0)) continue;
                            if (ph == 1) {
                                xor_byte(smem, off[j] + kPitch, kTop);
                                xor_byte(smem, off[j] + kPitch - 1, kNx);
                                xor_byte(smem, off[j], kNy);
                            } else {
                                smem[off[j] + kPitch] = (uint8_t)(sv[j] ^ kTop);
                                smem[off[j] + kPitch - 1] = (uint8_t)(l0 ^ kNx);
                                smem[off[j]] = (uint8_t)(d0 ^ kNy);
                            }
                        }
                        __syncthreads();
                    }
                } else {
                    bool cand[kCpt];
#pragma unroll
                    for (int j = 0; j < kCpt; ++j) {
                        asm volatile("" : "+v"(sv[j]));
                        cand[j] = candidate(j);
                        if (!kEager && cand[j]) {
                            lv[j] = smem[off[j] + kPitch - 1];
                            dv[j] = smem[off[j]];
                        }
                    }
#pragma unroll
                    for (int j = 0; j < kCpt; ++j) {
                        if (!cand[j]) continue;
                        asm volatile("" : "+v"(lv[j]), "+v"(dv[j]));
                        if (move_allowed<kMode>(sv[j], lv[j], dv[j])) {
                            // a growth flip only ever turns 0 (minimum) into kTop
                            smem[off[j] + kPitch] = (kMode == kGrowth) ? (uint8_t)kTop : (uint8_t)(sv[j] ^ kTop);
                            smem[off[j] + kPitch - 1] = (uint8_t)(lv[j] ^ kNx);
                            smem[off[j]] = (uint8_t)(dv[j] ^ kNy);
                        }
                    }
                    __syncthreads();
                }
                if (kDrawAccept && (e & 3) == 3) {
#pragma unroll
                    for (int j = 0; j < kCpt; ++j) {
                        aw[j][0] = nxa[j].x; aw[j][1] = nxa[j].y; aw[j][2] = nxa[j].z; aw[j][3] = nxa[j].w;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < kCpt; ++j) {
                sw[j][0] = nxt[j].x; sw[j][1] = nxt[j].y; sw[j][2] = nxt[j].z; sw[j][3] = nxt[j].w;
            }
        };
        // the last group apart: no branch inside a step
        for (int gs = 0; gs < kSteps / 8 - 1; ++gs) step_group(gs, std::true_type{});
        step_group(kSteps / 8 - 1, std::false_type{});
    };
    // A group of fewer than 1024 cells leaves whole waves without one.  They only
    // keep the barriers (one per step, three with delayed borders): on 32 x 32
    // 9.8 us per sweep against 12.6 us, on 96 x 96 11.9 against 13.0 us.
    if (kFixedB || __ballot(any_live) != 0) {
        run_steps(std::integral_constant<bool, kFixedB != 0 || !kLaneOrg>{});
    } else {
        for (int k = 0; k < kSteps * (kDelayed ? 3 : 1); ++k) __syncthreads();
    }

    // the store below is not on any step's critical path: back to low
    // priority, behind the steps of a co-resident workgroup
    __builtin_amdgcn_s_setprio(0);

    // ---- LDS -> HBM: bytes -> bits, aligned into the other copy -----------
    // (elements as in the load above)
    auto store_piece = [&](int e) {
        const int c = e & 7, R = e >> 3;
        const int k = c & (wpr - 1);
        const int v = R & (By - 1);
        const int g = kFixedB ? 0 : (((R >> lby) << lbpb) | (c >> lwpr));
        if (!kFixedB && g >= G) return;
        const int bi = kFixedB ? fbi : geo[3 * g + 2];
        int y = (kFixedB ? fy0 : geo[3 * g + 1]) + v;
        if (y >= a.Ly) y -= a.Ly;
        const uint4 *src = reinterpret_cast<const uint4 *>(smem + kPitch + R * kPitch + 32 * c);
        const uint4 q0 = src[0], q1 = src[1];
        const uint32_t d[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
        uint32_t bxw, byw;
        pack32(d, bxw, byw);
        if (has00) pre00 -= prefix00(g, v, k, bxw);
        const size_t col = (size_t)bi * wpr + k;
        if (kOneCopy) {
            // One lattice copy: the block goes back where it was read from,
            // its row segment starting at stored column xs (off = xs mod 32
            // is the same for every block of the sweep).  Blocks cover
            // disjoint sites and a block reads and writes only its own, so no
            // block sees another's update.  Segment word k takes tile word k
            // shifted up by off plus the top off bits of tile word k-1 (the
            // previous lane's).  The segment's first and one-past-last words
            // are shared with the left and right neighbour blocks, which the
            // host never puts in the same launch, so a plain read-modify-write
            // replaces only this block's bits.  With one block per row those
            // two words are one word, all of it this block's: the first lane
            // writes it whole, with the last lane's top bits.
            const int xs = kFixedB ? fxs : geo[3 * g];
            const uint32_t off = (uint32_t)(xs & 31);
            const uint32_t nx = ~bxw, ny = ~byw;
            const uint32_t px = __shfl_up(nx, 1, 64), py = __shfl_up(ny, 1, 64);
            const uint32_t lx = __shfl_down(nx, wpr - 1, 64), ly = __shfl_down(ny, wpr - 1, 64);
            uint32_t *rx = a.dst + (size_t)y * a.W, *ry = a.dst + ((size_t)a.Ly + y) * a.W;
            int gw = (xs >> 5) + k;
            if (gw >= a.W) gw -= a.W;
            if (off == 0) {
                rx[gw] = nx;
                ry[gw] = ny;
            } else if (k != 0) {
                rx[gw] = (nx << off) | (px >> (32 - off));
                ry[gw] = (ny << off) | (py >> (32 - off));
            } else if (a.nbx == 1) {
                rx[gw] = (nx << off) | (lx >> (32 - off));
                ry[gw] = (ny << off) | (ly >> (32 - off));
            } else {
                put_bits(rx + gw, nx << off, ~0u << off);
                put_bits(ry + gw, ny << off, ~0u << off);
            }
            if (k == wpr - 1 && off != 0 && a.nbx != 1) {
                int gl = gw + 1;
                if (gl == a.W) gl = 0;
                put_bits(rx + gl, nx >> (32 - off), (1u << off) - 1u);
                put_bits(ry + gl, ny >> (32 - off), (1u << off) - 1u);
            }
            return;
        }
        uint32_t *w0 = a.dst + (size_t)y * a.W + col, *w1 = w0 + plane;
        if (kStoreThrough && a.store_through) {
            __hip_atomic_store(w0, ~bxw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            __hip_atomic_store(w1, ~byw, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        } else {
            *w0 = ~bxw;  // back to sigma = +1 bits
            *w1 = ~byw;
        }
    };
    if (kFixedB) {
#pragma unroll
        for (int i = 0; i < (kFixedB ? kFixedB * 8 / kThreads : 1); ++i) store_piece(tid + i * kThreads);
    } else {
        for (int e = tid; e < nrows * 8; e += kThreads) store_piece(e);
    }
    // few lanes of one workgroup (a piece's change is at most 32 bonds)
    if (has00 && pre00 != 0)
        atomicAdd(reinterpret_cast<unsigned long long *>(a.h0), (unsigned long long)(2 * (int64_t)pre00));
}

}  // namespace core
}  // namespace okpz
