// CPU check of the spectrum's scratch (csrc/psd_plan.h): over the supported sides the
// plan of okpz_psd stays within the documented bytes, the plan of okpz_psd_noalloc
// within its 24 MiB up to 2^17 a side, and no two pieces of a plan that are in use at
// the same time overlap.  Prints "psd plans ok" or the first size that fails.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "psd_plan.h"

using namespace okpz;

static void check(int64_t Lx, int64_t Ly)
{
    auto fail = [&](const char *what, size_t bytes, size_t bound) {
        std::printf("%lld x %lld: %s (%zu bytes, %zu allowed)\n", (long long)Lx, (long long)Ly, what, bytes, bound);
        std::exit(1);
    };
    // the figures of okpz.h, not the library's own function of them
    const size_t most = (size_t)std::max(Lx, Ly);
    const size_t bound = std::min<size_t>(size_t(32) << 20, (size_t)Lx * Ly / 4) + 40 * most +
                         (pow2(Lx) && pow2(Ly) ? 0 : 128 * most) + 2048;
    PsdPlan plans[2] = {psd_plan(Lx, Ly), psd_plan_capped(Lx, Ly, size_t(24) << 20)};
    if (plans[0].bytes > bound) fail("okpz_psd's scratch", plans[0].bytes, bound);
    const bool small = Lx <= 1 << 17 && Ly <= 1 << 17;
    if (small && plans[1].bytes > size_t(24) << 20) fail("okpz_psd_noalloc's scratch", plans[1].bytes, size_t(24) << 20);
    for (int i = 0; i < (small ? 2 : 1); ++i) {
        const PsdPlan &p = plans[i];
        if ((int64_t)p.R * p.nch < Ly || (int64_t)p.R * (p.nch - 1) >= Ly) fail("chunks", p.R, p.nch);
        const size_t strips = (size_t)((Lx + kStripCols - 1) / kStripCols);
        auto al = [](size_t b) { return (b + 255) / 256 * 256; };
        // plane pass: column parts, row parts, then what the profiles write
        const size_t rowpart = p.tall ? 0 : strips * (size_t)Ly * 8;
        if ((size_t)p.nch * Lx * 4 > p.off_rowpart) fail("column parts", (size_t)p.nch * Lx * 4, p.off_rowpart);
        if (p.off_rowpart + rowpart > p.off_spec) fail("row parts", p.off_rowpart + rowpart, p.off_spec);
        // a wavefront counts at most kMaxWaveRows rows before its counters are added up
        if (!p.tall && p.R / kPlaneWaves > kMaxWaveRows) fail("rows per wavefront", p.R / kPlaneWaves, kMaxWaveRows);
        // transforms: plain buffers, then the Bluestein pairs
        const size_t zx = pow2(Lx) ? (size_t)Lx * 16 : 0, zy = pow2(Ly) ? (size_t)Ly * 16 : 0;
        if (p.off_zx + zx > p.off_zy || p.off_zy + zy > p.off_conv) fail("transforms", p.off_zy, p.off_conv);
        const size_t bx = pow2(Lx) ? 0 : 2 * (size_t)conv_len(Lx) * 16, by = pow2(Ly) ? 0 : 2 * (size_t)conv_len(Ly) * 16;
        const size_t conv = p.together ? bx + by : std::max(bx, by);
        if (p.off_conv + conv > p.off_spec) fail("Bluestein buffers", p.off_conv + conv, p.off_spec);
        const size_t spec = (size_t)(Lx / 2 + 1 + Ly / 2 + 1) * 8;
        if (p.off_spec + spec > p.off_prefix) fail("spectra", p.off_spec + spec, p.off_prefix);
        if (p.off_prefix + (size_t)Lx * 4 > p.off_blk) fail("prefix", p.off_prefix, p.off_blk);
        if (p.off_blk + al(2 * 8 * ((size_t)blocks_of(Lx) + blocks_of(Ly))) > p.bytes) fail("blocks", p.off_blk, p.bytes);
    }
}

int main()
{
    std::vector<int64_t> sides;
    for (int k = 5; k <= 20; ++k) {
        const int64_t n = int64_t(1) << k;
        for (int64_t v : {n - 32, n, n + 32, n + n / 2, n + n / 2 - 32})
            if (v >= 32 && v <= int64_t(1) << 20 && v % 32 == 0) sides.push_back(v);
    }
    for (int64_t Lx : sides)
        for (int64_t Ly : sides) check(Lx, Ly);
    std::mt19937_64 rng(7);
    std::uniform_int_distribution<int64_t> any(1, 32768);
    for (int i = 0; i < 200000; ++i) check(32 * any(rng), 32 * any(rng));
    std::printf("psd plans ok\n");
    return 0;
}
