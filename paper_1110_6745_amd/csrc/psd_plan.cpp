#include "psd_plan.h"

namespace okpz {
namespace {

constexpr int64_t kRowStep = kPlaneWaves * kGroupRows;
constexpr int64_t kMaxRows = (int64_t)kPlaneWaves * kMaxWaveRows;

// Scratch layout for R rows per workgroup of the plane pass (a multiple of
// kPlaneWaves * kGroupRows).  The transforms take the place of the plane pass's
// parts, which are added up by then.  together: both axes'
// Bluestein buffers at once.  tall: PsdPlan::tall.
PsdPlan plan_with_rows(int64_t Lx, int64_t Ly, int64_t R, bool together, bool tall)
{
    PsdPlan p{};
    p.tall = tall;
    p.R = (int32_t)R;
    p.nch = (int32_t)((Ly + R - 1) / R);
    auto al = [](size_t b) { return (b + 255) / 256 * 256; };
    const size_t strips = (size_t)((Lx + kStripCols - 1) / kStripCols);
    p.off_rowpart = al((size_t)p.nch * Lx * 4);
    const size_t parts = p.off_rowpart + (tall ? 0 : al(strips * (size_t)Ly * 8));
    p.off_zx = 0;
    p.off_zy = pow2(Lx) ? al((size_t)Lx * 16) : 0;
    p.off_conv = p.off_zy + (pow2(Ly) ? al((size_t)Ly * 16) : 0);
    const size_t Mx = pow2(Lx) ? 0 : (size_t)conv_len(Lx), My = pow2(Ly) ? 0 : (size_t)conv_len(Ly);
    p.together = together || Mx == 0 || My == 0;
    const size_t conv = p.together ? Mx + My : (Mx > My ? Mx : My);
    const size_t work = p.off_conv + al(2 * conv * 16);
    p.off_spec = parts > work ? parts : work;
    p.off_prefix = p.off_spec + al((size_t)(Lx / 2 + 1 + Ly / 2 + 1) * 8);
    p.off_blk = p.off_prefix + al((size_t)Lx * 4);
    p.bytes = p.off_blk + al((2 * ((size_t)blocks_of(Lx) + blocks_of(Ly))) * 8);
    return p;
}

}  // namespace

PsdPlan psd_plan_capped(int64_t Lx, int64_t Ly, size_t max_bytes)
{
    // enough workgroups to fill the device, then fewer and taller ones until the
    // parts fit the bytes; both axes' transforms at once if they fit too
    const int64_t strips = (Lx + kStripCols - 1) / kStripCols;
    const int64_t chunks = (kPlaneTarget + strips - 1) / strips;
    const int64_t want = ((Ly + chunks - 1) / chunks + kRowStep - 1) / kRowStep * kRowStep;
    for (int64_t R = want < kMaxRows ? want : kMaxRows;; R = 2 * R < kMaxRows ? 2 * R : kMaxRows) {
        for (int together = 1; together >= 0; --together) {
            const PsdPlan p = plan_with_rows(Lx, Ly, R, together != 0, false);
            if (p.bytes <= max_bytes) return p;
        }
        if (R >= Ly || R >= kMaxRows) break;
    }
    // the parts of the rows (8 bytes per strip and row) or those of the columns at
    // kMaxRows rows are too many bytes: from about 2^35 sites on
    for (int64_t R = want;; R *= 2) {
        for (int together = 1; together >= 0; --together) {
            const PsdPlan p = plan_with_rows(Lx, Ly, R, together != 0, true);
            if (p.bytes <= max_bytes) return p;
            if (!together && R >= Ly) return p;  // the caller checks .bytes
        }
    }
}

size_t psd_scratch_bound(int64_t Lx, int64_t Ly)
{
    const size_t n = (size_t)Lx * Ly, most = (size_t)(Lx > Ly ? Lx : Ly);
    const size_t parts = n / 4 < (size_t(32) << 20) ? n / 4 : size_t(32) << 20;
    return parts + 40 * most + (pow2(Lx) && pow2(Ly) ? 0 : 128 * most) + 2048;
}

PsdPlan psd_plan(int64_t Lx, int64_t Ly) { return psd_plan_capped(Lx, Ly, psd_scratch_bound(Lx, Ly)); }

}  // namespace okpz
