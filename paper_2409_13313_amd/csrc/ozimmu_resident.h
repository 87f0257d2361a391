// Which tile the kernel with resident chunk sums (ozimmu_resident.hip) uses for which schedule: shared by the kernel and
// by the host code that chooses between the ways to run a schedule.
#pragma once
#include <cstdint>

namespace ozr {

constexpr int MIN_K = 3, MAX_K = 16;  // slice counts the kernel is built for

// chunks of the schedule of Algorithm 6 for k slices and chunks of at most r products
constexpr int num_chunks(int k, int r)
{
    int w = 0;
    for (int g = 2; g <= k + 1; ++g) w += (g - 2) / r + 1;
    return w;
}

// A wave holds ta x tb tiles of 16 x 16 for every chunk, a workgroup 2 x 2 waves; depth = inner steps of operands in
// LDS; waves = workgroups that share a compute unit.  ta == 0: no such kernel.
struct Config {
    int ta, tb, depth, waves;
};
constexpr int lds_bytes(int k, const Config& c) { return c.depth * k * (c.ta + c.tb) * 2048 + 128 * (c.ta + c.tb); }

// variant 0: the largest tile whose chunk sums fit the 256 accumulation registers; 1: a small one for outputs that
// the large one would not spread over the chip
constexpr Config config(int k, int r, int variant)
{
    const int w = num_chunks(k, r);
    Config c{0, 0, 1, 1};
    if (variant == 0) {
        if (w <= 4) c.ta = 4, c.tb = 4;
        else if (w <= 8) c.ta = 2, c.tb = 4;
        else if (w <= 16) c.ta = 2, c.tb = 2;
        else if (w <= 21) c.ta = 1, c.tb = 3;
        else if (w <= 32) c.ta = 1, c.tb = 2;
        else if (w <= 64) c.ta = 1, c.tb = 1;
    } else {
        if (w <= 8) c.ta = 2, c.tb = 2, c.waves = 2;
    }
    if (c.ta == 0) return c;
    c.depth = 2;
    if (c.waves * lds_bytes(k, c) > 160 * 1024) c.depth = 1;
    if (lds_bytes(k, c) > 160 * 1024) c.ta = 0;
    return c;
}

constexpr int NUM_VARIANTS = 2;

// Estimate of the kernel's time in microseconds on a chip of num_cu compute units; -1 where it cannot run.
// Measured on MI355X: an MFMA of the main loop takes 7.3 ns plus 0.022 ns for every byte of operands that the
// compute unit brings in per MFMA (60 bytes at k = 16, 85 at k = 8 with tiles of 64 x 128, 152 at w = 20 with tiles of 32 x 96:
// 8.8, 9.0 and 11.2 ns), and a round of tiles 2 us plus 0.8 us per 16 x 16 tile of a wave for its start values and for
// writing D (8 us at k = 8, 16 us at k = 4); two workgroups on a compute unit cover part of that for each other.
inline double estimate_us(int k, int r, int variant, int64_t m, int64_t n, int64_t p, int num_cu)
{
    if (k < MIN_K || k > MAX_K || (r < k && r != 8 && r != 4 && r != 2 && r != 1)) return -1.0;
    const Config c = config(k, r < k ? r : k, variant);
    if (c.ta == 0 || num_cu < 1) return -1.0;
    const int64_t steps = (n + 63) / 64;
    const int64_t tiles = ((m + 32 * c.ta - 1) / (32 * c.ta)) * ((p + 32 * c.tb - 1) / (32 * c.tb));
    if (tiles >= ((int64_t)1 << 23) || steps >= ((int64_t)1 << 17)) return -1.0;  // grid size; 32-bit operand offsets
    const double mfmas = 0.5 * k * (k + 1) * c.ta * c.tb;
    const double copied = 4096.0 * ((2 * (c.ta + c.tb) + 3) / 4) * k;   // bytes per step
    const double step_us = mfmas * (0.0073 + 2.2e-5 * copied / (4.0 * mfmas));
    const double round_us = c.waves == 2 ? 7.0 : 2.0 + 0.8 * c.ta * c.tb;
    const int64_t slots = (int64_t)num_cu * c.waves, full = tiles / slots, left = tiles % slots;
    double us = (double)full * (steps * step_us * c.waves + round_us);
    if (left > 0) us += steps * step_us * (left > num_cu ? c.waves : 1) + round_us;
    return us;
}

}  // namespace ozr
