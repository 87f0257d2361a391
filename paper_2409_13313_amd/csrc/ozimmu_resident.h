// Which tile the kernel with resident chunk sums (ozimmu_resident.hip) uses for which schedule: shared by the kernel and
// by the host code that chooses between the ways to run a schedule.
#pragma once
#include "ozimmu_layout.h"
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
// LDS; waves = workgroups that share a compute unit; held = slices of A that k_held keeps in registers at a time (the other kernels:
// 0).  ta == 0: no such kernel.
struct Config {
    int ta, tb, depth, waves, held = 0;
};
// (k_held fetches slices 2 .. k - held of B twice a step, early and late: a second place each, or their copies had no time)
constexpr int lds_bytes(int k, const Config& c)
{
    return c.depth * k * (c.ta + c.tb) * 2048 + (c.held ? (k - c.held - 1) * c.tb * 2048 : 0) + 128 * (c.ta + c.tb);
}

constexpr int ACC_TILES = 64;    // tiles of 16 x 16 that the accumulation registers of a wave hold
constexpr int NUM_VARIANTS = 7, EXTENDED = 6;  // the last one is k_extended, the others k_resident
constexpr int HELD = 16;         // k_held, beside them
constexpr bool is_variant(int v) { return (v >= 0 && v < NUM_VARIANTS) || v == HELD; }
// for (int v = 0; is_variant(v); v = next_variant(v)): all of them, k_held last
constexpr int next_variant(int v) { return v + 1 == NUM_VARIANTS ? HELD : v + 1; }

// variant 0: the largest tile whose chunk sums fit the 256 accumulation registers; the others: smaller ones for outputs that
// the large one would not spread evenly over the chip; EXTENDED: the next larger tile whose chunk sums fit the ordinary registers
// too, beside fragments (those of the low slices and of two high ones) and about 24 more.  Shapes in the order of what they move per MFMA;
// others that fit (96 x 96, 64 x 160, 32 x 128) were no faster in k_extended.
constexpr Config config(int k, int r, int variant)
{
    const int w = num_chunks(k, r);
    Config c{0, 0, 1, 1};
    if (w <= 4) c.ta = 4, c.tb = 4;
    else if (w <= 8) c.ta = 2, c.tb = 4;
    else if (w <= 16) c.ta = 2, c.tb = 2;
    else if (w <= 21) c.ta = 1, c.tb = 3;
    else if (w <= 32) c.ta = 1, c.tb = 2;
    else if (w <= ACC_TILES) c.ta = 1, c.tb = 1;
    const int area = c.ta * c.tb;  // 16 x 16 tiles of a wave in the largest tile
    if (variant == HELD) {
        // The largest tile, in the order of what they move per MFMA, whose sums, held slices of A and two slices of B fit the registers (26
        // others), if it is larger than k_resident's and k_extended's.  An odd number held: see the kernel's order of a step.
        constexpr int shapes[4][2] = {{4, 4}, {3, 4}, {3, 3}, {2, 4}}, last[2] = {2, 3};
        const Config e = config(k, r, EXTENDED);
        const int least = e.ta * e.tb > area ? e.ta * e.tb : area;
        c.ta = 0;
        if (k < 5 || r == 1 || w > 26) return c;
        for (int x = 0; x < 5 && c.ta == 0; ++x) {
            const int ta = x < 4 ? shapes[x][0] : last[0], tb = x < 4 ? shapes[x][1] : last[1];
            for (int held = ((k + 1) / 2) | 1; held < k && c.ta == 0; held += 2) {
                const Config h{ta, tb, 1, 1, held};
                if (ta * tb > least && 4 * (w * ta * tb + held * ta + 2 * tb) + 26 <= 512 && lds_bytes(k, h) <= 160 * 1024) c = h;
            }
        }
        return c;
    }
    if (variant == EXTENDED) {
        constexpr int shapes[8][2] = {{4, 4}, {3, 4}, {2, 4}, {2, 3}, {2, 2}, {1, 3}, {1, 2}, {1, 1}};
        c.ta = 0;
        for (int x = 0; x < 8 && c.ta == 0; ++x) {
            const int ta = shapes[x][0], tb = shapes[x][1];
            const int more = 4 * (w * ta * tb - ACC_TILES), frag = 4 * (ta + tb) * ((k + 1) / 2 + 2);
            if (ta == 3 && k < 5) continue;  // (no faster: few MFMAs a step, 96 x 128 outputs to write)
            if (ta * tb > area && (more > 0 ? more : 0) + frag + 24 <= 256) c.ta = ta, c.tb = tb;
        }
    } else if (variant > 0) {
        const int ta = variant == 1 || variant == 2 ? 2 : 1, tb = variant == 1 ? 2 : variant == 2 || variant == 3 ? 3 : variant == 4 ? 2 : 1;
        c.ta = 0;
        if (w * ta * tb > ACC_TILES || (ta * tb >= area && !(w > 8 && ta * tb == 6))) return c;
        c.ta = ta, c.tb = tb;
        // two workgroups on a compute unit where the registers (accumulators; fragments of the low slices and of two high
        // ones, and about 25 more) and the LDS allow it
        const int frag = 4 * (ta + tb) * ((k + 1) / 2 + 2);
        if (w * ta * tb <= 32 && frag + 25 <= 128 && 2 * k * (ta + tb) * 2048 <= 158 * 1024) c.waves = 2;
    }
    c.depth = 2;
    if (c.waves * lds_bytes(k, c) > 160 * 1024) c.depth = 1;
    if (lds_bytes(k, c) > 160 * 1024) c.ta = 0;
    return c;
}

// config() of what the kernel is built for; ta == 0 for anything else
constexpr Config config_for(int k, int r, int variant)
{
    if (k < MIN_K || k > MAX_K || (r < k && r != 8 && r != 4 && r != 2 && r != 1)) return Config{0, 0, 1, 1};
    return config(k, r < k ? r : k, variant);
}
// Tiles for slices with one scale each (r = 1; k_per_slice): k_extended's only where there is no other.
constexpr bool per_slice_tile(int k, int variant) { return variant < EXTENDED || (variant == EXTENDED && config(k, 1, 0).ta == 0); }
// grid size; 32-bit operand offsets: a tile's rows lie in two row blocks at most, and an offset from the first one's begin is less than both
// of them (k_held; the others' are from a copy's own rows)
constexpr int64_t MAX_STEPS = ((int64_t)1 << 17) - 1;
static_assert(2 * (MAX_STEPS + 1) * ozl::TILE_BYTES + 2 * ozl::ROWPAD <= ((int64_t)1 << 32) && (MAX_STEPS + 1) % (ozl::KPAD / ozl::TILE_K) == 0, "");
constexpr bool in_range(int64_t m, int64_t n, int64_t p, int rows, int cols)
{
    return ((m + rows - 1) / rows) * ((p + cols - 1) / cols) < ((int64_t)1 << 23) && (n + 63) / 64 <= MAX_STEPS;
}

// Rows of the output that do not begin on 64 bytes leave pieces of lines at every tile's edge.  Streamed past L2 (non-temporal
// stores, 1 to 2 % faster for whole lines: 3000 x 64 x 3000, k = 4, 29.3 us, kept in L2 29.9) they are merged in memory, at a quarter of its
// rate; kept in L2 until the neighbouring tile has written the rest they are not: 6272 x 56 x 2842, k = 3, 98 -> 48 us,
// 3439 x 62 x 3552 into rows of 3553, k = 6, 74 -> 49, 2633 x 83 x 5709, k = 8, 113 -> 87.  Where the output is a small part of the work,
// what that evicts costs as much (pairs times inner steps at 3000 x 3003: 576, k = 8, n = 1024, 238.5 -> 234.4 us; 672,
// k = 6, n = 2048, 286.8 -> 276.5; 1152, k = 8, n = 2048, 443.8 -> 447.6; 1248, k = 12, n = 1024, 450 -> 454).
//
// What stays in L2 stays in the memory-side cache behind it too.  Where output, operands and slices (all of their padding is
// written) exceed its 256 MB, the operands of the next call and the slices of this one are evicted for it: 97567 x 95 x 106, k = 7, 148 us
// streamed and 158 kept; 68693 x 119 x 285, k = 8, 183 and 191; 280 x 3 x 77204, k = 12, 185 and 195.  It then pays only where the
// merging in memory, at 1.35 bytes per ps, is what the kernel waits for: 249 x 3 x 117287, k = 9, 301 and 262 us; 471 x 14 x
// 57084, k = 5, one addition per pair, 154 and 148; 374 x 114 x 84687, k = 4, per pair, with 78 MB of operands to evict, 210 and 167.
// us: the kernel's estimate.
constexpr bool may_merge_rows(int k, int64_t n) { return (int64_t)k * (k + 1) / 2 * ((n + 63) / 64) <= 700; }
inline bool merge_rows(int k, int64_t m, int64_t n, int64_t p, double us)
{
    if (!may_merge_rows(k, n)) return false;
    const double out = 8.0 * (double)m * (double)p, vectors = (double)m + (double)p, operands = 8.0 * vectors * (double)n;
    const double slices = vectors * (double)ozl::inner_padded(n) * k;
    return out + operands + slices <= 256e6 || out / 1.35e6 >= us * (operands > out / 8.0 ? 1.2 : 0.95);
}

// Tiles whose inner dimension may be cut among workgroups (k_cut): the smallest, which leave the fewest sums to exchange (at 15
// shapes of 41 to 1000 rows and columns one of these two was the best or within 4 % of it).
constexpr bool may_cut(int variant, const Config& c) { return variant < EXTENDED && c.ta * c.tb >= 1 && c.ta * c.tb <= 2; }
// Bytes of the chunk sums of `tiles` tiles (k_add_parts).
inline int64_t sums_bytes(int k, int r, const Config& c, int64_t tiles)
{
    return tiles * num_chunks(k, r < k ? r : k) * c.ta * c.tb * 4096;
}
// z_groups of k_add_parts: threads that share the parts of an element
constexpr int z_groups(int parts) { return parts > 8 ? 16 : 4; }
// What writing and adding the sums takes: every chunk costs a store in k_cut and a load and an addition in k_add_parts, one after the other
// (fitted to 8000 timings of 720 shapes of 500 to 60000 inner positions: four that are cut are slower than whole, by 2 to 6 %.  With
// the turns of the loop alone and a larger constant 24 were: 8 x 2054 x 8, k = 10, one addition per pair, 31.2 us whole, 45.2 in
// four parts; 33 x 3385 x 232 44.6 and 53.9; 44 x 1909 x 1, k = 7, 19.3 and 23.3 with its split).
inline double add_parts_us(int k, int r, const Config& c, int64_t tiles, int parts)
{
    const int zg = z_groups(parts), batch = zg == 4 ? 8 : 4, w = num_chunks(k, r < k ? r : k);
    const double trips = (double)((parts + zg - 1) / zg) * ((w + batch - 1) / batch);
    return 2.5 + 1.0 * trips + 0.3 * w + (double)sums_bytes(k, r, c, tiles) / 2.5e6;
}

// Estimate of the kernel's time in microseconds on a chip of num_cu compute units; -1 where it cannot run.
// Measured on MI355X: an inner step of a workgroup that has its compute unit to itself takes 7.5 ns per MFMA of a wave plus
// 0.1 to 0.2 us (k = 8, tiles of 64 x 64: 1.16 us, 32 x 32: 0.5 us; 64 x 128: 2.4 us; k = 4, 128 x 128: 1.42 us), one of two workgroups
// that share it 8.4 ns per MFMA of both plus 0.2 us; with several rounds of tiles the former becomes 0.27 us (32 x 32: 0.2; w = 45
// 0.52 us a step, 32 x 64 0.95).  A round of
// tiles adds start values, the first operands and the writing of D: 4 us plus 0.4 us per 16 x 16 tile of a wave.  Calls of
// milliseconds run at the clock the power budget leaves, and what an MFMA costs then grows with the bytes that are moved
// for it (4096^3: k = 9, 64 x 96 against 64 x 64 with half the fetches more, 1.85 and 1.91 ms; k = 10, 2.25 and 2.28;
// k = 5, two workgroups of 64 x 96 against one of 64 x 128, 0.75 and 0.80): 6.8 ns plus 0.02 ns per byte of operands that the
// compute unit brings in plus 5 ns per KiB of fragments that a wave fetches from LDS (k = 16, 64 x 64: 60 bytes, 0.12 KiB,
// 8.8 ns; k = 8, 64 x 128: 85, 0.17, 9.0; w = 20, 32 x 96: 152, 0.30, 11.2).  Two workgroups on a compute unit fill each
// other's barriers: 0.6 ns less (k = 5, two of 64 x 96 against one of 64 x 128: 5.44 and 5.94 ms at 8192^3, 44.0 and 46.4 at
// 16384^3; k = 8, two of 64 x 64 against one of 64 x 128: 11.84 and 11.44 at 8192^3, and the estimate keeps the latter).
// (The first of the two prices is used up to 1500 us: they differ there by 10 % for 64 x 128, k = 8, less for smaller tiles.)
//
// A step of few MFMAs waits for its operands instead.  How long depends on where they come from: the memory-side cache
// ("near") while it holds the operands and their slices (256 MiB), else memory ("far").  And on the ring: a copy has two thirds of a step to
// arrive with one step in LDS, one and a half with two (us a step, near / far: one, 40 KiB 0.6 / 0.9, 48 KiB 0.7 / 1.03, two
// intervals (k <= 4) 0.93 / 1.36; two, 12 KiB 0.2 / 0.33, 24 KiB 0.25 / 0.42, 48 KiB 0.68 / 0.76).  Without this the choice fell on
// tiles that were latency bound: 1473 x 13248 x 872, k = 4, 64 x 96 tiles 296 us (estimated 130), the chunk-parallel way
// 206; 1042 x 30250 x 1180, k = 4, whole call 1030 us, now 790; 615 x 31277 x 496, k = 7, 684, now 530.
//
// parts > 1: the inner dimension of every tile cut among that many workgroups (one round of them), whose sums k_add_parts adds up.
inline double estimate_us(int k, int r, int variant, int64_t m, int64_t n, int64_t p, int num_cu, int parts = 1)
{
    const Config c = config_for(k, r, variant);
    if (c.ta == 0 || num_cu < 1 || !in_range(m, n, p, 32 * c.ta, 32 * c.tb)) return -1.0;
    const int64_t steps = ((n + 63) / 64 + parts - 1) / parts;
    const int64_t tiles = parts * ((m + 32 * c.ta - 1) / (32 * c.ta)) * ((p + 32 * c.tb - 1) / (32 * c.tb));
    const double mfmas = 0.5 * k * (k + 1) * c.ta * c.tb;
    const double kib = 2.0 * k * (c.ta + c.tb);                               // operands of a step
    const double copied = 1024.0 * kib / (4.0 * mfmas);                      // bytes brought in per MFMA
    const double fetched = (c.held ? (double)(k * c.ta + (2 * k - c.held - 1) * c.tb) : 0.5 * kib) / mfmas;  // KiB fetched from LDS per MFMA and wave
    // (rows of D that begin inside a piece of 64 bytes leave pieces to be merged, in memory: 4224 x 4608 x 1611, k = 4, 128 x 128
    // tiles 296 us, 1608 columns 280)
    const double odd_us = p % 8 == 0 || may_merge_rows(k, n) ? 0.0 : c.ta * c.tb == 16 ? 0.6 : variant >= EXTENDED ? 0.3 : 0.0;
    // (k_extended has more start values to form and more sums to add up: 448 x 359 x 4480, k = 7, one addition per pair, 32 x 96
    // 39 us behind the split, three rounds of 5.4 us of steps)
    const double round_us = 4.0 + (variant >= EXTENDED ? 2.0 + 0.08 * c.ta * c.tb : 0.0) + (0.4 + odd_us) * c.ta * c.tb;
    const int64_t slots = (int64_t)num_cu * c.waves, full = tiles / slots, left = tiles % slots;
    // (32 x 32 tiles, two to a compute unit, several rounds: the steps of the one cover the ends of the other, half of them at most, and no
    // more than there are steps to cover with.  Whole calls, the tile that was chosen without this and 32 x 32: 9998 x 67 x 320, k = 14,
    // 73.9 and 61.0 us, 5000 x 200 x 500, k = 14, 74.8 and 62.2, 7552 x 80 x 393, k = 11, 48.0 and 45.4, 70484 x 1 x 109, k = 6, one
    // addition per pair, 128 and 119; it stays with the other at 1500 x 1000 x 1500, k = 12, 124.2 and 127.7, and, for the length of the
    // steps, at 127768 x 4 x 114, k = 16, 387 and 415, and 55 x 120 x 154014, k = 14, 314 and 326.  Of 260 shapes of up to 600
    // inner positions the choice took 1.8 % longer than the best tile on average, 4.7 % without this.)
    const bool covered = c.ta * c.tb == 1 && c.waves == 2 && full >= 2;
    auto total = [&](double alone_us, double all_us) {
        const double half_us = 0.5 * round_us, cover_us = 1.3 * (double)steps * all_us;
        double us = (double)full * ((double)steps * all_us + round_us - (!covered ? 0.0 : cover_us < half_us ? cover_us : half_us));
        if (left > 0) us += (double)steps * (left > num_cu ? all_us : alone_us) + round_us;
        return us;
    };
    // how much of the operands comes from memory
    const double bytes = (8.0 * (double)(m + p) + (double)k * (double)(ozl::rows_padded(m) + ozl::rows_padded(p))) * (double)n;
    const double far = bytes < 240e6 ? 0.0 : bytes > 320e6 ? 1.0 : (bytes - 240e6) / 80e6;
    auto at_least = [](double us, double least) { return us > least ? us : least; };
    double wait_us;                                                           // least time of a step, its operands' way
    if (c.depth == 1)
        wait_us = (0.05 + 0.0135 * kib + far * (0.40 - 0.002 * kib)) * (k <= 4 ? 1.5 : 1.0);
    else
        wait_us = (1.0 - far) * (0.15 + 0.0035 * kib) + far * at_least(0.24 + 0.0075 * kib, kib / 62.0);
    double wait2_us = wait_us;                                                // the same with all places taken
    if (far == 1.0 && n > 12000 && (c.waves == 2 || c.depth == 2)) wait2_us = at_least(wait_us, kib / (c.waves == 2 ? 34.0 : 58.0));
    if (far == 1.0 && c.waves == 2 && c.depth == 1 && k <= 4) wait2_us = at_least(wait2_us, 1.5);
    const double barrier_us = c.ta * c.tb == 1 ? 0.2 : 0.27;
    const double us = total(at_least(0.0075 * mfmas + 0.15, wait_us),
                            at_least(c.waves == 2 ? 0.0168 * mfmas + 0.2 : 0.0075 * mfmas + barrier_us, wait2_us));
    if (parts > 1) return us + add_parts_us(k, r, c, tiles, parts);
    if (us < 1500.0) return us;
    // (k_held's tiles of 96 rows 2 % more: in turn, 8192^3, k = 8, 96 x 128 11.58 ms, 64 x 128 11.42; 16384^3, k = 9, 96 x 96 114.2, 64 x 128
    // 111.2; still ahead at 16384^3, k = 8, 89.5 and 90.9, 6144^3 4.76 and 4.90)
    const double hot_us = mfmas * ((c.waves == 2 ? 0.0062 : 0.0068) + 2.0e-5 * copied + 0.005 * fetched) * (c.held && c.ta == 3 ? 1.02 : 1.0);
    return total(at_least(hot_us, wait_us), at_least(hot_us * c.waves, wait2_us));
}

// What k_held, estimated to take `us`, has to be ahead of the best other tile by to be taken instead.  The estimates know one workgroup's
// steps and ends after one another.  Two that share a compute unit cover each other's ends, by all that the steps of one last, 5 us a
// round at most (estimated less measured lead, us a round: 1 or 2 steps 1.5, 3 and 4 2.7, 5 to 8 4.0, 9 to 40 4.7), and their estimates run
// 6 % too long besides, 2 us at least; 32 x 32 tiles' 3 % more.  k_extended's ends are like k_held's own, the two level within 1 %, and
// the others' estimates within half a percent.
// (Whole calls with k_held and without: 8532 x 421 x 5453, k = 8, 613 and 532 us, 780 x 6178 x 1346, k = 14, 579 and 519,
// 1409 x 65 x 805, k = 13, 26.4 and 22.9, 2944 x 5595 x 3896, k = 7, A and B transposed, 1267 and 1189, 647 x 4 x 6747, k = 9, 47.7 and 43.7; still taken:
// 2017 x 193 x 824, k = 11, 34.3 and 39.5, 1537 x 2051 x 1283, k = 9, 149.0 and 157.3, 2705^3, k = 13, 1066 and 1211.  Of 500 random
// shapes for which it led by more than the first of these 33 were slower with it by more than 2 %, up to 9 %, and the average gained 4.0 %; with all of them it
// is taken at 444, twelve of them slower by more than 2 %, up to 7 %, and the average over the 500 is the same within 0.1 %.)
inline double held_lead_us(int k, int r, int other, double us, int64_t m, int64_t n, int64_t p, int num_cu)
{
    const Config h = config_for(k, r, HELD), o = config_for(k, r, other);
    if (o.waves < 2) return (other == EXTENDED ? 0.01 : 0.005) * us;
    const int64_t tiles = ((m + 32 * h.ta - 1) / (32 * h.ta)) * ((p + 32 * h.tb - 1) / (32 * h.tb));
    const double cover_us = 1.0 + 0.7 * (double)((n + 63) / 64), rounds = (double)((tiles + num_cu - 1) / num_cu);
    return rounds * (cover_us < 5.0 ? cover_us : 5.0) + (0.06 * us > 2.0 ? 0.06 * us : 2.0) + (o.ta * o.tb == 1 ? 0.03 * us : 0.0);
}

// Which tile workgroup b takes.  Workgroup b runs on XCD b % 8, and 256 consecutive workgroups run at about the same
// time; those of one XCD should share operand tiles in its L2, and the XCDs among each other in the memory-side cache.
// So 256 workgroups in a row ("round") get 256 consecutive places of the order below, XCD x the places 32 x .. 32 x + 31
// of them: an 8 x 4 patch of tiles, eight patches to a block of 16 x 16.  The order: all whole 16 x 16 blocks (rows of
// blocks back and forth), then what is left of the tile grid on the right, then below, in bands of 8 rows walked column
// by column.  A last round that is not full is cut into eight equal ranges.
__host__ __device__ inline void band_order(int lin, int rows, int& r, int& c, int cols)
{
    const int width = 8 * cols, band = lin / width, in_band = lin - band * width;
    const int h = rows - 8 * band < 8 ? rows - 8 * band : 8;
    r = 8 * band + in_band % h;
    c = in_band / h;
}
__host__ __device__ inline void tile_of_block(int b, int TM, int TP, int& tm, int& tp)
{
    const int T = TM * TP, x = b & 7, round = b >> 8;
    int lin;
    if (T - (round << 8) >= 256) {
        lin = (round << 8) + x * 32 + ((b >> 3) & 31);
    } else {
        const int left = T - (round << 8), base = left >> 3, rem = left & 7;
        lin = (round << 8) + x * base + (x < rem ? x : rem) + ((b & 255) >> 3);
    }
    const int BM = TM / 16, BP = TP / 16, whole = BM * BP * 256;
    if (lin < whole) {
        const int q = lin >> 8, u = lin & 255, br = q / BP, bc = q - br * BP;
        const int patch = u >> 5, mem = u & 31;
        tm = br * 16 + (patch >> 2) * 8 + (mem & 7);
        tp = ((br & 1) ? BP - 1 - bc : bc) * 16 + (patch & 3) * 4 + (mem >> 3);
        return;
    }
    lin -= whole;
    const int wr = TP - BP * 16;       // columns right of the blocks, over all rows
    if (lin < TM * wr) {
        band_order(lin, TM, tm, tp, wr);
        tp += BP * 16;
    } else {
        band_order(lin - TM * wr, TM - BM * 16, tm, tp, BP * 16);
        tm += BM * 16;
    }
}

}  // namespace ozr
