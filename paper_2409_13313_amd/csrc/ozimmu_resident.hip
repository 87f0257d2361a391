// Steps (iii) to (v) of the scheme with every chunk of a tile resident in registers.
//
// k_gemm (ozimmu_gemm.hip) runs the chunks of a tile one after the other and streams both operands' slices anew for
// every slice pair: k (k + 1) / 2 reads of an A tile and of a B tile per tile and inner step.  k_resident turns the
// loops round: for one inner step of 64 it takes ALL k slices of its rows of A and of its columns of B (2 k tiles
// instead of k (k + 1)) and runs all k (k + 1) / 2 slice pairs on them, each into the INT32 accumulators of its chunk.
// The w chunk sums of a tile (Algorithm 6) thus grow side by side in the accumulation registers, and when the inner
// dimension is through they are added up in FP64 in the order of Algorithm 6 - one rounded addition per chunk, as
// everywhere - and D is written once.  No INT32 blocks, no second pass, no counters between workgroups.
//
// What bounds it: the matrix cores, at the clock the chip's power budget allows.  Per MFMA the wave fetches 0.167 KiB of
// fragments from LDS (k = 8, tiles of 64 x 128; k_gemm 0.25), the compute unit brings in 85 bytes of operands (128), and
// the launch reads 137 GB from beyond L2 at 16384^3 (281).  All of that is energy that goes into clock instead:
// 16384^3, k = 8: 1.86 GHz at 92 % busy pipes against 1.68 GHz at 91.5 %, 86.9 against 95.6 ms on one box
// (3.5 to 3.7 POP/s, 86 to 90 % of what a register-only MFMA loop sustains on such bytes).  Small outputs gain more: their tiles
// need no blocks, no atomic adds and no second kernel, and 64 x 64 tiles spread a 1024^3 product over the whole chip
// (whole calls, k_gemm's ways and a split of three to seven launches -> this behind a split of one: 1024^3 k = 9
// 126 -> 43 us, 777 x 1001 x 513 k = 7 122 -> 29 us, 4096^3 k = 8 1.86 -> 1.50 ms, 4096^3 k = 9 with one addition per slice
// pair 4.13 -> 2.61 ms).
//
// Tried without gain: the MFMAs of a pair with A held and B changing (0.7 % slower at 16384^3, 1 % at 4096^3).
//
// k_extended is the same kernel with chunk sums in ordinary registers too, where the 64 tiles of 16 x 16 of the accumulation
// registers are too few for the next larger tile.  Its MFMAs are asm statements that read and write their sums in place: left to
// the compiler, sums of a full register file wander, and the moves that takes sit in the loop (64 x 96 at k = 12, 96 x 128 at k = 6:
// equal and 5 % slower than the smaller tile that way).  A larger tile moves fewer bytes per MFMA, from beyond L2, into LDS and out of
// it: 128 x 128 instead of two workgroups of 64 x 96 at k = 5, 4096^3 708 -> 658 us and 8192^3 5.62 -> 4.90 ms; 64 x 128 instead of 64 x 96 at
// k = 9 and 10, 1.84 -> 1.75 and 2.16 -> 2.06 ms at 4096^3, 14.5 -> 13.9 ms at 8192^3, k = 9.  One addition per slice pair, whose k (k + 1) / 2 sums
// leave small tiles only and whose bound is the way of the operands through LDS, gains most: 4096^3, k = 9, 32 x 64 instead of 32 x 32,
// 2.54 -> 2.25 ms, and k = 11 to 13, which had no resident tile at all, 5.95, 7.09, 8.32 -> 3.39, 3.77, 4.20 ms.
// No gain in k_extended's order: 96 x 96 and 64 x 160 at k = 7 and 8 (0 to 0.5 % at 8192^3 and 16384^3, 3 to 5 % slower where 4096 is no multiple of them).
//
// k_held is k_extended with another order of a step (HeldPlan): the lower slices of A stay in registers while those of B pass by, which takes
// fewer fragments at a time and leaves room for the sums of the next larger tile: 128 x 128 at k = 6, 96 x 128 at 7 and 8, 96 x 96 at 9 and
// 10, 64 x 128 at 11, 64 x 96 at 13, 14 and for the 16 chunks of k = 12 at r = 8.  What that saves is bytes that the compute units bring in (all of
// them compiled out, a working copy, 16384^3, k = 8, is 16 % of the time, half of the LDS fetches 0.5 %).  From beyond L2, the other tile and k_held's: 8192^3,
// k = 6, 12.4 and 9.7 GB, k = 11 38.7 and 28.5, 12288^3, k = 8, 58 and 51, 16384^3, k = 12, 530 to 590 and 374, but k = 8 138 to 143 and 143.  Whole calls, the two in turn: 8192^3,
// k = 6, 96 x 128 7.04 ms, 128 x 128 6.70; k = 11, 64 x 96 20.8 and 64 x 128 19.5; 12288^3, k = 8, 64 x 128 38.0, 96 x 128 36.9; 6144^3 4.90
// and 4.76.  At 16384^3, where the power budget sets the clock, little is left of it: k = 8 90.2 and 88.7, k = 12 191.0 and 187.2, where runs differ by 1 %.
// 1537 x 2051 x 1283, k = 9, one round of 96 x 96 instead of four of 32 x 32, 157 and 149 us.  Two to four barriers a step,
// copies spread wider, MFMAs with A held: the same within 0.5 %.
//
// Fragments: L = (k + 1) / 2 low slices of both operands stay in registers for a step, the high ones pass through two
// buffers, so that every fragment is fetched once per step and wave.  A wave holds as many 16 x 16 tiles as w chunk
// sums leave room for in the 256 accumulation registers (ozimmu_resident.h).
//
// This file is compiled once per slice count (OZ_RES_K = k).
#include "ozimmu_kernels.h"
#include "ozimmu_layout.h"
#include "ozimmu_resident.h"
#include <type_traits>
#include <utility>

#ifndef OZ_RES_K
#define OZ_RES_K 8
#endif

namespace {

using namespace ozl;

typedef int v4i __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const v4i* lds_v4i_ptr;

template <int... I, class F>
__device__ __attribute__((always_inline)) inline void static_for_impl(std::integer_sequence<int, I...>, F&& f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __attribute__((always_inline)) inline void static_for(F&& f)
{
    static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

template <int N>
__device__ inline void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is a 6-bit counter");
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// (the builtin, not asm: the compiler then knows that its own LDS reads have returned)
__device__ inline void wait_lds() { __builtin_amdgcn_s_waitcnt(0xc07f); }

using ozr::num_chunks;

// number (in schedule order) of the chunk that holds the pair (s, t)
constexpr int chunk_of(int s, int t, int r)
{
    int w = 0;
    for (int g = 2; g < s + t; ++g) w += (g - 2) / r + 1;
    return w + (s - 1) / r;
}

// chunk number c: s = s0 .. s1 of group g
struct Range {
    int g, s0, s1;
};
template <int K, int R>
constexpr Range chunk_range(int c)
{
    int n = 0;
    for (int g = 2; g <= K + 1; ++g)
        for (int s0 = 1; s0 <= g - 1; s0 += R, ++n)
            if (n == c) return Range{g, s0, (s0 + R - 1 < g - 1) ? s0 + R - 1 : g - 1};
    return Range{0, 0, 0};
}

// The order of one inner step, made at compile time.  With L = (k + 1) / 2 no pair has both slices above L.  Group
// number gi = 0 .. L - 1 belongs to j = L - gi: first the pairs of low slices whose larger one is j, then those of the
// high slice h = k + 1 - j (if h > L) with the low slices 1 .. j.  After it slice j is used up for this step: its
// registers take slice j of the NEXT step at the start of the next group.  The high slices pass through two buffers.
//
// Groups are gathered into intervals, each opened by a barrier: what an interval reads from LDS has landed before it, and
// the copies that replace what an interval has read go out in the one after.  Few of them, because a barrier costs some
// 80 ns (with one per group, one workgroup on a compute unit, 1024^3, k = 9: 1.76 us a step for 1.37 us of MFMAs): two for a ring
// of two steps, where a copy has a whole step to arrive; three for a ring of one - first group, second group, the rest -
// which leaves every copy some 2000 cycles; five beyond 13 slices,
// where the rest has grown too long (8192^3, k = 16: 40.0 ms with three, 38.4 with five; k = 12 23.7 and 24.3).
template <int K, int R, int TA, int TB, int D>
struct Plan {
    static constexpr int k = K, r = R, ta = TA, tb = TB, depth = D, HELD = 0;
    static constexpr int L = (K + 1) / 2;
    static constexpr int NP = K * (K + 1) / 2;
    static constexpr int W = num_chunks(K, R);
    static constexpr int TT = TA * TB;          // MFMAs of a pair
    static constexpr int NM = NP * TT;          // MFMAs of a step
    static constexpr int NF = TA + TB;          // fragments of a slice
    static constexpr int NC = (2 * NF + 3) / 4;  // copies (of 16 rows) per wave and slice
    static constexpr int NI = D == 2 ? 2 : (L < 3 ? L : (K > 13 ? 5 : 3));

    int s[NP] = {}, t[NP] = {};
    int group_at[L + 1] = {};        // first MFMA of a group
    int nread[L] = {}, read_slice[L][3] = {};  // slices whose fragments are fetched in a group
    bool read_next[L][3] = {};       // ... for the next step
    int first_group[NI + 1] = {};    // groups of an interval
    int nslot[NI] = {}, slot_slice[NI][K] = {};  // the same by interval
    bool slot_next[NI][K] = {};
    // per MFMA index: group, interval, the fragment fetches (read_at .. read_at + reads - 1 of the group's list) and the copies
    // (of the interval's list) that go out before it
    int read_at[NM] = {}, reads[NM] = {}, copy_at[NM] = {}, copies[NM] = {}, group_of[NM] = {}, interval_of[NM] = {};
    bool opens[NM] = {};             // first MFMA of an interval

    constexpr int high(int j) const { return K + 1 - j > L ? K + 1 - j : 0; }
    constexpr Plan()
    {
        int n = 0;
        for (int gi = 0; gi < L; ++gi) {
            const int j = L - gi;
            group_at[gi] = n * TT;
            s[n] = j, t[n++] = j;
            for (int q = j - 1; q >= 1; --q) {
                s[n] = j, t[n++] = q;
                s[n] = q, t[n++] = j;
            }
            const int h = high(j);
            if (h)
                for (int q = j; q >= 1; --q) {
                    s[n] = h, t[n++] = q;
                    s[n] = q, t[n++] = h;
                }
            auto add = [&](int sl, bool next) {
                read_slice[gi][nread[gi]] = sl;
                read_next[gi][nread[gi]++] = next;
            };
            if (gi == 0) {
                add(1, false);
                if (high(L)) add(high(L), false);
            } else {
                add(j + 1, true);
            }
            if (j >= 2 && high(j - 1)) add(high(j - 1), false);
        }
        group_at[L] = NM;
        if (D == 2) {
            // two intervals of about equal length
            int g = 1;
            while (g < L - 1 && 2 * group_at[g] < NM) ++g;
            first_group[1] = L == 1 ? 1 : g;
        } else {
            for (int v = 1; v < NI; ++v) first_group[v] = v;
        }
        first_group[NI] = L;
        for (int v = 0; v < NI; ++v)
            for (int gi = first_group[v]; gi < first_group[v + 1]; ++gi)
                for (int x = 0; x < nread[gi]; ++x) {
                    slot_slice[v][nslot[v]] = read_slice[gi][x];
                    slot_next[v][nslot[v]++] = read_next[gi][x];
                }
        auto spread = [](int len, int count, int most) {
            int sp = len / (count + 2);
            sp = sp > most ? most : sp;
            return sp < 1 ? 1 : sp;
        };
        for (int gi = 0; gi < L; ++gi) {
            const int len = group_at[gi + 1] - group_at[gi];
            for (int q = group_at[gi]; q < group_at[gi + 1]; ++q) group_of[q] = gi;
            const int nr = nread[gi] * NF, spr = spread(len, nr, TT <= 4 ? 2 : 4);
            for (int x = 0; x < nr; ++x) {
                const int q = group_at[gi] + (x * spr < len ? x * spr : len - 1);
                if (reads[q]++ == 0) read_at[q] = x;
            }
        }
        for (int v = 0; v < NI; ++v) {
            const int at = group_at[first_group[v]], len = group_at[first_group[v + 1]] - at;
            opens[at] = true;
            for (int q = at; q < at + len; ++q) interval_of[q] = v;
            const int nc = nslot[(v + NI - 1) % NI] * NC, spc = spread(len, nc, 4);
            for (int x = 0; x < nc; ++x) {
                const int q = at + (x * spc + 1 < len ? x * spc + 1 : len - 1);
                if (copies[q]++ == 0) copy_at[q] = x;
            }
        }
    }
};

// The order of one inner step of k_held, made at compile time: H = held slices of A (an odd number, at least K / 2) stay in registers, the
// slices of B pass by in two buffers.  First B_K with A_1, B_(K-1) with A_1 and A_2, ... down to B_1 with A_1 .. A_H; the others of A
// take the places of the held ones as those are used up, B_1 stays for them; then B_2 .. B_(K-H) once more.  2 K - H - 1 slices of B
// pass, an even number, so a slice finds the same buffer in every step.  Every slice of A is fetched once, B_2 .. B_(K-H) twice.
//
// A place in LDS holds one slice of a step; the copy of the next step's goes out once every wave has fetched it, at the next barrier,
// and has landed at the barrier before it is fetched.  B_2 .. B_(K-H), fetched last in one step and early in the next, have two places.
template <int K, int R, int TA, int TB, int H_>
struct HeldPlan {
    static constexpr int k = K, r = R, ta = TA, tb = TB, depth = 1, HELD = H_, H = H_;
    static constexpr int L = (K + 1) / 2, NC = 1, NF = TA + TB;
    static constexpr int NP = K * (K + 1) / 2, W = num_chunks(K, R), TT = TA * TB, NM = NP * TT;
    static constexpr int NI = 3;                             // intervals (barriers) of a step
    static constexpr int SEGS = 2 * K - H - 1;               // slices of B that pass
    static constexpr int CA = (2 * TA + 3) / 4, CB = (2 * TB + 3) / 4, NCOPY = K * (CA + CB);  // copies per wave (16 rows, or 8)
    static constexpr int ALT = K - H - 1;                    // slices of B with two places
    static constexpr int NR = K * TA + SEGS * TB;            // fragments
    static_assert(H % 2 == 1 && 2 * H >= K && H < K, "");

    // LDS, in bytes: A_1 .. A_K, then B: B_1, B_(K-H+1) .. B_K, B_2 .. B_(K-H), the second places of those
    static constexpr int A_BYTES = TA * 2048, B_BYTES = TB * 2048;
    static constexpr int BYTES = K * (A_BYTES + B_BYTES) + ALT * B_BYTES;
    static constexpr bool alternates(int t) { return t >= 2 && t <= K - H; }
    static constexpr int place_b(int t) { return t == 1 ? 0 : t > K - H ? t - (K - H) : H + 1 + t - 2; }
    // register place of a slice of A
    static constexpr int place_a(int s) { return s <= H ? s - 1 : K - s; }

    struct Read { int op = 0, slice = 0, frag = 0, to = 0, pos = 0; bool next = false; };
    struct Copy { int op = 0, slice = 0, part = 0, pos = 0, ahead = 0; };
    int s[NP] = {}, t[NP] = {}, seg[NP] = {};                // pairs
    int seg_t[SEGS] = {}, seg_at[SEGS + 1] = {};             // first MFMA
    Read reads[NR];
    int read_first[NM + 1] = {};
    Copy copies[NCOPY];
    int copy_first[NM + 1] = {};
    int border[NI + 1] = {}, wait[NI] = {};
    int most_ahead = 0;
    bool good = true;
    int from = 0;                                            // first copy of the step after next's data

    static constexpr int floor_div(int a, int b) { return a >= 0 ? a / b : -((b - 1 - a) / b); }
    constexpr int interval_of(int pos) const
    {
        int v = 0;
        while (v + 1 < NI && pos >= border[v + 1]) ++v;
        return v;
    }
    // number of the interval that holds MFMA x, counted from the first of step 0 (x < 0: the steps before)
    constexpr int interval_at(int x) const
    {
        const int step = floor_div(x, NM);
        return step * NI + interval_of(x - step * NM);
    }
    constexpr HeldPlan()
    {
        int n = 0, g = 0, end_of_a[K + 1] = {};              // end_of_a: behind the last MFMA that uses a slice of A
        auto pair = [&](int a, int b) {
            s[n] = a, t[n] = b, seg[n] = g;
            end_of_a[a] = ++n * TT;
        };
        auto open = [&](int b) { seg_t[g] = b, seg_at[g] = n * TT; };
        for (int b = K; b >= 1; --b) {
            open(b);
            for (int a = 1; a <= H && a <= K + 1 - b; ++a) pair(a, b);
            if (b == 1)
                for (int a = K; a > H; --a) pair(a, 1);
            ++g;
        }
        for (int b = 2; b <= K - H; ++b) {
            open(b);
            for (int a = K + 1 - b; a > H; --a) pair(a, b);
            ++g;
        }
        seg_at[SEGS] = NM;
        good = good && n == NP && g == SEGS;

        // fetches: a slice of B while the one before passes, a slice of A once its place is free
        int at[NM] = {}, count = 0;
        Read list[NR];
        auto put = [&](int op, int slice, int frag, int to, bool next, int from, int limit) {
            int pos = from;
            while (pos < limit - 1 && at[pos] > 0) ++pos;
            if (at[pos] > 0) pos = from;
            ++at[pos];
            list[count].op = op, list[count].slice = slice, list[count].frag = frag, list[count].to = to, list[count].next = next;
            list[count++].pos = pos;
            return pos;
        };
        int b_first[SEGS] = {}, b_last[SEGS] = {}, a_first[K + 1] = {}, a_last[K + 1] = {};
        for (int q = 0; q < SEGS; ++q) {
            const int before = q == 0 ? SEGS - 1 : q - 1, len = seg_at[before + 1] - seg_at[before];
            const int stride = len / (TB + 1) > 2 ? 2 : 1;
            int from = seg_at[before];
            for (int x = 0; x < TB; ++x) {
                const int pos = put(1, seg_t[q], x, q & 1, q == 0, from, seg_at[before + 1]);
                if (x == 0) b_first[q] = pos;
                b_last[q] = pos;
                from = pos + stride < seg_at[before + 1] ? pos + stride : seg_at[before + 1] - 1;
            }
        }
        for (int a = 1; a <= K; ++a) {
            // (its place belongs to K + 1 - a before)
            int from = a > H ? end_of_a[K + 1 - a] : a <= K - H ? end_of_a[K + 1 - a] : end_of_a[a];
            bool next = a <= H;
            if (from + 2 * TA >= NM) from = 0, next = false;  // (the place that comes free last: early in the step itself)
            for (int x = 0; x < TA; ++x) {
                const int pos = put(0, a, x, place_a(a), next, from, NM);
                if (x == 0) a_first[a] = pos;
                a_last[a] = pos;
                from = pos + 2 < NM ? pos + 2 : NM - 1;
            }
        }
        good = good && count == NR;
        // in the order of their places
        int out = 0;
        for (int q = 0; q < NM; ++q) {
            read_first[q] = out;
            for (int x = 0; x < NR; ++x)
                if (list[x].pos == q) reads[out++] = list[x];
        }
        read_first[NM] = out;

        // barriers: about a third of a step each, not where a slice is half fetched and best not just behind a fetch
        border[NI] = NM;
        for (int v = 1; v < NI; ++v) {
            int best = -1, best_cost = 0;
            for (int q = border[v - 1] + NM / (2 * NI); q < NM * v / NI + NM / (2 * NI); ++q) {
                int cost = q > NM * v / NI ? q - NM * v / NI : NM * v / NI - q;
                for (int x = 0; x < SEGS; ++x)
                    if (b_first[x] < q && q <= b_last[x]) cost += 1000;
                for (int a = 1; a <= K; ++a)
                    if (a_first[a] < q && q <= a_last[a]) cost += 1000;
                for (int x = read_first[q - 6 > 0 ? q - 6 : 0]; x < read_first[q]; ++x) cost += 8;
                if (best < 0 || cost < best_cost) best = q, best_cost = cost;
            }
            border[v] = best;
        }

        // copies: first and last fetch of a step's data, in MFMAs from the begin of that step
        int first[2 * K] = {}, last[2 * K] = {}, issue[2 * K] = {};
        for (int i = 0; i < 2 * K; ++i) first[i] = NM, last[i] = -NM;
        for (int x = 0; x < NR; ++x) {
            const int i = reads[x].op * K + reads[x].slice - 1, pos = reads[x].pos - (reads[x].next ? NM : 0);
            first[i] = pos < first[i] ? pos : first[i];
            last[i] = pos > last[i] ? pos : last[i];
        }
        for (int i = 0; i < 2 * K; ++i) {
            // (step 0's data goes out in this interval)
            issue[i] = interval_at(last[i]) - (i >= K && alternates(i - K + 1) ? 2 : 1) * NI + 1;
            good = good && issue[i] < interval_at(first[i]);
        }
        int seq[2 * K] = {}, nc = 0, before_interval[NI + 1] = {};
        for (int v = 0; v < NI; ++v) {
            before_interval[v] = nc;
            int total = 0, x = 0;
            for (int i = 0; i < 2 * K; ++i)
                if (issue[i] - floor_div(issue[i], NI) * NI == v) total += i < K ? CA : CB;
            const int len = border[v + 1] - border[v];
            int stride = len / (total + 2);
            stride = stride > 4 ? 4 : stride < 1 ? 1 : stride;
            for (int slack = 1; slack <= 3 * NI; ++slack)     // (what is needed first goes first)
                for (int i = 0; i < 2 * K; ++i) {
                    if (issue[i] - floor_div(issue[i], NI) * NI != v || interval_at(first[i]) - issue[i] != slack) continue;
                    for (int part = 0; part < (i < K ? CA : CB); ++part, ++x) {
                        Copy& c = copies[nc++];
                        c.op = i < K ? 0 : 1, c.slice = i % K + 1, c.part = part;
                        c.pos = border[v] + (x * stride + 1 < len ? x * stride + 1 : len - 1);
                        c.ahead = -floor_div(issue[i], NI);
                        most_ahead = c.ahead > most_ahead ? c.ahead : most_ahead;
                        good = good && c.ahead >= 0;
                    }
                    seq[i] = nc - 1;
                }
            good = good && x == total;
        }
        before_interval[NI] = nc;
        good = good && nc == NCOPY && most_ahead <= 2;
        while (from < NCOPY && copies[from].ahead < 2) ++from;
        int at_copy = 0;
        for (int q = 0; q < NM; ++q) {
            copy_first[q] = at_copy;
            while (at_copy < NCOPY && copies[at_copy].pos == q) ++at_copy;
        }
        copy_first[NM] = at_copy;
        good = good && at_copy == NCOPY;
        // copies that may still be on their way when an interval opens
        for (int v = 0; v < NI; ++v) wait[v] = 63;
        for (int i = 0; i < 2 * K; ++i) {
            const int f = interval_at(first[i]), step = floor_div(f, NI), v = f - step * NI;
            const int sent = step * NCOPY + before_interval[v], needed = floor_div(issue[i], NI) * NCOPY + seq[i] + 1;
            good = good && sent >= needed;
            if (sent - needed < wait[v]) wait[v] = sent - needed;
        }
    }
};

// The operands and the loop of k_held.  Copies: a slice's 2 TA or 2 TB pieces of 16 rows go to its place, TA / 2 or TB / 2 of them by each
// wave, all with one M0; of a last two, which four waves share, each brings half, with half of its lanes (6 pieces as 8, two of
// them brought twice, move a third more: 96 x 96 tiles, k = 9, then took as long as 64 x 128).
template <class P>
struct Held {
    static constexpr P plan{};
    static constexpr int K = P::k, TA = P::ta, TB = P::tb, H = P::H, WHOLE[2] = {TA / 2, TB / 2};
    const int8_t* base[2];                       // A, B: the row block of the tile's first row
    uint32_t from[2][2];                         // a lane's part of the wave's pieces from there: whole ones, the shared one
    uint32_t m0[2], m0_half[2];
    uint32_t even, odd, two_places;              // the slices of two places: that of the step's parity, the other one, both together
    uint64_t half;                               // lanes of a shared copy
    uint32_t at_a, at_b, at_two, at_two_sum;     // fragments of A, B, and B's slices of two places
    v4i fa[H][TA], fb[2][TB];

    template <int X>
    __device__ __attribute__((always_inline)) inline void copy(const ozk::ResidentArgs& a, bool second, uint32_t step)
    {
        constexpr auto c = plan.copies[X];
        constexpr int off = c.op ? P::place_b(c.slice) * P::B_BYTES : (c.slice - 1) * P::A_BYTES;
        const int8_t* const slice = base[c.op] + (int64_t)(c.slice - 1) * (c.op ? a.strideB : a.strideA);
        const uint32_t at = from[c.op][c.part == WHOLE[c.op] ? 1 : 0] + step;
        const uint32_t place = c.op && P::alternates(c.slice) ? (second ? odd : even) : 0u;
        if constexpr (c.part == WHOLE[c.op]) {
            const uint32_t m = m0_half[c.op] + place;
            const uint64_t lanes = half;
            // (all lanes take part in everything else)
            asm volatile("s_add_u32 m0, %0, %1\n\ts_mov_b64 exec, %4\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b64 exec, -1" ::"s"(m), "n"(off),
                         "v"(at), "s"(slice), "s"(lanes)
                         : "memory", "scc");
        } else if constexpr (c.part == 0) {
            const uint32_t m = m0[c.op] + place;
            asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3" ::"s"(m), "n"(off), "v"(at), "s"(slice)
                         : "memory", "scc");
        } else {
            // (the offset moves both addresses; two whole pieces a wave: tiles of 128, whose pieces lie one behind the other)
            asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" ::"v"(at), "s"(slice), "n"(c.part * 1024) : "memory");
        }
    }
    template <int X>
    __device__ __attribute__((always_inline)) inline void fetch()
    {
        constexpr auto r = plan.reads[X];
        if constexpr (r.op == 0)
            fa[r.to][r.frag] = *(lds_v4i_ptr)(uintptr_t)(at_a + ((r.slice - 1) * P::A_BYTES + r.frag * 1024));
        else if constexpr (P::alternates(r.slice))
            fb[r.to][r.frag] = *(lds_v4i_ptr)(uintptr_t)(at_two + ((r.slice - 2) * P::B_BYTES + r.frag * 1024));
        else
            fb[r.to][r.frag] = *(lds_v4i_ptr)(uintptr_t)(at_b + (P::place_b(r.slice) * P::B_BYTES + r.frag * 1024));
    }
    // addresses, and step 0's slices on their way
    __device__ __attribute__((always_inline)) inline void begin(const ozk::ResidentArgs& a, uint32_t lds_base, uint32_t row0, uint32_t col0,
                                                                int wave, int lane)
    {
        // (at most MAX_STEPS steps: a row block is 2 GiB at most, and a tile has rows in two)
        static_assert(32 * (TA > TB ? TA : TB) <= TILE_R, "");
        const uint32_t rowblk = (uint32_t)rowblock_bytes(a.KT);
#pragma unroll
        for (int o = 0; o < 2; ++o) {
            const uint32_t row0_o = o ? col0 : row0, top = (uint32_t)(o ? a.pstrideB : a.pstrideA) - 16u;  // (padded rows of the stack)
            const uint32_t block0 = (row0_o < top ? row0_o : top) / TILE_R;
            const int piece[2] = {wave * WHOLE[o], 4 * WHOLE[o] + (wave >> 1)};
            const uint32_t lds = lds_base + (o ? (uint32_t)(K * P::A_BYTES) : 0u);
            m0[o] = lds + (uint32_t)piece[0] * 1024u;
            m0_half[o] = lds + (uint32_t)piece[1] * 1024u;
            base[o] = (o ? a.SB : a.SA) + (int64_t)block0 * rowblk;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                uint32_t row = row0_o + (uint32_t)piece[q] * 16u;
                row = row < top ? row : top;  // a tile may reach past the padding: what it reads there is never stored
                from[o][q] = (row / TILE_R - block0) * rowblk + row % TILE_R * TILE_K + (uint32_t)lane * 16u;
            }
        }
        half = (wave & 1) ? 0xffffffff00000000ull : 0x00000000ffffffffull;
        even = 0, odd = P::ALT * P::B_BYTES, two_places = odd;
        asm volatile("" : "+s"(two_places), "+s"(half));
        const int chunk = (0x9c >> (2 * (lane >> 4))) & 3;  // 0, 3, 1, 2 (see run_tile)
        const int ra = (wave >> 1) * (16 * TA) + (lane & 15), rb = (wave & 1) * (16 * TB) + (lane & 15);
        at_a = lds_base + ra * TILE_K + swizzle(ra, chunk) * CHUNK;
        at_b = lds_base + K * P::A_BYTES + rb * TILE_K + swizzle(rb, chunk) * CHUNK;
        at_two = at_b + (H + 1) * P::B_BYTES;
        at_two_sum = 2 * at_two + P::ALT * P::B_BYTES;
        asm volatile("" : "+v"(at_a), "+v"(at_b), "+v"(at_two), "+v"(at_two_sum));
        // (but for those whose copies the loop's first interval sends out)
        static_for<P::NCOPY>([&](auto X) __attribute__((always_inline)) {
            constexpr int x = decltype(X)::value;
            if constexpr (plan.copies[x].ahead > 0) copy<x>(a, false, 0u);
        });
    }
    // (step 0's slices have landed, every wave's)
    template <class ACC>
    __device__ __attribute__((always_inline)) inline void loop(const ozk::ResidentArgs& a, ACC& acc, int KT)
    {
        static_assert(plan.good, "order of a step");
        auto step_off = [&](int kt) { return (uint32_t)(kt < KT - 1 ? kt : KT - 1) * (uint32_t)TILE_BYTES; };
        // What the step before would have fetched, and then its copies from the first of step 1's on, in the order of the loop, so that
        // its counted waits hold from the start (some bring the same bytes to the same place again).
        static_for<P::NR>([&](auto X) __attribute__((always_inline)) {
            constexpr int x = decltype(X)::value;
            if constexpr (plan.reads[x].next) fetch<x>();
        });
        wait_lds();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        static_for<P::NCOPY - plan.from>([&](auto X) __attribute__((always_inline)) {
            constexpr int x = plan.from + decltype(X)::value, ahead = plan.copies[x].ahead;
            if constexpr (ahead > 0) copy<x>(a, ahead == 2, step_off(ahead - 1));
        });
        // where the copies of a step read: this step, the next one, the one after (past the end: the last step again, never used)
        uint32_t s0 = 0, s1 = step_off(1), s2 = step_off(2);
        for (int kt = 0; kt < KT; ++kt) {
            static_for<P::NM>([&](auto Q) __attribute__((always_inline)) {
                constexpr int q = decltype(Q)::value, v = plan.interval_of(q);
                if constexpr (plan.border[v] == q) {
                    wait_lds();
                    wait_vmcnt<plan.wait[v]>();
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_sched_barrier(0);
                }
                static_for<plan.read_first[q + 1] - plan.read_first[q]>([&](auto X) __attribute__((always_inline)) {
                    fetch<plan.read_first[q] + decltype(X)::value>();
                });
                static_for<plan.copy_first[q + 1] - plan.copy_first[q]>([&](auto X) __attribute__((always_inline)) {
                    constexpr int x = plan.copy_first[q] + decltype(X)::value, ahead = plan.copies[x].ahead;
                    copy<x>(a, ahead == 1, ahead == 0 ? s0 : ahead == 1 ? s1 : s2);
                });
                constexpr int pr = q / P::TT, m = q % P::TT;
                constexpr int j = m / TA, i = (j & 1) ? TA - 1 - m % TA : m % TA;
                constexpr int c = chunk_of(plan.s[pr], plan.t[pr], P::r);
                const v4i x = fa[P::place_a(plan.s[pr])][i], y = fb[plan.seg[pr] & 1][j];
                // (in place, see k_extended: the compiler sees no matrix instruction)
                if constexpr ((c * TB + j) * TA + i >= ozr::ACC_TILES)
                    asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+v"(acc[c][i][j]) : "v"(x), "v"(y));
                else
                    asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+a"(acc[c][i][j]) : "v"(x), "v"(y));
                // (in gaps between two MFMAs, behind the last fetch of the slices of two places and behind the last copy)
                if constexpr (q == P::NM - 3) {
                    at_two = at_two_sum - at_two;
                    asm volatile("" : "+v"(at_two));
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            even = odd;
            odd = two_places - even;
            s0 = s1;
            s1 = s2;
            s2 = step_off(kt + 3);
        }
    }
};

// Copies of what interval V reads in `step` (a low slice for the step after).
template <class P, int V, int STEP, class COPY_SLICE, class STEP_OFF>
__device__ __attribute__((always_inline)) inline void copy_interval(COPY_SLICE&& copy_slice, STEP_OFF&& step_off, uint32_t m0_cur, uint32_t m0_nxt,
                                                                    uint32_t lv)
{
    static constexpr P plan{};
    static_for<plan.nslot[V]>([&](auto X) __attribute__((always_inline)) {
        constexpr int x = decltype(X)::value, data = STEP + (plan.slot_next[V][x] ? 1 : 0);
        copy_slice(std::integral_constant<int, plan.slot_slice[V][x]>{}, (data & 1) ? m0_nxt : m0_cur, lv + step_off(data));
    });
}

// What becomes of a tile's sums: added up into D with one exponent per row and column, or (r = 1) per row, column and slice; or left in
// memory as the sums of a part of the inner dimension.  Kernels of their own, each with one of them: an end that a call does not take
// costs it all the same (the second in the kernels of the first: 3 to 5 % of whole calls of short inner dimensions, 140388 x 4 x 8,
// k = 9, one addition per pair, 215.5 and 224 us; the third: spilled chunk sums).
enum class End { COMMON, PER_SLICE, PART };
// A workgroup's tile.  IN_PLACE: k_extended (see the head).
template <class P, int WAVES, bool IN_PLACE, End END>
__device__ __attribute__((always_inline)) inline void run_tile(const ozk::ResidentArgs& a)
{
    constexpr bool CUT = END == End::PART, PER_SLICE = END == End::PER_SLICE;
    static constexpr P plan{};
    constexpr int K = P::k, R = P::r, TA = P::ta, TB = P::tb, D = P::depth;
    constexpr int L = P::L, W = P::W, NF = P::NF, NI = P::NI, HELD = P::HELD;
    constexpr int RA = 32 * TA, RB = 32 * TB;               // rows and columns of the workgroup's tile
    constexpr int SLOT = (RA + RB) * TILE_K;                // one slice of both operands: A rows, then B columns
    constexpr int SET = [] {                                // all slices of an inner step
        if constexpr (P::HELD > 0)
            return P::BYTES;
        else
            return K * SLOT;
    }();
    extern __shared__ __align__(16) int8_t lds[];
    int* const lds_exp = reinterpret_cast<int*>(lds + D * SET);  // exponents of the tile's rows, then columns

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int wm = wave >> 1, wn = wave & 1;

    // workgroup b runs on XCD b % 8
    int tm, tp, block = (int)blockIdx.x, part = 0;
    if constexpr (CUT) {
        // (no padding to whole sets of XCDs: workgroups that end at once have others put two to a compute unit while some stay
        // idle, 659 x 11776 x 206, k = 6, 84 tiles in three parts, 115 instead of 91 us)
        part = block / (a.TM * a.TP);
        block -= part * a.TM * a.TP;
    }
    ozr::tile_of_block(block, a.TM, a.TP, tm, tp);
    tm = __builtin_amdgcn_readfirstlane(tm);
    tp = __builtin_amdgcn_readfirstlane(tp);
    const uint32_t row0 = (uint32_t)tm * RA, col0 = (uint32_t)tp * RB;

    // Operand copies: 16 rows (1 KiB) of a packed tile per instruction.  A slice's 2 TA pieces of A and 2 TB pieces of B
    // lie one behind the other in its LDS slot, wave w brings pieces w NC .. w NC + NC - 1 (where they do not divide among
    // four waves the last wave repeats some: the same bytes to the same place).  One M0 per slice: the instruction
    // offset moves the LDS and the global address alike, so the global base of piece q is taken q KiB lower.  (M0 is a
    // reserved register, no allocation puts a value there; that nothing else in the kernel names it is tested on the
    // assembly of every instance.  As an operand of the other copies it costs moves in two loops, k = 6, w = 8, 64 x 128 and
    // k = 16, 64 x 64.)
    constexpr int NC = P::NC;
    // inner steps of this part
    const int kt0 = CUT ? (int)((int64_t)a.steps * part / a.parts) : 0;
    const int KT = CUT ? (int)((int64_t)a.steps * (part + 1) / a.parts) - kt0 : a.steps;
    const int piece0 = wave * NC < 2 * NF - NC ? wave * NC : 2 * NF - NC;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)lds;
    uint32_t m0_cur = lds_base + (uint32_t)piece0 * 1024u, m0_nxt = m0_cur + (D - 1) * SET;
    const int64_t rowblk = rowblock_bytes(a.KT);
    const int8_t* gbase[NC];
    int64_t gstride[NC];
#pragma unroll
    for (int q = 0; q < NC; ++q) {
        const int pc = piece0 + q;
        const bool isb = pc >= 2 * TA;
        uint32_t row = isb ? col0 + (uint32_t)(pc - 2 * TA) * 16u : row0 + (uint32_t)pc * 16u;
        const uint32_t top = (uint32_t)(isb ? a.pstrideB : a.pstrideA) - 16u;  // (padded rows of the stack)
        row = row < top ? row : top;  // a tile may reach past the padding: what it reads there is never stored
        gbase[q] = (isb ? a.SB : a.SA) + (int64_t)(row / TILE_R) * rowblk + (int)(row % TILE_R) * TILE_K - q * 1024 +
                   (int64_t)kt0 * TILE_BYTES;
        gstride[q] = isb ? a.strideB : a.strideA;
    }

    // copy number q of slice s into the set at m0; voff = 16 lane + 16 KiB * inner step
    auto copy = [&](auto S, auto X, uint32_t m0, uint32_t voff) __attribute__((always_inline)) {
        constexpr int s = decltype(S)::value, q = decltype(X)::value;
        const int8_t* base = gbase[q] + (int64_t)(s - 1) * gstride[q];
        if constexpr (q == 0)
            asm volatile("s_add_u32 m0, %0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3" ::"s"(m0), "n"((s - 1) * SLOT),
                         "v"(voff), "s"(base)
                         : "memory", "scc");
        else
            asm volatile("global_load_lds_dwordx4 %0, %1 offset:%2" ::"v"(voff), "s"(base), "n"(q * 1024) : "memory");
    };
    auto copy_slice = [&](auto S, uint32_t m0, uint32_t voff) __attribute__((always_inline)) {
        static_for<NC>([&](auto X) __attribute__((always_inline)) { copy(S, X, m0, voff); });
    };

    // Fragment addresses (see k_gemm: one MFMA takes 64 inner bytes, the four lane groups of 16 supply the logical chunks
    // 0, 3, 1, 2, which keeps the fetches off each other's banks).  ds_read offsets are 16-bit immediates: a second base
    // serves what lies beyond (k = 16 with 64 x 64 tiles, 128 KiB a set, reaches past both: an addition per fetch there).
    constexpr int FAR = 49152;
    uint32_t fcur[2][2], fnxt[2][2];  // [A, B][near, far]
    {
        const int chunk = (0x9c >> (2 * (lane >> 4))) & 3;  // 0, 3, 1, 2
        const int ra = wm * (16 * TA) + (lane & 15), rb = wn * (16 * TB) + (lane & 15);
        const uint32_t oa = lds_base + ra * TILE_K + swizzle(ra, chunk) * CHUNK;
        const uint32_t ob = lds_base + RA * TILE_K + rb * TILE_K + swizzle(rb, chunk) * CHUNK;
#pragma unroll
        for (int f = 0; f < 2; ++f) {
            fcur[0][f] = oa + f * FAR;
            fcur[1][f] = ob + f * FAR;
            fnxt[0][f] = oa + f * FAR + (D - 1) * SET;
            fnxt[1][f] = ob + f * FAR + (D - 1) * SET;
        }
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                if (f == 1 && SET <= 61440) continue;
                asm volatile("" : "+v"(fcur[o][f]));
                if (D > 1) asm volatile("" : "+v"(fnxt[o][f]));
            }
    }
    v4i low[L + 1][NF], hi[2][NF];  // fragments: row tiles of A, then column tiles of B
    auto fetch = [&](auto S, auto X, auto NEXT) __attribute__((always_inline)) {
        constexpr int s = decltype(S)::value, x = decltype(X)::value;
        constexpr bool next = decltype(NEXT)::value && D > 1;
        constexpr bool isb = x >= TA;
        constexpr int off = (s - 1) * SLOT + (isb ? x - TA : x) * 1024;
        constexpr int f = off >= 61440 ? 1 : 0;
        const uint32_t base = next ? fnxt[isb][f] : fcur[isb][f];
        const v4i v = *(lds_v4i_ptr)(uintptr_t)(base + (off - f * FAR));
        if constexpr (s <= L)
            low[s][x] = v;
        else
            hi[(s - L - 1) & 1][x] = v;
    };

    v4i acc[W][TA][TB];
    // what the accumulation registers do not hold lies in ordinary ones (k_extended)
    constexpr auto ordinary = [](int c, int i, int j) { return (c * TB + j) * TA + i >= ozr::ACC_TILES; };

    const uint32_t lv = (uint32_t)lane * 16u;
    auto step_off = [&](int kt) { return (uint32_t)(kt < KT - 1 ? kt : KT - 1) * (uint32_t)TILE_BYTES; };
    static_assert(L >= 2, "at least three slices");
    // What the compiler loads itself goes out first - scale exponents and the prefix sums of the stored bytes for the start
    // values -, then the first copies; all of it is on its way before anything is waited for.  (With the loads behind the
    // copies and a branch on the offsets, three latencies in a row: 6.5 us from the first instruction to the loop at 4096^3,
    // k = 8; now 3.8 us, 2.8 us on an idle chip.)
    const int cA = !CUT || part == 0 ? a.cA[0] : 0, cB = !CUT || part == 0 ? a.cB[0] : 0;  // (start values: the first part's)
    int exp_row = 0, exp_col = 0;
    v4i pa[K][TA];
    int pb[K][TB];
    if (t < RA && row0 + t < a.m) exp_row = a.eA[row0 + t];
    if (t < RB && col0 + t < a.p) exp_col = a.eB[col0 + t];
    {
        // (row and column tiles past the padding take any sums: their results are never stored)
        uint32_t rr[TA], cc[TB];
#pragma unroll
        for (int i = 0; i < TA; ++i) {
            const uint32_t r0 = row0 + wm * (16 * TA) + 16 * i, top = (uint32_t)a.pstrideA - 16u;
            rr[i] = (r0 < top ? r0 : top) + 4 * (lane >> 4);
        }
#pragma unroll
        for (int j = 0; j < TB; ++j) {
            const uint32_t c0 = col0 + wn * (16 * TB) + 16 * j, top = (uint32_t)a.pstrideB - 16u;
            cc[j] = (c0 < top ? c0 : top) + (lane & 15);
        }
#pragma unroll
        for (int q = 0; q < K; ++q) {
#pragma unroll
            for (int i = 0; i < TA; ++i) pa[q][i] = *reinterpret_cast<const v4i*>(a.PA + (int64_t)q * a.pstrideA + rr[i]);
#pragma unroll
            for (int j = 0; j < TB; ++j) pb[q][j] = a.PB[(int64_t)q * a.pstrideB + cc[j]];
        }
    }
    // Copies of the first steps in the order of the loop, so that its counted waits hold from the start: what interval v
    // reads in `step` (a low slice for the step after).  Before that, the low slices 2 .. L of step 0 themselves.
    if constexpr (HELD == 0) {
        static_for<L - 1>([&](auto X) __attribute__((always_inline)) {
            copy_slice(std::integral_constant<int, L - decltype(X)::value>{}, m0_cur, lv);
        });
        static_for<D == 2 ? NI : 1>([&](auto V) __attribute__((always_inline)) { copy_interval<P, decltype(V)::value, 0>(copy_slice, step_off, m0_cur, m0_nxt, lv); });
    }
    std::conditional_t<(HELD > 0), Held<P>, int> held;
    if constexpr (HELD > 0) held.begin(a, lds_base, row0, col0, wave, lane);
    if (t < RA) lds_exp[t] = exp_row;
    if (t < RB) lds_exp[RA + t] = exp_col;
    // The accumulators of a chunk start at -(ra[row] + cb[column]) (see the head of ozimmu_gemm.hip); the inner positions
    // past the last step carry q = 0, i.e. the offsets themselves, in the stored sums.
    static_for<W>([&](auto C) __attribute__((always_inline)) {
        constexpr int c = decltype(C)::value;
        constexpr Range range = chunk_range<K, R>(c);
        constexpr int s0 = range.s0, s1 = range.s1, t0 = range.g - s1, t1 = range.g - s0;
        const uint32_t fix = (uint32_t)((s1 - s0 + 1) * cA * cB) * (uint32_t)((2 * a.KT - a.steps) * TILE_K);
        uint32_t cb[TB];
#pragma unroll
        for (int j = 0; j < TB; ++j) cb[j] = fix - (uint32_t)cA * (uint32_t)(pb[t1 - 1][j] - (t0 > 1 ? pb[t0 > 1 ? t0 - 2 : 0][j] : 0));
        static_for<TA>([&](auto I) __attribute__((always_inline)) {
            constexpr int i = decltype(I)::value;
            uint32_t ra[4];
#pragma unroll
            for (int r = 0; r < 4; ++r)
                ra[r] = (uint32_t)cB * (uint32_t)(pa[s1 - 1][i][r] - (s0 > 1 ? pa[s0 > 1 ? s0 - 2 : 0][i][r] : 0));
            static_for<TB>([&](auto J) __attribute__((always_inline)) {
                constexpr int j = decltype(J)::value;
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[c][i][j][r] = (int)(cb[j] - ra[r]);
                if constexpr (ordinary(c, i, j))
                    asm volatile("" : "+v"(acc[c][i][j]));
                else
                    asm volatile("" : "+a"(acc[c][i][j]));
            });
        });
    });
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if constexpr (HELD == 0) {
        static_for<L - 1>([&](auto X) __attribute__((always_inline)) {
            constexpr int s = L - decltype(X)::value;
            static_for<NF>([&](auto F) __attribute__((always_inline)) { fetch(std::integral_constant<int, s>{}, F, std::false_type{}); });
        });
        wait_lds();
        __builtin_amdgcn_s_barrier();  // every wave has the low slices of step 0: their slots are free
        asm volatile("" ::: "memory");
        if constexpr (D == 2)
            static_for<NI - 1>([&](auto V) __attribute__((always_inline)) { copy_interval<P, decltype(V)::value, 1>(copy_slice, step_off, m0_cur, m0_nxt, lv); });
        else if constexpr (NI > 2)
            static_for<NI - 2>([&](auto V) __attribute__((always_inline)) {
                copy_interval<P, decltype(V)::value + 1, 0>(copy_slice, step_off, m0_cur, m0_nxt, lv);
            });

        uint32_t m0_sum = m0_cur + m0_nxt, fsum[2][2];
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                fsum[o][f] = fcur[o][f] + fnxt[o][f];
                if (D == 2) asm volatile("" : "+v"(fsum[o][f]));
            }
        if (D == 2) asm volatile("" : "+s"(m0_sum));
        // where the copies of a step read: what is fetched for this step is followed by step kt + D in its place (v1), what is
        // fetched for the next one by step kt + 1 + D (v2; past the end: the last step again, never used)
        // (v0: v1 of the step before, for what the last interval of that step read for itself)
        uint32_t v0 = lv + step_off(D - 1), v1 = lv + step_off(D), v2 = v1;
        for (int kt = 0; kt < KT; ++kt) {
            static_for<P::NM>([&](auto Q) __attribute__((always_inline)) {
                constexpr int q = decltype(Q)::value;
                constexpr int gi = plan.group_of[q], v = plan.interval_of[q], vp = (v + NI - 1) % NI;
                if constexpr (plan.opens[q]) {
                    // what this interval reads has landed, and every wave has what the interval before read
                    wait_lds();
                    wait_vmcnt<P::NC * (D * K - plan.nslot[v] - plan.nslot[vp])>();
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_sched_barrier(0);
                }
                if constexpr (plan.group_at[0] + 2 == q) {
                    // what the step needs from its second group on, and the next step from its start (in a gap between two
                    // MFMAs: at the end of the loop it would make a bubble of a dozen instructions)
                    v2 = lv + step_off(kt + 1 + D);
                    asm volatile("" : "+v"(v2));
                }
                if constexpr (D == 2 && plan.group_at[0] + 3 == q) {
                    fnxt[0][0] = fsum[0][0] - fcur[0][0];
                    fnxt[1][0] = fsum[1][0] - fcur[1][0];
                    asm volatile("" : "+v"(fnxt[0][0]), "+v"(fnxt[1][0]));
                    if constexpr (SET > 61440) {
                        fnxt[0][1] = fsum[0][1] - fcur[0][1];
                        fnxt[1][1] = fsum[1][1] - fcur[1][1];
                        asm volatile("" : "+v"(fnxt[0][1]), "+v"(fnxt[1][1]));
                    }
                }
                static_for<plan.reads[q]>([&](auto X) __attribute__((always_inline)) {
                    constexpr int x = plan.read_at[q] + decltype(X)::value;
                    constexpr int sl = plan.read_slice[gi][x / NF];
                    // (the operand that is needed first comes first: B of a low slice, A of a high one)
                    constexpr int f = sl <= L ? (x % NF + TA) % NF : x % NF;
                    fetch(std::integral_constant<int, sl>{}, std::integral_constant<int, f>{},
                          std::integral_constant<bool, plan.read_next[gi][x / NF]>{});
                });
                static_for<plan.copies[q]>([&](auto X) __attribute__((always_inline)) {
                    constexpr int x = plan.copy_at[q] + decltype(X)::value, y = x / P::NC;
                    constexpr int sl = plan.slot_slice[vp][y];
                    // the first interval replaces what the last one of the step before read
                    constexpr bool next = plan.slot_next[vp][y];
                    constexpr int ahead = (next ? 1 : 0) - (v == 0 ? 1 : 0);  // -1, 0, 1: v0, v1, v2
                    copy(std::integral_constant<int, sl>{}, std::integral_constant<int, x % P::NC>{}, ahead == 0 ? m0_cur : m0_nxt,
                         ahead < 0 ? v0 : ahead == 0 ? v1 : v2);
                });
                constexpr int pr = q / P::TT, m = q % P::TT;
                constexpr int s = plan.s[pr], u = plan.t[pr];
                // (back and forth, so that consecutive MFMAs share an operand)
                constexpr int j = m / TA, i = (j & 1) ? TA - 1 - m % TA : m % TA;
                constexpr int c = chunk_of(s, u, R);
                const v4i fa = s <= L ? low[s <= L ? s : 0][i] : hi[(s - L - 1) & 1][i];
                const v4i fb = u <= L ? low[u <= L ? u : 0][TA + j] : hi[(u - L - 1) & 1][TA + j];
                // (in place: the compiler sees no matrix instruction; the wait states that its result asks for come after the loop)
                if constexpr (!IN_PLACE)
                    acc[c][i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa, fb, acc[c][i][j], 0, 0, 0);
                else if constexpr (ordinary(c, i, j))
                    asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+v"(acc[c][i][j]) : "v"(fa), "v"(fb));
                else
                    asm volatile("v_mfma_i32_16x16x64_i8 %0, %1, %2, %0" : "+a"(acc[c][i][j]) : "v"(fa), "v"(fb));
                // (an MFMA touches no memory: without a use in the order of the asm statements instruction selection may gather
                // all fetches and copies of the step in front of all MFMAs)
                // (with one set of operands it does not, and the use would cost moves of accumulators)
                if constexpr (D == 2 && !IN_PLACE) asm volatile("" ::"a"(acc[c][i][j]));
                __builtin_amdgcn_sched_barrier(0);
            });
            v0 = v1;
            v1 = v2;
            if constexpr (D == 2) {
                m0_cur = m0_nxt;
                m0_nxt = m0_sum - m0_cur;
                fcur[0][0] = fnxt[0][0], fcur[0][1] = fnxt[0][1];
                fcur[1][0] = fnxt[1][0], fcur[1][1] = fnxt[1][1];
            }
        }
    } else {
        held.loop(a, acc, KT);
    }
    wait_vmcnt<0>();  // no copy may still be writing LDS when the workgroup ends
    if constexpr (IN_PLACE) asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");

    if constexpr (CUT) {
        // the part's sums as they lie in the registers, 16 bytes a lane (k_add_parts reads them back); written through L2, which would
        // otherwise be written back between the two kernels (256 x 8192 x 256, k = 8, 48.4 -> 45.9 us a call with the slices)
        constexpr int TT = TA * TB, AGENT = 16;
        int32_t* const out = a.blocks + (int64_t)(block * a.parts + part) * (W * TT) * 1024;
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(out, 0, W * TT * 4096, 0x00020000);
        static_for<W * TT>([&](auto X) __attribute__((always_inline)) {
            constexpr int x = decltype(X)::value, c = x / TT, i = x % TT % TA, j = x % TT / TA;
            typedef unsigned v4u __attribute__((ext_vector_type(4)));
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, acc[c][i][j]), rsrc, t * 16, x * 4096, AGENT);
        });
        return;
    }
    // One scale per slice (Algorithm 5; a chunk is then one pair): the exponents of all slices of the tile's rows, then columns,
    // take the place of the operands.
    int* const slice_exp = reinterpret_cast<int*>(lds);
    if constexpr (PER_SLICE) {
        static_assert(R == 1, "");
        __syncthreads();
        for (int x = t; x < K * (RA + RB); x += 256) {
            const int s = x / (RA + RB), y = x - s * (RA + RB);
            const int64_t at = y < RA ? (int64_t)row0 + y : (int64_t)col0 + (y - RA), end = y < RA ? a.m : a.p;
            slice_exp[x] = at < end ? (y < RA ? a.eA : a.eB)[s * end + at] : 0;
        }
        __syncthreads();
    }

    // Steps (iv) and (v): per element the chunk sums in schedule order, one rounded addition each.  Register r of tile
    // (i, j) in lane l: row 4 (l / 16) + r, column l % 16.
    int lq = lane >> 4, lc = lane & 15;
    asm volatile("" : "+v"(lq), "+v"(lc));
    double* const obase = a.finish ? a.Cout : a.D;
    const int64_t opitch = a.finish ? a.ldco : a.ldd;
    const bool with_c = a.finish && a.cbeta != 0.0;
    int ea[TA][4], eb[TB];
    int emin = 0x7fffffff, emax = -0x7fffffff;
#pragma unroll
    for (int j = 0; j < TB; ++j) eb[j] = lds_exp[RA + wn * (16 * TB) + 16 * j + lc];
#pragma unroll
    for (int i = 0; i < TA; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) ea[i][r] = lds_exp[wm * (16 * TA) + 16 * i + 4 * lq + r];
#pragma unroll
    for (int j = 0; j < TB; ++j)
#pragma unroll
        for (int i = 0; i < TA; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int e = ea[i][r] + eb[j];
                emin = e < emin ? e : emin;
                emax = e > emax ? e : emax;
            }
    // Rounding does not see a common power of two: while every term is a normal number, the sum can be formed on the
    // integers scaled by 2^(beta (2 - g)) only (a term and its addition are then one fused multiply-add of an exact
    // product) and scaled by 2^(2 - 2 beta + ea + eb) at the end.  Otherwise term by term.
    const bool plain_range = emin + 2 - a.beta * (K + 1) >= -1022 && emax + 2 - 2 * a.beta + 40 <= 1023;
    const bool scaled = __ballot(plain_range) == ~0ull;
    // Four 16 x 16 tiles at a time: sixteen independent chains of additions per lane keep the FP64 unit busy.
    // Stores stay in L2 until its lines are whole (see ozr::merge_rows) or stream past it.  Where the registers allow it, that is asked around
    // every four stores: two whole ends, one for each, are 2 to 10 % of calls of short inner dimensions (554 x 5 x 20266, k = 10,
    // 96.0 and 94.9 us; 2947 x 1 x 756, k = 12, one addition per pair, 76.3 and 73.0).  Elsewhere it spills sums, and asked around
    // every store it costs more than it saves (4096 x 256 x 4096, k = 9, per pair, 329 and 344 us).
    enum { STREAMED, KEPT, ASK };
    auto finish_tile = [&](auto SCALED, auto STORE) __attribute__((always_inline)) {
        constexpr int TT = TA * TB, BATCH = TT < 4 ? TT : 4;
        const double step = ldexp(1.0, -a.beta);
        static_for<(TT + BATCH - 1) / BATCH>([&](auto Q) __attribute__((always_inline)) {
            constexpr int first = decltype(Q)::value * BATCH, n = TT - first < BATCH ? TT - first : BATCH;
            double cold[n][4], d[n][4];
            if (with_c)
#pragma unroll
                for (int x = 0; x < n; ++x) {
                    const int i = (first + x) % TA, j = (first + x) / TA;
                    const int64_t col = (int64_t)col0 + wn * (16 * TB) + 16 * j + lc;
                    const int64_t row = (int64_t)row0 + wm * (16 * TA) + 16 * i + 4 * lq;
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        cold[x][r] = (col < a.p && row + r < a.m) ? __builtin_nontemporal_load(obase + (row + r) * opitch + col) : 0.0;
                }
            double scale = 1.0;
            static_for<W>([&](auto C) __attribute__((always_inline)) {
                constexpr int c = decltype(C)::value;
                constexpr int g = chunk_range<K, R>(c).g, s = chunk_range<K, R>(c).s0;
                if constexpr (c > 0)
                    if constexpr (g != chunk_range<K, R>(c - 1).g) scale *= step;
#pragma unroll
                for (int x = 0; x < n; ++x) {
                    const int i = (first + x) % TA, j = (first + x) / TA;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const double v = (double)acc[c][i][j][r];
                        if constexpr (decltype(SCALED)::value) {
                            d[x][r] = c == 0 ? v : __builtin_fma(v, scale, d[x][r]);
                        } else if constexpr (PER_SLICE) {
                            const int es = slice_exp[(s - 1) * (RA + RB) + wm * (16 * TA) + 16 * i + 4 * lq + r];
                            const int et = slice_exp[(g - s - 1) * (RA + RB) + RA + wn * (16 * TB) + 16 * j + lc];
                            const double term = ldexp(v, es + et + 2 - 2 * a.beta);
                            d[x][r] = c == 0 ? term : d[x][r] + term;
                        } else {
                            const double term = ldexp(v, ea[i][r] + eb[j] + 2 - a.beta * g);
                            d[x][r] = c == 0 ? term : d[x][r] + term;
                        }
                    }
                }
            });
#pragma unroll
            for (int x = 0; x < n; ++x) {
                const int i = (first + x) % TA, j = (first + x) / TA;
                const int64_t col = (int64_t)col0 + wn * (16 * TB) + 16 * j + lc;
                const int64_t row = (int64_t)row0 + wm * (16 * TA) + 16 * i + 4 * lq;
                auto finish = [&](int r) __attribute__((always_inline)) {
                    if constexpr (decltype(SCALED)::value) d[x][r] = ldexp(d[x][r], ea[i][r] + eb[j] + 2 - 2 * a.beta);
                    if (a.finish) {
                        d[x][r] = a.alpha * d[x][r];
                        if (with_c) d[x][r] = d[x][r] + a.cbeta * cold[x][r];
                    }
                };
                if constexpr (decltype(STORE)::value == ASK) {
                    auto store = [&](auto KEEP) __attribute__((always_inline)) {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (col < a.p && row + r < a.m) {
                                double* const out = obase + (row + r) * opitch + col;
                                if constexpr (decltype(KEEP)::value)
                                    *out = d[x][r];
                                else
                                    __builtin_nontemporal_store(d[x][r], out);
                            }
                    };
#pragma unroll
                    for (int r = 0; r < 4; ++r) finish(r);
                    // (the comments in asm keep the compiler from making one ordinary store of two)
                    if (a.keep) {
                        store(std::true_type{});
                    } else {
                        asm volatile("; streamed");
                        store(std::false_type{});
                        asm volatile("; streamed");
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        finish(r);
                        if (col < a.p && row + r < a.m) {
                            double* const out = obase + (row + r) * opitch + col;
                            if constexpr (decltype(STORE)::value == KEPT)
                                *out = d[x][r];
                            else
                                __builtin_nontemporal_store(d[x][r], out);
                        }
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    constexpr bool ROOM = W * TA * TB < (WAVES == 1 ? 60 : 32);
    constexpr std::integral_constant<int, ROOM ? ASK : STREAMED> asked{};
    constexpr std::integral_constant<int, ROOM ? ASK : KEPT> kept{};
    if constexpr (PER_SLICE)
        finish_tile(std::false_type{}, kept);
    else if (!scaled)
        finish_tile(std::false_type{}, asked);
    else if (ROOM || !a.keep)
        finish_tile(std::true_type{}, asked);
    else if constexpr (!ROOM)
        finish_tile(std::true_type{}, kept);
}

template <int K, int R, int TA, int TB, int D, int WAVES>
__global__ __launch_bounds__(256, WAVES) void k_resident(ozk::ResidentArgs a)
{
    run_tile<Plan<K, R, TA, TB, D>, WAVES, false, End::COMMON>(a);
}
// Few tiles of a long inner dimension would leave most of the chip idle: each is cut among a.parts workgroups, whose INT32 sums
// k_add_parts (ozimmu_gemm.hip) adds up.  What bounds it is the latency of a step and of the sums' way (whole calls, k = 8: 47 x 11948 x 48 119 -> 62 us, 43 of it the split; 256 x 8192 x 256
// 83 -> 63; 67 x 25614 x 69, k = 4, 148 -> 96).
template <int K, int R, int TA, int TB, int D, int WAVES>
__global__ __launch_bounds__(256, WAVES) void k_cut(ozk::ResidentArgs a)
{
    run_tile<Plan<K, R, TA, TB, D>, WAVES, false, End::PART>(a);
}
template <int K, int R, int TA, int TB, int D>
__global__ __launch_bounds__(256, 1) void k_extended(ozk::ResidentArgs a)
{
    run_tile<Plan<K, R, TA, TB, D>, 1, true, End::COMMON>(a);
}
// k_extended's way with H slices of A held and those of B passing by (HeldPlan).
template <int K, int R, int TA, int TB, int H>
__global__ __launch_bounds__(256, 1) void k_held(ozk::ResidentArgs a)
{
    run_tile<HeldPlan<K, R, TA, TB, H>, 1, true, End::COMMON>(a);
}
// One scale per slice: k_resident or k_extended with the exponents of every slice.
template <int K, int TA, int TB, int D, int WAVES, bool IN_PLACE>
__global__ __launch_bounds__(256, WAVES) void k_per_slice(ozk::ResidentArgs a)
{
    run_tile<Plan<K, 1, TA, TB, D>, WAVES, IN_PLACE, End::PER_SLICE>(a);
}

template <int K, int R, int V>
hipError_t launch(const ozk::ResidentArgs& a_in, hipStream_t st)
{
    constexpr ozr::Config c = ozr::config(K, R, V);
    if constexpr (c.ta == 0) {
        return a_in.setup ? hipSuccess : hipErrorInvalidValue;
    } else {
        ozk::ResidentArgs a = a_in;
        constexpr int RA = 32 * c.ta, RB = 32 * c.tb;
        a.TM = (int)((a.m + RA - 1) / RA);
        a.TP = (int)((a.p + RB - 1) / RB);
        const unsigned tiles = (unsigned)a.TM * (unsigned)a.TP;
        constexpr int smem = ozr::lds_bytes(K, c);
        static_assert(smem <= 160 * 1024, "LDS of a compute unit");
        // [0]: whole tiles, one exponent per row and column; then, where there is one, the kernel for a scale per slice, for parts
        const void* kernels[3] = {};
        if constexpr (V == ozr::HELD)
            kernels[0] = reinterpret_cast<const void*>(&k_held<K, R, c.ta, c.tb, c.held>);
        else if constexpr (V == ozr::EXTENDED)
            kernels[0] = reinterpret_cast<const void*>(&k_extended<K, R, c.ta, c.tb, c.depth>);
        else
            kernels[0] = reinterpret_cast<const void*>(&k_resident<K, R, c.ta, c.tb, c.depth, c.waves>);
        if constexpr (R == 1 && ozr::per_slice_tile(K, V))
            kernels[1] = reinterpret_cast<const void*>(&k_per_slice<K, c.ta, c.tb, c.depth, c.waves, V == ozr::EXTENDED>);
        if constexpr (ozr::may_cut(V, c))
            kernels[2] = reinterpret_cast<const void*>(&k_cut<K, R, c.ta, c.tb, c.depth, c.waves>);
        if (a.setup) {
            for (const void* kernel : kernels) {
                const hipError_t e = kernel ? hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, smem) : hipSuccess;
                if (e != hipSuccess) return e;
            }
            return hipSuccess;
        }
        const void* const kernel = kernels[a.parts > 1 ? 2 : a.per_slice ? 1 : 0];
        if (!kernel || (a.parts > 1 && a.per_slice)) return hipErrorInvalidValue;
        void* args[] = {&a};
        return ozk::launch_status(hipLaunchKernel(kernel, dim3(a.parts > 1 ? tiles * (unsigned)a.parts : tiles), dim3(256), args, smem, st));
    }
}

template <int K, int R>
hipError_t launch_r(const ozk::ResidentArgs& a, int variant, hipStream_t st)
{
    switch (variant) {
        case 0: return launch<K, R, 0>(a, st);
        case 1: return launch<K, R, 1>(a, st);
        case 2: return launch<K, R, 2>(a, st);
        case 3: return launch<K, R, 3>(a, st);
        case 4: return launch<K, R, 4>(a, st);
        case 5: return launch<K, R, 5>(a, st);
        case ozr::EXTENDED: return launch<K, R, ozr::EXTENDED>(a, st);
        case ozr::HELD: return launch<K, R, ozr::HELD>(a, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

namespace ozk {

template <>
hipError_t launch_resident_k<OZ_RES_K>(const ResidentArgs& a, int r, int variant, hipStream_t st)
{
    constexpr int K = OZ_RES_K;
    if (r >= K) return launch_r<K, K>(a, variant, st);
    if constexpr (K > 8)
        if (r == 8) return launch_r<K, 8>(a, variant, st);
    if constexpr (K > 4)
        if (r == 4) return launch_r<K, 4>(a, variant, st);
    if (r == 2) return launch_r<K, 2>(a, variant, st);
    if (r == 1) return launch_r<K, 1>(a, variant, st);
    return hipErrorInvalidValue;
}

}  // namespace ozk
