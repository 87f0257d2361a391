// C ABI of the library (declared in include/ozimmu.h): argument checks, the
// host-side schedule of Algorithm 6 (groups g = 2..k+1, chunks of at most r
// consecutive s), workspace carving and kernel launches.  No allocation, no
// host synchronisation.  The only state kept between calls is what the one-time
// set-up of a device leaves behind (ozimmu_init).
#include "../../include/ozimmu.h"
#include "ozimmu_kernels.h"
#include "ozimmu_layout.h"
#include "ozimmu_resident.h"
#include <cmath>
#include <mutex>

namespace {

// m, p <= 2^22 - 256: every grid dimension stays within the HIP limits (the column split launches
// rows_padded(p) / 64 <= 65535 workgroups along y)
constexpr int64_t MAX_OUTER = ((int64_t)1 << 22) - 256;
constexpr int64_t MAX_INNER = (int64_t)1 << 29;   // beta >= 1 (Section 2)
constexpr int64_t MAX_LD = ((int64_t)1 << 30) - 1;  // the kernels form 4 * ld in 32 bits

// Workspace of ozimmu_dgemm_static: device memory of the library itself, one copy on every GPU the library
// is loaded on.  In host code this name is only a handle for hipGetSymbolAddress; the address kernels and
// launchers get is DeviceState::static_ws.
static __device__ __align__(256) unsigned char scratch[OZIMMU_STATIC_WORKSPACE_BYTES];

constexpr int MAX_DEVICES = 64;
struct DeviceState {
    bool ready;
    int num_cu;       // compute units: size of the persistent grid
    void* static_ws;  // device address of `scratch` on this device
};
std::mutex g_state_mutex;
DeviceState g_state[MAX_DEVICES];

// State of the current device, set up on first use.
int device_state(DeviceState* out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return OZIMMU_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_state_mutex);
    DeviceState& s = g_state[dev];
    if (!s.ready) {
        if (ozk::setup_gemm_kernels() != hipSuccess || ozk::setup_small() != hipSuccess) return OZIMMU_ERR_HIP;
        int ncu = 0;
        if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || ncu < 1)
            return OZIMMU_ERR_HIP;
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return OZIMMU_ERR_HIP;
        s.num_cu = ncu;
        s.static_ws = ptr;
        s.ready = true;
    }
    *out = s;
    return OZIMMU_OK;
}

inline int64_t align256(int64_t x) { return (x + 255) / 256 * 256; }

int beta_of(int64_t n)
{
    // floor((31 - log2 n)/2) >= b  <=>  n * 4^b <= 2^31
    int beta = 0;
    while (beta < 7 && (n << (2 * (beta + 1))) <= ((int64_t)1 << 31)) ++beta;
    return beta;
}

int64_t r_of(int64_t n, int beta)
{
    int L = 0;  // ceil(log2 n)
    while (((int64_t)1 << L) < n) ++L;
    const int ex = 31 - 2 * beta - L;
    return ex > 0 ? ((int64_t)1 << ex) : 1;
}

// largest power of two r_w with r_w * n * (2^(beta-1))^2 <= 2^31 - 1 (round-to-nearest slices obey |q| <= 2^(beta-1))
int64_t r_wide_of(int64_t n, int beta)
{
    int64_t r = 1;
    const int64_t lim = ((int64_t)1 << 31) - 1;
    while (2 * r * n * ((int64_t)1 << (2 * beta - 2)) <= lim) r *= 2;
    return r;
}

// most products of a chunk, by accumulate mode
int64_t r_of_mode(int64_t n, int accumulate_mode)
{
    if (accumulate_mode == OZIMMU_ACCUM_PER_PAIR) return 1;
    return accumulate_mode == OZIMMU_ACCUM_WIDE ? r_wide_of(n, beta_of(n)) : r_of(n, beta_of(n));
}

int dgemm_impl(int64_t m, int64_t n, int64_t p, const double* A, int64_t lda, const double* B, int64_t ldb,
               double* D, int64_t ldd, int k, int split_mode, int accumulate_mode, void* workspace,
               size_t workspace_bytes, void* stream, void* const* events, int resident_tile = -1, int parts = 1);

// The split-inner way of running the schedule (see run_schedule) works on at most this many 256 x 256 tiles
// at a time: outputs that small as a whole, or the last, partly filled round of tiles of a larger output
// (half the 256 compute units of the chip this is written for: every tile can then be cut at least in two).
// A constant, so that the workspace size does not depend on the device.
constexpr int64_t SPLIT_INNER_MAX_TILES = 128;
inline int64_t output_tiles(int64_t m, int64_t p)
{
    return (ozl::rows_padded(m) / ozl::TILE_R) * (ozl::rows_padded(p) / ozl::TILE_R);
}
// The chunk-parallel way (see run_schedule) keeps one block per (chunk, tile): used for outputs of fewer tiles than
// the chip has compute units whose tiles times chunks stay within this many blocks (1 GiB).
constexpr int64_t CHUNK_PARALLEL_MAX_BLOCKS = 4096;
// Inner dimensions above this make the persistent kernel wait for the whole grid at chunk starts.
constexpr int64_t GRID_WAIT_MIN_INNER = 8192 + 512;
// Sets of blocks the rounds of the queue schedule take in turn (see run_schedule).
constexpr int64_t QUEUE_SETS = 3;
// Outputs of at least this many tiles take the queue by default, unless they are one round of tiles (one per compute
// unit at most) whose blocks fit the chunk-parallel way.
constexpr int64_t QUEUE_MIN_TILES = 96;
constexpr int64_t QUEUE_XCD_WORDS = 8 * 40;  // per-XCD ticket batches of the queue (see k_gemm)
constexpr int64_t BLOCK_BYTES = 4 * 256 * 256;
// Room for the sums of tiles whose inner dimension is cut (ozr::estimate_us with parts): asked for where that may pay.
constexpr int64_t CUT_MAX_TILES = 16, CUT_MIN_INNER = 1024, CUT_BLOCKS = 128;
inline int64_t chunks_of(int k, int64_t r)
{
    int64_t w = 0;
    for (int g = 2; g <= k + 1; ++g) w += ((g - 1) + r - 1) / r;
    return w;
}
// INT32 blocks of 256 x 256 behind the slice stacks: what the split-inner way needs at least ...
inline int64_t min_partial_blocks(int64_t m, int64_t p)
{
    const int64_t T = output_tiles(m, p);
    return T < SPLIT_INNER_MAX_TILES ? T : SPLIT_INNER_MAX_TILES;
}
// ... and what ozimmu_workspace_bytes asks for, so that the chunk-parallel way can be used where it applies
inline int64_t partial_blocks(int64_t m, int64_t n, int64_t p, int k)
{
    const int64_t base = min_partial_blocks(m, p);
    if (n < 1 || n > MAX_INNER || k < 1) return base;
    // (the chunk-parallel way takes the tiles that do not fill a round of the 256 compute units of the chip this is
    // written for; the queue, which takes outputs of QUEUE_MIN_TILES tiles and more, wants up to QUEUE_SETS sets of chunks x 256
    // blocks and a counter per tile and round)
    const int64_t T = output_tiles(m, p);
    const int64_t w = chunks_of(k, r_of(n, beta_of(n)));
    const int64_t items = (T <= 256 ? T : T % 256) * w;
    int64_t blocks = (items <= CHUNK_PARALLEL_MAX_BLOCKS && items > base) ? items : base;
    if (T <= CUT_MAX_TILES && n >= CUT_MIN_INNER && blocks < CUT_BLOCKS) blocks = CUT_BLOCKS;
    if (T >= QUEUE_MIN_TILES && w * 256 * BLOCK_BYTES < ((int64_t)1 << 31) && T * w < ((int64_t)1 << 30)) {
        const int64_t rounds = (T + 255) / 256;
        const int64_t queue = (rounds < QUEUE_SETS ? rounds : QUEUE_SETS) * w * (T < 256 ? T : 256) +
                              (4 * (T + rounds + 2 + QUEUE_XCD_WORDS) + BLOCK_BYTES - 1) / BLOCK_BYTES;
        if (queue > blocks) blocks = queue;
    }
    return blocks;
}
// the least a call of ozimmu_dgemm can run in (no room for the chunk-parallel blocks)
inline size_t min_workspace_bytes(int64_t m, int64_t n, int64_t p, int k)
{
    return (size_t)(align256(OZIMMU_SCRATCH_BYTES) + align256(4 * m) + align256(4 * p)) +
           (size_t)ozl::stack_bytes(m, n, k) + (size_t)ozl::stack_bytes(p, n, k) +
           (size_t)(min_partial_blocks(m, p) * BLOCK_BYTES);
}

inline int hip_status(hipError_t e) { return e == hipSuccess ? OZIMMU_OK : OZIMMU_ERR_HIP; }

int check_gemm_args(int64_t m, int64_t n, int64_t p, const void* SA, int kA, const void* SB, int kB, int g, int s0,
                    int s1)
{
    if (m < 0 || n < 0 || p < 0 || m > MAX_OUTER || p > MAX_OUTER || n > MAX_INNER) return OZIMMU_ERR_DIM;
    if (kA < 1 || kA > OZIMMU_MAX_SLICES || kB < 1 || kB > OZIMMU_MAX_SLICES) return OZIMMU_ERR_SLICES;
    if (s0 < 1 || s1 < s0 || s1 > kA || g - s1 < 1 || g - s0 > kB) return OZIMMU_ERR_SLICES;
    if (m == 0 || n == 0 || p == 0) return OZIMMU_OK;
    if (!SA || !SB) return OZIMMU_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(SA) % 256 || reinterpret_cast<uintptr_t>(SB) % 256) return OZIMMU_ERR_WORKSPACE;
    return OZIMMU_OK;
}

// Offset of the stored bytes (see ozimmu_layout.h): round-to-nearest slices obey |q| <= 2^(beta-1), so the offset
// 2^(beta-1) - 1 (63 for beta = 7) moves them into [-1, 2^beta - 1]: inside the magnitude 2^beta - 1 for which the
// paper derives the chunk length r, so no INT32 sum of a chunk can overflow with the stored bytes either.  Bit-mask
// slices (|q| <= 2^beta - 1) have no room for an offset, and neither have the wide chunks, whose length is derived
// from |q| <= 2^(beta-1).
inline int rn_offset(int beta) { return (1 << (beta - 1)) - 1; }

// Products so short that the offsets do not matter (a compute unit at work for 100 us or so does not reach the power limit).
inline bool short_product(int64_t m, int64_t n, int64_t p, int k)
{
    return (double)m * (double)n * (double)p * k * (k + 1) <= 3.2e11;
}

// single chunk (s0 > 0): g, s = s0..s1; full schedule (s0 == 0): g = g_lo..g_hi, chunks of r.
// SA / SB are whole stacks of kA / kB slices (slices, prefix row sums, trailer).
ozk::GemmArgs make_args(int64_t m, int64_t n, int64_t p, const int8_t* SA, int kA, const int8_t* SB, int kB, int g_lo,
                        int g_hi, int r, int s0, int s1, void* scratch, int num_cu)
{
    ozk::GemmArgs a{};
    a.num_cu = num_cu;
    a.SA = SA;
    a.SB = SB;
    a.PA = reinterpret_cast<const int32_t*>(SA + ozl::sums_offset(m, n, kA));
    a.PB = reinterpret_cast<const int32_t*>(SB + ozl::sums_offset(p, n, kB));
    a.pstrideA = ozl::rows_padded(m);
    a.pstrideB = ozl::rows_padded(p);
    a.cA = reinterpret_cast<const int32_t*>(SA + ozl::trailer_offset(m, n, kA));
    a.cB = reinterpret_cast<const int32_t*>(SB + ozl::trailer_offset(p, n, kB));
    a.strideA = ozl::slice_bytes(m, n);
    a.strideB = ozl::slice_bytes(p, n);
    a.KT = (int)(ozl::inner_padded(n) / ozl::TILE_K);
    a.g_lo = g_lo;
    a.g_hi = g_hi;
    a.r = r;
    a.s0 = s0;
    a.s1 = s1;
    a.m = m;
    a.p = p;
    a.beta = beta_of(n);
    a.tile_begin = 0;
    a.tile_count = (int)((ozl::rows_padded(m) / ozl::TILE_R) * (ozl::rows_padded(p) / ozl::TILE_R));
    a.zsplit = 1;
    a.sync = static_cast<unsigned*>(scratch);
    a.spin_limit = 64;  // polls (about 0.1 us each) before a workgroup stops waiting for its team
    // the grid-wide wait pays only when the operand panels are long (see arrive_and_wait2)
    a.grid_spin_limit = n > GRID_WAIT_MIN_INNER ? 64 : 0;
    a.sync_epoch = 0;
    a.alpha = 1.0;
    return a;
}

// Step (v) applied by the last chunk of every tile: out = fl(fl(alpha d) + fl(cbeta c_old)).
struct Finish {
    bool on;
    double alpha, cbeta;
    double* Cout;   // == D when cbeta == 0 (the sum is formed in C itself)
    int64_t ldco;
};

// How steps (iii) to (v) are run.
struct Way {
    enum Kind { RESIDENT, QUEUE, TILES } kind = TILES;
    int tile = -1, parts = 1;        // RESIDENT: which tile; workgroups that share its inner dimension
    int64_t sets = 0;                // QUEUE
    int64_t cp_tail = 0, tail = 0;   // TILES: the last cp_tail tiles go the chunk-parallel way, or the last `tail` the split-inner
    int cp_z = 1, Z = 1;             // way, cut in cp_z / Z; the others to the persistent launch
};

// The choice among the ways that run_schedule lists.  A function of the sizes, the room for blocks (`capacity`, of BLOCK_BYTES; with one
// scale per slice no way that needs any is taken: they know one exponent per row and column) and the number of compute units only: no GPU is asked, so tests check it without one.
Way choose_way(int64_t m, int64_t n, int64_t p, int k, int r_eff, bool per_slice, int schedule, int64_t capacity, int num_cu)
{
    const int KT = (int)(ozl::inner_padded(n) / ozl::TILE_K);
    const int64_t T = output_tiles(m, p);
    const int64_t w = chunks_of(k, r_eff);
    Way way;
    auto queue_way = [&](int64_t sets) {
        way.kind = Way::QUEUE;
        way.sets = sets;
        return way;
    };

    // The queue, for the tiles [0, tiles) of the band order: one launch whose work items are all
    // (chunk, tile) pairs, handed out round by round (256 tiles) through a counter; an item leaves its INT32 sums
    // in a block, and the workgroup that stores the last block of a tile adds the tile's chunks up (steps (iv),
    // (v)).  Needs sets x chunks x min(tiles, 256) blocks (the rounds take the sets in turn) and a counter per
    // tile and round.  Against the persistent launch with the fused epilogue it moves 4 + 4 bytes per element
    // and chunk instead of 16, and no workgroup ever waits for another (measured 3 to 4 % faster at 16384^3,
    // 2 % at 8192^3, k = 8).  queue_sets: how many sets fit (0: the way cannot be used for that many tiles).
    auto queue_sets = [&](int64_t tiles) -> int64_t {
        if (per_slice || tiles < 1 || tiles * w >= ((int64_t)1 << 30)) return 0;
        const int64_t stride = tiles < ozk::QUEUE_ROUND_TILES ? tiles : ozk::QUEUE_ROUND_TILES;
        if (w * stride * BLOCK_BYTES >= ((int64_t)1 << 31)) return 0;  // 32-bit byte offsets inside a set of blocks
        const int64_t rounds = (tiles + ozk::QUEUE_ROUND_TILES - 1) / ozk::QUEUE_ROUND_TILES;
        const int64_t counter_blocks = (4 * (tiles + rounds + 2 + QUEUE_XCD_WORDS) + BLOCK_BYTES - 1) / BLOCK_BYTES;
        int64_t sets = rounds < QUEUE_SETS ? rounds : QUEUE_SETS;
        while (sets > 1 && sets * w * stride + counter_blocks > capacity) --sets;
        if (sets * w * stride + counter_blocks > capacity) return 0;
        return (sets >= 2 || rounds == 1) ? sets : 0;
    };
    // An output of one round of tiles whose blocks fit goes the chunk-parallel way rather than through the queue: every
    // compute unit gets items from the first moment, and the one accumulation kernel at the end costs less than the
    // queue's ramp (k = 8, chunk-parallel against queue: 2560^3, 100 tiles, 0.53 against 0.58 ms; 3072^3 0.87 against
    // 0.92; 4096^3, 256 tiles, 1.87 against 1.89; 5120^3, 400 tiles, with the queue for the full round only: 3.60
    // against 3.43).
    const bool one_round_fits = !per_slice && T <= num_cu && T * w <= CHUNK_PARALLEL_MAX_BLOCKS &&
                                T * w <= capacity;
    const int64_t sets_all = queue_sets(T);
    if (schedule == OZIMMU_SCHEDULE_QUEUE && sets_all > 0) return queue_way(sets_all);

    // Chunk-parallel, for outputs of few tiles, or the tiles of a partly filled last round (`cand`, the last ones in band
    // order): ONE launch whose work items are (chunk, inner part, tile), every chunk writing (or, when cut,
    // atomically adding) its INT32 sums to a block of its own per tile, and one kernel that adds the chunks of every
    // element in the order of Algorithm 6.  All chunks of all those tiles run side by side, so a 1024^3 product
    // occupies 128 compute units instead of 16; the price is 4 bytes of workspace per element and chunk.
    const int64_t cand = num_cu > 0 ? (T <= num_cu ? T : T % num_cu) : 0;  // tiles of the last round, if not full or the only one
    int64_t cp_tail = 0;  // tiles that go this way
    int cp_z = 1;
    double cp_us = 0.0;
    if (!per_slice && cand >= 1 && cand * w <= CHUNK_PARALLEL_MAX_BLOCKS && cand * w <= capacity &&
        schedule != OZIMMU_SCHEDULE_ONE_LAUNCH && schedule != OZIMMU_SCHEDULE_SPLIT_INNER) {
        // (measured on MI355X: a stage 0.58 us; prologue + epilogue of an item 12 us, 19 us when the epilogue adds
        // with atomics; clearing the blocks 5 us + 0.065 us per block; the accumulation kernel 15 us + 0.058 us
        // per block)
        const double stage_us = 0.58;
        const double pairs = (double)k * (k + 1) / 2;
        const int longest = r_eff < k ? r_eff : k;  // pairs of the longest chunk
        const double blocks = (double)(cand * w);
        // one more round of the persistent launch: every tile at once, chunks in sequence, each with a fused
        // epilogue in which all workgroups update D at the same time (measured 2.0 ms at 4096^3, k = 8)
        const double one_launch_us = 0.60 * pairs * KT + 50.0 * (double)w;
        double best = 0.0;
        int best_z = 0;
        const int zmax = KT / 4 > 0 ? KT / 4 : 1;
        for (int z = 1; z <= zmax; z *= 2) {
            const double item_us = z > 1 ? 19.0 : 12.0;
            const double total = (double)cand * (stage_us * pairs * KT + item_us * (double)w * z);
            const double longest_item = stage_us * longest * KT / z + item_us;
            // items are handed out longest first to whichever workgroup is free: the last ones end unevenly
            double t = total / (double)num_cu + 0.25 * longest_item;
            if (t < longest_item) t = longest_item;
            t += 15.0 + 0.058 * blocks;               // the accumulation kernel
            if (z > 1) t += 5.0 + 0.065 * blocks;     // clearing the blocks for the atomic adds
            if (best_z == 0 || t < best) {
                best = t;
                best_z = z;
            }
        }
        if (schedule == OZIMMU_SCHEDULE_CHUNK_PARALLEL || best < 0.97 * one_launch_us) {
            cp_tail = cand;
            cp_z = best_z;
            cp_us = best;
        }
    }
    // (where the model prefers the persistent launch to the chunk-parallel way, the queue beats that one)
    const bool queue_pays = schedule == 0 && T >= QUEUE_MIN_TILES && sets_all > 0 && !(one_round_fits && cp_tail > 0);

    // tiles [0, T - tail) go to the persistent launch, the last `tail` tiles (band order) are cut Z ways
    int64_t tail = 0;
    int Z = 1;
    double tail_us = 0.0;
    if (!per_slice && cp_tail == 0 && !queue_pays && schedule != OZIMMU_SCHEDULE_ONE_LAUNCH &&
        schedule != OZIMMU_SCHEDULE_CHUNK_PARALLEL) {
        const int64_t ncu = num_cu;
        const int64_t zmax = KT / 4;  // every part gets at least one group of 4 stages of the shortest chunk
        if (cand >= 1 && cand <= SPLIT_INNER_MAX_TILES && zmax >= 2) {
            // Time per chunk in microseconds, from measurements on MI355X: a stage of the main loop takes
            // 0.58 us; the fused path pays about 35 us per chunk and tile for epilogue and prologue, a part of
            // the cut path about 15 us (atomic epilogue, prologue), and every chunk of the cut path about 15 us
            // of launches plus the accumulation pass over the tail tiles (20 bytes per element at 4.5 TB/s).
            const double chunk_us = 0.58 * (double)k * (k + 1) / 2 * KT / (double)w;  // average chunk of one tile
            const double fused_us = chunk_us + 35.0;  // one more round of the persistent launch
            const double fixed_us = 15.0 + 0.29 * (double)cand;
            double best = 0.0;
            int64_t best_z = 0;
            // one round only: cutting finer and running the parts in several rounds measured slower than the
            // fused path even where this model favours it (3072 x 16384 x 3072: 8.0 against 6.0 ms)
            for (int64_t z = 2; z <= zmax && cand * z <= ncu; ++z) {
                const double t = chunk_us / (double)z + 15.0 + fixed_us;
                if (best_z == 0 || t < best) {
                    best = t;
                    best_z = z;
                }
            }
            if (best_z && (schedule == OZIMMU_SCHEDULE_SPLIT_INNER || best < 0.9 * fused_us)) {
                tail = cand;
                Z = (int)best_z;
                tail_us = best * (double)w;
            }
        }
    }

    // Resident: all chunks of a tile resident in registers (ozimmu_resident.h).  It reads every slice once per tile
    // where the other ways read it once per slice pair, and it writes nothing but D, so it is the fastest wherever
    // its tiles (of 32 x 32 to 128 x 128 outputs) fill the chip and their chunk sums fit the registers without
    // making the tiles so small that the operands' way through LDS becomes the bound.
    if (schedule == 0) {
        const double pairs = (double)k * (k + 1) / 2, rounds = (double)((T - tail - cp_tail + num_cu - 1) / num_cu);
        // what the ways above take: the queue 0.64 us per stage of 64 inner positions and 17 us per work item of a tile
        // (measured 96.5 ms at 16384^3, k = 8; 36.7 ms at 4096 x 65536 x 4096, k = 10; 7.4 ms at 8192^3, k = 6).  Both
        // sides at some shapes, whole calls, queue or chunk-parallel against the chosen resident variant: 4096^3 k = 3
        // 0.46 / 0.36 ms, k = 8 1.78 / 1.48, k = 16 5.91 / 4.87; 1024 x 16384 x 1024 k = 8 0.61 / 0.54;
        // 2048 x 65536 x 2048 k = 6 (12 chunks) 5.08 / 4.96; 4096 x 65536 x 4096 k = 10 (30 chunks) 39.7 / 40.3.
        // Beyond 16384 inner positions the chunk-parallel way takes longer than its estimate (by 1.04 at 20000, 1.15 at 40000, 1.2
        // to 1.35 at 80000, less with few chunks).  The split-inner way takes 2.0 to 2.3 times its own from 140000 on, where it wins
        // (23 x 309890 x 14, k = 3, 561 us, k_resident 1588; 7 x 196852 x 184, k = 10, 2970 and 2896), and more before (474 x
        // 37065 x 351, k = 3, 308 and 179).
        double other_us = queue_pays ? (0.64 * pairs * KT + 17.0 * (double)w) * (double)T / num_cu
                                     : cp_us + 1.9 * tail_us + rounds * (0.60 * pairs * KT + 50.0 * (double)w);
        if (!queue_pays && n > 16384) {
            const double slower = 0.02 + 0.004 * (double)w;
            other_us *= 1.0 + (slower < 0.08 ? slower : 0.08) * log2((double)n / 16384.0);
        }
        int variant = -1, parts = 1;
        for (int v = 0; ozr::is_variant(v); v = ozr::next_variant(v)) {
            if (per_slice && !ozr::per_slice_tile(k, v)) continue;
            const double us = ozr::estimate_us(k, r_eff, v, m, n, p, num_cu);
            if (us < 0.0) continue;
            if (v == ozr::HELD && variant >= 0 && parts == 1 &&
                us + ozr::held_lead_us(k, r_eff, variant, us, m, n, p, num_cu) >= other_us)
                continue;
            if (us < other_us) {
                other_us = us;
                variant = v;
                parts = 1;
            }
            // Tiles that leave half of the chip idle or more, cut along the inner dimension (below 16 us there is nothing to gain,
            // and the estimates themselves take time)
            if (us < 16.0) continue;
            const ozr::Config c = ozr::config_for(k, r_eff, v);
            const int64_t tiles = ((m + 32 * c.ta - 1) / (32 * c.ta)) * ((p + 32 * c.tb - 1) / (32 * c.tb));
            const int64_t room = capacity * BLOCK_BYTES, steps = (n + ozl::TILE_K - 1) / ozl::TILE_K;
            for (int z = 2; !per_slice && ozr::may_cut(v, c) && z <= 64 && tiles * z <= (int64_t)num_cu * c.waves && 2 * z <= steps &&
                            ozr::sums_bytes(k, r_eff, c, tiles * z) <= room;
                 z += z < 4 ? 1 : z / 2) {
                const double cut_us = ozr::estimate_us(k, r_eff, v, m, n, p, num_cu, z);
                if (cut_us + 1.0 < other_us) {
                    other_us = cut_us;
                    variant = v;
                    parts = z;
                }
            }
        }
        if (variant >= 0) {
            way.kind = Way::RESIDENT;
            way.tile = variant;
            way.parts = parts;
            return way;
        }
    }
    if (queue_pays) return queue_way(sets_all);
    way.cp_tail = cp_tail;
    way.cp_z = cp_z;
    way.tail = tail;
    way.Z = Z;
    return way;
}

// Steps (iii) + (iv) (+ (v), see Finish) for the whole schedule of Algorithm 6 (groups g = 2..k+1 ascending, chunks
// of at most r consecutive s), into D.  Five ways to run it, with bit-identical results (which one: see
// choose_way):
//  * resident: one launch, all chunk sums of a tile side by side in registers, D written once -- the default where its
//    estimate is the lowest (nearly everywhere at 3 to 16 slices and at most 16 chunks); few tiles of a long inner dimension
//    cut along it, a second launch adding the parts up, where the workspace has room for their sums;
//  * the queue: one launch whose work items are the (chunk, tile) pairs, an INT32 block per item, the tile's chunks
//    added up by the workgroup that completes it -- the default for outputs of more tiles than compute units (and
//    from QUEUE_MIN_TILES tiles on where the chunk-parallel way has no room) when the workspace holds the blocks;
//  * one persistent launch with the accumulation fused into the GEMM epilogue (mode 1, or 2 for per-slice
//    scales): one workgroup per compute unit takes tile after tile, all chunks of a tile in turn -- needs no
//    blocks;
//  * chunk-parallel, for outputs of few tiles or the last, partly filled round after a persistent launch: one
//    launch whose work items are (chunk, inner part, tile), a block per chunk and tile, then one accumulation
//    kernel over those tiles;
//  * split-inner, for the same tiles when there is room for one block per tile only: per chunk, the chunk GEMM
//    with its inner range cut into Z parts on Z workgroups per tile, which add their partial sums to zeroed
//    per-tile INT32 blocks with integer atomics, then the accumulation kernel over those tiles, which also clears
//    the blocks again.
// schedule: 0 = choose, or one of the OZIMMU_SCHEDULE_* flags (honoured when possible).  resident_tile >= 0: the resident
// way with that tile, cut in `parts` (the caller has checked that there is one, and the room for its sums).
int run_schedule(int64_t m, int64_t n, int64_t p, const int8_t* SA, const int8_t* SB, const int32_t* eA,
                 const int32_t* eB, int k, int64_t r, bool per_slice, int schedule, double* D, int64_t ldd,
                 const Finish& fin, int32_t* partial, int64_t partial_capacity, void* scratch, int num_cu, hipStream_t st,
                 bool sync_clean = false, int resident_tile = -1, int parts = 1)
{
    // sync_clean: the caller has already zeroed the soft-barrier counters in `scratch` (the first GEMM launch
    // then need not; later ones of the same call find them used and do)
    auto take_clean = [&]() -> int {
        const int c = sync_clean ? 1 : 0;
        sync_clean = false;
        return c;
    };
    const int beta = beta_of(n);
    const int r_eff = (int)(r < k ? r : k);
    const int KT = (int)(ozl::inner_padded(n) / ozl::TILE_K);
    const int64_t T = output_tiles(m, p);
    const int64_t w = chunks_of(k, r_eff);

    auto launch_resident = [&](int variant, int z) -> int {
        const ozk::GemmArgs g = make_args(m, n, p, SA, k, SB, k, 2, k + 1, r_eff, 0, 0, scratch, num_cu);
        ozk::ResidentArgs a{};
        a.SA = g.SA;
        a.SB = g.SB;
        a.PA = g.PA;
        a.PB = g.PB;
        a.pstrideA = g.pstrideA;
        a.pstrideB = g.pstrideB;
        a.cA = g.cA;
        a.cB = g.cB;
        a.strideA = g.strideA;
        a.strideB = g.strideB;
        a.KT = KT;
        a.steps = (int)((n + ozl::TILE_K - 1) / ozl::TILE_K);
        a.m = m;
        a.p = p;
        a.D = D;
        a.ldd = ldd;
        a.eA = eA;
        a.eB = eB;
        a.beta = beta;
        a.finish = fin.on ? 1 : 0;
        a.alpha = fin.alpha;
        a.cbeta = fin.cbeta;
        a.Cout = fin.Cout;
        a.ldco = fin.ldco;
        a.per_slice = per_slice ? 1 : 0;
        a.parts = z;
        a.blocks = partial;
        double* const out = fin.on ? fin.Cout : D;
        a.keep = (reinterpret_cast<uintptr_t>(out) % 64 != 0 || (fin.on ? fin.ldco : ldd) % 8 != 0) &&
                 ozr::merge_rows(k, m, n, p, ozr::estimate_us(k, r_eff, variant, m, n, p, num_cu));
        const hipError_t e = ozk::launch_resident(a, k, r_eff, variant, st);
        if (e != hipSuccess || z == 1) return hip_status(e);
        const ozr::Config c = ozr::config_for(k, r_eff, variant);
        const ozk::AddPartsArgs add = {partial, k,      r_eff,     beta,     z, c.ta, c.tb,
                                       m,       p,      eA,        eB,       a.finish, fin.alpha, fin.cbeta,
                                       out,     fin.on ? fin.ldco : ldd};
        return hip_status(ozk::launch_add_parts(add, st));
    };
    if (resident_tile >= 0) return launch_resident(resident_tile, parts);

    const Way way = choose_way(m, n, p, k, r_eff, per_slice, schedule, partial ? partial_capacity : 0, num_cu);
    if (way.kind == Way::RESIDENT) return launch_resident(way.tile, way.parts);

    auto launch_queue = [&](int64_t tiles, int64_t sets) -> int {
        const int64_t stride = tiles < ozk::QUEUE_ROUND_TILES ? tiles : ozk::QUEUE_ROUND_TILES;
        const int64_t rounds = (tiles + ozk::QUEUE_ROUND_TILES - 1) / ozk::QUEUE_ROUND_TILES;
        int32_t* const ctr = partial + sets * w * stride * (BLOCK_BYTES / 4);
        // counters: one per tile, one per round, the flag; then, 8-byte aligned, the per-XCD ticket batches
        const int64_t xq_at = (tiles + rounds + 2) & ~(int64_t)1;
        hipError_t e = ozk::launch_fill_zero_i32(xq_at + QUEUE_XCD_WORDS, ctr, st);
        if (e != hipSuccess) return OZIMMU_ERR_HIP;
        ozk::GemmArgs a = make_args(m, n, p, SA, k, SB, k, 2, k + 1, r_eff, 0, 0, scratch, num_cu);
        a.tile_count = (int)tiles;
        a.C = partial;
        a.zsplit = 1;
        a.nchunks = (int)w;
        a.queue_sets = (int)sets;
        a.queue_stride = (int)stride;
        const int64_t TM = ozl::rows_padded(m) / ozl::TILE_R, TP = ozl::rows_padded(p) / ozl::TILE_R;
        a.queue_block_rounds = (tiles == T && TM % 16 == 0 && TP % 16 == 0) ? 1 : 0;
        a.done = reinterpret_cast<unsigned*>(ctr);
        // batches of 32 tickets per XCD when every compute unit of the 8-XCD chip this is written for has a workgroup
        a.xq = (tiles >= num_cu && num_cu == 256) ? reinterpret_cast<unsigned*>(ctr) + xq_at : nullptr;
        a.D = D;
        a.ldd = ldd;
        a.eA = eA;
        a.eB = eB;
        a.finish = fin.on ? 1 : 0;
        a.alpha = fin.alpha;
        a.cbeta = fin.cbeta;
        a.Cout = fin.Cout;
        a.ldco = fin.ldco;
        a.spin_limit = 0;  // the items of a team are different chunks: nothing to line up
        a.grid_spin_limit = 0;
        a.sync_zeroed = take_clean();
        return hip_status(ozk::launch_gemm(a, 3, st));
    };
    if (way.kind == Way::QUEUE) return launch_queue(T, way.sets);
    const int64_t tail = way.tail, cp_tail = way.cp_tail;
    const int Z = way.Z, cp_z = way.cp_z;

    if (T - tail - cp_tail > 0) {
        ozk::GemmArgs a = make_args(m, n, p, SA, k, SB, k, 2, k + 1, r_eff, 0, 0, scratch, num_cu);
        a.tile_count = (int)(T - tail - cp_tail);
        a.D = D;
        a.ldd = ldd;
        a.eA = eA;
        a.eB = eB;
        a.estrideA = m;
        a.estrideB = p;
        a.first = 1;
        a.finish = fin.on ? 1 : 0;
        a.alpha = fin.alpha;
        a.cbeta = fin.cbeta;
        a.Cout = fin.Cout;
        a.ldco = fin.ldco;
        a.sync_zeroed = take_clean();
        const hipError_t e = ozk::launch_gemm(a, per_slice ? 2 : 1, st);
        if (e != hipSuccess) return OZIMMU_ERR_HIP;
    }
    if (cp_tail > 0) {
        hipError_t e = hipSuccess;
        if (cp_z > 1) e = ozk::launch_fill_zero_i32(cp_tail * w * 256 * 256, partial, st);
        if (e != hipSuccess) return OZIMMU_ERR_HIP;
        ozk::GemmArgs a = make_args(m, n, p, SA, k, SB, k, 2, k + 1, r_eff, 0, 0, scratch, num_cu);
        a.tile_begin = (int)(T - cp_tail);
        a.tile_count = (int)cp_tail;
        a.C = partial;
        a.zsplit = cp_z;
        a.nchunks = (int)w;
        a.spin_limit = 0;  // the items of a team are different chunks: nothing to line up
        a.grid_spin_limit = 0;
        a.sync_zeroed = take_clean();
        e = ozk::launch_gemm(a, 3, st);
        if (e != hipSuccess) return OZIMMU_ERR_HIP;
        ozk::TileAccArgs t{};
        t.tile_begin = (int)(T - cp_tail);
        t.tile_count = (int)cp_tail;
        t.m = m;
        t.p = p;
        t.Ct = partial;
        t.parts = cp_z;
        t.eA = eA;
        t.eB = eB;
        t.D = D;
        t.ldd = ldd;
        t.finish = fin.on ? 1 : 0;
        t.alpha = fin.alpha;
        t.cbeta = fin.cbeta;
        t.Cout = fin.Cout;
        t.ldco = fin.ldco;
        return hip_status(ozk::launch_accumulate_chunks(t, k, r_eff, beta, st));
    }
    if (tail == 0) return OZIMMU_OK;
    int first = 1;
    int epoch = 0;
    hipError_t e = ozk::launch_fill_zero_i32(tail * 256 * 256, partial, st);  // later chunks find it cleared
    if (e != hipSuccess) return OZIMMU_ERR_HIP;
    for (int g = 2; g <= k + 1; ++g)
        for (int s0 = 1; s0 <= g - 1; s0 += r_eff) {
            const int s1 = s0 + r_eff - 1 < g - 1 ? s0 + r_eff - 1 : g - 1;
            ozk::GemmArgs a = make_args(m, n, p, SA, k, SB, k, g, g, s1 - s0 + 1, s0, s1, scratch, num_cu);
            a.tile_begin = (int)(T - tail);
            a.tile_count = (int)tail;
            a.C = partial;
            a.zsplit = Z;
            a.sync_epoch = epoch++;
            a.sync_zeroed = take_clean();
            e = ozk::launch_gemm(a, 3, st);
            if (e != hipSuccess) return OZIMMU_ERR_HIP;
            ozk::TileAccArgs t{};
            t.tile_begin = (int)(T - tail);
            t.tile_count = (int)tail;
            t.m = m;
            t.p = p;
            t.Ct = partial;
            t.parts = Z;
            t.eA = eA;
            t.eB = eB;
            t.shift = 2 - beta * g;
            t.first = first;
            t.D = D;
            t.ldd = ldd;
            const bool last = (g == k + 1 && s1 == g - 1);
            t.finish = (fin.on && last) ? 1 : 0;
            t.alpha = fin.alpha;
            t.cbeta = fin.cbeta;
            t.Cout = fin.Cout;
            t.ldco = fin.ldco;
            e = ozk::launch_accumulate_tiles(t, st);
            if (e != hipSuccess) return OZIMMU_ERR_HIP;
            first = 0;
        }
    return OZIMMU_OK;
}

// The whole call in one launch (k_small) for small outputs of a short inner dimension.
inline bool overlap(const double* x, int64_t rows, int64_t cols, int64_t ldx, const double* y, int64_t ysize)
{
    const uintptr_t x0 = reinterpret_cast<uintptr_t>(x), y0 = reinterpret_cast<uintptr_t>(y);
    return x0 < y0 + 8 * (uintptr_t)ysize && y0 < x0 + 8 * (uintptr_t)((rows - 1) * ldx + cols);
}
// One round of its workgroups, two to a compute unit where LDS holds their slices (us a call in a graph, two launches and one, k = 8:
// 64^3 8.9 and 5.2, 128^3 9.6 and 5.7, 256^3 10.6 and 7.2, 320 x 256 x 320, 400 workgroups, 10.7 and 9.3, 352 x 256 x 352, 484, 10.7 and 9.6;
// k = 14: 256^3 14.2 and 9.4; at 70 sizes of up to 420 x 256 x 700 never slower in one.  Beyond, before either way was shortened by about a fifth: 400 x 256 x
// 400, 625, 12.4 and 16.1; 512 x 64 x 512, 1024, 10.1 and 10.7).
inline bool small_sizes(int64_t m, int64_t n, int64_t p, int k, int64_t r, int num_cu)
{
    if (n > ozk::SMALL_MAX_INNER || k < ozk::SMALL_MIN_K || k > ozk::SMALL_MAX_K || r < k) return false;
    const int64_t room = 2 * (2 * k * ((n + 63) / 64) * 1024 + 2048) <= 160 * 1024 ? 2 : 1;
    return ((m + 15) / 16) * ((p + 15) / 16) <= room * num_cu;
}
inline bool small_way(const ozk::SmallArgs& a, int k, int64_t r, int num_cu)
{
    const ozk::SmallArgs::Op &A = a.op[0], &B = a.op[1];
    if (!small_sizes(A.rows, a.n, B.rows, k, r, num_cu)) return false;
    // the operands are read while the output is written
    const int64_t size = (A.rows - 1) * a.ldo + B.rows;
    return !overlap(A.X, A.by_col ? a.n : A.rows, A.by_col ? A.rows : a.n, A.ld, a.out, size) &&
           !overlap(B.X, B.by_col ? a.n : B.rows, B.by_col ? B.rows : a.n, B.ld, a.out, size);
}

}  // namespace

extern "C" {

const char* ozimmu_status_string(int status)
{
    switch (status) {
        case OZIMMU_OK: return "ok";
        case OZIMMU_ERR_NULL: return "null pointer argument";
        case OZIMMU_ERR_DIM: return "invalid dimension or leading dimension";
        case OZIMMU_ERR_SLICES: return "invalid slice count or slice range";
        case OZIMMU_ERR_WORKSPACE: return "workspace too small or misaligned";
        case OZIMMU_ERR_HIP: return "HIP launch error";
        default: return "unknown status";
    }
}

int ozimmu_params(int64_t n, int* beta, int64_t* r)
{
    if (n < 1 || n > MAX_INNER) return OZIMMU_ERR_DIM;
    const int b = beta_of(n);
    if (beta) *beta = b;
    if (r) *r = r_of(n, b);
    return OZIMMU_OK;
}

int64_t ozimmu_num_chunks(int64_t n, int k)
{
    if (n < 1 || n > MAX_INNER || k < 1) return 0;
    const int64_t r = r_of(n, beta_of(n));
    int64_t w = 0;
    for (int g = 2; g <= k + 1; ++g) w += ((g - 1) + r - 1) / r;
    return w;
}

size_t ozimmu_slices_bytes(int64_t rows, int64_t n, int k)
{
    if (rows < 0 || n < 0 || k < 0) return 0;
    return (size_t)ozl::stack_bytes(rows, n, k);
}

size_t ozimmu_workspace_bytes(int64_t m, int64_t n, int64_t p, int k)
{
    if (m < 0 || n < 0 || p < 0 || k < 0) return 0;
    return (size_t)(align256(OZIMMU_SCRATCH_BYTES) + align256(4 * m) + align256(4 * p)) +
           ozimmu_slices_bytes(m, n, k) + ozimmu_slices_bytes(p, n, k) + (size_t)(partial_blocks(m, n, p, k) * BLOCK_BYTES);
}

size_t ozimmu_workspace_bytes_min(int64_t m, int64_t n, int64_t p, int k)
{
    if (m < 0 || n < 0 || p < 0 || k < 0) return 0;
    return min_workspace_bytes(m, n, p, k);
}

int ozimmu_split_A(int64_t m, int64_t n, const double* A, int64_t lda, int k, int8_t* SA, int32_t* eA, void* stream)
{
    if (m < 0 || n < 0 || m > MAX_OUTER || n > MAX_INNER || lda < n || lda > MAX_LD) return OZIMMU_ERR_DIM;
    if (k < 1 || k > OZIMMU_MAX_SLICES) return OZIMMU_ERR_SLICES;
    if (m == 0 || n == 0) return OZIMMU_OK;
    if (!A || !SA || !eA) return OZIMMU_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(SA) % 256) return OZIMMU_ERR_WORKSPACE;
    const ozk::SplitIn op = {A, lda, m, n, 0, rn_offset(beta_of(n)), SA, eA};
    return hip_status(ozk::launch_split(&op, 1, k, beta_of(n), 0, (hipStream_t)stream));
}

int ozimmu_split_B(int64_t n, int64_t p, const double* B, int64_t ldb, int k, int8_t* SB, int32_t* eB, void* stream)
{
    if (p < 0 || n < 0 || p > MAX_OUTER || n > MAX_INNER || ldb < p || ldb > MAX_LD) return OZIMMU_ERR_DIM;
    if (k < 1 || k > OZIMMU_MAX_SLICES) return OZIMMU_ERR_SLICES;
    if (p == 0 || n == 0) return OZIMMU_OK;
    if (!B || !SB || !eB) return OZIMMU_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(SB) % 256) return OZIMMU_ERR_WORKSPACE;
    const ozk::SplitIn op = {B, ldb, p, n, 1, rn_offset(beta_of(n)), SB, eB};
    return hip_status(ozk::launch_split(&op, 1, k, beta_of(n), 0, (hipStream_t)stream));
}

int ozimmu_gemm_group(int64_t m, int64_t n, int64_t p, const int8_t* SA, int kA, const int8_t* SB, int kB, int g,
                      int s0, int s1, int32_t* C, int64_t ldc, void* scratch, void* stream)
{
    int st = check_gemm_args(m, n, p, SA, kA, SB, kB, g, s0, s1);
    if (st != OZIMMU_OK) return st;
    if (ldc < p || ldc > MAX_LD) return OZIMMU_ERR_DIM;
    if (m == 0 || p == 0) return OZIMMU_OK;
    if (!C) return OZIMMU_ERR_NULL;
    if (n == 0) return hip_status(ozk::launch_fill_zero_i32_2d(m, p, C, ldc, (hipStream_t)stream));  // empty sum
    if (!scratch) return OZIMMU_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(scratch) % 4) return OZIMMU_ERR_WORKSPACE;
    DeviceState ds;
    st = device_state(&ds);
    if (st != OZIMMU_OK) return st;
    const int num_cu = ds.num_cu;
    ozk::GemmArgs a = make_args(m, n, p, SA, kA, SB, kB, g, g, s1 - s0 + 1, s0, s1, scratch, num_cu);
    a.C = C;
    a.ldc = ldc;
    return hip_status(ozk::launch_gemm(a, 0, (hipStream_t)stream));
}

int ozimmu_accumulate(int64_t m, int64_t p, const int32_t* C, int64_t ldc, const int32_t* eA, const int32_t* eB,
                      int beta, int g, int first, double* D, int64_t ldd, void* stream)
{
    if (m < 0 || p < 0 || m > MAX_OUTER || p > MAX_OUTER || ldc < p || ldd < p || ldc > MAX_LD || ldd > MAX_LD)
        return OZIMMU_ERR_DIM;
    if (beta < 1 || beta > 7 || g < 2 || g > 2 * OZIMMU_MAX_SLICES) return OZIMMU_ERR_SLICES;
    if (m == 0 || p == 0) return OZIMMU_OK;
    if (!C || !eA || !eB || !D) return OZIMMU_ERR_NULL;
    return hip_status(
        ozk::launch_accumulate(m, p, C, ldc, eA, eB, 2 - beta * g, first, D, ldd, (hipStream_t)stream));
}

int ozimmu_gemm_group_accumulate(int64_t m, int64_t n, int64_t p, const int8_t* SA, int kA, const int8_t* SB, int kB,
                                 int g, int s0, int s1, const int32_t* eA, const int32_t* eB, int first, double* D,
                                 int64_t ldd, void* scratch, void* stream)
{
    int st = check_gemm_args(m, n, p, SA, kA, SB, kB, g, s0, s1);
    if (st != OZIMMU_OK) return st;
    if (ldd < p || ldd > MAX_LD) return OZIMMU_ERR_DIM;
    if (m == 0 || p == 0) return OZIMMU_OK;
    if (!D) return OZIMMU_ERR_NULL;
    if (n == 0)  // empty sum: D <- D + 0, or D <- +0 when D is taken to be zero
        return first ? hip_status(ozk::launch_fill_zero_f64(m, p, D, ldd, (hipStream_t)stream)) : OZIMMU_OK;
    if (!eA || !eB || !scratch) return OZIMMU_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(scratch) % 4) return OZIMMU_ERR_WORKSPACE;
    DeviceState ds;
    st = device_state(&ds);
    if (st != OZIMMU_OK) return st;
    const int num_cu = ds.num_cu;
    ozk::GemmArgs a = make_args(m, n, p, SA, kA, SB, kB, g, g, s1 - s0 + 1, s0, s1, scratch, num_cu);
    a.D = D;
    a.ldd = ldd;
    a.eA = eA;
    a.eB = eB;
    a.first = first;
    return hip_status(ozk::launch_gemm(a, 1, (hipStream_t)stream));
}

int ozimmu_export_slices(int64_t rows, int64_t n, int k, const int8_t* packed, int8_t* out, void* stream)
{
    if (rows < 0 || n < 0 || rows > MAX_OUTER || n > MAX_INNER) return OZIMMU_ERR_DIM;
    if (k < 1 || k > OZIMMU_MAX_SLICES) return OZIMMU_ERR_SLICES;
    if (rows == 0 || n == 0) return OZIMMU_OK;
    if (!packed || !out) return OZIMMU_ERR_NULL;
    return hip_status(ozk::launch_export(rows, n, k, packed, out, (hipStream_t)stream));
}

size_t ozimmu_workspace_bytes_ex(int64_t m, int64_t n, int64_t p, int k)
{
    if (m < 0 || n < 0 || p < 0 || k < 0) return 0;
    return ozimmu_workspace_bytes(m, n, p, k) + (size_t)align256(8 * m * p);
}

int ozimmu_gemm_ex(int transA, int transB, int64_t m, int64_t n, int64_t p, double alpha, const double* A,
                   int64_t lda, const double* B, int64_t ldb, double beta, double* C, int64_t ldc, int k,
                   void* workspace, size_t workspace_bytes, void* stream)
{
    if (m < 0 || n < 0 || p < 0 || m > MAX_OUTER || p > MAX_OUTER || n > MAX_INNER) return OZIMMU_ERR_DIM;
    if (lda < (transA ? m : n) || ldb < (transB ? n : p) || ldc < p) return OZIMMU_ERR_DIM;
    if (lda > MAX_LD || ldb > MAX_LD || ldc > MAX_LD) return OZIMMU_ERR_DIM;
    if (k < 1 || k > OZIMMU_MAX_SLICES) return OZIMMU_ERR_SLICES;
    if (m == 0 || p == 0) return OZIMMU_OK;
    if (!C) return OZIMMU_ERR_NULL;
    hipStream_t st = (hipStream_t)stream;
    if (n == 0) {  // empty product: C <- beta C
        if (beta == 0.0) return hip_status(ozk::launch_fill_zero_f64(m, p, C, ldc, st));
        return hip_status(ozk::launch_axpby(m, p, 0.0, nullptr, 0, beta, C, ldc, st));
    }
    if (!A || !B || !workspace) return OZIMMU_ERR_NULL;
    // beta == 0: the sum is formed in C itself, no m x p buffer
    const size_t need = min_workspace_bytes(m, n, p, k) + (beta == 0.0 ? (size_t)0 : (size_t)align256(8 * m * p));
    if (reinterpret_cast<uintptr_t>(workspace) % 256 || workspace_bytes < need) return OZIMMU_ERR_WORKSPACE;

    DeviceState ds;
    const int drc = device_state(&ds);
    if (drc != OZIMMU_OK) return drc;
    const int bt = beta_of(n);
    const int64_t r = r_of(n, bt);
    if (n <= ozk::SMALL_MAX_INNER) {
        const ozk::SmallArgs a = {{{A, lda, m, transA ? 1 : 0}, {B, ldb, p, transB ? 0 : 1}}, (int)n, (int)((n + 63) / 64), bt,
                                  !(alpha == 1.0 && beta == 0.0), alpha, beta, C, ldc};
        if (small_way(a, k, r, ds.num_cu)) return hip_status(ozk::launch_small(a, k, st));
    }
    char* ws = static_cast<char*>(workspace);
    void* scratch = ws;
    ws += align256(OZIMMU_SCRATCH_BYTES);
    int32_t* eA = reinterpret_cast<int32_t*>(ws);
    ws += align256(4 * m);
    int32_t* eB = reinterpret_cast<int32_t*>(ws);
    ws += align256(4 * p);
    int8_t* SA = reinterpret_cast<int8_t*>(ws);
    ws += ozimmu_slices_bytes(m, n, k);
    int8_t* SB = reinterpret_cast<int8_t*>(ws);
    ws += ozimmu_slices_bytes(p, n, k);
    double* Dw = reinterpret_cast<double*>(ws);  // beta != 0 only
    if (beta != 0.0) ws += align256(8 * m * p);
    int32_t* partial = reinterpret_cast<int32_t*>(ws);  // the rest: INT32 blocks, as many as there is room for
    const int64_t blocks = (int64_t)((static_cast<char*>(workspace) + workspace_bytes - ws) / BLOCK_BYTES);

    // op(A): one scale per row of op(A).  Stored transposed (n x m), those rows are the columns of the
    // stored matrix, which the column-wise split handles; likewise for op(B).
    const ozk::SplitIn ops[2] = {{A, lda, m, n, transA ? 1 : 0, rn_offset(bt), SA, eA},
                                 {B, ldb, p, n, transB ? 0 : 1, rn_offset(bt), SB, eB}};
    const hipError_t e = ozk::launch_split(ops, 2, k, bt, 0, st, static_cast<uint32_t*>(scratch), ozk::SYNC_WORDS,
                                           short_product(m, n, p, k) ? partial : nullptr, (size_t)(blocks * BLOCK_BYTES));
    if (e != hipSuccess) return OZIMMU_ERR_HIP;

    // Step (v) rides on the epilogue of every tile's last chunk.  beta == 0: the running sum lives in C and the
    // last chunk stores fl(alpha d) there.  Otherwise the running sum lives in the workspace buffer and the last
    // chunk reads the old C and writes the new one.
    const bool in_place = beta == 0.0;
    const Finish fin = {!(alpha == 1.0 && beta == 0.0), alpha, beta, C, ldc};
    return run_schedule(m, n, p, SA, SB, eA, eB, k, r, false, 0, in_place ? C : Dw, in_place ? ldc : p, fin, partial,
                        blocks, scratch, ds.num_cu, st, true);
}

int ozimmu_dgemm(int64_t m, int64_t n, int64_t p, const double* A, int64_t lda, const double* B, int64_t ldb,
                 double* D, int64_t ldd, int k, void* workspace, size_t workspace_bytes, void* stream)
{
    return ozimmu_dgemm_profiled(m, n, p, A, lda, B, ldb, D, ldd, k, workspace, workspace_bytes, stream, nullptr);
}

int ozimmu_dgemm_profiled(int64_t m, int64_t n, int64_t p, const double* A, int64_t lda, const double* B,
                          int64_t ldb, double* D, int64_t ldd, int k, void* workspace, size_t workspace_bytes,
                          void* stream, void* const* events)
{
    return dgemm_impl(m, n, p, A, lda, B, ldb, D, ldd, k, OZIMMU_SPLIT_NEAREST, OZIMMU_ACCUM_GROUPED, workspace,
                      workspace_bytes, stream, events);
}

size_t ozimmu_remainder_bytes(int64_t rows, int64_t n, int by_col)
{
    if (rows < 0 || n < 0) return 0;
    return (size_t)8 * (size_t)rows * (size_t)(by_col ? n : ozl::inner_padded(n));
}

size_t ozimmu_workspace_bytes_variant(int64_t m, int64_t n, int64_t p, int k, int split_mode)
{
    if (m < 0 || n < 0 || p < 0 || k < 0) return 0;
    if (split_mode == OZIMMU_SPLIT_NEAREST || split_mode == OZIMMU_SPLIT_BITMASK)
        return ozimmu_workspace_bytes(m, n, p, k);
    if (split_mode != OZIMMU_SPLIT_NEAREST_PER_SLICE) return 0;
    return (size_t)(align256(OZIMMU_SCRATCH_BYTES) + align256(4 * (int64_t)k * m) + align256(4 * (int64_t)k * p)) +
           ozimmu_slices_bytes(m, n, k) + ozimmu_slices_bytes(p, n, k) +
           (size_t)align256((int64_t)ozimmu_remainder_bytes(m, n, 0)) +
           (size_t)align256((int64_t)ozimmu_remainder_bytes(p, n, 1));
}

int ozimmu_split_A_per_slice(int64_t m, int64_t n, const double* A, int64_t lda, int k, int8_t* SA, int32_t* eA,
                             double* rem, void* stream)
{
    if (m < 0 || n < 0 || m > MAX_OUTER || n > MAX_INNER || lda < n || lda > MAX_LD) return OZIMMU_ERR_DIM;
    if (k < 1 || k > OZIMMU_MAX_SLICES) return OZIMMU_ERR_SLICES;
    if (m == 0 || n == 0) return OZIMMU_OK;
    if (!A || !SA || !eA || !rem) return OZIMMU_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(SA) % 256 || reinterpret_cast<uintptr_t>(rem) % 16) return OZIMMU_ERR_WORKSPACE;
    return hip_status(ozk::launch_split_A_per_slice(m, n, A, lda, k, beta_of(n), SA, eA, rem, (hipStream_t)stream));
}

int ozimmu_split_B_per_slice(int64_t n, int64_t p, const double* B, int64_t ldb, int k, int8_t* SB, int32_t* eB,
                             double* rem, void* stream)
{
    if (p < 0 || n < 0 || p > MAX_OUTER || n > MAX_INNER || ldb < p || ldb > MAX_LD) return OZIMMU_ERR_DIM;
    if (k < 1 || k > OZIMMU_MAX_SLICES) return OZIMMU_ERR_SLICES;
    if (p == 0 || n == 0) return OZIMMU_OK;
    if (!B || !SB || !eB || !rem) return OZIMMU_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(SB) % 256 || reinterpret_cast<uintptr_t>(rem) % 16) return OZIMMU_ERR_WORKSPACE;
    return hip_status(ozk::launch_split_B_per_slice(n, p, B, ldb, k, beta_of(n), SB, eB, rem, (hipStream_t)stream));
}

int ozimmu_dgemm_variant(int64_t m, int64_t n, int64_t p, const double* A, int64_t lda, const double* B, int64_t ldb,
                         double* D, int64_t ldd, int k, int split_mode, int accumulate_mode, void* workspace,
                         size_t workspace_bytes, void* stream)
{
    const int flags = accumulate_mode & ~0xff, amode = accumulate_mode & 0xff;
    if (split_mode < OZIMMU_SPLIT_NEAREST || split_mode > OZIMMU_SPLIT_NEAREST_PER_SLICE) return OZIMMU_ERR_SLICES;
    if (amode < OZIMMU_ACCUM_GROUPED || amode > OZIMMU_ACCUM_WIDE) return OZIMMU_ERR_SLICES;
    if (flags != 0 && flags != OZIMMU_SCHEDULE_ONE_LAUNCH && flags != OZIMMU_SCHEDULE_SPLIT_INNER &&
        flags != OZIMMU_SCHEDULE_CHUNK_PARALLEL && flags != OZIMMU_SCHEDULE_QUEUE)
        return OZIMMU_ERR_SLICES;
    if (amode == OZIMMU_ACCUM_WIDE && split_mode != OZIMMU_SPLIT_NEAREST) return OZIMMU_ERR_SLICES;
    if (split_mode == OZIMMU_SPLIT_NEAREST_PER_SLICE && amode != OZIMMU_ACCUM_PER_PAIR) return OZIMMU_ERR_SLICES;
    return dgemm_impl(m, n, p, A, lda, B, ldb, D, ldd, k, split_mode, accumulate_mode, workspace, workspace_bytes,
                      stream, nullptr);
}

int ozimmu_resident_tile(int64_t n, int k, int accumulate_mode, int tile, int* rows, int* cols)
{
    if (n < 1 || n > MAX_INNER) return OZIMMU_ERR_DIM;
    if (accumulate_mode < OZIMMU_ACCUM_GROUPED || accumulate_mode > OZIMMU_ACCUM_WIDE) return OZIMMU_ERR_SLICES;
    if (k < 1 || k > OZIMMU_MAX_SLICES || !ozr::is_variant(tile)) return OZIMMU_ERR_SLICES;
    const int64_t r = r_of_mode(n, accumulate_mode);
    const ozr::Config c = ozr::config_for(k, (int)(r < k ? r : k), tile);
    if (c.ta == 0) return OZIMMU_ERR_SLICES;
    if (rows) *rows = 32 * c.ta;
    if (cols) *cols = 32 * c.tb;
    return OZIMMU_OK;
}

int ozimmu_dgemm_resident(int64_t m, int64_t n, int64_t p, const double* A, int64_t lda, const double* B, int64_t ldb,
                          double* D, int64_t ldd, int k, int split_mode, int accumulate_mode, int tile, void* workspace,
                          size_t workspace_bytes, void* stream)
{
    if (split_mode != OZIMMU_SPLIT_NEAREST && split_mode != OZIMMU_SPLIT_BITMASK) return OZIMMU_ERR_SLICES;
    if (accumulate_mode == OZIMMU_ACCUM_WIDE && split_mode != OZIMMU_SPLIT_NEAREST) return OZIMMU_ERR_SLICES;
    int rows = 0, cols = 0;
    const int st = ozimmu_resident_tile(n, k, accumulate_mode, tile, &rows, &cols);
    if (st != OZIMMU_OK) return st;
    if (m < 0 || p < 0 || m > MAX_OUTER || p > MAX_OUTER || !ozr::in_range(m, n, p, rows, cols)) return OZIMMU_ERR_DIM;
    return dgemm_impl(m, n, p, A, lda, B, ldb, D, ldd, k, split_mode, accumulate_mode, workspace, workspace_bytes, stream,
                      nullptr, tile);
}

// blocks behind the slice stacks in a workspace of that many bytes
static int64_t block_capacity(int64_t m, int64_t n, int64_t p, int k, size_t workspace_bytes)
{
    const size_t before = (size_t)(align256(OZIMMU_SCRATCH_BYTES) + align256(4 * m) + align256(4 * p)) +
                          ozimmu_slices_bytes(m, n, k) + ozimmu_slices_bytes(p, n, k);
    return workspace_bytes < before ? 0 : (int64_t)((workspace_bytes - before) / BLOCK_BYTES);
}

int ozimmu_dgemm_tile(int64_t m, int64_t n, int64_t p, const double* A, int64_t lda, const double* B, int64_t ldb,
                      double* D, int64_t ldd, int k, int split_mode, int accumulate_mode, int tile, int parts,
                      void* workspace, size_t workspace_bytes, void* stream)
{
    const bool per_slice = split_mode == OZIMMU_SPLIT_NEAREST_PER_SLICE;
    if (!per_slice) {
        if (parts == 1)
            return ozimmu_dgemm_resident(m, n, p, A, lda, B, ldb, D, ldd, k, split_mode, accumulate_mode, tile, workspace,
                                         workspace_bytes, stream);
        if (split_mode != OZIMMU_SPLIT_NEAREST && split_mode != OZIMMU_SPLIT_BITMASK) return OZIMMU_ERR_SLICES;
        if (accumulate_mode == OZIMMU_ACCUM_WIDE && split_mode != OZIMMU_SPLIT_NEAREST) return OZIMMU_ERR_SLICES;
    } else if (accumulate_mode != OZIMMU_ACCUM_PER_PAIR || parts != 1) {
        return OZIMMU_ERR_SLICES;
    }
    int rows = 0, cols = 0;
    const int st = ozimmu_resident_tile(n, k, accumulate_mode, tile, &rows, &cols);
    if (st != OZIMMU_OK) return st;
    if (m < 0 || p < 0 || m > MAX_OUTER || p > MAX_OUTER || !ozr::in_range(m, n, p, rows, cols)) return OZIMMU_ERR_DIM;
    if (per_slice) {
        if (!ozr::per_slice_tile(k, tile)) return OZIMMU_ERR_SLICES;
    } else {
        const int r = (int)(r_of_mode(n, accumulate_mode) < k ? r_of_mode(n, accumulate_mode) : k);
        const ozr::Config c = ozr::config_for(k, r, tile);
        const int64_t tiles = ((m + rows - 1) / rows) * ((p + cols - 1) / cols);
        if (!ozr::may_cut(tile, c) || parts < 1 || parts > 64 || 2 * (int64_t)parts > (n + ozl::TILE_K - 1) / ozl::TILE_K)
            return OZIMMU_ERR_SLICES;
        if (tiles * parts > ((int64_t)1 << 18)) return OZIMMU_ERR_DIM;  // (grids of k_cut and k_add_parts)
        if (ozr::sums_bytes(k, r, c, tiles * parts) > block_capacity(m, n, p, k, workspace_bytes) * BLOCK_BYTES)
            return OZIMMU_ERR_WORKSPACE;
    }
    return dgemm_impl(m, n, p, A, lda, B, ldb, D, ldd, k, split_mode, accumulate_mode, workspace, workspace_bytes, stream,
                      nullptr, tile, parts);
}

int ozimmu_split_way(int transA, int transB, int64_t m, int64_t n, int64_t p, int k, size_t workspace_bytes)
{
    if (m < 1 || n < 1 || p < 1 || m > MAX_OUTER || p > MAX_OUTER || n > MAX_INNER) return OZIMMU_ERR_DIM;
    if (k < 1 || k > OZIMMU_MAX_SLICES) return OZIMMU_ERR_SLICES;
    const ozk::SplitIn ops[2] = {{nullptr, n, m, n, transA != 0, 0, nullptr, nullptr}, {nullptr, p, p, n, transB == 0, 0, nullptr, nullptr}};
    const int64_t capacity = block_capacity(m, n, p, k, workspace_bytes);
    switch (ozk::split_cut(ops, 2, k, (size_t)(capacity * BLOCK_BYTES), short_product(m, n, p, k))) {
        case 1: return OZIMMU_SPLIT_WAY_CUT;
        case 2: return OZIMMU_SPLIT_WAY_CUT_COLUMNS;
        default: return OZIMMU_SPLIT_WAY_WHOLE;
    }
}

int ozimmu_choose(int64_t m, int64_t n, int64_t p, int k, int split_mode, int accumulate_mode, size_t workspace_bytes, int num_cu,
                  ozimmu_choice* out)
{
    if (m < 1 || n < 1 || p < 1 || m > MAX_OUTER || p > MAX_OUTER || n > MAX_INNER) return OZIMMU_ERR_DIM;
    if (k < 1 || k > OZIMMU_MAX_SLICES || num_cu < 1) return OZIMMU_ERR_SLICES;
    if (split_mode < OZIMMU_SPLIT_NEAREST || split_mode > OZIMMU_SPLIT_NEAREST_PER_SLICE ||
        accumulate_mode < OZIMMU_ACCUM_GROUPED || accumulate_mode > OZIMMU_ACCUM_WIDE)
        return OZIMMU_ERR_SLICES;
    if (!out) return OZIMMU_ERR_NULL;
    const bool per_slice = split_mode == OZIMMU_SPLIT_NEAREST_PER_SLICE;
    const int64_t r = r_of_mode(n, accumulate_mode);
    *out = ozimmu_choice{OZIMMU_WAY_ONE_LAUNCH, -1, 1, OZIMMU_SPLIT_WAY_WHOLE, 0};
    if (split_mode == OZIMMU_SPLIT_NEAREST && small_sizes(m, n, p, k, r, num_cu)) {
        out->way = OZIMMU_WAY_SMALL;
        out->split_way = OZIMMU_SPLIT_WAY_NONE;
        return OZIMMU_OK;
    }
    const int64_t capacity = block_capacity(m, n, p, k, workspace_bytes);
    if (per_slice) {
        out->split_way = n <= ozk::PER_SLICE_MAX_INNER ? OZIMMU_SPLIT_WAY_WHOLE : OZIMMU_SPLIT_WAY_PASSES;
    } else {
        out->split_way = ozimmu_split_way(0, 0, m, n, p, k, workspace_bytes);
    }
    const Way way = choose_way(m, n, p, k, (int)(r < k ? r : k), per_slice, 0, capacity, num_cu);
    if (way.kind == Way::RESIDENT) {
        out->way = OZIMMU_WAY_RESIDENT;
        out->tile = way.tile;
        out->parts = way.parts;
        const double us = ozr::estimate_us(k, (int)(r < k ? r : k), way.tile, m, n, p, num_cu);
        out->merge_rows = way.parts == 1 && ozr::merge_rows(k, m, n, p, us) ? 1 : 0;
    } else if (way.kind == Way::QUEUE) {
        out->way = OZIMMU_WAY_QUEUE;
    } else if (way.cp_tail > 0) {
        out->way = OZIMMU_WAY_CHUNK_PARALLEL;
    } else if (way.tail > 0) {
        out->way = OZIMMU_WAY_SPLIT_INNER;
    }
    return OZIMMU_OK;
}

int ozimmu_split_A_variant(int64_t m, int64_t n, const double* A, int64_t lda, int k, int split_mode, int8_t* SA,
                           int32_t* eA, void* stream)
{
    if (m < 0 || n < 0 || m > MAX_OUTER || n > MAX_INNER || lda < n || lda > MAX_LD) return OZIMMU_ERR_DIM;
    if (k < 1 || k > OZIMMU_MAX_SLICES || (split_mode != 0 && split_mode != 1)) return OZIMMU_ERR_SLICES;
    if (m == 0 || n == 0) return OZIMMU_OK;
    if (!A || !SA || !eA) return OZIMMU_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(SA) % 256) return OZIMMU_ERR_WORKSPACE;
    const ozk::SplitIn op = {A, lda, m, n, 0, split_mode == 0 ? rn_offset(beta_of(n)) : 0, SA, eA};
    return hip_status(ozk::launch_split(&op, 1, k, beta_of(n), split_mode, (hipStream_t)stream));
}

int ozimmu_split_B_variant(int64_t n, int64_t p, const double* B, int64_t ldb, int k, int split_mode, int8_t* SB,
                           int32_t* eB, void* stream)
{
    if (p < 0 || n < 0 || p > MAX_OUTER || n > MAX_INNER || ldb < p || ldb > MAX_LD) return OZIMMU_ERR_DIM;
    if (k < 1 || k > OZIMMU_MAX_SLICES || (split_mode != 0 && split_mode != 1)) return OZIMMU_ERR_SLICES;
    if (p == 0 || n == 0) return OZIMMU_OK;
    if (!B || !SB || !eB) return OZIMMU_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(SB) % 256) return OZIMMU_ERR_WORKSPACE;
    const ozk::SplitIn op = {B, ldb, p, n, 1, split_mode == 0 ? rn_offset(beta_of(n)) : 0, SB, eB};
    return hip_status(ozk::launch_split(&op, 1, k, beta_of(n), split_mode, (hipStream_t)stream));
}

int ozimmu_init(void)
{
    DeviceState ds;
    return device_state(&ds);
}

int ozimmu_dgemm_static(int64_t m, int64_t n, int64_t p, const double* A, int64_t lda, const double* B, int64_t ldb,
                        double* D, int64_t ldd, int k, void* stream)
{
    if (m < 0 || n < 0 || p < 0 || m > MAX_OUTER || p > MAX_OUTER || n > MAX_INNER) return OZIMMU_ERR_DIM;
    if (k < 1 || k > OZIMMU_MAX_SLICES) return OZIMMU_ERR_SLICES;
    if (min_workspace_bytes(m, n, p, k) > (size_t)OZIMMU_STATIC_WORKSPACE_BYTES) return OZIMMU_ERR_WORKSPACE;
    if (m == 0 || p == 0) return OZIMMU_OK;
    DeviceState ds;
    const int rc = device_state(&ds);
    if (rc != OZIMMU_OK) return rc;
    return dgemm_impl(m, n, p, A, lda, B, ldb, D, ldd, k, OZIMMU_SPLIT_NEAREST, OZIMMU_ACCUM_GROUPED, ds.static_ws,
                      (size_t)OZIMMU_STATIC_WORKSPACE_BYTES, stream, nullptr);
}

int64_t ozimmu_r_wide(int64_t n)
{
    if (n < 1 || n > MAX_INNER) return 0;
    return r_wide_of(n, beta_of(n));
}

}  // extern "C"

namespace {

int dgemm_impl(int64_t m, int64_t n, int64_t p, const double* A, int64_t lda, const double* B, int64_t ldb,
               double* D, int64_t ldd, int k, int split_mode, int accumulate_mode, void* workspace,
               size_t workspace_bytes, void* stream, void* const* events, int resident_tile, int parts)
{
    if (m < 0 || n < 0 || p < 0 || m > MAX_OUTER || p > MAX_OUTER || n > MAX_INNER) return OZIMMU_ERR_DIM;
    if (lda < n || ldb < p || ldd < p || lda > MAX_LD || ldb > MAX_LD || ldd > MAX_LD) return OZIMMU_ERR_DIM;
    if (k < 1 || k > OZIMMU_MAX_SLICES) return OZIMMU_ERR_SLICES;
    if (m == 0 || p == 0) return OZIMMU_OK;
    if (!D) return OZIMMU_ERR_NULL;
    hipStream_t st = (hipStream_t)stream;
    if (n == 0) return hip_status(ozk::launch_fill_zero_f64(m, p, D, ldd, st));
    if (!A || !B || !workspace) return OZIMMU_ERR_NULL;
    if (reinterpret_cast<uintptr_t>(workspace) % 256 ||
        workspace_bytes < (split_mode == OZIMMU_SPLIT_NEAREST_PER_SLICE
                               ? ozimmu_workspace_bytes_variant(m, n, p, k, split_mode)
                               : min_workspace_bytes(m, n, p, k)))
        return OZIMMU_ERR_WORKSPACE;
    DeviceState ds;
    const int drc = device_state(&ds);
    if (drc != OZIMMU_OK) return drc;

    const int schedule =
        accumulate_mode & (OZIMMU_SCHEDULE_ONE_LAUNCH | OZIMMU_SCHEDULE_SPLIT_INNER | OZIMMU_SCHEDULE_CHUNK_PARALLEL |
                           OZIMMU_SCHEDULE_QUEUE);
    accumulate_mode &= 0xff;
    const int beta = beta_of(n);
    const bool per_slice = split_mode == OZIMMU_SPLIT_NEAREST_PER_SLICE;
    if (split_mode == OZIMMU_SPLIT_NEAREST && schedule == 0 && resident_tile < 0 && !events && n <= ozk::SMALL_MAX_INNER) {
        const ozk::SmallArgs a = {{{A, lda, m, 0}, {B, ldb, p, 1}}, (int)n, (int)((n + 63) / 64), beta, 0, 1.0, 0.0, D, ldd};
        if (small_way(a, k, r_of_mode(n, accumulate_mode), ds.num_cu)) return hip_status(ozk::launch_small(a, k, st));
    }
    const int64_t ne = per_slice ? k : 1;  // exponent arrays per operand
    const int64_t r = r_of_mode(n, accumulate_mode);
    char* ws = static_cast<char*>(workspace);
    void* scratch = ws;
    ws += align256(OZIMMU_SCRATCH_BYTES);
    int32_t* eA = reinterpret_cast<int32_t*>(ws);
    ws += align256(4 * ne * m);
    int32_t* eB = reinterpret_cast<int32_t*>(ws);
    ws += align256(4 * ne * p);
    int8_t* SA = reinterpret_cast<int8_t*>(ws);
    ws += ozimmu_slices_bytes(m, n, k);
    int8_t* SB = reinterpret_cast<int8_t*>(ws);
    ws += ozimmu_slices_bytes(p, n, k);
    double* remA = reinterpret_cast<double*>(ws);  // per-slice split only
    double* remB = reinterpret_cast<double*>(ws + align256((int64_t)ozimmu_remainder_bytes(m, n, 0)));

    auto mark = [&](int i) -> hipError_t {
        return (events && events[i]) ? hipEventRecord((hipEvent_t)events[i], st) : hipSuccess;
    };
    hipError_t e = mark(0);
    if (e != hipSuccess) return OZIMMU_ERR_HIP;
    const int offset = (split_mode == OZIMMU_SPLIT_NEAREST && accumulate_mode != OZIMMU_ACCUM_WIDE) ? rn_offset(beta) : 0;
    if (per_slice && n <= ozk::PER_SLICE_MAX_INNER) {
        const ozk::SplitIn ops[2] = {{A, lda, m, n, 0, 0, SA, eA}, {B, ldb, p, n, 1, 0, SB, eB}};
        e = ozk::launch_split_per_slice(ops, k, beta, st);
    } else if (per_slice) {
        e = ozk::launch_split_A_per_slice(m, n, A, lda, k, beta, SA, eA, remA, st);
        if (e != hipSuccess) return OZIMMU_ERR_HIP;
        e = ozk::launch_split_B_per_slice(n, p, B, ldb, k, beta, SB, eB, remB, st);
    } else {
        const ozk::SplitIn ops[2] = {{A, lda, m, n, 0, offset, SA, eA}, {B, ldb, p, n, 1, offset, SB, eB}};
        char* const room = reinterpret_cast<char*>(SB) + ozimmu_slices_bytes(p, n, k);
        e = ozk::launch_split(ops, 2, k, beta, split_mode, st, static_cast<uint32_t*>(scratch), ozk::SYNC_WORDS,
                              short_product(m, n, p, k) ? room : nullptr, static_cast<char*>(workspace) + workspace_bytes - room);
    }
    if (e != hipSuccess) return OZIMMU_ERR_HIP;
    e = mark(1);
    if (e != hipSuccess) return OZIMMU_ERR_HIP;

    int32_t* partial = nullptr;  // INT32 partial sums of few-tile outputs, behind the slices
    if (!per_slice) partial = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(SB) + ozimmu_slices_bytes(p, n, k));
    const Finish no_finish = {false, 1.0, 0.0, D, ldd};
    // blocks of 256 x 256 INT32 the rest of the workspace holds (decides whether the chunk-parallel way fits)
    int64_t capacity = 0;
    if (partial)
        capacity = (int64_t)((static_cast<char*>(workspace) + workspace_bytes - reinterpret_cast<char*>(partial)) /
                             BLOCK_BYTES);
    const int rc = run_schedule(m, n, p, SA, SB, eA, eB, k, r, per_slice, schedule, D, ldd, no_finish, partial,
                                capacity, scratch, ds.num_cu, st, !per_slice, resident_tile, parts);
    if (rc != OZIMMU_OK) return rc;
    return hip_status(mark(2));
}

}  // namespace
