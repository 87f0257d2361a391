// Steps (i) and (ii) of the scheme: power-of-two scale exponents and INT8
// slices, written in the packed tile-major layout of ozimmu_layout.h.
//
// What is computed (Algorithm 8 of the paper, with its scale mu'' = 2^e * 2^(1-beta)):
//   e      = ceil(log2 max |x|) over a row of A / a column of B (0 if all zero)
//   slice s (s = 1..k) of x = the integer nearest (ties to even) to
//            remainder / 2^(e + 1 - s beta), remainder reduced accordingly.
// How: the kernels scale once,
//   y = x * 2^(beta - 1 - e)  (exact, |y| <= 2^(beta-1)),
// and then round the remainder to one grid after the other, 1, 2^-beta, 2^(-2 beta), ... (see digits4).
// The kernels are HBM-bound: 8 bytes read (16 where a vector does not stay in
// registers or cache) and k bytes written per element.
// The bytes stored are q_s + c (c = offset of the stack, see ozimmu_layout.h;
// inner padding counts as a real zero; padding rows are not written at all: what they hold only reaches outputs that are
// never stored); with them go the prefix sums over the slices
// of the row sums of the stored bytes, which the GEMM needs to take the
// offsets out again.
#include "ozimmu_kernels.h"
#include "ozimmu_layout.h"

namespace {
using namespace ozl;

constexpr int OZIMMU_MAX_SLICES_DEV = 20;  // OZIMMU_MAX_SLICES of the C ABI

// ceil(log2 x) key of a positive finite double given as its bit pattern,
// monotone in x so that maxima can be taken on keys:
// key = 2 * (t + 1100) + (f != 0.5) with x = f * 2^t, f in [0.5, 1); 0 for x == 0.
__device__ inline uint32_t exp_key(uint64_t absbits)
{
    if (absbits == 0) return 0u;
    double x = __longlong_as_double((long long)absbits);
    int t;
    double f = frexp(x, &t);
    return (uint32_t)(2 * (t + 1100) + (f != 0.5 ? 1 : 0));
}
// MASK = false: ceil(log2 x) (round-to-nearest split); MASK = true: floor(log2 x) = t - 1 (bit-mask split)
template <bool MASK>
__device__ inline int key_to_exp(uint32_t key)
{
    if (key == 0u) return 0;
    int t = (int)(key >> 1) - 1100;
    if (MASK) return t - 1;
    return (key & 1u) ? t : t - 1;
}
// digit of one slice: nearest integer, ties to even (Algorithm 8) or truncation toward zero (Algorithm 3)
template <bool MASK>
__device__ inline double digit(double y)
{
    return MASK ? __builtin_trunc(y) : __builtin_rint(y);
}

__device__ inline uint64_t abs_bits(double x)
{
    return (uint64_t)__double_as_longlong(x) & 0x7fffffffffffffffull;
}

__device__ inline uint64_t wave_max_u64(uint64_t v)
{
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        uint64_t o = __shfl_xor(v, off, 64);
        v = o > v ? o : v;
    }
    return v;
}

// Sums and maxima over lanes without the way through LDS that a shuffle takes (four to six of those one after the other for every slice:
// 100000 x 100 x 64, k = 6, 114 -> 102 us a call, 300^3, k = 8, 12.6 -> 11.8, 777 x 1001 x 513, k = 7, 26.3 -> 25.5, 1024^3, k = 12, 59.7 -> 58.3).
// moved: inside 16 lanes; swapped: the halves of 32 or of 64.
template <int CTRL>
__device__ inline int moved(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ inline double moved(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)moved<CTRL>((int)(uint32_t)b), hi = (uint32_t)moved<CTRL>((int)(uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
struct Sum {
    __device__ int operator()(int a, int b) const { return a + b; }
};
struct Max {
    __device__ double operator()(double a, double b) const { return fmax(a, b); }
};
// v of a lane with the one 16 or 32 lanes away
template <int BY, class OP>
__device__ inline int swapped(int v, OP op)
{
    const auto r = BY == 16 ? __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false)
                            : __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    return op((int)r[0], (int)r[1]);
}
template <int BY, class OP>
__device__ inline double swapped(double v, OP op)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const unsigned l = (unsigned)b, h = (unsigned)(b >> 32);
    const auto lo = BY == 16 ? __builtin_amdgcn_permlane16_swap(l, l, false, false) : __builtin_amdgcn_permlane32_swap(l, l, false, false);
    const auto hi = BY == 16 ? __builtin_amdgcn_permlane16_swap(h, h, false, false) : __builtin_amdgcn_permlane32_swap(h, h, false, false);
    return op(__longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0])), __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1])));
}
// over groups of LANES (16, 32 or 64) neighbours
template <int LANES, class T, class OP>
__device__ inline T over_neighbours(T v, OP op)
{
    static_assert(LANES >= 16, "");
    v = op(v, moved<0xb1>(v));   // lane ^ 1
    v = op(v, moved<0x4e>(v));   // lane ^ 2
    v = op(v, moved<0x141>(v));  // mirrored in 8: the other four
    v = op(v, moved<0x140>(v));  // mirrored in 16: the other eight
    if (LANES >= 32) v = swapped<16>(v, op);
    if (LANES >= 64) v = swapped<32>(v, op);
    return v;
}
// over the lanes of the same number modulo FIRST (4, 8 or 16)
template <int FIRST, class T, class OP>
__device__ inline T over_strided(T v, OP op)
{
    static_assert(FIRST >= 4, "");
    if (FIRST <= 8) v = op(v, moved<0x128>(v));  // rotated by 8 in 16
    if (FIRST <= 4) v = op(v, moved<0x124>(v));  // by 4
    v = swapped<16>(v, op);
    return swapped<32>(v, op);
}

// One slice of 4 consecutive inner elements: digits of y[], remainders updated in place, the 4 stored
// bytes (digit + c, c = the stack's offset) packed into a dword.  Returns the dword; *sum receives the sum
// of the 4 stored bytes.  Inner padding (l >= n) enters as y = 0 like a real zero and is stored as c.
template <bool MASK>
__device__ inline uint32_t slice_word4(double* y, int c, double two_beta, int* sum)
{
    uint32_t w = 0;
    int sm = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const double q = digit<MASK>(y[j]);
        const int b = (int)q + c;
        w |= ((uint32_t)b & 0xffu) << (8 * j);
        sm += b;
        y[j] = (y[j] - q) * two_beta;
    }
    *sum = sm;
    return w;
}

// ---------------------------------------------------------------------------
// Rows of A and columns of B in one launch.
//
// Rows: a workgroup of 8 waves (4 for short ones alone) takes ROWS consecutive vectors (4, 2 or 1); a wave
// covers 256 / ROWS inner positions of them at a time, a lane 4 consecutive ones,
// so that a slice goes out in runs of 64 ROWS bytes.  Columns: a workgroup takes
// COLS of them (16, 8 or 4); a wave covers 1024 / COLS inner positions, a lane 16
// consecutive ones of one column, which is exactly one 16-byte chunk of the packed
// tile per slice: nothing has to be transposed, and 16 columns x 64 positions are
// written in one piece of 1 KiB.  (Reads: 8 COLS contiguous bytes per inner position.)
// Either way a thread keeps up to 16 elements (rows: DBR) in registers: what a
// workgroup cannot keep it walks in batches of that size, the last batch of the
// maximum's walk staying in the registers, the others being read again (from L2 or the
// memory-side cache when they are still there).
//
// Bound by HBM where there is enough of it, by latency below: what matters is loads in flight, so more and smaller
// workgroups with 16 elements a thread beat fewer with more of the row in registers up to inner dimensions of 8192.
// Measured against the five launches this took before (one pass over A, fill, column maxima, split of B, prefix sums),
// both operands, k = 8: 256^2 27.6 -> 8.8 us, 1024^2 (k = 9) 41 -> 16, 2048^2 55 -> 29, 4096^2 194 -> 132;
// rows alone 16384^2 962 -> 907 us (4.7 TB/s, what a plain copy reaches), 65536 x 4096 (k = 10) 1.86 -> 1.23 ms; columns
// alone, read twice, 4096^2 108 -> 59, 16384^2 1.52 -> 1.34 ms.
// ---------------------------------------------------------------------------
typedef __attribute__((address_space(1))) const double* global_f64;
typedef double f64x2_a8 __attribute__((ext_vector_type(2), aligned(8)));
typedef __attribute__((address_space(1))) const f64x2_a8* global_f64x2;

struct SplitOp {
    const double* X;      // rows: vector i at X + i ld; columns: vector j at X + j, its elements ld apart
    int64_t ld, rows, n;
    int8_t* S;
    int32_t* e;
    int32_t* P;
    int32_t* trailer;
    int64_t Rpad, slice_stride;
    int KT, c;
    int by_col;
    int per;              // vectors per workgroup: rows 1, 2 or 4, columns 4, 8 or 16
    int blocks;           // workgroups
};

// Digits of 4 consecutive elements for one slice, packed (digit of element j in byte j); the elements become the
// remainders.  Nearest, ties to even: adding sig = 1.5 * 2^52 grids rounds to the grid and leaves the digit in the low
// bits of the sum (the published sequence (a + sigma) - sigma; the digit needs no conversion, the remainder no scaling).
// Truncation: the remainder is scaled to the next grid (step = 2^beta; exact), which stays 1 (scaling the digit instead of
// the remainder costs an operation more: 12 rows of 768, k = 16, 10.0 instead of 8.6 us).
template <bool MASK>
__device__ inline uint32_t digits4(double* y, double sig, double step)
{
    uint32_t q[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (MASK) {
            const double d = __builtin_trunc(y[j]);
            q[j] = (uint32_t)__double_as_longlong(d + 6755399441055744.0);
            y[j] = (y[j] - d) * step;
        } else {
            const double t = y[j] + sig;
            q[j] = (uint32_t)__double_as_longlong(t);
            y[j] -= t - sig;
        }
    }
    // (remainders now, four elements at a time: left to the compiler, the sums of all that a thread holds wait in registers
    // until after the store, and half as many waves fit)
    asm volatile("" : "+v"(y[0]), "+v"(y[1]), "+v"(y[2]), "+v"(y[3]));
    return __builtin_amdgcn_perm(q[1], q[0], 0x0c0c0400u) | __builtin_amdgcn_perm(q[3], q[2], 0x04000c0cu);
}
// The same to the nearest where a digit has 7 bits (inner dimensions up to 2^17), without the remainders: with N_s the integer nearest to y
// in grids of slice s, digit s is N_s - 128 N_(s-1) (128 N_(s-1) is even, rounding to nearest even does not see it), and its byte that
// of N_s with the top bit turned where N_(s-1) is odd.  One addition an element and slice instead of three, for DIRECT slices: then N_s no
// longer fits the sum, the elements become their remainders (next_digits) and N starts from zero again.  (In k_small, which is bound by them: 256^3,
// k = 8, 7.2 -> 6.7 us a call, 200 x 250 x 300, k = 15, 10.7 -> 9.9.  The splits, which wait for memory and for the lanes' sums, gain nothing: 512^3,
// k = 8, 14.2 and 14.6.)
constexpr int DIRECT = 7;
__device__ inline uint32_t digits4_direct(const double* y, double& sig, uint32_t* before)
{
    asm volatile("" : "+v"(sig));  // (four elements at a time, as in digits4)
    uint32_t q[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) q[j] = (uint32_t)__double_as_longlong(y[j] + sig);
    const uint32_t w = __builtin_amdgcn_perm(q[1], q[0], 0x0c0c0400u) | __builtin_amdgcn_perm(q[3], q[2], 0x04000c0cu);
    const uint32_t v = w ^ ((*before & 0x01010101u) << 7);
    *before = w;
    asm volatile("" : "+v"(*before));
    return v;
}
// sig: of the last slice taken
__device__ inline void next_digits(double* y, double sig, uint32_t* before)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) y[j] -= (y[j] + sig) - sig;
    *before = 0;
}
// the stored bytes digit + c (no carry between bytes: digit + 128 + c stays below 256), and their sum added to *sum
__device__ inline uint32_t with_offset(uint32_t w, uint32_t c4, int* sum)
{
    w = ((w ^ 0x80808080u) + c4) ^ 0x80808080u;
    *sum = __builtin_amdgcn_sdot4((int)w, 0x01010101, *sum, false);
    return w;
}

// Slices are written through L2.  Left there they are written back when the kernel ends, before the product may start: 2 to 6 us in
// which nothing runs (start of the product after the last workgroup of the split, left in L2 and written through: 777 x 1001 x 513, k = 7,
// 6.3 and 1.1 us, a call 30.2 and 26.9; 512^3, k = 8, 3.6 and 1.8, 16.2 and 14.0; 1024^3, k = 9, 4.4 and 0.9, 45.2 and 42.7).  They stay in the
// memory-side cache, which non-temporal stores would not do (the product then takes 4 us longer at 777 x 1001 x 513).
// NEAR: left there, for the few vectors whose workgroups and the product's only tile run on one XCD (see launch_split).
template <bool NEAR = false>
__device__ __attribute__((always_inline)) inline void store_slices(int8_t* out, uint32_t v)
{
    if constexpr (NEAR)
        *reinterpret_cast<uint32_t*>(out) = v;
    else
        __hip_atomic_store(reinterpret_cast<uint32_t*>(out), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <bool NEAR = false>
__device__ __attribute__((always_inline)) inline void store_slices(int8_t* out, uint32_t x, uint32_t y, uint32_t z, uint32_t w)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = {x, y, z, w};
    if constexpr (NEAR) {
        *reinterpret_cast<u32x4*>(out) = v;
        return;
    }
    // (one store: as two of 8 bytes each memory line would be written twice.  Behind a store of more than 8 bytes a vector instruction may
    // write its registers again from the third wait state on; the compiler, which sees no store here, would not keep that distance)
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(out), "v"(v) : "memory");
}

template <bool MASK>
__device__ inline int exponent_of(double mx)
{
    return key_to_exp<MASK>(exp_key(abs_bits(mx)));
}

template <int DB, int ROWS, bool MASK, bool NEAR = false>
__device__ inline void split_rows(const SplitOp& o, int64_t block, int k, int beta, double (*red)[16], int (*lsum)[16])
{
    constexpr int LPR = 64 / ROWS;        // lanes of a row
    constexpr int TPW = 4 / ROWS;         // inner tiles of 64 a wave covers at a time
    constexpr int U = DB / 4;
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), nw = blockDim.x >> 6;
    const int64_t R = block * ROWS + lane / LPR;
    const int li = (lane % LPR) * 4;
    const bool ok = R < o.rows;
    const global_f64 row = (global_f64)o.X + (ok ? R : o.rows - 1) * o.ld;  // (lanes past the edge read along and store nothing)
    const int groups = o.KT / TPW, per_batch = nw * U, nb = (groups + per_batch - 1) / per_batch;
    double y[U][4];
    double mx = 0.0;
    auto load = [&](int b) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int gq = b * per_batch + u * nw + w;
            const int64_t l = (int64_t)gq * (64 * TPW) + li;
            if ((int64_t)(gq + 1) * (64 * TPW) <= o.n) {  // (uniform)
                // (16-byte loads want 4-byte alignment only: any row and leading dimension will do.  An odd one with 8-byte loads,
                // each with its own bounds: 6 rows of 2036013, k = 1, 1316 instead of 424 us, 22 of 1813697, k = 8, 2084 and 1213)
                const f64x2_a8 p = *(global_f64x2)(row + l), q = *(global_f64x2)(row + l + 2);
                y[u][0] = p.x, y[u][1] = p.y, y[u][2] = q.x, y[u][3] = q.y;
            } else if ((int64_t)gq * (64 * TPW) < o.n) {  // (uniform; what lies wholly in the padding is not loaded)
                const int left = (int)(o.n - (int64_t)gq * (64 * TPW));
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    y[u][j] = 0.0;
                    if (li + j < left) y[u][j] = row[l + j];
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) y[u][j] = 0.0;
            }
        }
    };
    for (int b = nb - 1; b >= 0; --b) {
        load(b);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) mx = fmax(mx, fabs(y[u][j]));
    }
    mx = over_neighbours<LPR>(mx, Max{});
    if (lane % LPR == 0) red[w][lane / LPR] = mx;
    for (int i = t; i < k * ROWS; i += blockDim.x) lsum[i / ROWS][i % ROWS] = 0;
    __syncthreads();
    for (int q = 0; q < nw; ++q) mx = fmax(mx, red[q][lane / LPR]);
    const int e = exponent_of<MASK>(mx);
    const int sc = beta - 1 - e;
    const uint32_t c4 = (uint32_t)o.c * 0x01010101u;
    const double inv_step = ldexp(1.0, -beta), step = (double)(1 << beta);
    if (w == 0 && lane % LPR == 0 && ok) o.e[R] = e;
    for (int b = 0; b < nb; ++b) {
        if (b > 0) load(b);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) y[u][j] = ldexp(y[u][j], sc);
        double sig = 6755399441055744.0;
        int8_t* out = o.S + packed_offset(R, (int64_t)(b * per_batch + w) * (64 * TPW) + li, o.KT);
        for (int s = 0; s < k; ++s) {
            int sum = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (b * per_batch + u * nw + w < groups) {
                    const uint32_t v = with_offset(digits4<MASK>(y[u], sig, step), c4, &sum);
                    if (ok) store_slices<NEAR>(out + (int64_t)u * nw * (TPW * TILE_BYTES), v);
                }
            }
            out += o.slice_stride;
            sig *= inv_step;
            sum = over_neighbours<LPR>(sum, Sum{});
            if (lane % LPR == 0) atomicAdd(&lsum[s][lane / LPR], sum);
        }
    }
    __syncthreads();
    if (t < ROWS && block * ROWS + t < o.rows) {
        int run = 0;
        for (int s = 0; s < k; ++s) {
            run += lsum[s][t];
            o.P[(int64_t)s * o.Rpad + block * ROWS + t] = run;
        }
    }
}

template <int DB, int COLS, bool MASK, bool NEAR>
__device__ inline void split_cols(const SplitOp& o, int64_t block, int k, int beta, double (*red)[16], int (*lsum)[16])
{
    constexpr int TPW = 16 / COLS;        // inner tiles of 64 a wave covers at a time
    constexpr int U = DB / 16;
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), nw = blockDim.x >> 6;
    const int cl = lane % COLS, lb = lane / COLS;
    const int64_t R = block * COLS + cl;  // column = packed row
    const bool ok = R < o.rows;
    const int64_t col = ok ? R : o.rows - 1;  // (lanes past the edge read along and store nothing)
    const int groups = o.KT / TPW, per_batch = nw * U, nb = (groups + per_batch - 1) / per_batch;
    double y[U][16];
    double mx = 0.0;
    auto load = [&](int b) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int gq = b * per_batch + u * nw + w;
            const int64_t l = (int64_t)gq * (64 * TPW) + lb * 16;
            if ((int64_t)(gq + 1) * (64 * TPW) <= o.n) {      // (uniform)
                // (one running pointer, opaque to the optimiser: sixteen addresses at once cost a third of the registers)
                global_f64 p = (global_f64)o.X + l * o.ld + col;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    y[u][i] = *p;
                    p += o.ld;
                    asm volatile("" : "+v"(p));
                }
            } else if ((int64_t)gq * (64 * TPW) < o.n) {      // (uniform; what lies wholly in the padding is not loaded)
                const int left = (int)(o.n - (int64_t)gq * (64 * TPW));
                global_f64 p = (global_f64)o.X + l * o.ld + col;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    y[u][i] = 0.0;
                    if (lb * 16 + i < left) y[u][i] = *p;
                    p += o.ld;
                    asm volatile("" : "+v"(p));
                }
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) y[u][i] = 0.0;
            }
        }
    };
    for (int b = nb - 1; b >= 0; --b) {
        load(b);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < 16; ++i) mx = fmax(mx, fabs(y[u][i]));
    }
    mx = over_strided<COLS>(mx, Max{});
    if (lane < COLS) red[w][lane] = mx;
    for (int i = t; i < k * COLS; i += blockDim.x) lsum[i / COLS][i % COLS] = 0;
    __syncthreads();
    for (int q = 0; q < nw; ++q) mx = fmax(mx, red[q][cl]);
    const int e = exponent_of<MASK>(mx);
    const int sc = beta - 1 - e;
    const uint32_t c4 = (uint32_t)o.c * 0x01010101u;
    const double inv_step = ldexp(1.0, -beta), step = (double)(1 << beta);
    if (w == 0 && lane < COLS && ok) o.e[R] = e;
    for (int b = 0; b < nb; ++b) {
        if (b > 0) load(b);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < 16; ++i) y[u][i] = ldexp(y[u][i], sc);
        double sig = 6755399441055744.0;
        int8_t* out = o.S + packed_offset(R, (int64_t)(b * per_batch + w) * (64 * TPW) + lb * 16, o.KT);
        for (int s = 0; s < k; ++s) {
            int sum = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (b * per_batch + u * nw + w < groups) {
                    uint4 v;
                    v.x = with_offset(digits4<MASK>(y[u], sig, step), c4, &sum);
                    v.y = with_offset(digits4<MASK>(y[u] + 4, sig, step), c4, &sum);
                    v.z = with_offset(digits4<MASK>(y[u] + 8, sig, step), c4, &sum);
                    v.w = with_offset(digits4<MASK>(y[u] + 12, sig, step), c4, &sum);
                    if (ok) store_slices<NEAR>(out + (int64_t)u * nw * (TPW * TILE_BYTES), v.x, v.y, v.z, v.w);
                }
            }
            out += o.slice_stride;
            sig *= inv_step;
            sum = over_strided<COLS>(sum, Sum{});
            if (lane < COLS) atomicAdd(&lsum[s][lane], sum);
        }
    }
    __syncthreads();
    if (t < COLS && block * COLS + t < o.rows) {
        int run = 0;
        for (int s = 0; s < k; ++s) {
            run += lsum[s][t];
            o.P[(int64_t)s * o.Rpad + block * COLS + t] = run;
        }
    }
}

// ---------------------------------------------------------------------------
// Few long vectors in two launches: the inner dimension cut among workgroups.
//
// k_split_both's workgroups own whole vectors, which leaves most of the chip idle here, each working through one latency after
// the other (48 columns and 47 rows of 11948, k = 8: 40 us).  k_cut_maxima takes the maxima of pieces (as 16-bit keys; no atomics,
// nothing to clear), k_cut_split reduces those of its vectors and splits its piece.  Stored without offset: there are no sums of bytes
// to collect.  (That costs clock in long products, and is used where the product is short: launch_split.)
// A piece: 8 waves of 64 positions of 16 columns, or 8 waves of 4 x 64 positions of 4 rows.
// ---------------------------------------------------------------------------
// Marks a column entry of eB that still holds the key of the column maximum rather than the exponent decoded
// from it (k_split_B and k_cut_columns decode on the fly and store the exponents): exponents are small, keys carry this bit.
constexpr uint32_t RAW_KEY_TAG = 0x40000000u;
constexpr int CUT_COLS = 16, CUT_ROWS = 4, CUT_WAVES = 8;
__host__ __device__ inline int cut_vectors(int by_col) { return by_col ? CUT_COLS : CUT_ROWS; }
__host__ __device__ inline int cut_inner(int by_col) { return by_col ? CUT_WAVES * 64 : CUT_WAVES * 256; }

struct CutOp {
    const double* X;
    int64_t ld, rows, n;
    int8_t* S;
    int32_t* e;
    int32_t* trailer;
    uint16_t* keys;       // [piece][vector]
    int64_t slice_stride;
    int KT, by_col, groups, pieces;
};

// 16 elements a thread: columns, column lane % 16, positions 16 (lane / 16) + 0 .. 15 of a tile of 64; rows, row lane / 16, positions
// 4 (lane % 16) + 0 .. 3 of four tiles.
__device__ inline void cut_load(const CutOp& o, int group, int piece, double (*y)[4])
{
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    if (o.by_col) {
        int64_t R = (int64_t)group * CUT_COLS + (lane & 15);
        R = R < o.rows ? R : o.rows - 1;
        const int64_t l = (int64_t)piece * (CUT_WAVES * 64) + w * 64 + (lane >> 4) * 16;
        global_f64 p = (global_f64)o.X + l * o.ld + R;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            y[i / 4][i % 4] = 0.0;
            if (l + i < o.n) y[i / 4][i % 4] = *p;
            p += o.ld;
        }
    } else {
        int64_t R = (int64_t)group * CUT_ROWS + (lane >> 4);
        R = R < o.rows ? R : o.rows - 1;
        const global_f64 row = (global_f64)o.X + R * o.ld;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t l = (int64_t)piece * (CUT_WAVES * 256) + (u * CUT_WAVES + w) * 64 + (lane & 15) * 4;
            if (l + 4 <= o.n) {
                const f64x2_a8 p = *(global_f64x2)(row + l), q = *(global_f64x2)(row + l + 2);
                y[u][0] = p.x, y[u][1] = p.y, y[u][2] = q.x, y[u][3] = q.y;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    y[u][j] = 0.0;
                    if (l + j < o.n) y[u][j] = row[l + j];
                }
            }
        }
    }
}
// the largest of the workgroup's values per vector, in every thread of that vector
template <class T>
__device__ inline T cut_max(T v, bool by_col, T (*red)[16])
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int off = 0; off < 4; ++off) {
        if (by_col && off >= 2) break;
        const T x = __shfl_xor(v, by_col ? 16 << off : 1 << off, 64);
        v = x > v ? x : v;
    }
    const int at = by_col ? lane & 15 : lane >> 4;
    if (by_col ? lane < 16 : (lane & 15) == 0) red[w][at] = v;
    __syncthreads();
    for (int q = 0; q < CUT_WAVES; ++q) v = red[q][at] > v ? red[q][at] : v;
    return v;
}

// TAGGED: merged into the exponents' place, which holds RAW_KEY_TAG
template <bool TAGGED>
__device__ inline void cut_maxima(const CutOp& o, int block, double (*red)[16])
{
    const int group = block % o.groups, piece = block / o.groups, lane = threadIdx.x & 63;
    double y[4][4], mx = 0.0;
    cut_load(o, group, piece, y);
#pragma unroll
    for (int i = 0; i < 16; ++i) mx = fmax(mx, fabs(y[i / 4][i % 4]));
    mx = cut_max(mx, o.by_col, red);
    const int64_t R = (int64_t)group * cut_vectors(o.by_col) + (o.by_col ? lane & 15 : lane >> 4);
    if (threadIdx.x < 64 && (o.by_col ? lane < 16 : (lane & 15) == 0) && R < o.rows) {
        const uint32_t key = exp_key(abs_bits(mx));
        if constexpr (TAGGED) {
            if (key) atomicMax(reinterpret_cast<uint32_t*>(o.e) + R, RAW_KEY_TAG | key);
        } else {
            o.keys[piece * o.rows + R] = (uint16_t)key;
        }
    }
}
__global__ __launch_bounds__(64 * CUT_WAVES) void k_cut_maxima(CutOp a, CutOp b)
{
    __shared__ double red[CUT_WAVES][16];
    const int first = a.groups * a.pieces, second = (int)blockIdx.x >= first;
    const CutOp o = second ? b : a;
    cut_maxima<false>(o, (int)blockIdx.x - (second ? first : 0), red);
}

template <bool MASK>
__global__ __launch_bounds__(64 * CUT_WAVES) void k_cut_split(CutOp a, CutOp b, int k, int beta, uint32_t* zero, int zero_count)
{
    __shared__ int red[CUT_WAVES][16];
    const int first = a.groups * a.pieces, second = (int)blockIdx.x >= first, block = (int)blockIdx.x - (second ? first : 0);
    const CutOp o = second ? b : a;
    const int group = block % o.groups, piece = block / o.groups;
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    if (block == 0 && t == 0) o.trailer[0] = 0;
    if (blockIdx.x == 0 && t < zero_count) zero[t] = 0u;
    double y[4][4];
    cut_load(o, group, piece, y);
    // (threads of a vector: 4 lanes or 16 of each wave)
    const int64_t R = (int64_t)group * cut_vectors(o.by_col) + (o.by_col ? lane & 15 : lane >> 4);
    const bool ok = R < o.rows;
    const int share = o.by_col ? w * 4 + (lane >> 4) : w * 16 + (lane & 15), shares = CUT_WAVES * (o.by_col ? 4 : 16);
    int key = 0;
    for (int z = share; z < o.pieces; z += shares) {
        const int x = o.keys[z * o.rows + (ok ? R : o.rows - 1)];
        key = x > key ? x : key;
    }
    key = cut_max(key, o.by_col, red);
    const int e = key_to_exp<MASK>((uint32_t)key), sc = beta - 1 - e;
    if (piece == 0 && share == 0 && ok) o.e[R] = e;
#pragma unroll
    for (int i = 0; i < 16; ++i) y[i / 4][i % 4] = ldexp(y[i / 4][i % 4], sc);
    const double inv_step = ldexp(1.0, -beta), step = (double)(1 << beta);
    double sig = 6755399441055744.0;
    const int64_t l0 = (int64_t)piece * cut_inner(o.by_col) + w * 64 + (o.by_col ? (lane >> 4) * 16 : (lane & 15) * 4);
    int8_t* out = o.S + packed_offset(R, l0, o.KT);
    for (int s = 0; s < k; ++s) {
        uint32_t v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = digits4<MASK>(y[u], sig, step);
        if (ok) {
            if (o.by_col) {
                if (l0 < (int64_t)o.KT * TILE_K) store_slices(out, v[0], v[1], v[2], v[3]);
            } else {
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (l0 + u * (CUT_WAVES * 64) < (int64_t)o.KT * TILE_K)
                        store_slices(out + (int64_t)u * CUT_WAVES * TILE_BYTES, v[u]);
            }
        }
        out += o.slice_stride;
        sig *= inv_step;
    }
}

constexpr int SPLIT_WAVES = 8;
// DBR: elements of a row a thread holds (columns: 16); COLS: the launch may have columns.  Vectors per workgroup are each
// operand's own: both sides of a product may be columns (A transposed), one of many vectors and one of few.
// (With 64 elements a thread one kernel for both numbers of rows would spill: ROWS is fixed there.)
template <int DBR, int ROWS, bool COLS, bool MASK, bool NEAR = false>
__global__ __launch_bounds__(64 * SPLIT_WAVES, DBR == 16 ? 6 : DBR == 32 ? 4 : 2) void k_split_both(SplitOp a, SplitOp b, int k, int beta, uint32_t* zero, int zero_count)
{
    __shared__ double red[SPLIT_WAVES][16];
    __shared__ int lsum[OZIMMU_MAX_SLICES_DEV][16];  // sums of the stored bytes per slice and vector
    const bool second = (int)blockIdx.x >= a.blocks;
    // (field by field: a reference to one of the two would have the fields loaded into vector registers)
    SplitOp o;
    o.X = second ? b.X : a.X, o.ld = second ? b.ld : a.ld, o.rows = second ? b.rows : a.rows, o.n = second ? b.n : a.n;
    o.S = second ? b.S : a.S, o.e = second ? b.e : a.e, o.P = second ? b.P : a.P, o.trailer = second ? b.trailer : a.trailer;
    o.Rpad = second ? b.Rpad : a.Rpad, o.slice_stride = second ? b.slice_stride : a.slice_stride;
    o.KT = second ? b.KT : a.KT, o.c = second ? b.c : a.c, o.by_col = second ? b.by_col : a.by_col;
    o.per = second ? b.per : a.per;
    int block = second ? (int)blockIdx.x - a.blocks : (int)blockIdx.x;
    if (block == 0 && threadIdx.x == 0) o.trailer[0] = o.c;
    if (blockIdx.x == 0 && (int)threadIdx.x < zero_count) zero[threadIdx.x] = 0u;
    // (the grid holds whole sets of 32 workgroups per operand: four neighbours share memory lines and run on one XCD)
    block = (block >> 5) * 32 + (block & 7) * 4 + ((block >> 3) & 3);
    if ((int64_t)block * o.per >= o.rows) return;
    if (COLS && o.by_col) {
        if (o.per == 16)
            split_cols<16, 16, MASK, NEAR>(o, block, k, beta, red, lsum);
        else if (o.per == 8)
            split_cols<16, 8, MASK, NEAR>(o, block, k, beta, red, lsum);
        else
            split_cols<16, 4, MASK, NEAR>(o, block, k, beta, red, lsum);
    } else {
        if constexpr (ROWS > 0) {
            split_rows<DBR, ROWS, MASK, NEAR>(o, block, k, beta, red, lsum);
        } else {
            if (DBR == 16 && o.per == 4)
                split_rows<DBR, 4, MASK, NEAR>(o, block, k, beta, red, lsum);
            else if (o.per == 2)
                split_rows<DBR, 2, MASK, NEAR>(o, block, k, beta, red, lsum);
            else
                split_rows<DBR, 1, MASK, NEAR>(o, block, k, beta, red, lsum);
        }
    }
}

// ---------------------------------------------------------------------------
// Columns of a long inner dimension cut along it, with their offsets.
//
// A workgroup that owns 4 to 16 whole columns walks them twice, and what it takes is not memory alone: the digits of 8 columns of 16384 are
// 55 us of vector instructions of a compute unit.  Where whole columns leave compute units idle at the end, they are cut into
// pieces: behind a fill of maxima and sums, k_split_and_maxima splits the operand taken by rows, if there is one, and takes the maxima of
// the pieces of columns on the side; k_cut_columns splits the pieces.  (1024 x 16384 x 1024, k = 8: split
// 174 -> 138 us, 671 MB in all.)
// ---------------------------------------------------------------------------
struct ColumnsOp : CutOp {
    int32_t* P;           // prefix sums
    int64_t Rpad;
    int c;                // offset
};
template <int DBR, int ROWS, bool MASK>
__global__ __launch_bounds__(64 * SPLIT_WAVES, DBR == 16 ? 6 : 2) void k_split_and_maxima(SplitOp a, ColumnsOp b, ColumnsOp c, int k, int beta,
                                                                                         uint32_t* zero, int zero_count)
{
    __shared__ double red[SPLIT_WAVES][16];
    __shared__ int lsum[OZIMMU_MAX_SLICES_DEV][16];
    const int t = threadIdx.x;
    if (blockIdx.x == 0 && t < zero_count) zero[t] = 0u;
    int block = (int)blockIdx.x;
    if (block < a.blocks) {
        if (block == 0 && t == 0) a.trailer[0] = a.c;
        block = (block >> 5) * 32 + (block & 7) * 4 + ((block >> 3) & 3);  // (see k_split_both)
        if ((int64_t)block * ROWS < a.rows) split_rows<DBR, ROWS, MASK>(a, block, k, beta, red, lsum);
        return;
    }
    block -= a.blocks;
    const int first = b.groups * b.pieces, second = block >= first;
    const ColumnsOp o = second ? c : b;
    block -= second ? first : 0;
    if (block == 0 && t == 0) o.trailer[0] = o.c;
    cut_maxima<true>(o, block, red);
}

template <bool MASK>
__global__ __launch_bounds__(64 * CUT_WAVES) void k_cut_columns(ColumnsOp b, ColumnsOp c, int k, int beta)
{
    __shared__ int lsum[OZIMMU_MAX_SLICES_DEV][16];
    const int first = b.groups * b.pieces, second = (int)blockIdx.x >= first, block = (int)blockIdx.x - (second ? first : 0);
    const ColumnsOp o = second ? c : b;
    const int group = block % o.groups, piece = block / o.groups;
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    double y[4][4];
    cut_load(o, group, piece, y);
    const int64_t R = (int64_t)group * CUT_COLS + (lane & 15);
    const bool ok = R < o.rows;
    for (int i = t; i < k * 16; i += 64 * CUT_WAVES) lsum[i / 16][i % 16] = 0;
    // (the tagged key of the column's maximum, or already the exponent that the first piece's workgroup puts in its place: see k_split_B)
    int e = 0;
    if (ok) {
        const uint32_t v = __hip_atomic_load(reinterpret_cast<uint32_t*>(o.e) + R, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        e = (v & 0xc0000000u) == RAW_KEY_TAG ? key_to_exp<MASK>(v - RAW_KEY_TAG) : (int)v;
        if (piece == 0 && w == 0 && lane < 16)
            __hip_atomic_store(reinterpret_cast<uint32_t*>(o.e) + R, (uint32_t)e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const int sc = beta - 1 - e;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) y[i / 4][i % 4] = ldexp(y[i / 4][i % 4], sc);
    const double inv_step = ldexp(1.0, -beta), step = (double)(1 << beta);
    const uint32_t c4 = (uint32_t)o.c * 0x01010101u;
    double sig = 6755399441055744.0;
    const int64_t l0 = (int64_t)piece * cut_inner(1) + w * 64 + (lane >> 4) * 16;
    const bool inside = l0 < (int64_t)o.KT * TILE_K;
    int8_t* out = o.S + packed_offset(R, l0, o.KT);
    for (int s = 0; s < k; ++s) {
        uint32_t v[4];
        int sum = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = with_offset(digits4<MASK>(y[u], sig, step), c4, &sum);
        if (ok && inside) store_slices(out, v[0], v[1], v[2], v[3]);
        out += o.slice_stride;
        sig *= inv_step;
        sum = inside ? sum : 0;
        sum = over_strided<16>(sum, Sum{});
        if (lane < 16) atomicAdd(&lsum[s][lane], sum);
    }
    if (o.c == 0) return;  // (nobody asks for the sums)
    __syncthreads();
    // integers: their order does not matter
    for (int i = t; i < k * 16; i += 64 * CUT_WAVES) {
        const int s = i / 16;
        const int64_t col = (int64_t)group * CUT_COLS + i % 16;
        int run = 0;
        for (int q = 0; q <= s; ++q) run += lsum[q][i % 16];
        if (col < o.rows) atomicAdd(&o.P[(int64_t)s * o.Rpad + col], run);
    }
}

// ---------------------------------------------------------------------------
// B, pass 1: column maxima.  A workgroup covers 64 columns x LCH inner rows;
// lane = column, so each wave reads 512 contiguous bytes per inner row.  The
// per-column maximum is merged into keys[] with a 32-bit atomic max (order
// free, hence deterministic).
// ---------------------------------------------------------------------------
constexpr int LCH = 512;  // rows of B per workgroup of the column-maximum kernel (fewer for small B)

__global__ __launch_bounds__(256) void k_colmax_B(int64_t n, int64_t p, const double* __restrict__ B, int64_t ldb,
                                                  uint32_t* __restrict__ keys, int lch, uint32_t tag)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t j = (int64_t)blockIdx.y * 64 + lane;
    const int64_t l0 = (int64_t)blockIdx.x * lch;
    const int64_t l1 = l0 + lch < n ? l0 + lch : n;
    __shared__ uint64_t part[4][64];
    uint64_t mx = 0;
    if (j < p) {
        for (int64_t l = l0 + w; l < l1; l += 4) {
            uint64_t b = abs_bits(B[l * ldb + j]);
            mx = b > mx ? b : mx;
        }
    }
    part[w][lane] = mx;
    __syncthreads();
    if (w == 0 && j < p) {
        for (int q = 1; q < 4; ++q) mx = part[q][lane] > mx ? part[q][lane] : mx;
        uint32_t key = exp_key(mx);
        if (key) atomicMax(keys + j, tag | key);
    }
}

// rows per workgroup of k_colmax_B: LCH, halved while that leaves the chip short of workgroups
inline int colmax_rows(int64_t n, int64_t p)
{
    int lch = LCH;
    while (lch > 16 && ((n + lch - 1) / lch) * ((p + 63) / 64) < 1024) lch /= 2;
    return lch;
}

// two fills in one launch: x[0, cx) = vx and y[0, cy) = vy
__global__ void k_fill2_u32(int64_t cx, uint32_t* x, uint32_t vx, int64_t cy, uint32_t* y, uint32_t vy)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < cx) x[i] = vx;
    if (i < cy) y[i] = vy;
}

__global__ void k_fill_u32(int64_t count, uint32_t* x, uint32_t v)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) x[i] = v;
}

__global__ void k_decode_keys(int64_t count, int32_t* e)
{
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) e[i] = key_to_exp<false>((uint32_t)e[i]);
}

// per-slice sums of a stack (k arrays of Rpad entries) -> prefix sums over the slices, in place
__global__ void k_prefix_sums(int64_t Rpad, int k, int32_t* P)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= Rpad) return;
    int run = 0;
    for (int s = 0; s < k; ++s) {
        run += P[(int64_t)s * Rpad + i];
        P[(int64_t)s * Rpad + i] = run;
    }
}

// ---------------------------------------------------------------------------
// B, pass 2: slices, transposed so that the inner index becomes contiguous.
// A workgroup handles 128 inner rows x 64 columns.  Reads: lane = column
// (512 contiguous bytes per wave and inner row).  Each thread keeps its 32
// remainders in registers, emits slices in batches of SBATCH through LDS
// (row pitch 33 dwords: conflict-free column-wise dword stores), and the
// batch is written out with lane = 16-byte chunk along the inner index, i.e.
// full 128-byte lines (two adjacent rows of a tile) per slice.
// ---------------------------------------------------------------------------
constexpr int SBATCH = 4;
constexpr int PITCH = 33;  // dwords per column row in LDS (32 data + 1 pad)

template <bool MASK, bool KEEP>
__global__ __launch_bounds__(256) void k_split_B(int64_t n, int64_t p, const double* __restrict__ B, int64_t ldb,
                                                 int k, int beta, int c, int8_t* __restrict__ SB,
                                                 int32_t* eB, int32_t* __restrict__ P,
                                                 int32_t* __restrict__ trailer, int64_t Npad, int64_t Rpad,
                                                 int64_t slice_stride, int blocks_per_wg)
{
    __shared__ uint32_t tile[SBATCH][64 * PITCH];
    __shared__ int colsum[OZIMMU_MAX_SLICES_DEV][64];  // sums of the stored bytes per slice and column
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t j0 = (int64_t)blockIdx.y * 64;      // first column (= packed row)
    const int64_t j = j0 + lane;
    const int64_t KT = Npad / TILE_K;
    const double two_beta = (double)(1 << beta);
    const bool col_ok = j < p;
    // eB[j] holds the tagged key of the column maximum until the workgroups of the first inner block have
    // replaced it by the exponent; a workgroup that reads it meanwhile gets one or the other, and both give e
    int e = 0;
    if (col_ok) {
        const uint32_t v = __hip_atomic_load(reinterpret_cast<uint32_t*>(eB) + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        e = (v & 0xc0000000u) == RAW_KEY_TAG ? key_to_exp<MASK>(v - RAW_KEY_TAG) : (int)v;
        if (blockIdx.x == 0 && w == 0)
            __hip_atomic_store(reinterpret_cast<uint32_t*>(eB) + j, (uint32_t)e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const int sc = beta - 1 - e;
    if (blockIdx.x == 0 && blockIdx.y == 0 && t == 0) trailer[0] = c;
    for (int i = t; i < k * 64; i += 256) colsum[i / 64][i % 64] = 0;
    // write-out mapping: 8 lanes per column row, 32 column rows per pass
    const int oc = t & 7, orow = t >> 3;
    __syncthreads();

    // blocks_per_wg consecutive blocks of 128 inner rows (fewer atomics on the sums than one block each)
    for (int blk = 0; blk < blocks_per_wg; ++blk) {
        const int64_t l0 = ((int64_t)blockIdx.x * blocks_per_wg + blk) * 128;  // inner offset of this block
        if (l0 >= Npad) break;
        double y[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            const int64_t l = l0 + w * 32 + i;
            const double v = (col_ok && l < n) ? B[l * ldb + j] : 0.0;
            y[i] = ldexp(v, sc);
        }
        for (int sb = 0; sb < k; sb += SBATCH) {
            const int ns = (k - sb) < SBATCH ? (k - sb) : SBATCH;
            for (int s = 0; s < ns; ++s) {
                int tsum = 0;
#pragma unroll
                for (int ii = 0; ii < 8; ++ii) {
                    int sm;
                    tile[s][lane * PITCH + w * 8 + ii] = slice_word4<MASK>(&y[4 * ii], c, two_beta, &sm);
                    tsum += sm;
                }
                atomicAdd(&colsum[sb + s][lane], tsum);
            }
            __syncthreads();
            for (int s = 0; s < ns; ++s) {
#pragma unroll
                for (int pass = 0; pass < 2; ++pass) {
                    int jr = orow + 32 * pass;
                    const uint32_t* src = &tile[s][jr * PITCH + oc * 4];
                    uint4 v = make_uint4(src[0], src[1], src[2], src[3]);
                    int8_t* dst = SB + (int64_t)(sb + s) * slice_stride + packed_offset(j0 + jr, l0 + oc * CHUNK, KT);
                    // Whole 128-byte lines.  KEEP: the memory-side cache holds the slices until the products read them, whose
                    // steps otherwise wait on memory (41 x 25165 x 94, k = 6, 32 x 32 tiles: 159 us and 105); where they
                    // are too many, non-temporal, 4 % faster here (1024 columns of 65536, k = 8).
                    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
                    const u32x4 vv = {v.x, v.y, v.z, v.w};
                    if constexpr (KEEP)
                        store_slices(dst, v.x, v.y, v.z, v.w);
                    else
                        __builtin_nontemporal_store(vv, reinterpret_cast<u32x4*>(dst));
                }
            }
            __syncthreads();
        }
    }
    // integer sums: order-free, hence deterministic (P was zeroed; k_prefix_sums finishes)
    for (int i = t; i < k * 64; i += 256)
        if (colsum[i / 64][i % 64] != 0) atomicAdd(&P[(int64_t)(i / 64) * Rpad + j0 + (i % 64)], colsum[i / 64][i % 64]);
}

// ---------------------------------------------------------------------------
// Algorithm 5 (one scale per slice), A: one wave per padded row.
// The scale of slice s+1 comes from the largest remainder after slice s, so the
// row is walked k times; what is left of it lives in `rem` (row pitch Npad) and
// every lane re-reads only the elements it wrote itself.  With
//   y = remainder * 2^(beta-1-e_s)  (exact),  q_s = rint(y),
//   remainder <- (y - q_s) * 2^(e_s+1-beta)  (both exact).
// HBM-bound: about 16 k bytes per element (remainder read and written per slice).
// ---------------------------------------------------------------------------
template <bool VEC>
__global__ __launch_bounds__(256) void k_split_A_ps(int64_t m, int64_t n, const double* __restrict__ A, int64_t lda,
                                                    int k, int beta, int8_t* __restrict__ SA,
                                                    int32_t* __restrict__ eA, double* __restrict__ rem,
                                                    int32_t* __restrict__ trailer, int64_t Npad,
                                                    int64_t slice_stride)
{
    const int lane = threadIdx.x & 63;
    const int64_t R = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t KT = Npad / TILE_K;
    if (blockIdx.x == 0 && threadIdx.x == 0) trailer[0] = 0;  // slices with a scale each are stored without offset

    if (R >= m) {  // padding row: zeros in every slice
        for (int64_t l = 4 * lane; l < Npad; l += 256)
            for (int s = 0; s < k; ++s)
                *reinterpret_cast<uint32_t*>(SA + s * slice_stride + packed_offset(R, l, KT)) = 0u;
        return;
    }
    const double* row = A + R * lda;
    double* rrow = rem + R * Npad;

    auto load4 = [&](int64_t l, double* v) {
        if (VEC && l + 3 < n) {
            double2 a = *reinterpret_cast<const double2*>(row + l);
            double2 b = *reinterpret_cast<const double2*>(row + l + 2);
            v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = (l + j < n) ? row[l + j] : 0.0;
        }
    };

    uint64_t mx = 0;
    for (int64_t l = 4 * lane; l < n; l += 256) {
        double v[4];
        load4(l, v);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint64_t b = abs_bits(v[j]);
            mx = b > mx ? b : mx;
        }
    }
    int e = key_to_exp<false>(exp_key(wave_max_u64(mx)));

    for (int s = 0; s < k; ++s) {
        if (lane == 0) eA[(int64_t)s * m + R] = e;
        const int sc = beta - 1 - e;
        const bool keep = s + 1 < k;
        mx = 0;
        for (int64_t l = 4 * lane; l < Npad; l += 256) {
            double v[4];
            if (s == 0) {
                load4(l, v);
            } else {
                double2 a = *reinterpret_cast<const double2*>(rrow + l);
                double2 b = *reinterpret_cast<const double2*>(rrow + l + 2);
                v[0] = a.x; v[1] = a.y; v[2] = b.x; v[3] = b.y;
            }
            uint32_t w = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double y = ldexp(v[j], sc);
                const double q = __builtin_rint(y);
                w |= ((uint32_t)(int)q & 0xffu) << (8 * j);
                v[j] = ldexp(y - q, -sc);
                const uint64_t b = abs_bits(v[j]);
                mx = b > mx ? b : mx;
            }
            *reinterpret_cast<uint32_t*>(SA + s * slice_stride + packed_offset(R, l, KT)) = w;
            if (keep) {
                *reinterpret_cast<double2*>(rrow + l) = make_double2(v[0], v[1]);
                *reinterpret_cast<double2*>(rrow + l + 2) = make_double2(v[2], v[3]);
            }
        }
        e = key_to_exp<false>(exp_key(wave_max_u64(mx)));
    }
}

// ---------------------------------------------------------------------------
// Algorithm 5, vectors that stay in the registers of a workgroup: both operands in one launch, read once.
//
// A workgroup of THREADS has V vectors, rows or columns, 16 U elements a thread: 16 U THREADS / V inner positions.  The remainders
// stay where they are from slice to slice; only their maximum travels, between lanes and, where a vector is on several waves,
// through LDS.  V by the length (see launch_split_per_slice): elements past the end cost as much as real ones, so short vectors share a
// workgroup (a wave skips a quad or chunk that lies past the padding).  Bound by HBM for large operands (8 + k bytes an element; the
// kernels above and below move 16 k), by k reductions for small ones.
// Whole calls, us, k + 4 launches; one launch with a row to each workgroup of 512 threads whatever its length; and this: 176 x 38 x 702,
// k = 9, 74, 23.1, 15.3; 2006 x 768 x 615, k = 8, 168, 109, 72; 3892^3, k = 12, 4400, 3690, 3470; 100000 x 50 x 10, k = 6, 1215, 1682, 72.
// ---------------------------------------------------------------------------
struct PsOp {
    const double* X;
    int64_t ld, rows, n;
    int8_t* S;
    int32_t* e;
    int32_t* trailer;
    int64_t slice_stride;
    int KT, by_col, blocks;
};

// BY_COL: vector t % V, a thread has U chunks of 16 consecutive positions; else vector t / (threads of a vector), U times 4 quads,
// neighbouring threads beside each other.
template <int THREADS, int U, int V, bool BY_COL>
__device__ inline void split_ps(const PsOp& o, int block, int k, int beta, double (*red)[THREADS / 64][64])
{
    constexpr int TPV = THREADS / V;                       // threads of a vector
    constexpr int LANES = BY_COL ? 64 / (V < 64 ? V : 64) : TPV < 64 ? TPV : 64;   // of a vector in a wave
    constexpr int WAVES = BY_COL ? THREADS / 64 : TPV / LANES;                     // that a vector is on
    constexpr int FIRST = BY_COL ? V : 1;                  // distance of a vector's lanes
    constexpr int GROUP = BY_COL ? 4 : 2;                  // quads at a time: a column's chunk of 16 bytes
    static_assert(V <= 64 && TPV * V == THREADS, "");
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int v = BY_COL ? t % V : t / TPV, tv = BY_COL ? t / V : t % TPV;
    const int64_t R = (int64_t)block * V + v;
    const bool ok = R < o.rows;
    const int64_t at = ok ? R : o.rows - 1;                // (vectors past the edge read along, their results are not stored)
    const int n = (int)o.n, end = o.KT * TILE_K;
    // position of quad q (4 consecutive elements)
    auto place = [&](int q) -> int { return BY_COL ? (q / 4) * (TPV * 16) + tv * 16 + (q % 4) * 4 : q * (TPV * 4) + tv * 4; };
    double y[4 * U][4], mx = 0.0;
    if constexpr (BY_COL) {
        const global_f64 x = (global_f64)o.X + at;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            global_f64 p = x + (int64_t)place(4 * u) * o.ld;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                y[4 * u + i / 4][i % 4] = 0.0;
                if (place(4 * u) + i < n) y[4 * u + i / 4][i % 4] = *p;
                p += o.ld;
                asm volatile("" : "+v"(p));                // (one running pointer: see split_cols)
            }
        }
    } else {
        const global_f64 x = (global_f64)o.X + at * o.ld;
#pragma unroll
        for (int q = 0; q < 4 * U; ++q) {
            const int l = place(q), l0 = q * (TPV * 4) + (WAVES > 1 ? w % WAVES * 256 : 0);  // (the wave's first: uniform)
            if (l0 + 4 * LANES <= n) {
                const f64x2_a8 a = *(global_f64x2)(x + l), b = *(global_f64x2)(x + l + 2);
                y[q][0] = a.x, y[q][1] = a.y, y[q][2] = b.x, y[q][3] = b.y;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    y[q][j] = 0.0;
                    if (l + j < n) y[q][j] = x[l + j];
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < 4 * U; ++q)
#pragma unroll
        for (int j = 0; j < 4; ++j) mx = fmax(mx, fabs(y[q][j]));
    for (int s = 0; s < k; ++s) {
#pragma unroll
        for (int off = FIRST; off < FIRST * LANES; off <<= 1) mx = fmax(mx, __shfl_xor(mx, off, 64));
        if constexpr (WAVES > 1) {
            // (two places for the maxima in turn: one barrier a slice)
            constexpr int SLOTS = BY_COL ? V : 1;
            if (lane < SLOTS) red[s & 1][w][lane] = mx;
            __syncthreads();
            const int w0 = BY_COL ? 0 : w / WAVES * WAVES;
#pragma unroll
            for (int z = 0; z < WAVES; ++z) mx = fmax(mx, red[s & 1][w0 + z][BY_COL ? v : 0]);
        }
        const int e = exponent_of<false>(mx), sc = beta - 1 - e;
        if (ok && tv == 0) o.e[(int64_t)s * o.rows + R] = e;
        mx = 0.0;
        int8_t* out = o.S + s * o.slice_stride;
        // (under one condition GROUP quads: each by itself they would wait for each other's latencies)
#pragma unroll
        for (int q0 = 0; q0 < 4 * U; q0 += GROUP) {
            uint32_t word[GROUP] = {};
            if (place(q0) < n) {
#pragma unroll
                for (int g = 0; g < GROUP; ++g)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const double ys = ldexp(y[q0 + g][j], sc), d = __builtin_rint(ys);
                        word[g] |= ((uint32_t)(int)d & 0xffu) << (8 * j);
                        y[q0 + g][j] = ldexp(ys - d, -sc);
                        mx = fmax(mx, fabs(y[q0 + g][j]));
                    }
            }
            // (Through L2, see store_slices.  A chunk of a column in one store: in four of 4 bytes each goes through by itself.  Four, one and left in
            // L2, whole calls: 36 x 1885 x 5453, k = 8, 172.3, 114.9 and 116.7 us, 303 x 380 x 10162, k = 6, 86.2, 71.0 and 74.0;
            // one and left in L2: 700 x 500 x 900, k = 8, 36.9 and 40.9, 700 x 8000 x 900 256.7 and 261.5.)
            if constexpr (BY_COL) {
                if (ok && place(q0) < end) store_slices(out + packed_offset(R, place(q0), o.KT), word[0], word[1], word[2], word[3]);
            } else {
#pragma unroll
                for (int g = 0; g < GROUP; ++g)
                    if (ok && place(q0 + g) < end) store_slices(out + packed_offset(R, place(q0 + g), o.KT), word[g]);
            }
        }
    }
}

template <int THREADS, int U, int V>
__global__ __launch_bounds__(THREADS) void k_split_ps(PsOp a, PsOp b, int k, int beta)
{
    __shared__ double red[2][THREADS / 64][64];
    const bool second = (int)blockIdx.x >= a.blocks;
    const PsOp o = second ? b : a;
    const int block = second ? (int)blockIdx.x - a.blocks : (int)blockIdx.x;
    if (block == 0 && threadIdx.x == 0) o.trailer[0] = 0;  // slices with a scale each are stored without offset
    if (o.by_col)
        split_ps<THREADS, U, V, true>(o, block, k, beta, red);
    else
        split_ps<THREADS, U, V, false>(o, block, k, beta, red);
}

// ---------------------------------------------------------------------------
// Algorithm 5, B: one launch per slice (the column maxima of the remainder need
// a grid-wide reduction between slices).  Tiling and write-out as in k_split_B;
// src is B for the first slice and the remainder buffer (pitch p) afterwards.
// The maxima of the new remainder are merged into keys_next for the next launch.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_split_B_ps(int64_t n, int64_t p, const double* src, int64_t ld, int beta,
                                                    int8_t* __restrict__ SBs, const uint32_t* __restrict__ keys,
                                                    uint32_t* __restrict__ keys_next, double* rem, int64_t Npad)
{
    __shared__ uint32_t tile[64 * PITCH];
    __shared__ uint64_t part[4][64];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t l0 = (int64_t)blockIdx.x * 128;
    const int64_t j0 = (int64_t)blockIdx.y * 64;
    const int64_t j = j0 + lane;
    const int64_t KT = Npad / TILE_K;
    const bool col_ok = j < p;
    const int sc = beta - 1 - (col_ok ? key_to_exp<false>(keys[j]) : 0);

    double y[32];
#pragma unroll
    for (int i = 0; i < 32; ++i) {
        const int64_t l = l0 + w * 32 + i;
        y[i] = (col_ok && l < n) ? src[l * ld + j] : 0.0;
    }
    uint64_t mx = 0;
#pragma unroll
    for (int ii = 0; ii < 8; ++ii) {
        uint32_t wv = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int i = 4 * ii + b;
            const double ys = ldexp(y[i], sc);
            const double q = __builtin_rint(ys);
            wv |= ((uint32_t)(int)q & 0xffu) << (8 * b);
            y[i] = ldexp(ys - q, -sc);
            const uint64_t ab = abs_bits(y[i]);
            mx = ab > mx ? ab : mx;
        }
        tile[lane * PITCH + w * 8 + ii] = wv;
    }
    if (keys_next) {
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            const int64_t l = l0 + w * 32 + i;
            if (col_ok && l < n) rem[l * p + j] = y[i];
        }
    }
    part[w][lane] = mx;
    __syncthreads();
    const int oc = t & 7, orow = t >> 3;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        const int jr = orow + 32 * pass;
        const uint32_t* sp = &tile[jr * PITCH + oc * 4];
        uint4 v = make_uint4(sp[0], sp[1], sp[2], sp[3]);
        *reinterpret_cast<uint4*>(SBs + packed_offset(j0 + jr, l0 + oc * CHUNK, KT)) = v;
    }
    if (keys_next && w == 0 && col_ok) {
        for (int q = 1; q < 4; ++q) mx = part[q][lane] > mx ? part[q][lane] : mx;
        const uint32_t key = exp_key(mx);
        if (key) atomicMax(keys_next + j, key);
    }
}

// ---------------------------------------------------------------------------
// The whole call (steps (i) to (v)) in one launch, for small outputs of an inner dimension of at most 256.
//
// A workgroup has one 16 x 16 tile of the output: it splits the 16 rows and 16 columns itself, into LDS (the packed layout's
// swizzle, signed digits without offset), each wave multiplies one inner step of 64 into its k chunk sums (r >= k there: a chunk is a
// group), and the sums of the waves meet in LDS, where each thread adds up one element.  Every vector is split again
// by all the tiles in its row or column; what it saves is what such a call consists of: a launch and the wait between two
// dependent ones (k = 8, in a graph: 64^3 8.9 us for two launches, 5.2 for this one, 256^3 10.6 and 7.2).  What bounds it is one latency after the other:
// operands, maxima, digits (a thread makes those of 32 elements), fragments, sums.
// ---------------------------------------------------------------------------
template <int K>
__global__ __launch_bounds__(256) void k_small(ozk::SmallArgs a)
{
    typedef int v4i __attribute__((ext_vector_type(4)));
    extern __shared__ __align__(16) int8_t lds[];
    __shared__ double red[2][4][16];
    __shared__ int lds_exp[2][16];
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int steps = a.steps, slice = steps * 1024;  // bytes of a slice of one operand's 16 vectors
    const int64_t row0 = (int64_t)blockIdx.y * 16, col0 = (int64_t)blockIdx.x * 16;

    // thread (vector v, place q) holds the positions 64 j + 4 q + 0 .. 3 of step j: neighbouring threads read neighbouring memory
    double y[2][4][4];
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        const ozk::SmallArgs::Op& op = a.op[o];
        const int v = op.by_col ? (t & 15) : (t >> 4), q = op.by_col ? (t >> 4) : (t & 15);
        int64_t R = (o == 0 ? row0 : col0) + v;
        R = R < op.rows ? R : op.rows - 1;  // (vectors past the edge read along, their results are not stored)
        const global_f64 x = (global_f64)op.X + (op.by_col ? R : R * op.ld);
        const int64_t pitch = op.by_col ? op.ld : 1;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int l = 64 * j + 4 * q;
            if (!op.by_col && l + 4 <= a.n) {
                const f64x2_a8 p = *(global_f64x2)(x + l), r = *(global_f64x2)(x + l + 2);
                y[o][j][0] = p.x, y[o][j][1] = p.y, y[o][j][2] = r.x, y[o][j][3] = r.y;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    y[o][j][i] = 0.0;
                    if (l + i < a.n) y[o][j][i] = x[(l + i) * pitch];
                }
            }
        }
    }
    double mx[2];
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        mx[o] = 0.0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) mx[o] = fmax(mx[o], fabs(y[o][j][i]));
        if (a.op[o].by_col) {
            mx[o] = over_strided<16>(mx[o], Max{});
            if (lane < 16) red[o][w][lane] = mx[o];
        } else {
            mx[o] = over_neighbours<16>(mx[o], Max{});
        }
    }
    __syncthreads();
    const double inv_step = ldexp(1.0, -a.beta);
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        const bool by_col = a.op[o].by_col;
        const int v = by_col ? (t & 15) : (t >> 4), q = by_col ? (t >> 4) : (t & 15);
        if (by_col)
#pragma unroll
            for (int z = 0; z < 4; ++z) mx[o] = fmax(mx[o], red[o][z][v]);
        const int e = exponent_of<false>(mx[o]), sc = a.beta - 1 - e;
        if (q == 0) lds_exp[o][v] = e;
        int8_t* out = lds + o * K * slice + v * TILE_K + swizzle(v, q >> 2) * CHUNK + 4 * (q & 3);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j >= steps) break;
#pragma unroll
            for (int i = 0; i < 4; ++i) y[o][j][i] = ldexp(y[o][j][i], sc);
            double sig = 6755399441055744.0;
            uint32_t before = 0;                     // (at most 256 inner positions: digits of 7 bits)
#pragma unroll
            for (int s = 0; s < K; ++s) {
                if (s > 0 && s % DIRECT == 0) next_digits(y[o][j], sig * 128.0, &before);
                *reinterpret_cast<uint32_t*>(out + s * slice + j * 1024) = digits4_direct(y[o][j], sig, &before);
                sig *= inv_step;
            }
        }
    }
    __syncthreads();
    v4i acc[K] = {};
    if (w < steps) {
        const int chunk = (0x9c >> (2 * (lane >> 4))) & 3;  // 0, 3, 1, 2: see k_resident
        const int8_t* in = lds + w * 1024 + (lane & 15) * TILE_K + swizzle(lane & 15, chunk) * CHUNK;
        v4i f[2][K];
#pragma unroll
        for (int s = 0; s < K; ++s) {
            f[0][s] = *reinterpret_cast<const v4i*>(in + s * slice);
            f[1][s] = *reinterpret_cast<const v4i*>(in + (K + s) * slice);
        }
#pragma unroll
        for (int g = 0; g < K; ++g)
#pragma unroll
            for (int s = 0; s <= g; ++s) acc[g] = __builtin_amdgcn_mfma_i32_16x16x64_i8(f[0][s], f[1][g - s], acc[g], 0, 0, 0);
    }
    __syncthreads();  // every wave has its fragments: their place takes the sums (zeros past the last step)
#pragma unroll
    for (int g = 0; g < K; ++g) *reinterpret_cast<v4i*>(lds + (w * K + g) * 1024 + lane * 16) = acc[g];
    __syncthreads();
    // Thread t adds up integer t of every sum: register t % 4 of lane t / 4, row 4 (lane / 16) + register, column lane % 16.  Always four
    // waves' sums, all of them on their way at once (a loop over the steps waited for one after the other: 256^3, k = 8, 1.7 us of 8.4).
    const int i = 4 * w + (t & 3), j = lane >> 2;
    const int e = lds_exp[0][i] + lds_exp[1][j] + 2;
    int v[4][K];
#pragma unroll
    for (int z = 0; z < 4; ++z)
#pragma unroll
        for (int g = 0; g < K; ++g) v[z][g] = *reinterpret_cast<const int*>(lds + (z * K + g) * 1024 + 4 * t);
    double d = 0.0;
#pragma unroll
    for (int g = 0; g < K; ++g) {
        const double term = ldexp((double)(v[0][g] + v[1][g] + (v[2][g] + v[3][g])), e - a.beta * (g + 2));
        d = g == 0 ? term : d + term;
    }
    if (row0 + i < a.op[0].rows && col0 + j < a.op[1].rows) {
        double* const out = a.out + (row0 + i) * a.ldo + col0 + j;
        if (a.finish) {
            d = a.alpha * d;
            if (a.cbeta != 0.0) d = d + a.cbeta * *out;
        }
        *out = d;
    }
}

// Unpack: one thread per output byte, out[s][row][l].
__global__ __launch_bounds__(256) void k_export(int64_t rows, int64_t n, int k, const int8_t* __restrict__ packed,
                                                const int32_t* __restrict__ trailer, int8_t* __restrict__ out,
                                                int64_t KT, int64_t slice_stride)
{
    int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int64_t total = (int64_t)k * rows * n;
    if (idx >= total) return;
    int64_t l = idx % n, R = (idx / n) % rows, s = idx / (n * rows);
    out[idx] = (int8_t)(packed[s * slice_stride + packed_offset(R, l, KT)] - trailer[0]);  // stored byte = q + c
}

}  // namespace

namespace ozk {

// k_set_i32: one INT32 (the offset in the trailer of a stack whose split kernels do not write it themselves)
}  // namespace ozk
namespace {
__global__ void k_set_i32(int32_t* x, int32_t v) { x[0] = v; }
}  // namespace
namespace ozk {

// The columns of an operand with the inner dimension cut across workgroups: for few long columns, which would otherwise
// leave most of the chip idle (128 columns of 65536, k = 8: 87 against 198 us).
static hipError_t launch_split_cols_cut(const SplitIn& i, int k, int beta, int split_mode, hipStream_t st)
{
    const int64_t n = i.n, p = i.rows;
    const int64_t Rpad = ozl::rows_padded(p), Npad = ozl::inner_padded(n);
    const int64_t stride = ozl::slice_bytes(p, n);
    int32_t* P = reinterpret_cast<int32_t*>(i.S + ozl::sums_offset(p, n, k));
    int32_t* trailer = reinterpret_cast<int32_t*>(i.S + ozl::trailer_offset(p, n, k));
    const int64_t nsums = (int64_t)k * Rpad, nfill = nsums > p ? nsums : p;
    hipLaunchKernelGGL(k_fill2_u32, dim3((unsigned)((nfill + 255) / 256)), dim3(256), 0, st, p,
                       reinterpret_cast<uint32_t*>(i.e), RAW_KEY_TAG, nsums, reinterpret_cast<uint32_t*>(P), 0u);
    const int lch = colmax_rows(n, p);
    dim3 gmax((unsigned)((n + lch - 1) / lch), (unsigned)((p + 63) / 64));
    hipLaunchKernelGGL(k_colmax_B, gmax, dim3(256), 0, st, n, p, i.X, i.ld, reinterpret_cast<uint32_t*>(i.e), lch,
                       RAW_KEY_TAG);
    // a workgroup takes 4 consecutive blocks of 128 inner rows once there are enough blocks to fill the chip anyway
    const int64_t blocks = Npad / 128;
    const int per_wg = blocks >= 32 ? 4 : 1;
    dim3 grid((unsigned)((blocks + per_wg - 1) / per_wg), (unsigned)(Rpad / 64));
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, n, p, i.X, i.ld, k, beta, i.offset, i.S, i.e, P, trailer, Npad, Rpad,
                           stride, per_wg);
    };
    const bool mask = split_mode != 0, keep = (8.0 + k) * (double)n * (double)p <= 260e6;
    if (keep)
        mask ? launch(k_split_B<true, true>) : launch(k_split_B<false, true>);
    else
        mask ? launch(k_split_B<true, false>) : launch(k_split_B<false, false>);
    hipLaunchKernelGGL(k_prefix_sums, dim3((unsigned)((Rpad + 255) / 256)), dim3(256), 0, st, Rpad, k, P);
    return hipGetLastError();
}

static SplitOp make_op(const SplitIn& i, int k)
{
    SplitOp o{};
    o.X = i.X;
    o.ld = i.ld;
    o.rows = i.rows;
    o.n = i.n;
    o.S = i.S;
    o.e = i.e;
    o.P = reinterpret_cast<int32_t*>(i.S + ozl::sums_offset(i.rows, i.n, k));
    o.trailer = reinterpret_cast<int32_t*>(i.S + ozl::trailer_offset(i.rows, i.n, k));
    o.Rpad = ozl::rows_padded(i.rows);
    o.slice_stride = ozl::slice_bytes(i.rows, i.n);
    o.KT = (int)(ozl::inner_padded(i.n) / ozl::TILE_K);
    o.c = i.offset;
    o.by_col = i.by_col;
    return o;
}

// Columns a workgroup of k_split_both takes (16, 8 or 4), or 0 where they are better cut along the inner dimension
// (launch_split_cols_cut); 0 for rows.  By the least sum of microseconds over the operands of a call, which share a launch unless
// they are cut.  Fitted to 64 to 8192 columns of 4096 to 2^18, k = 1, 4, 8 and 16, each form forced, operands beyond 64 MB in
// no cache (smaller ones are usually still there from whatever made them, unless both together are beyond 128 MB).
//  * Whole, 16 + k bytes an element (read twice): a compute unit moves 25, 20, 16.5 bytes per ns with 16, 8, 4 columns a
//    workgroup, however many workgroups it holds (26 with 4 of an operand in the caches), all of them 4.4, 3.9, 2.9 (4.2)
//    per ps (k = 8, us with 16, 8, 4: 4096 columns of 4096 97, 108, 124; 2017 of 16384 254, 214, 240; 1024 of 4096 54, 42, 37;
//    one workgroup too many for the compute units: 2117 of 80064, k = 2, 878, 1141, 1315).
//  * Cut: four launches and their merging, 65 + 2.4 k us; 6 bytes per ps where the operand stays in the memory-side cache for the
//    second time, else 4.1; padding columns are written too.  Against the best whole, k = 8: 64 columns of 16384 90 and 72 us,
//    500 of 65536 219 and 354, 1024 of 65536 434 and 513, 2017 of 65536 824 and 711, 8192 of 16384 807 and 713.
//  * Rows beside or instead: 8 + k bytes an element (16 + k beyond 16384 positions) at 4.5 per ps, a row at 25 per ns.
// Up to 256 inner positions, where a wave does not share a tile of 64 with others, 16 (1024 columns of 64: 6.4 us, with 4 7.6).
static double choose_columns(const SplitIn* ops, int count, int k, int* per)
{
    constexpr int FORMS = 4, columns_of[FORMS] = {16, 8, 4, 0};
    for (int q = 0; q < count; ++q) per[q] = ops[q].by_col && ops[q].n <= 256 ? 16 : 0;
    if (ops[0].n <= 256) return 0.0;
    const double n = (double)ops[0].n, both = (double)ops[0].rows + (count == 2 ? (double)ops[1].rows : 0.0);
    const int forms0 = ops[0].by_col ? FORMS : 1, forms1 = count == 2 && ops[1].by_col ? FORMS : 1;
    double least = -1.0;
    for (int form = 0; form < forms0 * forms1; ++form) {
        const int f[2] = {form % forms0, form / forms0};
        double cut_us = 0.0, all_us = 0.0, longest_us = 0.0, rows_us = 0.0, groups = 0.0, group_us = 0.0;  // of the launch they share
        bool shared = false;
        for (int q = 0; q < count; ++q) {
            const double vectors = (double)ops[q].rows;
            const int c = columns_of[f[q]];
            if (!ops[q].by_col) {
                const double row_us = n * (16 + k) / 25e3;
                rows_us = n * vectors * (n > 16384 ? 16 + k : 8 + k) / 4.5e6;
                all_us += rows_us;
                longest_us = longest_us > row_us ? longest_us : row_us;
                shared = true;
            } else if (c == 0) {
                const double bytes = n * (16.0 * vectors + (double)k * (double)ozl::rows_padded(ops[q].rows));
                cut_us += 65.0 + 2.4 * k + bytes / (8.0 * n * vectors <= 2.7e8 ? 6e6 : 4.1e6);
            } else {
                const bool cached = 8.0 * n * vectors <= 64e6 && 8.0 * n * both <= 128e6;
                const double w = (double)((ops[q].rows + c - 1) / c);
                const double us = n * (16 + k) * c / (c == 16 ? 25e3 : c == 8 ? 20e3 : cached ? 26e3 : 16.5e3);
                all_us += n * vectors * (16 + k) / (c == 16 ? 4.4e6 : c == 8 ? 3.9e6 : cached ? 4.2e6 : 2.9e6);
                groups += w, group_us += w * us;
                longest_us = longest_us > us ? longest_us : us;
                shared = true;
            }
        }
        double us = cut_us;
        if (shared) {
            // (short workgroups share compute units, long ones each bind one's rate)
            const double rounds = n > 4096.0 ? (double)(((int64_t)groups + 255) / 256) : groups / 256.0;
            double own_us = groups > 0.0 ? rounds * group_us / groups : 0.0;
            own_us = own_us > all_us ? own_us : all_us;
            // (a long workgroup of columns has less of the memory while rows take most of it: 39 columns of 189760 beside 1024
            // rows, k = 4, 1167 us, cut 816)
            const double slowed_us = longest_us + 0.25 * rows_us;
            own_us = own_us > slowed_us ? own_us : slowed_us;
            us += 6.0 + own_us;
        }
        if (least < 0.0 || us < least) {
            least = us;
            for (int q = 0; q < count; ++q) per[q] = ops[q].by_col ? columns_of[f[q]] : 0;
        }
    }
    return least;
}

static CutOp make_cut(const SplitIn& i, int k, uint16_t* keys)
{
    CutOp o{};
    o.X = i.X;
    o.ld = i.ld;
    o.rows = i.rows;
    o.n = i.n;
    o.S = i.S;
    o.e = i.e;
    o.trailer = reinterpret_cast<int32_t*>(i.S + ozl::trailer_offset(i.rows, i.n, k));
    o.keys = keys;
    o.slice_stride = ozl::slice_bytes(i.rows, i.n);
    o.KT = (int)(ozl::inner_padded(i.n) / ozl::TILE_K);
    o.by_col = i.by_col;
    o.groups = (int)((i.rows + cut_vectors(i.by_col) - 1) / cut_vectors(i.by_col));
    o.pieces = (int)((ozl::inner_padded(i.n) + cut_inner(i.by_col) - 1) / cut_inner(i.by_col));
    return o;
}

// Both operands in two launches (k_cut_maxima, k_cut_split), where that is estimated to take less than `us`: 12.5 us (0.4 more for
// each slice less than six: `us` is then too large by that) and 8 bytes per
// ps while the operands are still in the memory-side cache for the second, else 3.8 (whole calls, one launch or the cut columns'
// four and two, k = 8: 47 x 11948 x 48 58.4 and 31.4, 256 x 8192 x 256 63.6 and 48.9, 600 x 20000 x 200 203 and 185, 75 x 2212 x 512 30.2 and
// 29.1, 500 x 1024 x 500 23.2 and 26.1; k = 4: 100 x 262144 x 100 488 and 370, 1000 x 2000 x 1000 35.2 and 40.6).  Not for many columns of
// moderate length: whole ones fill the chip then, and read what does not fit their registers again from near by (12 x 1982 x
// 3483, k = 8, 47.7 and 61.2, 8 x 2369 x 4391, k = 3, 55.2 and 66.4, 31 x 4960 x 3851, k = 1, 96.0 and 126.5; 12 x 17700 x 942, k = 14, 246 and
// 212), and from 2048 positions on, a workgroup's registers full with one row (37 x 2031 x 130, k = 8, 21.7 and 23.7, 22 x 2240 x 170,
// k = 13, 38.4 and 35.4).  Of 488 shapes of many columns or of few vectors this takes 0.3 % longer than the faster of the two on average, without
// the exception 1.0 %.
static bool cut_pays(const SplitIn* ops, int count, int k, double us, size_t room)
{
    if (count != 2 || ops[0].n < 2048) return false;
    double vectors = 0.0;
    int64_t columns = 0;
    size_t keys = 0;
    for (int q = 0; q < 2; ++q) {
        const CutOp o = make_cut(ops[q], k, nullptr);
        if ((int64_t)o.groups * o.pieces >= ((int64_t)1 << 22)) return false;
        keys += 2 * (size_t)o.pieces * (size_t)o.rows;
        vectors += (double)o.rows;
        columns += o.by_col ? o.rows : 0;
    }
    if (keys > room || (columns > 1300 && ops[0].n <= 14500)) return false;
    const double bytes = vectors * (double)ops[0].n * (16 + k), near = bytes < 160e6 ? bytes : 160e6;
    return 12.5 + (k < 6 ? 0.4 * (6 - k) : 0.0) + near / 8e6 + (bytes - near) / 3.8e6 < us;
}

// The columns of a call cut (k_split_and_maxima, k_cut_columns), where that is estimated to take clearly less than `us`:
// 12 us, rows as in choose_columns at 5.5 bytes per ps, 16 + k / 2 bytes an element of columns at 4.5 (whole calls, without and with,
// k = 8: 1024 x 16384 x 1024 535 and 505 us, 523 x 31110 x 815 737 and 673, 256 x 145408 x 512 1364 and 1184; k = 4, A transposed, 256 x 58880 x
// 1152 719 and 523; left whole: 1024^3 39.5 and 44.0, 3000 x 2900 x 3100 613 and 631, 14 x 16060 x 3607, k = 12, 510 and 550, 16384^3,
// k = 3, 18.55 and 18.79 ms).
// 17 to 300 columns of 8192 and more, whose whole ones walk far longer than the rows beside them, have to be ahead by a sixth
// (640 x 14848 x 256, k = 8, 141 and 129 us, 909 x 14947 x 85, k = 4, 88 and 72), others by 20 us and an eighth: whole columns of
// moderate length then fill the chip, and `us` is up to 30 us too long (11 x 7698 x 2231, k = 5, 93 and 118 us, 10 x 5261 x 2140, k = 4, 58 and
// 73, 704 x 13298 x 1524, k = 5, 331 and 362, 1045 x 8580 x 8, k = 4, 45.6 and 52.2).  Of 629 shapes of 2000 to 200000 positions for which it is estimated
// at less than 0.84 `us` this takes 289, of which five are slower by more than 2 %, and is 2.1 % faster on average over all 629 where the best choice
// would be 2.7 %; with the sixth alone 120 were, by up to 26 %, and the average 1.3 %.
// From 12 slices on beside 256 rows and more the sixth is enough again: the error of `us` is small beside all that is written (1300 x 8190 x 901,
// k = 20, whole 2001 us, cut 1971, 488 x 7153 x 1075, k = 17, 653 and 615, 1500 x 9579 x 308, k = 17, 999 and 1024; 28 shapes that the twenty us had
// left whole, cut: 1.0 % faster on average, one slower by more than 1 %.  With fewer rows 44 x 5720 x 1762, k = 16, 144 and 164, with fewer slices 325 x
// 7969 x 1875, k = 6, 171 and 191).
static bool cut_columns_pay(const SplitIn* ops, int count, int k, double us)
{
    if (count != 2 || ops[0].n < 2048) return false;
    const double n = (double)ops[0].n;
    double cut_us = 12.0;
    int64_t columns = 0, rows = 0;
    for (int q = 0; q < 2; ++q) {
        const double vectors = (double)ops[q].rows;
        if (!ops[q].by_col) {
            rows += ops[q].rows;
            const double all_us = n * vectors * (n > 16384.0 ? 16 + k : 8 + k) / 5.5e6, row_us = n * (16 + k) * (n > 8192.0 ? 2 : 1) / 25e3;
            cut_us += all_us > row_us ? all_us : row_us;
            continue;
        }
        const CutOp o = make_cut(ops[q], k, nullptr);
        if ((int64_t)o.groups * o.pieces >= ((int64_t)1 << 22)) return false;
        cut_us += n * vectors * (16.0 + 0.5 * k) / 4.5e6;
        columns += ops[q].rows;
    }
    if (columns < 1 || columns > 2400) return false;
    const bool by_a_sixth = (columns > 16 && columns <= 300 && ops[0].n >= 8192) || (k >= 12 && rows >= 256);
    return by_a_sixth ? cut_us < 0.84 * us : cut_us + 20.0 < 0.88 * us;
}

static hipError_t launch_cut_columns(const SplitIn* ops, int count, int k, int beta, int split_mode, hipStream_t st, uint32_t* also_zero,
                                     int also_zero_count)
{
    SplitOp rows{};
    ColumnsOp columns[2]{};
    int n_columns = 0;
    for (int q = 0; q < count; ++q) {
        if (!ops[q].by_col) {
            rows = make_op(ops[q], k);
            continue;
        }
        ColumnsOp& o = columns[n_columns++];
        static_cast<CutOp&>(o) = make_cut(ops[q], k, nullptr);
        o.P = reinterpret_cast<int32_t*>(ops[q].S + ozl::sums_offset(o.rows, o.n, k));
        o.Rpad = ozl::rows_padded(o.rows);
        o.c = ops[q].offset;
        const int64_t sums = (int64_t)k * o.Rpad, most = sums > o.rows ? sums : o.rows;
        hipLaunchKernelGGL(k_fill2_u32, dim3((unsigned)((most + 255) / 256)), dim3(256), 0, st, o.rows, reinterpret_cast<uint32_t*>(o.e),
                           RAW_KEY_TAG, sums, reinterpret_cast<uint32_t*>(o.P), 0u);
    }
    const bool wide = rows.n > 8192;
    if (rows.rows > 0) {
        rows.per = 2;
        rows.blocks = (int)(((rows.rows + rows.per - 1) / rows.per + 31) / 32 * 32);
    }
    const unsigned pieces = (unsigned)(columns[0].groups * columns[0].pieces + columns[1].groups * columns[1].pieces);
    auto launch = [&](auto first, auto second) {
        hipLaunchKernelGGL(first, dim3((unsigned)rows.blocks + pieces), dim3(64 * SPLIT_WAVES), 0, st, rows, columns[0], columns[1], k, beta,
                           also_zero, also_zero_count);
        hipLaunchKernelGGL(second, dim3(pieces), dim3(64 * CUT_WAVES), 0, st, columns[0], columns[1], k, beta);
    };
    if (split_mode != 0)
        wide ? launch(k_split_and_maxima<64, 2, true>, k_cut_columns<true>) : launch(k_split_and_maxima<16, 2, true>, k_cut_columns<true>);
    else
        wide ? launch(k_split_and_maxima<64, 2, false>, k_cut_columns<false>) : launch(k_split_and_maxima<16, 2, false>, k_cut_columns<false>);
    return hipGetLastError();
}

int split_cut(const SplitIn* ops, int count, int k, size_t room_bytes, bool short_product)
{
    int per[2] = {0, 0};
    const double us = choose_columns(ops, count, k, per);
    if (short_product && cut_pays(ops, count, k, us, room_bytes)) return 1;
    return cut_columns_pay(ops, count, k, us) ? 2 : 0;
}

hipError_t launch_split(const SplitIn* ops, int count, int k, int beta, int split_mode, hipStream_t st, uint32_t* also_zero,
                        int also_zero_count, void* room, size_t room_bytes)
{
    SplitOp op[2]{};
    int used = 0, per[2] = {0, 0};
    bool columns = false;
    const double whole_us = choose_columns(ops, count, k, per);
    if (room && cut_pays(ops, count, k, whole_us, room_bytes)) {
        const CutOp a = make_cut(ops[0], k, static_cast<uint16_t*>(room));
        const CutOp b = make_cut(ops[1], k, a.keys + (int64_t)a.pieces * a.rows);
        const dim3 grid((unsigned)(a.groups * a.pieces + b.groups * b.pieces)), block(64 * CUT_WAVES);
        hipLaunchKernelGGL(k_cut_maxima, grid, block, 0, st, a, b);
        if (split_mode != 0)
            hipLaunchKernelGGL(k_cut_split<true>, grid, block, 0, st, a, b, k, beta, also_zero, also_zero_count);
        else
            hipLaunchKernelGGL(k_cut_split<false>, grid, block, 0, st, a, b, k, beta, also_zero, also_zero_count);
        return hipGetLastError();
    }
    if (cut_columns_pay(ops, count, k, whole_us)) return launch_cut_columns(ops, count, k, beta, split_mode, st, also_zero, also_zero_count);
    for (int q = 0; q < count; ++q) {
        if (ops[q].by_col && per[q] == 0) {
            const hipError_t e = launch_split_cols_cut(ops[q], k, beta, split_mode, st);
            if (e != hipSuccess) return e;
            continue;
        }
        columns = columns || ops[q].by_col;
        op[used] = make_op(ops[q], k);
        op[used++].per = per[q];
    }
    // Columns first beyond 1024 inner positions: their workgroups are the longer ones (1537 x 2051 x 1283, k = 9, a call 174.1 us,
    // columns first 170.0; up to there they are not: 777 x 1001 x 513, k = 7, 29.5 and 30.1)
    if (used == 2 && op[1].by_col && !op[0].by_col && op[0].n > 1024) {
        const SplitOp rows = op[0];
        op[0] = op[1];
        op[1] = rows;
    }
    if (used == 0) {
        if (also_zero_count > 0)
            hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)((also_zero_count + 255) / 256)), dim3(256), 0, st, also_zero_count,
                               also_zero, 0u);
        return hipGetLastError();
    }
    const int64_t n = op[0].n;
    int waves = 4, dbr = 16;
    if (columns) {
        // (the 4 tiles of an inner dimension of up to 256 keep four waves busy: 262144 columns of 64, k = 8, 178 us, with
        // eight 216)
        if (n > 256) waves = SPLIT_WAVES;
        // Rows beside columns: by two where a row keeps 8 waves busy (4096 rows of 4096: 49 us, by four 58; 1024 rows of
        // 1024: 9.0 and 7.9), one by one where there are few (256 rows of 16384: 21 us, by two 24).  Beyond 8192 inner
        // positions a row is kept in 64 registers a thread (16384^2 907 us, with 16 of them 993).
        for (int q = 0; q < used; ++q) {
            if (op[q].by_col) continue;
            op[q].per = n < 2048 ? 4 : (n > 8192 && op[q].rows <= 512) ? 1 : 2;
            if (n > 8192) dbr = 64;
        }
    } else {
        // Rows alone, up to 16384 inner positions: a workgroup of as few waves and registers as hold its rows, so that several
        // share a compute unit - all eight waves where there are few rows, for the time of one (16 rows of 2048, k = 16: 9.3 us,
        // with four waves 10.4).  One row a workgroup from 2048 positions on; more, whose longer pieces of a packed tile are whole
        // memory lines, where the slices leave the caches (us, by one and by two: 4096 rows of 4096 k = 8 47.8 and 48.3, k = 16
        // 129 and 90; 2048 of 8192 k = 1 24.0 and 25.2, k = 16 127 and 91; 2048 of 12288 k = 1 34.8 and 45.1; 4096 of 16384
        // k = 16 447 and 380; a row of just over 8192 wastes the wide form's registers: 16384 of 9216 k = 8 540 and 568).
        // Beyond, one by one where there are few, as beside columns.
        for (int q = 0; q < used; ++q) {
            const bool few = op[q].rows <= (n > 16384 ? 512 : 256);
            const double slices = (double)k * (double)op[q].rows * (double)n;
            const bool one = n > 16384 ? few : n > 10240 ? slices <= 200e6 : n > 8192 || slices <= 150e6;
            op[q].per = n <= 1024 ? 4 : n > 2048 ? (one ? 1 : 2) : few ? 1 : one ? 2 : 4;
            if (few ? n > 256 : op[q].per * n > 64 * 16 * 4) waves = SPLIT_WAVES;
            const int hold = n <= 4096 || (one && n <= 8192) ? 16 : n <= 8192 || (one && n <= 16384) ? 32 : 64;
            dbr = hold > dbr ? hold : dbr;
        }
    }
    if (dbr == 64) {  // one number of rows a launch
        int rows = 2;
        for (int q = 0; q < used; ++q) rows = !op[q].by_col && op[q].per < rows ? op[q].per : rows;
        for (int q = 0; q < used; ++q) op[q].per = op[q].by_col ? op[q].per : rows;
        dbr += rows;
    }
    // whole sets of 32 workgroups per operand (see k_split_both)
    for (int q = 0; q < used; ++q) op[q].blocks = (int)(((op[q].rows + op[q].per - 1) / op[q].per + 31) / 32 * 32);
    const dim3 grid((unsigned)(op[0].blocks + op[1].blocks)), block(64 * waves);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, st, op[0], op[1], k, beta, also_zero, also_zero_count);
    };
    const bool mask = split_mode != 0;
    // The first four workgroups of an operand run on XCD 0 (see k_split_both), and so does the product's only tile, which finds slices left in that L2
    // near by.  Written through it waits for them: 11 x 1176 x 9, k = 5, 11.9 and 13.4 us a call, 5 x 772 x 7, k = 11, 17.2 and 19.4, 3 x
    // 2304 x 6, k = 3, 14.1 and 16.6 (300 random calls of up to 16 x 16 outputs: 6.5 % slower on average, up to 22 %).  Also where the next four hold
    // rows (300 calls of 17 to 32 x 1 to 16: 0.8 % on average, up to 25 %, eight gain, 2.3 % at most); not with more columns (4 x 640 x 32,
    // k = 12, 18.0 and 17.7).
    auto beside_the_tile = [](const SplitOp& o) { return o.rows <= (o.by_col ? 4 : 8) * o.per; };
    const bool near = used == 2 && dbr == 16 && beside_the_tile(op[0]) && beside_the_tile(op[1]);
    if (near && columns)
        mask ? launch(k_split_both<16, 0, true, true, true>) : launch(k_split_both<16, 0, true, false, true>);
    else if (near)
        mask ? launch(k_split_both<16, 0, false, true, true>) : launch(k_split_both<16, 0, false, false, true>);
    else if (columns && dbr == 16)
        mask ? launch(k_split_both<16, 0, true, true>) : launch(k_split_both<16, 0, true, false>);
    else if (columns && dbr == 65)
        mask ? launch(k_split_both<64, 1, true, true>) : launch(k_split_both<64, 1, true, false>);
    else if (columns)
        mask ? launch(k_split_both<64, 2, true, true>) : launch(k_split_both<64, 2, true, false>);
    else if (dbr == 16)
        mask ? launch(k_split_both<16, 0, false, true>) : launch(k_split_both<16, 0, false, false>);
    else if (dbr == 32)
        mask ? launch(k_split_both<32, 0, false, true>) : launch(k_split_both<32, 0, false, false>);
    else if (dbr == 65)
        mask ? launch(k_split_both<64, 1, false, true>) : launch(k_split_both<64, 1, false, false>);
    else
        mask ? launch(k_split_both<64, 2, false, true>) : launch(k_split_both<64, 2, false, false>);
    return hipGetLastError();
}

hipError_t launch_split_A_per_slice(int64_t m, int64_t n, const double* A, int64_t lda, int k, int beta, int8_t* SA,
                                    int32_t* eA, double* rem, hipStream_t st)
{
    const int64_t Rpad = ozl::rows_padded(m), Npad = ozl::inner_padded(n);
    const int64_t stride = ozl::slice_bytes(m, n);
    int32_t* trailer = reinterpret_cast<int32_t*>(SA + ozl::trailer_offset(m, n, k));
    const bool vec = (reinterpret_cast<uintptr_t>(A) % 16 == 0) && (lda % 2 == 0);
    dim3 grid((unsigned)(Rpad / 4)), block(256);
    if (vec)
        hipLaunchKernelGGL((k_split_A_ps<true>), grid, block, 0, st, m, n, A, lda, k, beta, SA, eA, rem, trailer, Npad,
                           stride);
    else
        hipLaunchKernelGGL((k_split_A_ps<false>), grid, block, 0, st, m, n, A, lda, k, beta, SA, eA, rem, trailer, Npad,
                           stride);
    return hipGetLastError();
}

template <int THREADS, int U, int V>
static hipError_t launch_split_ps(const SplitIn* ops, int k, int beta, hipStream_t st)
{
    PsOp op[2]{};
    for (int q = 0; q < 2; ++q) {
        const SplitIn& i = ops[q];
        op[q].X = i.X;
        op[q].ld = i.ld;
        op[q].rows = i.rows;
        op[q].n = i.n;
        op[q].S = i.S;
        op[q].e = i.e;
        op[q].trailer = reinterpret_cast<int32_t*>(i.S + ozl::trailer_offset(i.rows, i.n, k));
        op[q].slice_stride = ozl::slice_bytes(i.rows, i.n);
        op[q].KT = (int)(ozl::inner_padded(i.n) / ozl::TILE_K);
        op[q].by_col = i.by_col;
        op[q].blocks = (int)((i.rows + V - 1) / V);
    }
    hipLaunchKernelGGL((k_split_ps<THREADS, U, V>), dim3((unsigned)(op[0].blocks + op[1].blocks)), dim3(THREADS), 0, st, op[0], op[1],
                       k, beta);
    return hipGetLastError();
}
hipError_t launch_split_per_slice(const SplitIn* ops, int k, int beta, hipStream_t st)
{
    // As many vectors to a workgroup as the padding of the slices (to 256 positions, stored too) allows; from 2048 positions on that
    // would be 32 elements a thread, which few vectors, a compute unit to each workgroup, have to wait for: 30 x 4008 x 10,
    // k = 10, 57.5 us, with two vectors to a workgroup 52.2; 200 x 3000 x 200, k = 8, 40.3 and 39.4.  (Two columns are 16 bytes of a
    // memory line at a time: 30 x 4000 x 300, k = 5, 37.3 and 39.7.)
    const int64_t n = ozl::inner_padded(ops[0].n);
    if (n <= 256) return launch_split_ps<256, 1, 16>(ops, k, beta, st);
    if (n <= 512) return launch_split_ps<512, 1, 16>(ops, k, beta, st);
    if (n <= 2048) return launch_split_ps<512, 1, 4>(ops, k, beta, st);
    if (n <= 4096 && ops[0].rows <= 256 && ops[1].rows <= 256) return launch_split_ps<512, 1, 2>(ops, k, beta, st);
    if (n <= 4096) return launch_split_ps<512, 2, 4>(ops, k, beta, st);
    return launch_split_ps<1024, 2, 4>(ops, k, beta, st);
}

hipError_t launch_split_B_per_slice(int64_t n, int64_t p, const double* B, int64_t ldb, int k, int beta, int8_t* SB,
                                    int32_t* eB, double* rem, hipStream_t st)
{
    const int64_t Rpad = ozl::rows_padded(p), Npad = ozl::inner_padded(n);
    const int64_t stride = ozl::slice_bytes(p, n);
    hipLaunchKernelGGL(k_set_i32, dim3(1), dim3(1), 0, st,
                       reinterpret_cast<int32_t*>(SB + ozl::trailer_offset(p, n, k)), 0);
    uint32_t* keys = reinterpret_cast<uint32_t*>(eB);  // k arrays of p keys, decoded in place at the end
    const int64_t nk = (int64_t)k * p;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)((nk + 255) / 256)), dim3(256), 0, st, nk, keys, 0u);
    dim3 gmax((unsigned)((n + LCH - 1) / LCH), (unsigned)((p + 63) / 64));
    hipLaunchKernelGGL(k_colmax_B, gmax, dim3(256), 0, st, n, p, B, ldb, keys, LCH, 0u);
    dim3 grid((unsigned)(Npad / 128), (unsigned)(Rpad / 64));
    for (int s = 0; s < k; ++s)
        hipLaunchKernelGGL(k_split_B_ps, grid, dim3(256), 0, st, n, p, s == 0 ? B : rem, s == 0 ? ldb : p, beta,
                           SB + (int64_t)s * stride, keys + (int64_t)s * p,
                           s + 1 < k ? keys + (int64_t)(s + 1) * p : nullptr, rem, Npad);
    hipLaunchKernelGGL(k_decode_keys, dim3((unsigned)((nk + 255) / 256)), dim3(256), 0, st, nk, eB);
    return hipGetLastError();
}

template <int K>
static hipError_t launch_small_k(const SmallArgs* a, int k, hipStream_t st)
{
    if constexpr (K <= SMALL_MAX_K) {
        if (k != K) return launch_small_k<K + 1>(a, k, st);
        const void* kernel = reinterpret_cast<const void*>(&k_small<K>);
        if (!a) return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 2 * K * 4 * 1024);
        void* args[] = {const_cast<SmallArgs*>(a)};
        const dim3 grid((unsigned)((a->op[1].rows + 15) / 16), (unsigned)((a->op[0].rows + 15) / 16));
        // (the operands' slices, then the sums of four waves)
        return ozk::launch_status(hipLaunchKernel(kernel, grid, dim3(256), args, (a->steps > 2 ? 2 * a->steps : 4) * K * 1024, st));
    }
    return hipErrorInvalidValue;
}
hipError_t launch_small(const SmallArgs& a, int k, hipStream_t st) { return launch_small_k<SMALL_MIN_K>(&a, k, st); }
hipError_t setup_small()
{
    for (int k = SMALL_MIN_K; k <= SMALL_MAX_K; ++k) {
        const hipError_t e = launch_small_k<SMALL_MIN_K>(nullptr, k, nullptr);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_export(int64_t rows, int64_t n, int k, const int8_t* packed, int8_t* out, hipStream_t st)
{
    const int64_t Npad = ozl::inner_padded(n);
    const int64_t total = (int64_t)k * rows * n;
    if (total == 0) return hipSuccess;
    hipLaunchKernelGGL(k_export, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, rows, n, k, packed,
                       reinterpret_cast<const int32_t*>(packed + ozl::trailer_offset(rows, n, k)), out,
                       Npad / ozl::TILE_K, ozl::slice_bytes(rows, n));
    return hipGetLastError();
}

}  // namespace ozk
