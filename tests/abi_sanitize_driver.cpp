// Drives the host side of the C-ABI library without a GPU, for a build whose host pass carries
// AddressSanitizer + UndefinedBehaviorSanitizer (tests/test_sanitizers.py): the parameter formulas, the size
// functions over the whole admissible range (64-bit products of sizes), and every argument check.  No call
// below reaches a kernel launch: each fails validation first or has nothing to do.
#include "../include/ozimmu.h"
#include <cstdio>
#include <cstdlib>

#define EXPECT(call, want)                                                                    \
    do {                                                                                      \
        const long long got_ = (long long)(call);                                             \
        if (got_ != (long long)(want)) {                                                      \
            std::printf("line %d: %s = %lld, expected %lld\n", __LINE__, #call, got_, (long long)(want)); \
            ++failures;                                                                       \
        }                                                                                     \
    } while (0)

int main()
{
    int failures = 0;
    const int64_t top = ((int64_t)1 << 22) - 256, inner_max = (int64_t)1 << 29;
    void* fake = reinterpret_cast<void*>(4096);  // never dereferenced
    double* fd = static_cast<double*>(fake);
    int8_t* f8 = static_cast<int8_t*>(fake);
    int32_t* f32 = static_cast<int32_t*>(fake);

    for (int64_t n = 1; n <= inner_max; n = n * 2 + ((n & 1) ? 0 : 1)) {
        int beta = 0;
        int64_t r = 0;
        EXPECT(ozimmu_params(n, &beta, &r), OZIMMU_OK);
        if (beta < 1 || beta > 7 || r < 1) ++failures;
        for (int k = 1; k <= OZIMMU_MAX_SLICES; ++k)
            if (ozimmu_num_chunks(n, k) < k) ++failures;
        if (ozimmu_r_wide(n) < r) ++failures;
    }
    EXPECT(ozimmu_params(0, nullptr, nullptr), OZIMMU_ERR_DIM);
    EXPECT(ozimmu_params(inner_max + 1, nullptr, nullptr), OZIMMU_ERR_DIM);
    // the size functions at the corners of the admissible range (no overflow in their 64-bit arithmetic)
    const int64_t sizes[] = {0, 1, 255, 256, 257, 65536, top};
    for (int64_t m : sizes)
        for (int64_t p : sizes)
            for (int64_t n : {(int64_t)0, (int64_t)1, (int64_t)300, inner_max})
                for (int k : {1, 8, OZIMMU_MAX_SLICES}) {
                    const size_t w = ozimmu_workspace_bytes(m, n, p, k);
                    if (ozimmu_workspace_bytes_ex(m, n, p, k) < w) ++failures;
                    for (int mode = 0; mode < 3; ++mode)
                        if (ozimmu_workspace_bytes_variant(m, n, p, k, mode) < (mode == 2 ? 0 : w)) ++failures;
                    (void)ozimmu_slices_bytes(m, n, k);
                    (void)ozimmu_remainder_bytes(m, n, 0);
                    (void)ozimmu_remainder_bytes(p, n, 1);
                }
    EXPECT(ozimmu_workspace_bytes(-1, 1, 1, 1), 0);
    for (int s = 1; s >= -6; --s)
        if (!ozimmu_status_string(s)) ++failures;

    // argument checks of every entry point
    EXPECT(ozimmu_dgemm(-1, 4, 4, fd, 4, fd, 4, fd, 4, 8, fake, 1 << 30, nullptr), OZIMMU_ERR_DIM);
    EXPECT(ozimmu_dgemm(4, 4, 4, fd, 3, fd, 4, fd, 4, 8, fake, 1 << 30, nullptr), OZIMMU_ERR_DIM);
    EXPECT(ozimmu_dgemm(4, 4, 4, fd, (int64_t)1 << 30, fd, 4, fd, 4, 8, fake, 1 << 30, nullptr), OZIMMU_ERR_DIM);
    EXPECT(ozimmu_dgemm(top + 1, 4, 4, fd, 4, fd, 4, fd, 4, 8, fake, 1 << 30, nullptr), OZIMMU_ERR_DIM);
    EXPECT(ozimmu_dgemm(4, inner_max + 1, 4, fd, inner_max + 1, fd, 4, fd, 4, 8, fake, 1 << 30, nullptr), OZIMMU_ERR_DIM);
    EXPECT(ozimmu_dgemm(4, 4, 4, fd, 4, fd, 4, fd, 4, 0, fake, 1 << 30, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_dgemm(4, 4, 4, fd, 4, fd, 4, fd, 4, 21, fake, 1 << 30, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_dgemm(4, 4, 4, nullptr, 4, fd, 4, fd, 4, 8, fake, 1 << 30, nullptr), OZIMMU_ERR_NULL);
    EXPECT(ozimmu_dgemm(4, 4, 4, fd, 4, fd, 4, fd, 4, 8, fake, 16, nullptr), OZIMMU_ERR_WORKSPACE);
    EXPECT(ozimmu_dgemm(4, 4, 4, fd, 4, fd, 4, fd, 4, 8, reinterpret_cast<void*>(4097), (size_t)1 << 30, nullptr),
           OZIMMU_ERR_WORKSPACE);
    EXPECT(ozimmu_dgemm(0, 4, 4, nullptr, 4, nullptr, 4, nullptr, 4, 8, nullptr, 0, nullptr), OZIMMU_OK);
    EXPECT(ozimmu_dgemm(top, inner_max, top, fd, inner_max, fd, top, fd, top, 20, fake, 16, nullptr), OZIMMU_ERR_WORKSPACE);
    EXPECT(ozimmu_dgemm_variant(4, 4, 4, fd, 4, fd, 4, fd, 4, 8, 3, 0, fake, 1 << 30, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_dgemm_variant(4, 4, 4, fd, 4, fd, 4, fd, 4, 8, 0, 3, fake, 1 << 30, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_dgemm_variant(4, 4, 4, fd, 4, fd, 4, fd, 4, 8, 1, OZIMMU_ACCUM_WIDE, fake, 1 << 30, nullptr),
           OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_dgemm_variant(4, 4, 4, fd, 4, fd, 4, fd, 4, 8, 2, OZIMMU_ACCUM_GROUPED, fake, 1 << 30, nullptr),
           OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_dgemm_variant(4, 4, 4, fd, 4, fd, 4, fd, 4, 8, 0, 0x300, fake, 1 << 30, nullptr), OZIMMU_ERR_SLICES);
    for (int k = 0; k <= 21; ++k)
        for (int tile = -1; tile <= OZIMMU_RESIDENT_TILES; ++tile)
            for (int64_t n : {(int64_t)0, (int64_t)1, (int64_t)8200, (int64_t)40000, inner_max, inner_max + 1}) {
                int rows = 0, cols = 0;
                const int st = ozimmu_resident_tile(n, k, OZIMMU_ACCUM_GROUPED, tile, &rows, &cols);
                EXPECT(st == OZIMMU_OK ? (rows >= 32 && rows <= 128 && cols >= 32 && cols <= 128) : rows == 0, 1);
                EXPECT(st != OZIMMU_OK || (k >= 3 && k <= 16 && tile >= 0 && tile < OZIMMU_RESIDENT_TILES && n >= 1 && n <= inner_max), 1);
            }
    EXPECT(ozimmu_resident_tile(64, 8, 3, 0, nullptr, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_resident_tile(64, 8, 0, 0, nullptr, nullptr), OZIMMU_OK);
    EXPECT(ozimmu_dgemm_resident(4, 4, 4, fd, 4, fd, 4, fd, 4, 2, 0, 0, 0, fake, 1 << 30, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_dgemm_resident(4, 4, 4, fd, 4, fd, 4, fd, 4, 8, 2, 1, 0, fake, 1 << 30, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_dgemm_resident(4, inner_max, 4, fd, inner_max, fd, 4, fd, 4, 8, 0, 1, 0, fake, 1 << 30, nullptr), OZIMMU_ERR_DIM);
    EXPECT(ozimmu_dgemm_resident(4, 4, 4, fd, 3, fd, 4, fd, 4, 8, 0, 0, 0, fake, 1 << 30, nullptr), OZIMMU_ERR_DIM);
    EXPECT(ozimmu_dgemm_resident(4, 4, 4, fd, 4, fd, 4, fd, 4, 8, 0, 0, 0, fake, 16, nullptr), OZIMMU_ERR_WORKSPACE);
    // forced parts: one scale per slice is never cut, parts of less than two steps, tiles that are not cut, room for the sums
    EXPECT(ozimmu_dgemm_tile(4, 4096, 4, fd, 4096, fd, 4, fd, 4, 8, 2, 1, 0, 2, fake, 1 << 30, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_dgemm_tile(4, 4096, 4, fd, 4096, fd, 4, fd, 4, 8, 2, 0, 5, 1, fake, 1 << 30, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_dgemm_tile(4, 4096, 4, fd, 4096, fd, 4, fd, 4, 8, 0, 0, 5, 33, fake, 1 << 30, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_dgemm_tile(4, 4096, 4, fd, 4096, fd, 4, fd, 4, 8, 0, 0, 5, 0, fake, 1 << 30, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_dgemm_tile(4, 4096, 4, fd, 4096, fd, 4, fd, 4, 8, 0, 0, 0, 2, fake, 1 << 30, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_dgemm_tile(4, 4096, 4, fd, 4096, fd, 4, fd, 4, 8, 1, OZIMMU_ACCUM_WIDE, 5, 2, fake, 1 << 30, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_dgemm_tile(4, 4096, 4, fd, 4096, fd, 4, fd, 4, 8, 0, 0, 5, 2, fake, 16, nullptr), OZIMMU_ERR_WORKSPACE);
    EXPECT(ozimmu_dgemm_tile(200000, 4096, 400, fd, 4096, fd, 400, fd, 400, 8, 0, 0, 5, 2, fake, 1 << 30, nullptr), OZIMMU_ERR_WORKSPACE);
    EXPECT(ozimmu_dgemm_tile(top, 4096, 400, fd, 4096, fd, 400, fd, 400, 8, 0, 0, 5, 2, fake, 1 << 30, nullptr), OZIMMU_ERR_DIM);
    EXPECT(ozimmu_dgemm_tile(4, 4, 4, fd, 4, fd, 4, fd, 4, 2, 0, 0, 0, 1, fake, 1 << 30, nullptr), OZIMMU_ERR_SLICES);
    // the choice, over the admissible range
    ozimmu_choice choice;
    for (int64_t m : sizes)
        for (int64_t p : sizes)
            for (int64_t n : {(int64_t)0, (int64_t)1, (int64_t)300, (int64_t)20000, inner_max})
                for (int k = 1; k <= OZIMMU_MAX_SLICES; ++k)
                    for (int mode = 0; mode < 3; ++mode)
                        for (size_t bytes : {(size_t)0, ozimmu_workspace_bytes_min(m, n, p, k), ozimmu_workspace_bytes(m, n, p, k)}) {
                            const int accumulate = mode == 2 ? OZIMMU_ACCUM_PER_PAIR : OZIMMU_ACCUM_GROUPED;
                            const int st = ozimmu_choose(m, n, p, k, mode, accumulate, bytes, 256, &choice);
                            EXPECT(st, m && n && p ? OZIMMU_OK : OZIMMU_ERR_DIM);
                            for (int trans = 0; trans < 4; ++trans) {
                                const int split = ozimmu_split_way(trans & 1, trans >> 1, m, n, p, k, bytes);
                                EXPECT(m && n && p ? split >= OZIMMU_SPLIT_WAY_WHOLE : split == OZIMMU_ERR_DIM, 1);
                                if (trans == 0 && st == OZIMMU_OK && mode < 2 && choice.way != OZIMMU_WAY_SMALL) EXPECT(split, choice.split_way);
                            }
                            if (st != OZIMMU_OK) continue;
                            EXPECT(choice.way == OZIMMU_WAY_RESIDENT ? choice.tile >= 0 && choice.parts >= 1 : choice.tile == -1, 1);
                            EXPECT(choice.parts > 1 && (mode == 2 || 2 * choice.parts > (n + 63) / 64), 0);
                        }
    EXPECT(ozimmu_choose(4, 4, 4, 8, 0, 0, 0, 256, nullptr), OZIMMU_ERR_NULL);
    EXPECT(ozimmu_choose(4, 4, 4, 8, 3, 0, 0, 256, &choice), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_choose(4, 4, 4, 8, 0, 0, 0, 0, &choice), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_split_way(0, 0, 4, 4, 4, 0, 0), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_gemm_ex(0, 0, 4, 4, 4, 1.0, fd, 3, fd, 4, 0.0, fd, 4, 8, fake, 1 << 30, nullptr), OZIMMU_ERR_DIM);
    EXPECT(ozimmu_gemm_ex(1, 0, 5, 4, 4, 1.0, fd, 4, fd, 4, 0.0, fd, 4, 8, fake, 1 << 30, nullptr), OZIMMU_ERR_DIM);
    EXPECT(ozimmu_gemm_ex(0, 1, 4, 5, 4, 1.0, fd, 5, fd, 4, 0.0, fd, 4, 8, fake, 1 << 30, nullptr), OZIMMU_ERR_DIM);
    EXPECT(ozimmu_gemm_ex(0, 0, 4, 4, 4, 1.0, fd, 4, fd, 4, 0.0, nullptr, 4, 8, fake, 1 << 30, nullptr), OZIMMU_ERR_NULL);
    EXPECT(ozimmu_gemm_ex(0, 0, 4, 4, 4, 1.0, fd, 4, fd, 4, 0.5, fd, 4, 8, fake, 16, nullptr), OZIMMU_ERR_WORKSPACE);
    EXPECT(ozimmu_split_A(4, 4, fd, 3, 8, f8, f32, nullptr), OZIMMU_ERR_DIM);
    EXPECT(ozimmu_split_A(4, 4, fd, 4, 8, reinterpret_cast<int8_t*>(4097), f32, nullptr), OZIMMU_ERR_WORKSPACE);
    EXPECT(ozimmu_split_A(4, 4, nullptr, 4, 8, f8, f32, nullptr), OZIMMU_ERR_NULL);
    EXPECT(ozimmu_split_B(4, top + 1, fd, top + 1, 8, f8, f32, nullptr), OZIMMU_ERR_DIM);
    EXPECT(ozimmu_split_B(4, 4, fd, 4, 0, f8, f32, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_split_A_variant(4, 4, fd, 4, 8, 2, f8, f32, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_split_B_variant(4, 4, fd, 4, 8, -1, f8, f32, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_split_A_per_slice(4, 4, fd, 4, 8, f8, f32, nullptr, nullptr), OZIMMU_ERR_NULL);
    EXPECT(ozimmu_split_B_per_slice(4, 4, fd, 4, 8, f8, f32, reinterpret_cast<double*>(4104), nullptr),
           OZIMMU_ERR_WORKSPACE);
    EXPECT(ozimmu_gemm_group(4, 4, 4, f8, 2, f8, 2, 5, 1, 1, f32, 4, fake, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_gemm_group(4, 4, 4, f8, 2, f8, 2, 3, 2, 1, f32, 4, fake, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_gemm_group(4, 4, 4, f8, 2, f8, 2, 3, 1, 2, f32, 3, fake, nullptr), OZIMMU_ERR_DIM);
    EXPECT(ozimmu_gemm_group(4, 4, 4, f8, 2, f8, 2, 3, 1, 2, nullptr, 4, fake, nullptr), OZIMMU_ERR_NULL);
    EXPECT(ozimmu_gemm_group(4, 4, 4, f8, 2, f8, 2, 3, 1, 2, f32, 4, reinterpret_cast<void*>(4098), nullptr),
           OZIMMU_ERR_WORKSPACE);
    EXPECT(ozimmu_gemm_group_accumulate(4, 4, 4, f8, 2, f8, 2, 3, 1, 2, f32, f32, 1, fd, 3, fake, nullptr), OZIMMU_ERR_DIM);
    EXPECT(ozimmu_gemm_group_accumulate(4, 4, 4, f8, 2, f8, 2, 3, 1, 2, nullptr, f32, 1, fd, 4, fake, nullptr),
           OZIMMU_ERR_NULL);
    EXPECT(ozimmu_accumulate(4, 4, f32, 4, f32, f32, 0, 2, 1, fd, 4, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_accumulate(4, 4, f32, 4, f32, f32, 7, 1, 1, fd, 4, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_accumulate(4, 4, nullptr, 4, f32, f32, 7, 2, 1, fd, 4, nullptr), OZIMMU_ERR_NULL);
    EXPECT(ozimmu_export_slices(4, 4, 0, f8, f8, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_export_slices(4, 4, 2, nullptr, f8, nullptr), OZIMMU_ERR_NULL);
    EXPECT(ozimmu_dgemm_static(4096, 4096, 4096, fd, 4096, fd, 4096, fd, 4096, 8, nullptr), OZIMMU_ERR_WORKSPACE);
    EXPECT(ozimmu_dgemm_static(4, 4, 4, fd, 4, fd, 4, fd, 4, 21, nullptr), OZIMMU_ERR_SLICES);
    EXPECT(ozimmu_dgemm_static(0, 4, 4, nullptr, 4, nullptr, 4, nullptr, 4, 8, nullptr), OZIMMU_OK);

    if (failures) {
        std::printf("abi sanitize driver: %d failure(s)\n", failures);
        return 1;
    }
    std::printf("abi sanitize driver ok\n");
    return 0;
}
