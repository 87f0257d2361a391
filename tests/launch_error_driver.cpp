// A launch that fails is reported by the launcher and by nobody after it (tests/test_launch_errors.py).  The runtime's launch is
// replaced by one that fails, so this runs the launchers' error path and nothing on a GPU.
#include "../paper_2409_13313_amd/csrc/ozimmu_kernels.h"
#include <cstdio>

static hipError_t last_error = hipSuccess;

extern "C" hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t)
{
    return last_error = hipErrorLaunchOutOfResources;
}
// (what a launch in triple brackets goes through first; without a GPU the runtime's own fail before they come to it)
extern "C" hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
extern "C" hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
extern "C" hipError_t hipGetLastError(void)
{
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}

int main()
{
    int failures = 0;
    auto expect = [&](const char* what, hipError_t e) {
        const hipError_t left = hipGetLastError();
        if (e != hipErrorLaunchOutOfResources || left != hipSuccess) {
            std::printf("%s: returned %d, left %d behind\n", what, (int)e, (int)left);
            ++failures;
        }
    };
    ozk::SmallArgs small{};
    small.op[0].rows = small.op[1].rows = 16;
    small.n = 64;
    small.steps = 1;
    small.beta = 7;
    for (int k = ozk::SMALL_MIN_K; k <= ozk::SMALL_MAX_K; ++k) expect("launch_small", ozk::launch_small(small, k, nullptr));
    ozk::ResidentArgs a{};
    a.m = a.p = 32;
    a.steps = 4;
    for (int k = 3; k <= 16; ++k)
        for (int parts = 1; parts <= 2; ++parts) {
            a.parts = parts;
            expect("launch_resident", ozk::launch_resident(a, k, k, 5, nullptr));
        }
    a.parts = 1;
    a.per_slice = 1;
    expect("launch_resident, one scale per slice", ozk::launch_resident(a, 5, 1, 5, nullptr));
    // the split: whole vectors, the same of a few, both operands in two launches, columns cut beside rows and columns alone (several launches)
    const struct { int64_t m, n, p; int a_by_col, room, way; } splits[] = {{300, 600, 300, 0, 0, 0}, {4, 600, 4, 0, 0, 0},
                                                                           {47, 11948, 48, 0, 1, 1}, {523, 31111, 815, 0, 0, 2}, {256, 40001, 700, 1, 0, 2}};
    for (const auto& s : splits)
        for (int mode = 0; mode < 2; ++mode) {
            ozk::SplitIn ops[2] = {};                   // (nothing is dereferenced: the launches fail)
            ops[0].rows = s.m, ops[0].ld = s.a_by_col ? s.m : s.n, ops[0].by_col = s.a_by_col;
            ops[1].rows = ops[1].ld = s.p, ops[1].by_col = 1;
            ops[0].n = ops[1].n = s.n;
            static char room[1 << 20];
            if (ozk::split_cut(ops, 2, 8, s.room ? sizeof(room) : 0, s.room != 0) != s.way) {
                std::printf("split of %d x %d x %d: another way\n", (int)s.m, (int)s.n, (int)s.p);
                ++failures;
            }
            expect("launch_split", ozk::launch_split(ops, 2, 8, 7, mode, nullptr, nullptr, 0, s.room ? room : nullptr, s.room ? sizeof(room) : 0));
        }
    if (!failures) std::printf("launch error driver ok\n");
    return failures != 0;
}
