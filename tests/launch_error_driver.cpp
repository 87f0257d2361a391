// A launch that fails is reported by the launcher and by nobody after it (tests/test_launch_errors.py).  The runtime's launch is
// replaced by one that fails, so this runs the launchers' error path and nothing on a GPU.
#include "../paper_2409_13313_amd/csrc/ozimmu_kernels.h"
#include <cstdio>

static hipError_t last_error = hipSuccess;

extern "C" hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t)
{
    return last_error = hipErrorLaunchOutOfResources;
}
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
    if (!failures) std::printf("launch error driver ok\n");
    return failures != 0;
}
