// Readback of small pieces of device state: one kernel gathers what a host call
// asks for (a discharge's state, its counters, a profile) and writes it to
// pinned host memory, in stream order, so a call costs one launch and one wait.
// Bound by those two latencies: 11 us a call, where the same pieces took 35-50 us
// as three to five synchronous copies through the runtime's staging.
#include "pic_internal.h"
#include "pic_kernels.h"

#include <algorithm>

namespace pic {

namespace {

constexpr int kRT = 256;

__global__ __launch_bounds__(kRT) void read_kernel(ReadArgs a)
{
    const uint32_t total = a.first[a.n];
    for (uint32_t i = blockIdx.x * kRT + threadIdx.x; i < total; i += gridDim.x * kRT) {
        int e = 0;
        while (i >= a.first[e + 1]) ++e;
        a.dst[i] = a.src[e][i - a.first[e]];
    }
}

}  // namespace

// by the launch's own status: an error that some other call of the program has
// left behind is not this one's
hipError_t launch_read(const ReadArgs& a, hipStream_t st)
{
    const unsigned grid = std::max(1u, std::min((a.first[a.n] + kRT - 1) / kRT, 64u));
    ReadArgs copy = a;
    void* args[] = {&copy};
    return hipLaunchKernel(reinterpret_cast<const void*>(read_kernel), dim3(grid), dim3(kRT), args, 0, st);
}

}  // namespace pic
