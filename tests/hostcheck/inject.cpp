// With hipstub.cpp (compiled with -DhipLaunchKernel=stub_hipLaunchKernel
// -DhipEventSynchronize=stub_hipEventSynchronize): launches are recorded, and an
// event wait can be made to fail.
#include <hip/hip_runtime_api.h>

extern "C" {
hipError_t stub_hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t);
hipError_t stub_hipEventSynchronize(hipEvent_t);

static const void* last_fn[2];
static unsigned last_grid[2];
static int waits_until_failure = -1;

hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t n, hipStream_t s) {
    last_fn[0] = last_fn[1];
    last_grid[0] = last_grid[1];
    last_fn[1] = f;
    last_grid[1] = g.x;
    return stub_hipLaunchKernel(f, g, b, args, n, s);
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    if (waits_until_failure == 0) return hipErrorUnknown;
    if (waits_until_failure > 0) --waits_until_failure;
    return stub_hipEventSynchronize(e);
}
// which = 1: the last launch, 0: the one before it
const void* inject_launch_fn(int which) { return last_fn[which]; }
unsigned inject_launch_grid(int which) { return last_grid[which]; }
// Event waits succeed `waits` more times, then fail (negative: never).
void inject_failing_wait(int waits) { waits_until_failure = waits; }
}
