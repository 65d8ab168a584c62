// Stands in for the HIP runtime's launch call, so that a test without a GPU sees what the library would
// launch: grid, block, the first pointer of the kernel's argument block, and the kernel.  Loaded into the global scope
// before the library.
#include <hip/hip_runtime_api.h>

namespace {
struct Launch {
    unsigned grid_x, grid_y, block_x, reserved;
    const void *first, *kernel;
};
constexpr int kMax = 4096;
Launch g_launches[kMax];
int g_count, g_refuse_at = -1;
}  // namespace

extern "C" {

hipError_t hipLaunchKernel(const void *kernel, dim3 grid, dim3 block, void **args, size_t, hipStream_t) {
    // the runtime refuses a grid of 2^32 threads and more
    if (g_count == g_refuse_at || (unsigned long long)grid.x * block.x >> 32) return hipErrorInvalidConfiguration;
    if (g_count < kMax) g_launches[g_count] = Launch{grid.x, grid.y, block.x, 0, *static_cast<const void *const *>(args[0]), kernel};
    ++g_count;
    return hipSuccess;
}

hipError_t hipGetDevice(int *device) {
    *device = 0;
    return hipSuccess;
}

hipError_t hipDeviceGetAttribute(int *value, hipDeviceAttribute_t, int) {
    *value = 160 * 1024;    // LDS of a compute unit
    return hipSuccess;
}

int recorded(const Launch **launches) {
    *launches = g_launches;
    return g_count;
}

void record_anew(int refuse_at) {
    g_count = 0;
    g_refuse_at = refuse_at;
}
}
