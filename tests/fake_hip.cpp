// Stands in for the few HIP calls that a launch makes, for tests without a GPU: loaded ahead of the
// HIP runtime, it answers for as many devices as a test names, starts nothing, and notes what each
// launch asked for.  A CU holds 32 waves and 160 KB of LDS; a kernel has 64 KB until it is given more
// on the device it is launched on, as documented for the attribute.
#include <hip/hip_runtime.h>

#include <map>
#include <set>
#include <utility>

static int g_device = 0, g_queries = 0;
static unsigned g_grid, g_block, g_launches;
static size_t g_lds;
static hipError_t g_last = hipSuccess;
static std::set<std::pair<int, const void*>> g_raised;
static std::map<const void*, int> g_answers;   // of the last question about a kernel: its workgroups per CU
static int g_scarce = 0;                       // of every g_scarce kernels asked about, the last has one per CU
static unsigned g_resident;

extern "C" {
void fake_use(int device) { g_device = device; }
unsigned fake_grid() { return g_grid; }
unsigned fake_block() { return g_block; }
unsigned fake_lds() { return (unsigned)g_lds; }
unsigned fake_launches() { return g_launches; }
int fake_queries() { return g_queries; }
void fake_scarce(int every) { g_scarce = every; }
// What the device was said to keep of the kernel launched last; 0 if nobody asked about it.
unsigned fake_resident() { return g_resident; }

hipError_t hipGetDevice(int* dev) {
    *dev = g_device;
    return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int) {
    p->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* value, hipDeviceAttribute_t, int) {
    *value = 256;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* blocks, const void* kernel, int threads, size_t lds) {
    ++g_queries;
    const int by_waves = 32 / (threads / 64), by_lds = lds ? (int)(163840 / lds) : 32;
    *blocks = by_waves < by_lds ? by_waves : by_lds;
    if (g_scarce && !g_answers.count(kernel) && (int)g_answers.size() % g_scarce == g_scarce - 1) *blocks = 1;
    else if (g_scarce && g_answers.count(kernel)) *blocks = g_answers[kernel];
    g_answers[kernel] = *blocks;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* kernel, hipFuncAttribute, int) {
    g_raised.insert({g_device, kernel});
    return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t) {
    g_grid = grid.x;
    g_block = block.x;
    g_lds = lds;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
    *grid = dim3(g_grid);
    *block = dim3(g_block);
    *lds = g_lds;
    *stream = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* kernel, dim3, dim3, void**, size_t lds, hipStream_t) {
    if (lds > 65536 && !g_raised.count({g_device, kernel})) return g_last = hipErrorInvalidValue;
    ++g_launches;
    g_resident = g_answers.count(kernel) ? 256u * g_answers[kernel] : 0u;
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = g_last;
    g_last = hipSuccess;
    return e;
}
}
