// A stand-in for the part of the HIP runtime that librr.so calls on the host,
// preloaded by stream_memory_calls.py and loglik_plan_calls.py on a machine
// without a GPU: memory comes from malloc, kernels are not run, and every
// allocation, release and launch is recorded with its stream in call order.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <new>
#include <vector>

namespace {
struct Event { char op; hipStream_t stream; void* ptr; long blocks = 0, lds = 0; };
std::vector<Event> g_log;
char g_symbol[1 << 22];
dim3 g_grid, g_block;                    // of the launch being made
size_t g_lds;
hipStream_t g_stream;
bool g_no_memory = false;                // operator new throws
hipError_t allocate(char op, void** p, size_t n, hipStream_t s) {
    *p = std::malloc(n);
    g_log.push_back({op, s, *p});
    return hipSuccess;
}
}  // namespace

void* operator new(std::size_t n) {
    void* p = g_no_memory ? nullptr : std::malloc(n);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

extern "C" {
void recorder_no_memory(int on) {
    g_log.reserve(g_log.size() + 64);    // what is recorded meanwhile has its place
    g_no_memory = on != 0;
}
int recorder_size() { return int(g_log.size()); }
void recorder_get(int i, char* op, void** stream, void** ptr) {
    *op = g_log[size_t(i)].op;
    *stream = g_log[size_t(i)].stream;
    *ptr = g_log[size_t(i)].ptr;
}

void recorder_launch(int i, long* blocks, long* lds) {
    *blocks = g_log[size_t(i)].blocks;
    *lds = g_log[size_t(i)].lds;
}

hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 160 << 10;
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) {
    *n = 8;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = g_symbol; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { return allocate('M', p, n, nullptr); }
hipError_t hipFree(void* p) { g_log.push_back({'F', nullptr, p}); return hipSuccess; }
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t s) { return allocate('m', p, n, s); }
hipError_t hipFreeAsync(void* p, hipStream_t s) { g_log.push_back({'f', s, p}); return hipSuccess; }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t) {
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = reinterpret_cast<hipStream_t>(0x100);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) {
    *c = hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
    g_grid = grid;
    g_block = block;
    g_lds = lds;
    g_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
    *grid = g_grid;
    *block = g_block;
    *lds = g_lds;
    *s = g_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3 grid, dim3, void**, size_t lds, hipStream_t s) {
    g_log.push_back({'L', s, nullptr, long(grid.x) * grid.y * grid.z, long(lds)});
    return hipSuccess;
}
}
