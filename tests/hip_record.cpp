// Host-side stand-in for the HIP runtime calls that libacm makes, for tests on
// a machine without a GPU: device memory is host memory, kernels are recorded
// (name, grid, integer arguments) instead of run, and a chosen launch can be
// made to fail.  Loaded with RTLD_GLOBAL before libacm.so, so that its
// definitions come first.
#include <cstddef>
#include <cstdint>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Dim3 {
    uint32_t x, y, z;
};
struct Launch {
    std::string name;
    Dim3 grid;
    int args[3];
};
std::map<const void*, std::string> kernels;
std::vector<Launch> launches;
long fail_in = -1;  // launches until one fails (-1: none does)
int last_error = 0;
Dim3 cfg_grid, cfg_block;
char dummy[256];
constexpr int FAILURE = 719;  // hipErrorLaunchFailure

// integers after (coefficients, in, out) of the march kernels
int int_args(const std::string& n)
{
    if (n.find("march3d_kernel") != std::string::npos) return 3;
    if (n.find("march2d_kernel") != std::string::npos || n.find("twophase_march_kernel") != std::string::npos) return 2;
    return 0;
}
}  // namespace

extern "C" {
void rec_reset(long fail) { launches.clear(), fail_in = fail, last_error = 0; }
long rec_count() { return (long)launches.size(); }
const char* rec_name(long i) { return launches[i].name.c_str(); }
int rec_grid(long i) { return (int)launches[i].grid.x; }
int rec_arg(long i, int k) { return launches[i].args[k]; }

void** __hipRegisterFatBinary(const void*) { return reinterpret_cast<void**>(dummy); }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    kernels[host] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t, void*)
{
    cfg_grid = grid, cfg_block = block;
    return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* shmem, void** stream)
{
    *grid = cfg_grid, *block = cfg_block, *shmem = 0, *stream = nullptr;
    return 0;
}
int hipLaunchKernel(const void* f, Dim3 grid, Dim3, void** args, size_t, void*)
{
    if (fail_in == 0) return last_error = FAILURE;
    if (fail_in > 0) --fail_in;
    Launch l{kernels[f], grid, {0, 0, 0}};
    for (int k = 0; k < int_args(l.name); ++k) l.args[k] = *static_cast<int*>(args[3 + k]);
    launches.push_back(l);
    return 0;
}
int hipGetLastError()
{
    const int e = last_error;
    last_error = 0;
    return e;
}
const char* hipGetErrorString(int) { return "recorded error"; }
int hipGetDevice(int* d) { return *d = 0; }
int hipDeviceGetAttribute(int* v, int, int)
{
    *v = 256;  // compute units
    return 0;
}
int hipGetSymbolAddress(void** p, const void*)
{
    *p = dummy;
    return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t)
{
    *n = 2;
    return 0;
}
int hipStreamCreateWithFlags(void** s, unsigned)
{
    *s = dummy;
    return 0;
}
int hipStreamDestroy(void*) { return 0; }
int hipStreamSynchronize(void*) { return 0; }
int hipStreamBeginCapture(void*, int) { return 0; }
int hipStreamEndCapture(void*, void** g)
{
    *g = dummy;
    return 0;
}
int hipGraphInstantiate(void** e, void*, void**, char*, size_t)
{
    *e = dummy;
    return 0;
}
int hipGraphLaunch(void*, void*) { return 0; }
int hipGraphDestroy(void*) { return 0; }
int hipGraphExecDestroy(void*) { return 0; }
int hipEventCreate(void** e)
{
    *e = dummy;
    return 0;
}
int hipEventDestroy(void*) { return 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipEventElapsedTime(float* ms, void*, void*)
{
    *ms = 1.f;
    return 0;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int, void*)
{
    std::memcpy(d, s, n);
    return 0;
}
int hipMemsetAsync(void* d, int v, size_t n, void*)
{
    std::memset(d, v, n);
    return 0;
}
}
