// A stand-in for the few runtime entries that the library launches through, loaded ahead of the runtime: launches are written
// down and not made, so what a call would launch can be read on a machine without a GPU.
#include <cxxabi.h>
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <map>
#include <string>

namespace {
std::map<const void*, std::string>& names()
{
    static std::map<const void*, std::string> m;      // (kernels are registered by constructors)
    return m;
}
std::string log_text;
struct { dim3 grid, block; size_t lds; hipStream_t stream; } config;

void note(const char* what, const void* kernel, size_t grid, size_t bytes)
{
    log_text += std::string(what) + "\t" + names()[kernel] + "\t" + std::to_string(grid) + "\t" + std::to_string(bytes) + "\n";
}
}  // namespace

extern "C" {
const char* launch_log() { return log_text.c_str(); }
void launch_log_clear() { log_text.clear(); }

void __hipRegisterFunction(void*, const void* host, char*, const char* device, unsigned, void*, void*, void*, void*, int*)
{
    int status;
    char* plain = abi::__cxa_demangle(device, nullptr, nullptr, &status);
    names()[host] = plain ? plain : device;
    free(plain);
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream)
{
    config = {grid, block, lds, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream)
{
    *grid = config.grid;
    *block = config.block;
    *lds = config.lds;
    *stream = config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* kernel, dim3 grid, dim3, void**, size_t lds, hipStream_t)
{
    note("launch", kernel, (size_t)grid.x * grid.y * grid.z, lds);
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* kernel, hipFuncAttribute, int bytes)
{
    note("allow", kernel, 0, (size_t)bytes);
    return hipSuccess;
}
hipError_t hipGetDevice(int* device)
{
    *device = 0;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
}
