// A HIP runtime that only writes down which kernels were launched, as a shared library: loaded in front of libagattn.so it
// answers the library's calls in place of the real one, so that a test without a GPU sees which kernel a call takes and with how
// many workgroups.  TEST INFRASTRUCTURE ONLY: nothing is run.  A stream handle of n stands for a stream of n CUs, NULL for all.
#include <cxxabi.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>

struct dim3 { uint32_t x, y, z; };

namespace {
std::map<const void*, std::string>& names() { static std::map<const void*, std::string> n; return n; }
std::string& log_text() { static std::string l; return l; }
struct { dim3 grid, block; size_t lds; void* stream; } pushed;
int cus = 256;
}  // namespace

extern "C" {
void launch_log_cus(int n) { cus = n; }
// the launches since the last call, one "kernel<arguments> workgroups" a line
const char* launch_log_take()
{
    static std::string out;
    out.swap(log_text());
    log_text().clear();
    return out.c_str();
}

void** __hipRegisterFatBinary(const void*) { static void* module; return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    std::string s = name;
    for (size_t at; (at = s.find("DF16b")) != std::string::npos;) s.replace(at, 5, "6__bf16");       // (older demanglers do not know the type)
    int st = 0;
    char* d = abi::__cxa_demangle(s.c_str(), nullptr, nullptr, &st);
    if (d) s = d;
    free(d);
    const std::string space = "(anonymous namespace)::";
    for (size_t at; (at = s.find(space)) != std::string::npos;) s.erase(at, space.size());
    const size_t paren = s.find('(');
    if (paren != std::string::npos) s.erase(paren);
    if (s.compare(0, 5, "void ") == 0) s.erase(0, 5);
    for (size_t at; (at = s.find("ag::")) != std::string::npos;) s.erase(at, 4);
    for (size_t at; (at = s.find(' ')) != std::string::npos;) s.erase(at, 1);
    names()[host] = s;
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream) { pushed = {grid, block, lds, stream}; return 0; }
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream)
{
    *grid = pushed.grid, *block = pushed.block, *lds = pushed.lds, *stream = pushed.stream;
    return 0;
}
int hipLaunchKernel(const void* f, dim3 grid, dim3, void**, size_t, void*)
{
    log_text() += names()[f] + " " + std::to_string(grid.x) + "\n";
    return 0;
}
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "no device"; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipDeviceGetAttribute(int* v, int, int) { *v = cus; return 0; }
int hipExtStreamGetCUMask(void* stream, uint32_t words, uint32_t* mask)
{
    memset(mask, 0, 4 * words);
    for (int i = 0; i < (stream ? (int)(intptr_t)stream : cus); ++i) mask[i / 32] |= 1u << (i % 32);
    return 0;
}
int hipGetSymbolAddress(void** p, const void*) { *p = (void*)4096; return 0; }
// not part of a launch
int hipEventCreate(void**) { return 1; }
int hipEventCreateWithFlags(void**, unsigned) { return 1; }
int hipEventDestroy(void*) { return 1; }
int hipEventElapsedTime(float*, void*, void*) { return 1; }
int hipEventQuery(void*) { return 1; }
int hipEventRecord(void*, void*) { return 1; }
int hipEventSynchronize(void*) { return 1; }
int hipExtStreamCreateWithCUMask(void**, uint32_t, const uint32_t*) { return 1; }
int hipGetDevicePropertiesR0600(void*, int) { return 1; }
int hipMemcpy(void*, const void*, size_t, int) { return 1; }
int hipStreamDestroy(void*) { return 1; }
int hipStreamSynchronize(void*) { return 1; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 1; }
}
