// A HIP runtime that launches nothing (test infrastructure): linked with the library's own objects it records which kernel
// every call would have launched, with its grid, workgroup and LDS size, so that dispatch rules can be checked without a GPU.
#include <cxxabi.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
struct Dim { uint32_t x, y, z; };
struct Config { Dim grid, block; size_t lds; void* stream; };
std::map<const void*, std::string>& names() { static std::map<const void*, std::string> m; return m; }
// a demangled name without return type, namespaces and parameters
std::string plain(std::string k) {
    for (const char* drop : {"void ", "bimask::", "(anonymous namespace)::"})
        for (size_t at; (at = k.find(drop)) != std::string::npos;) k.erase(at, std::strlen(drop));
    k.resize(k.find('('));
    return k;
}
Config pending;
std::string record;                                      // one line per launch
bool refuse_lds = false;
char device_array[16];
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* handle; return &handle; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* device_name, unsigned, void*, void*, void*, void*, int*) {
    int status = 0;
    char* d = abi::__cxa_demangle(device_name, nullptr, nullptr, &status);
    names()[host] = status == 0 ? d : device_name;
    std::free(d);
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim grid, Dim block, size_t lds, void* stream) { pending = {grid, block, lds, stream}; return 0; }
int __hipPopCallConfiguration(Dim* grid, Dim* block, size_t* lds, void** stream) {
    *grid = pending.grid; *block = pending.block; *lds = pending.lds; *stream = pending.stream;
    return 0;
}
int hipLaunchKernel(const void* f, Dim grid, Dim block, void**, size_t lds, void*) {
    const std::string k = plain(names()[f]);
    char line[160];
    std::snprintf(line, sizeof line, "|%u,%u,%u|%u|%zu\n", grid.x, grid.y, grid.z, block.x * block.y * block.z, lds);
    record += k + line;
    return 0;
}
int hipFuncSetAttribute(const void*, int, int) { return refuse_lds ? 1 : 0; }
int hipGetDevice(int* d) { *d = refuse_lds ? 1 : 0; return 0; }       // (what was granted is remembered per device)
int hipGetLastError() { return 0; }
int hipGetSymbolAddress(void** p, const void*) { *p = device_array; return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { *n = 2; return 0; }

__attribute__((visibility("default"))) const char* stub_launches() { return record.c_str(); }
__attribute__((visibility("default"))) const char* stub_kernels() {         // every kernel of the library, one a line
    static std::string all;
    if (all.empty())
        for (const auto& n : names()) all += plain(n.second) + "\n";
    return all.c_str();
}
__attribute__((visibility("default"))) void stub_clear() { record.clear(); }
__attribute__((visibility("default"))) void stub_refuse_lds(int on) { refuse_lds = on != 0; }
}
