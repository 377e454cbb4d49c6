// Stands in for the HIP runtime in a process without a GPU: the library's launches are written down instead of carried
// out, so that its dispatch rules can be tested on the host.  Defines the runtime functions libhq.so calls.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <cxxabi.h>
#include <map>
#include <string>
#include <utility>

struct Dim { unsigned x, y, z; };

static std::map<const void *, std::string> names;                       // host stub -> kernel
static std::map<std::pair<int, const void *>, int> allowed;             // (device, host stub) -> dynamic LDS allowed
static std::string record;                                              // one line per launch
static struct { Dim grid, block; size_t lds; void *stream; } pending;
static int device;

extern "C" {

void recorder_reset(int dev) { record.clear(); device = dev; }
const char *recorder_lines() { return record.c_str(); }

void **__hipRegisterFatBinary(const void *) { static void *module; return &module; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *stub, char *, const char *name, unsigned, void *, void *, Dim *, Dim *, int *)
{
    int status = 0;
    char *plain = abi::__cxa_demangle(name, nullptr, nullptr, &status);
    std::string s = status == 0 ? plain : name;
    free(plain);
    const size_t at = s.find("::") == std::string::npos ? 0 : s.find("::") + 2;      // (kernels live in an unnamed namespace)
    names[stub] = s.substr(at, s.find('(', at) - at);
}
int __hipPushCallConfiguration(Dim grid, Dim block, size_t lds, void *stream)
{
    pending = {grid, block, lds, stream};
    return 0;
}
int __hipPopCallConfiguration(Dim *grid, Dim *block, size_t *lds, void **stream)
{
    *grid = pending.grid; *block = pending.block; *lds = pending.lds; *stream = pending.stream;
    return 0;
}
int hipLaunchKernel(const void *stub, Dim grid, Dim block, void **, size_t lds, void *)
{
    const auto a = allowed.find({device, stub});
    char line[512];
    snprintf(line, sizeof line, "%s\t%llu\t%u\t%zu\t%d\n", names[stub].c_str(), (unsigned long long)grid.x * grid.y * grid.z,
             block.x * block.y * block.z, lds, a == allowed.end() ? 0 : a->second);
    record += line;
    return 0;
}
int hipFuncSetAttribute(const void *stub, int, int value) { allowed[{device, stub}] = value; return 0; }
int hipGetDevice(int *d) { *d = device; return 0; }
int hipGetLastError() { return 0; }
int hipGetSymbolAddress(void **p, const void *) { *p = reinterpret_cast<void *>(0x10000); return 0; }

} // extern "C"
