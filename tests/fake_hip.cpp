// A HIP runtime that launches nothing and writes down what it was asked to do: the launches (kernel, grid, block, LDS) and the LDS
// limits set, as text lines.  Loaded with RTLD_GLOBAL ahead of libtri.so it takes the place of the real one, so that tests without a
// GPU see which kernels a call would launch and how.
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>

#include <map>
#include <mutex>
#include <string>

struct Dim3 {
    uint32_t x, y, z;
};

namespace {
std::mutex mutex_;
std::map<const void *, std::string> names;
std::string log_;
thread_local struct {
    Dim3 grid, block;
    size_t lds;
    void *stream;
} config;

std::string name_of(const void *f)
{
    auto it = names.find(f);
    return it == names.end() ? "?" : it->second;
}
}  // namespace

extern "C" {

const char *fake_log(void)
{
    static std::string out;
    std::lock_guard<std::mutex> lock(mutex_);
    out.swap(log_);
    log_.clear();
    return out.c_str();
}

void **__hipRegisterFatBinary(const void *)
{
    static void *handle;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, void *, void *, int *)
{
    std::lock_guard<std::mutex> lock(mutex_);
    names[host] = device;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}

int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void *stream)
{
    config = {grid, block, lds, stream};
    return 0;
}
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *lds, void **stream)
{
    *grid = config.grid, *block = config.block, *lds = config.lds, *stream = config.stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim3 grid, Dim3 block, void **, size_t lds, void *)
{
    char line[96];
    snprintf(line, sizeof line, " %u %u %u %u %zu\n", grid.x, grid.y, grid.z, block.x * block.y * block.z, lds);
    std::lock_guard<std::mutex> lock(mutex_);
    log_ += "launch " + name_of(f) + line;
    return 0;
}
int hipFuncSetAttribute(const void *f, int, int value)
{
    std::lock_guard<std::mutex> lock(mutex_);
    log_ += "limit " + name_of(f) + " " + std::to_string(value) + "\n";
    return 0;
}
int hipGetDevice(int *dev)
{
    *dev = 0;
    return 0;
}
int hipDeviceGetAttribute(int *value, int, int)   // (the library asks for the compute units only)
{
    *value = 256;
    return 0;
}
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *blocks, const void *, int, size_t)
{
    *blocks = 1;
    return 0;
}
int hipGetSymbolAddress(void **p, const void *)
{
    static char at[256] __attribute__((aligned(256)));
    *p = at;
    return 0;
}
int hipGetLastError(void) { return 0; }
const char *hipGetErrorString(int) { return "none"; }
int hipEventRecord(void *, void *) { return 0; }
}
