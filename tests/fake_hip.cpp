// Stands in for the HIP runtime in a process without a GPU: keeps the names of the kernels that the library
// registers and, of every launch, the kernel's name, its grid and its block.  Nothing runs.
#include <cstdint>
#include <cstdio>
#include <map>
#include <string>

#include "kernels.hpp"

namespace {
struct Dim3 { uint32_t x, y, z; };
struct Call { Dim3 grid, block; size_t lds; void *stream; };
std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> n;
    return n;
}
std::string launches;
Call pending;
}

extern "C" {

void **__hipRegisterFatBinary(const void *) { static void *module; return &module; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, void *, void *, int *)
{
    names()[host] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void *stream) { pending = {grid, block, lds, stream}; return 0; }
int __hipPopCallConfiguration(Dim3 *grid, Dim3 *block, size_t *lds, void **stream)
{
    *grid = pending.grid;
    *block = pending.block;
    *lds = pending.lds;
    *stream = pending.stream;
    return 0;
}
int hipLaunchKernel(const void *host, Dim3 g, Dim3 b, void **, size_t, void *)
{
    char dims[96];
    std::snprintf(dims, sizeof dims, " %u %u %u %u\n", g.x, g.y, g.z, b.x * b.y * b.z);
    launches += names()[host] + dims;
    return 0;
}
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipGetDevice(int *device) { *device = 0; return 0; }
const char *hipGetErrorString(int) { return "fake"; }
int hipGetLastError() { return 0; }
int hipGetSymbolAddress(void **p, const void *) { *p = reinterpret_cast<void *>(uintptr_t(4096)); return 0; }
int hipMemcpyAsync(void *, const void *, size_t, int, void *) { return 0; }
int hipStreamSynchronize(void *) { return 0; }

// The launches since the last call, a line each: mangled name, grid, threads of a block.
const char *fake_launches()
{
    static std::string taken;
    taken.swap(launches);
    launches.clear();
    return taken.c_str();
}

// codec::launch_merge for one request of four heads with the given reduction form.
int fake_reduction(int (*launch)(const codec::MergeParams &, int, int, void *), int head_dim, int split_waves)
{
    codec::MergeParams p{};
    p.num_requests = 1;
    p.h_q = 4;
    p.group = 1;
    p.split_waves = split_waves;
    return launch(p, CODEC_DTYPE_BF16, head_dim, nullptr);
}

}
