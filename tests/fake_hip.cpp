// The HIP calls and kernel launchers that csrc/api.cpp uses, on the CPU: device
// memory is numbers, a launch or a copy leaves its stream's device busy until it
// is waited for.  For tests of the library's host side (memory, devices).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <map>

#include "kernels.h"

namespace {

constexpr int kDevices = 2;
struct Stream {
    int dev;
};
int g_dev = 0;
size_t g_total = 0, g_others[kDevices];
bool g_busy[kDevices];
uintptr_t g_next = 1 << 20;
int g_mallocs = 0;
std::map<uintptr_t, std::pair<int, size_t>> g_blocks;

size_t live(int dev) {
    size_t sum = 0;
    for (const auto& b : g_blocks)
        if (b.second.first == dev) sum += b.second.second;
    return sum;
}
size_t unused(int dev) { return g_total - g_others[dev] - live(dev); }
hipError_t work(hipStream_t s) {
    g_busy[s ? ((Stream*)s)->dev : g_dev] = true;
    return hipSuccess;
}

}  // namespace

extern "C" {

void fake_reset(long long total) {
    g_total = (size_t)total;
    for (int d = 0; d < kDevices; ++d) g_others[d] = 0, g_busy[d] = false;
    g_dev = 0;
}
void fake_others(int dev, long long bytes) { g_others[dev] = (size_t)bytes; }
long long fake_live(int dev) { return (long long)live(dev); }
int fake_blocks() { return (int)g_blocks.size(); }
int fake_mallocs() { return g_mallocs; }
int fake_busy(int dev) { return g_busy[dev]; }

hipError_t hipGetDevice(int* d) { return *d = g_dev, hipSuccess; }
hipError_t hipSetDevice(int d) { return g_dev = d, hipSuccess; }
hipError_t hipMemGetInfo(size_t* fr, size_t* tot) { return *fr = unused(g_dev), *tot = g_total, hipSuccess; }
hipError_t hipMalloc(void** p, size_t bytes) {
    if (bytes > unused(g_dev)) return hipErrorOutOfMemory;
    ++g_mallocs;
    *p = (void*)g_next;
    g_blocks[g_next] = {g_dev, bytes};
    g_next += (bytes + 511) / 256 * 256;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    const auto it = g_blocks.find((uintptr_t)p);
    if (it == g_blocks.end()) return hipErrorInvalidValue;
    g_busy[it->second.first] = false;
    g_blocks.erase(it);
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipStreamCreate(hipStream_t* s) { return *s = (hipStream_t) new Stream{g_dev}, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { return delete (Stream*)s, hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return g_busy[s ? ((Stream*)s)->dev : g_dev] = false, hipSuccess; }
hipError_t hipDeviceSynchronize() { return g_busy[g_dev] = false, hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return *e = nullptr, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { return *ms = 0, hipSuccess; }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t s) { return work(s); }

}  // extern "C"

namespace pm {

int win_depth(int, int, int, bool) { return 2; }
int adj_depth(int) { return 2; }
hipError_t launch_tables(const double*, const double*, const double*, double*, GridDesc, double, bool, hipStream_t s) { return work(s); }
hipError_t launch_tables_f32(const double*, float*, long long, hipStream_t s) { return work(s); }
hipError_t launch_sweep_win(int, void*, StateOffs, const double*, const float*, int, Aniso, WinArgs, GridDesc, hipStream_t s) { return work(s); }
hipError_t launch_sweep_low(int, int, int, void*, StateOffs, const double*, const float*, int, const LowArgs&, const GridDesc&, hipStream_t s) { return work(s); }
hipError_t launch_adj_low(int, int, int, void*, StateOffs, double*, const double*, int, double, int, const LowArgs&, const GridDesc&, hipStream_t s) { return work(s); }
int low_passes(int, int) { return 1; }
hipError_t low_load() { return hipSuccess; }
bool low_use(int, int N, long long) { return N >= 1 && N <= 4; }
bool tile_use(int, int, const GridDesc&, TileGeom&) { return false; }
bool tile_use_adj(int, int, const GridDesc&, TileGeom&) { return false; }
int tile_depth(int, int, bool) { return 4; }
hipError_t tile_load() { return hipSuccess; }
hipError_t launch_sweep_tile(int, void*, StateOffs, const double*, const float*, int, const TileArgs&, const TileGeom&, const GridDesc&, hipStream_t s) { return work(s); }
hipError_t launch_adj_tile(int, void*, StateOffs, double*, const double*, int, double, int, const TileArgs&, const TileGeom&, const GridDesc&, hipStream_t s) { return work(s); }
hipError_t launch_adj_win(int, void*, StateOffs, double*, const double*, int, Aniso, WinArgs, GridDesc, hipStream_t s) { return work(s); }
hipError_t launch_adj_seed(int, const double*, void*, const void*, const void*, const double*, bool, double, double*, long long, hipStream_t s) { return work(s); }
hipError_t launch_grad_sum(const double*, int, double*, long long, hipStream_t s) { return work(s); }
hipError_t launch_to_f64(int, const void*, double*, long long, hipStream_t s) { return work(s); }
hipError_t launch_from_f64(int, const double*, void*, long long, hipStream_t s) { return work(s); }
hipError_t launch_sum(int, const void*, long long, double*, int, double*, hipStream_t s) { return work(s); }
hipError_t launch_check(int, const void*, int, GridDesc, double*, unsigned long long*, int, double*, unsigned long long*, hipStream_t s) { return work(s); }
hipError_t launch_grad_final(const double*, double*, double*, GridDesc, bool, hipStream_t s) { return work(s); }
hipError_t launch_fill_zero(void*, long long, hipStream_t s) { return work(s); }
hipError_t scratch_device(void**) { return hipErrorNotSupported; }
int scratch_partials() { return 0; }
hipError_t launch_halo(int, bool, void*, void*, const int*, HaloFaces, GridDesc, hipStream_t s) { return work(s); }

}  // namespace pm
