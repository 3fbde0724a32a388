// The runtime calls of libcacnn.so without a device: loaded in front of the runtime's own library, it notes what is launched, on which device and stream,
// refuses a launch whose LDS the kernel was not given on that device, and keeps a clock that a launch moves on by what its kernel is said to
// cost.  Nothing runs.
#ifndef _GNU_SOURCE
#define _GNU_SOURCE
#endif
#include <dlfcn.h>
#include <stdint.h>
#include <string.h>

#include <map>
#include <set>
#include <string>
#include <vector>

struct Dim3 {
    uint32_t x, y, z;
};

namespace {
int g_device = 0, g_last = 0;
double g_clock = 0.0;
std::set<std::pair<int, const void*>> g_raised;                 // (device, kernel) whose dynamic LDS limit was raised
std::vector<std::pair<std::string, double>> g_costs;            // part of a kernel's name, milliseconds; the first that fits counts
std::map<void*, double> g_events;
std::string g_log;
struct {
    Dim3 grid, block;
    size_t lds;
    void* stream;
} g_configuration;

const char* name_of(const void* kernel) {
    Dl_info info;
    return dladdr(kernel, &info) && info.dli_sname ? info.dli_sname : "?";
}
}  // namespace

extern "C" {
// ---- for the test
void stand_in_device(int device) { g_device = device; }
void stand_in_cost(const char* part, double ms) { g_costs.emplace_back(part, ms); }
// the kernels launched since the last call, one a line
const char* stand_in_launches() {
    static std::string log;
    log.swap(g_log);
    g_log.clear();
    return log.c_str();
}

// ---- for the library
int hipGetDeviceCount(int* n) {
    *n = 4;
    return 0;
}
int hipGetDevice(int* device) {
    *device = g_device;
    return 0;
}
int hipGetLastError() {
    const int e = g_last;
    g_last = 0;
    return e;
}
int hipFuncSetAttribute(const void* kernel, int, int) {
    g_raised.insert({g_device, kernel});
    return 0;
}
int __hipPushCallConfiguration(Dim3 grid, Dim3 block, size_t lds, void* stream) {
    g_configuration = {grid, block, lds, stream};
    return 0;
}
int __hipPopCallConfiguration(Dim3* grid, Dim3* block, size_t* lds, void** stream) {
    *grid = g_configuration.grid;
    *block = g_configuration.block;
    *lds = g_configuration.lds;
    *stream = g_configuration.stream;
    return 0;
}
int hipLaunchKernel(const void* kernel, Dim3 grid, Dim3 block, void**, size_t lds, void*) {
    if (lds > 65536 && !g_raised.count({g_device, kernel})) return g_last = 1;
    if (!grid.x || (uint64_t)grid.x * block.x >= (1ull << 32)) return g_last = 9;
    const std::string name = name_of(kernel);
    g_log += name + "\n";
    for (const auto& c : g_costs)
        if (name.find(c.first) != std::string::npos) {
            g_clock += c.second;
            break;
        }
    return 0;
}
int hipEventCreate(void** e) {
    *e = new char;
    return 0;
}
int hipEventDestroy(void* e) {
    delete (char*)e;
    return 0;
}
int hipEventRecord(void* e, void*) {
    g_events[e] = g_clock;
    return 0;
}
int hipEventSynchronize(void*) { return 0; }
int hipEventElapsedTime(float* ms, void* from, void* to) {
    *ms = (float)(g_events[to] - g_events[from]);
    return 0;
}
}
