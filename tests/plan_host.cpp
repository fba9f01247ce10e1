// The plan's host code (plan.cpp) over a HIP runtime of its own that keeps memory on the host
// and knows which device every allocation and stream belongs to.  Plain C++, no GPU.
//
// usage: plan_host device
//   device: the projector's lists go to the plan's device whatever device is current, which
//           stays current
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>

#include "common.h"

namespace {
int g_current = 0, g_bad = 0;
std::map<void*, int> g_memory;  // allocation -> device
std::set<hipStream_t> g_streams;

void expect(bool ok, const char* what) {
    if (!ok) std::printf("failed: %s\n", what), ++g_bad;
}
}  // namespace

extern "C" {
hipError_t hipGetDevice(int* d) { return *d = g_current, hipSuccess; }
hipError_t hipSetDevice(int d) { return g_current = d, hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) {
    *p = std::malloc(n ? n : 1);
    g_memory[*p] = g_current;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (p) {
        expect(g_memory.erase(p) == 1, "free of an allocation");
        std::free(p);
    }
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    return std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = reinterpret_cast<hipStream_t>(new int(g_current));
    g_streams.insert(*s);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
    g_streams.erase(s);
    delete reinterpret_cast<int*>(s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t on) {
    expect(g_memory[d] == *reinterpret_cast<int*>(on), "a copy's stream is on its device");
    return std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode*) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
}

int main(int argc, char** argv) {
    using namespace dect;
    dect_geometry g{};
    g.kind = DECT_FAN;
    g.nx = g.ny = 20;
    g.n_views = 24;
    g.n_det = 30;
    g.pixel_cm = 0.5;
    g.det_cm = 0.8;
    g.src_iso_cm = 20.0;
    g.src_det_cm = 35.0;
    g.span = 6.283185307179586;
    const double s[3] = {1.0, 2.0, 1.0}, f[3] = {0.5, 0.4, 0.3};
    const dect_spectra spec{3, f, s, s, f, f};
    dect_plan* p = nullptr;
    g_current = 1;
    expect(dect_plan_create(&g, &spec, DECT_F32, &p) == DECT_OK, "plan");
    const auto before = g_memory;
    const int* order[2] = {nullptr, nullptr};
    int blocks[2] = {0, 0};
    if (argc > 1 && !std::strcmp(argv[1], "device")) {
        g_current = 0;
        expect(proj_order_for(p, 4, 3, order, blocks) == DECT_OK, "lists");
        expect(g_current == 0, "the current device stays current");
        int made = 0;
        for (const auto& m : g_memory) {
            expect(m.second == 1, "every allocation is on the plan's device");
            made += before.count(m.first) == 0;
        }
        expect(made == 2, "two lists");
    }
    g_current = 1;
    dect_plan_destroy(p);
    expect(g_memory.empty() && g_streams.empty(), "the plan gives everything back");
    std::printf(g_bad ? "FAILED\n" : "OK\n");
    return g_bad != 0;
}
