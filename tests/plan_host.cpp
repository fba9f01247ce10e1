// The plan's host code (plan.cpp) over a HIP runtime of its own that keeps memory on the host
// and knows which device every allocation and stream belongs to.  Plain C++, no GPU.
//
// usage: plan_host device | nomem | threads
//   device: the projector's lists go to the plan's device whatever device is current, which
//           stays current
//   nomem:  lists or a plan that host memory does not suffice for are an error, not an
//           exception, and nothing leaks
//   threads: while several threads choose launch shapes, the current shape is always one
//           shape with its own lists, and each shape's are built once
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <set>
#include <thread>
#include <utility>

#include "common.h"

namespace {
int g_current = 0, g_bad = 0;
std::map<void*, int> g_memory;  // allocation -> device
std::set<hipStream_t> g_streams;
std::recursive_mutex g_mu;    // guards the above
long g_fail_after = -1;  // host allocations left before one fails; -1: none does

void expect(bool ok, const char* what) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    if (!ok) std::printf("failed: %s\n", what), ++g_bad;
}
void* host_alloc(std::size_t n) {
    if (g_fail_after >= 0 && g_fail_after-- == 0) return nullptr;
    return std::malloc(n ? n : 1);
}
}  // namespace

void* operator new(std::size_t n) {
    if (void* p = host_alloc(n)) return p;
    throw std::bad_alloc();
}
// A sort's buffer may be missing: it then does without.
void* operator new(std::size_t n, const std::nothrow_t&) noexcept { return std::malloc(n); }
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

extern "C" {
hipError_t hipGetDevice(int* d) { return *d = g_current, hipSuccess; }
hipError_t hipSetDevice(int d) { return g_current = d, hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    const long left = std::exchange(g_fail_after, -1);  // not for this runtime's own
    *p = std::malloc(n ? n : 1);
    g_memory[*p] = g_current;
    g_fail_after = left;
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (p) {
        std::lock_guard<std::recursive_mutex> lk(g_mu);
        expect(g_memory.erase(p) == 1, "free of an allocation");
        std::free(p);
    }
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
    return std::memcpy(d, s, n), hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    const long left = std::exchange(g_fail_after, -1);
    *s = reinterpret_cast<hipStream_t>(new int(g_current));
    g_streams.insert(*s);
    g_fail_after = left;
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
    g_streams.erase(s);
    delete reinterpret_cast<int*>(s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t on) {
    std::lock_guard<std::recursive_mutex> lk(g_mu);
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
    auto before = g_memory;
    const char* what = argc > 1 ? argv[1] : "";
    if (!std::strcmp(what, "device")) {
        g_current = 0;
        expect(dect_plan_set_launch(p, 4, 8, 4, 3) == DECT_OK, "lists");
        expect(g_current == 0, "the current device stays current");
        int made = 0;
        for (const auto& m : g_memory) {
            expect(m.second == 1, "every allocation is on the plan's device");
            made += before.count(m.first) == 0;
        }
        expect(made == 2, "two lists");
    } else if (!std::strcmp(what, "threads")) {
        std::map<std::pair<int, int>, std::vector<int>> want[2];
        for (int views : {1, 2, 4, 8})
            for (int chunk = 1; chunk <= 16; ++chunk)
                for (int R = 1; R <= 2; ++R)
                    want[R - 1][{views, chunk}] = proj_launch_order(
                        g, p->Vb, p->splits.data(), R * views, R * R * views, chunk);
        std::atomic<int> running{4};
        std::vector<std::thread> pool;
        for (int t = 0; t < 4; ++t)
            pool.emplace_back([&, t] {
                for (int n = 0; n < 256; ++n) {
                    const int k = (n * (2 * t + 1) + 17 * t) % 64;
                    expect(dect_plan_set_launch(p, 2 << n % 3, 8, 1 << k % 4, 1 + k / 4) ==
                           DECT_OK, "a shape is set");
                }
                --running;
            });
        while (running > 0) {
            const dect_plan::ProjOrder* o = p->pj_shape;
            for (int r = 0; r < 2; ++r) {
                const std::vector<int>& w = want[r][{o->views, o->chunk}];
                expect(o->blocks[r] == (int)w.size() &&
                           !std::memcmp(o->order[r], w.data(), w.size() * sizeof(int)),
                       "a shape's own lists");
            }
        }
        for (auto& t : pool) t.join();
        expect(p->pj_orders.size() == 64, "each shape once");
    } else {
        // Each host allocation of the two calls in turn fails.
        for (int call = 0; call < 2; ++call) {
            long fails = 0;
            dect_plan* q = nullptr;
            for (long n = 0; !g_bad; ++n) {
                g_fail_after = n;
                dect_status st = DECT_E_DEVICE;
                try {
                    st = call == 0 ? dect_plan_set_launch(p, 4, 8, 8, 2)
                                   : dect_plan_create(&g, &spec, DECT_F64, &q);
                } catch (...) {
                    expect(false, "nothing is thrown");
                }
                const bool failed = g_fail_after < 0;
                g_fail_after = -1;
                if (!failed) {
                    expect(st == DECT_OK, "the call succeeds");
                    break;
                }
                ++fails;
                expect(st == DECT_E_NOMEM, "out of memory is reported");
                expect(call == 1 ? !q : p->pj_shape.load()->views == 2, "no result");
                expect(g_streams.empty() && g_memory == before, "nothing leaks");
            }
            expect(fails > 0, "allocations failed");
            if (call == 0) {
                expect(p->pj_shape.load()->views == 8, "the shape is set");
                before = g_memory;
            } else {
                dect_plan_destroy(q);
            }
        }
    }
    g_current = 1;
    dect_plan_destroy(p);
    expect(g_memory.empty() && g_streams.empty(), "the plan gives everything back");
    std::printf(g_bad ? "FAILED\n" : "OK\n");
    return g_bad != 0;
}
