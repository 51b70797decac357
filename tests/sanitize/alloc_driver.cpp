// Failed allocations in the edge index, on a machine without a GPU (built and run by
// tests/test_alloc_cpu.py).
//
// The program defines the HIP runtime calls that the index makes, which replace the runtime's:
// device memory is host memory under a budget or with the n-th allocation failing, copies are
// memcpy, launches run nothing.  The graph is a descriptor of given sizes.  After a failed call
// the graph must hold no part of the index, nothing may have leaked, and the next call must
// build it; the optional per-entry rows must give way to what the index cannot do without.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>

#include "../../paper_2201_11655_amd/csrc/vdmc_internal.h"

namespace {
std::map<void*, size_t> g_live;
size_t g_used = 0, g_peak = 0, g_budget = ~(size_t)0;
long g_calls = 0, g_fail_at = -1, g_sync_fails = 0;
bool g_failed = false;

int fails = 0;
void expect(bool ok, const char* what, long i) {
    if (ok) return;
    std::fprintf(stderr, "%s (case %ld): %s\n", what, i, vdmc_last_error());
    fails++;
}
void reset(size_t budget, long fail_at) {
    g_used = g_peak = 0;
    g_budget = budget;
    g_calls = 0;
    g_fail_at = fail_at;
    g_failed = false;
    g_live.clear();
}
}  // namespace

extern "C" {
#undef hipGetDeviceProperties
hipError_t hipMalloc(void** p, size_t bytes) {
    if (g_calls++ == g_fail_at || g_used + bytes > g_budget) {
        g_failed = true;
        return hipErrorOutOfMemory;
    }
    *p = std::calloc(1, bytes);
    g_live[*p] = bytes;
    g_used += bytes;
    g_peak = std::max(g_peak, g_used);
    return hipSuccess;
}
hipError_t hipFree(void* p) {
    if (!p) return hipSuccess;
    g_used -= g_live.at(p);
    g_live.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* st) {
    *g = *b = dim3(1);
    *s = 0;
    *st = nullptr;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) {
    if (g_sync_fails > 0 && --g_sync_fails == 0) {
        g_failed = true;
        return hipErrorUnknown;
    }
    return hipSuccess;
}
int hipGetStreamDeviceId(hipStream_t) { return 0; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeWarpSize ? 64 : (a == hipDeviceAttributeMultiprocessorCount ? 256 : 65536);
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_t* p, int) {
    std::memset(p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950");
    p->warpSize = 64;
    p->multiProcessorCount = 256;
    p->maxThreadsPerBlock = 1024;
    p->sharedMemPerBlock = 65536;
    return hipSuccess;
}
}

int main() {
    const int64_t n = 5000, P = 40000;
    int32_t* lo = (int32_t*)std::malloc(P * 4);
    int32_t* hi = (int32_t*)std::malloc(P * 4);
    auto graph = [&] {
        auto* g = new vdmc_graph_s();
        g->n = n;
        g->pairs = P;
        return g;
    };
    auto empty = [](const vdmc_graph_s* g) { return !g->epid && !g->elo && !g->ehi && !g->ework; };
    auto held = [](const vdmc_graph_s* g) {   // allocations the graph owns
        return (size_t)((g->ehash != nullptr) + (g->epid != nullptr) + (g->elo != nullptr) + (g->ehi != nullptr) +
                        (g->ework != nullptr));
    };
    auto drop = [](vdmc_graph_s* g) {
        for (void* p : {(void*)g->ehash, (void*)g->epid, (void*)g->elo, (void*)g->ehi, (void*)g->ework}) (void)hipFree(p);
        delete g;
    };
    // the index with and without the optional rows
    reset(~(size_t)0, -1);
    vdmc_graph_s* g = graph();
    expect(vdmc_edge_list(g, lo, hi) == VDMC_OK, "build", 0);
    expect(g->epid && g->elo && g->ehi && g->ework && g->ehash, "complete", 0);
    expect(g_live.size() == held(g), "leak", 0);
    const long calls = g_calls;
    const size_t peak = g_peak, optional = g_live.at(g->ework);
    drop(g);
    // every allocation in turn fails, then the next call builds the index
    long without = 0;
    for (long i = 0; i < calls; i++) {
        reset(~(size_t)0, i);
        g = graph();
        const vdmc_status st = vdmc_edge_list(g, lo, hi);
        if (st == VDMC_OK) {   // the optional rows alone may fail
            expect(g_failed && g->epid && g->elo && g->ehi && !g->ework, "built without the rows", i);
            without++;
        } else {
            expect(st == VDMC_ERR_OUT_OF_MEMORY, "status", i);
            expect(empty(g), "no part of a failed index stays with the graph", i);
            expect(g_live.size() == held(g), "leak after a failure", i);
            expect(vdmc_edge_list(g, lo, hi) == VDMC_OK && g->epid && g->ework, "next call", i);
        }
        expect(g_live.size() == held(g), "leak", i);
        drop(g);
    }
    expect(without == 1, "one allocation is optional", without);
    // a failure after the allocations (the work itself): of the hash, of the index
    for (long i = 1; i <= 2; i++) {
        reset(~(size_t)0, -1);
        g = graph();
        g_sync_fails = i;
        expect(vdmc_edge_list(g, lo, hi) == VDMC_ERR_DEVICE, "device failure", i);
        expect(empty(g) && (g->ehash != nullptr) == (i == 2), "nothing of a failed build stays", i);
        expect(g_live.size() == held(g), "leak after a device failure", i);
        expect(vdmc_edge_list(g, lo, hi) == VDMC_OK && g->epid, "next call", i);
        drop(g);
    }
    // memory for all but the optional rows: built without them
    reset(peak - optional, -1);
    g = graph();
    expect(vdmc_edge_list(g, lo, hi) == VDMC_OK, "the optional rows take no room from the rest", 0);
    expect(g->epid && !g->ework, "built without the rows", 0);
    drop(g);
    std::free(lo);
    std::free(hi);
    if (fails) return 1;
    std::printf("allocation failures ok: %ld allocations\n", calls);
    return 0;
}
