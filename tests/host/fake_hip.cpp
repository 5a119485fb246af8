// Stands in for the HIP runtime and the kernels under csrc/headkv_abi.cpp, so
// that its host logic runs on the CPU ("device" memory is host memory; every
// call has ended when it returns).  Counts what the tests look at.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <set>

#include "../../include/headkv.h"
#include "../../paper_2605_20600_amd/csrc/layout.h"
#include "../../paper_2605_20600_amd/csrc/scratch.h"

namespace {

std::mutex mu;
std::set<void*> live;  // pinned buffers
struct Counts {
    long mallocs, frees, unsafe_calls, copies, live_buffers, live_bytes, max_live;
} counts;
size_t live_bytes = 0;
bool pin_fails = false;
thread_local hipError_t last_error = hipSuccess;
int fail_wait = 0;              // which of the next stream waits fails (1: the next)
const void* last_host = nullptr;  // where the last k_budgets wrote for the host
void (*on_budgets)() = nullptr;
headkv::AttnPlan last_plan{};  // of the last attention launch
thread_local hipStreamCaptureMode mode = hipStreamCaptureModeGlobal;

void unsafe() {  // refused by the runtime while any thread captures in global mode
    if (mode != hipStreamCaptureModeRelaxed) ++counts.unsafe_calls;
}

}  // namespace

extern "C" {

Counts fake_counts() {
    std::lock_guard<std::mutex> lock(mu);
    Counts c = counts;
    c.live_buffers = (long)live.size();
    c.live_bytes = (long)live_bytes;
    return c;
}
void fake_pin_fails(int yes) { pin_fails = yes != 0; }
void fake_fail_wait(int n) { fail_wait = n; }
const void* fake_last_host() { return last_host; }
int fake_plan(int* tpr, int* items) {  // its threads
    *tpr = last_plan.tpr;
    *items = last_plan.items;
    return last_plan.threads;
}
void fake_on_budgets(void (*f)()) { on_budgets = f; }

hipError_t hipHostMalloc(void** p, size_t bytes, unsigned int) {
    std::lock_guard<std::mutex> lock(mu);
    ++counts.mallocs;
    unsafe();
    if (pin_fails) return last_error = hipErrorOutOfMemory;
    *p = std::malloc(bytes + 16);
    *static_cast<size_t*>(*p) = bytes;
    *p = static_cast<char*>(*p) + 16;
    live.insert(*p);
    live_bytes += bytes;
    counts.max_live = std::max(counts.max_live, (long)live.size());
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}
hipError_t hipHostFree(void* p) {
    std::lock_guard<std::mutex> lock(mu);
    ++counts.frees;
    unsafe();
    live.erase(p);
    char* b = static_cast<char*>(p) - 16;
    live_bytes -= *reinterpret_cast<size_t*>(b);
    std::free(b);
    return hipSuccess;
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
    std::swap(mode, *m);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
    return fail_wait > 0 && --fail_wait == 0 ? hipErrorStreamCaptureUnsupported : hipSuccess;
}
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t) {
    std::lock_guard<std::mutex> lock(mu);
    ++counts.copies;
    std::memcpy(dst, src, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t) {
    std::memset(p, v, n);
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "fake error"; }
hipError_t hipEventCreate(hipEvent_t*) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
    *ms = 0;
    return hipSuccess;
}

}  // extern "C"

namespace headkv {

int launch_prefill(const LayerDev&, const Shape&, const uint16_t*, const uint16_t*, int64_t, int,
                   int, void*) {
    return 0;
}
int launch_append(const LayerDev&, const Shape&, const AppendArgs&, void*) { return 0; }
int launch_prefill_attn(const LayerDev&, const Shape&, const uint16_t*, const uint16_t*,
                        const uint16_t*, float*, int64_t, int, int, void*, void*, void*) {
    return 0;
}
int launch_score(const LayerDev&, const Shape&, const uint16_t*, int32_t*, uint8_t*, int, double,
                 double, int, void*) {
    return 0;
}
// the caller's budgets (override mode), and as labels their lowest bits
int launch_budgets(const LayerDev& L, const Shape& s, const uint8_t*, const int32_t* override_b,
                   int32_t* budgets, int, int, int, int, int, int, int32_t* host, void*) {
    for (int i = 0; i < s.BH; ++i) {
        budgets[i] = L.budget[i] = override_b[i];
        L.label[i] = override_b[i] & 1;
        if (host) {
            host[i] = budgets[i];
            host[s.BH + i] = L.label[i];
        }
    }
    last_host = host;
    if (on_budgets) on_budgets();
    return (int)hipGetLastError();  // as the kernels' launchers do
}
int launch_tables(const LayerDev& L, const Shape& s, const LayoutTables& t, void*) {
    std::copy(t.seg_off, t.seg_off + s.BH, L.seg_off);
    std::copy(t.cap, t.cap + s.BH, L.cap);
    std::copy(t.order, t.order + s.BH, L.order);
    std::copy(t.item_start, t.item_start + s.BH + 1, L.item_start);
    std::copy(t.items, t.items + t.n_items, L.items);
    return 0;
}
int launch_update(const LayerDev&, const Shape&, const AppendArgs&, const char*, int, int64_t, int,
                  int, int, int, int, int, int, double, void*, void*, void*) {
    return 0;
}
int launch_update_attn(const LayerDev&, const Shape&, const AppendArgs&, int, int, int, int, int,
                       int, double, const uint16_t*, float*, int, int, int, int, void*, void*,
                       void*) {
    return 0;
}
size_t update_lds_bytes(int, int, int, int, bool, int) { return 0; }
int launch_attn_layers(const LayersArg&, int, const MetaLayout&, const Shape&, int, int, void*) {
    return 0;
}
int launch_attn(const LayerDev&, const Shape&, const AppendArgs&, const uint16_t*, float*,
                uint64_t*, const AttnPlan& p, void*, void*, void*) {
    last_plan = p;
    return 0;
}
int launch_zero_words(uint64_t*, size_t, void*) { return 0; }
int launch_export(const LayerDev&, const Shape&, uint8_t*, int32_t*, void*) { return 0; }
int scratch_address(void** p) {
    *p = nullptr;
    return 0;
}

}  // namespace headkv
