// The host side of the plan and one-shot calls against a stand-in HIP runtime:
// device memory is host memory, launches are recorded and not run.  Built with
// AddressSanitizer and UndefinedBehaviorSanitizer on the host code; no GPU.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <numeric>
#include <vector>

#include <hip/hip_runtime.h>

#include "lora.h"
#include "lora_internal.h"
#include "lora_plan.h"

namespace lora {
hipError_t launch_shrink(const KernelArgs&, const uint32_t*, int, hipStream_t) { return hipSuccess; }
hipError_t launch_expand(const KernelArgs&, const uint32_t*, int, hipStream_t) { return hipSuccess; }
hipError_t launch_reduce(const KernelArgs&, const uint32_t*, hipStream_t) { return hipSuccess; }
hipError_t launch_step(const KernelArgs&, const uint32_t*, int, hipStream_t) { return hipSuccess; }
hipError_t launch_fill(uint32_t* p, uint32_t v, uint64_t n, hipStream_t);
hipError_t launch_base(const BaseArgs&, int, hipStream_t) { return hipSuccess; }
}  // namespace lora

// The runtime calls of the library's host code (defined here, they take the
// place of the HIP library's).
extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeNumberOfXccs ? 8 : 256;
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { return (*p = std::aligned_alloc(256, (n + 255) / 256 * 256)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned);
hipError_t hipHostFree(void* p);
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m);
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { *d = h; return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { return hipMalloc(p, 1 << 24); }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) { *c = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipGetLastError();
// a <<<>>> launch: its configuration pushed, popped by the kernel's stub, then the launch
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t);
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s);
hipError_t hipLaunchKernel(const void*, dim3 grid, dim3, void**, size_t, hipStream_t);
}

namespace {

// of the kernel that writes the work list: how many (the g_fail_at-th from now on
// fails), their workgroups, the generation the list's header holds after them
int g_launches, g_workgroups, g_fail_at;
bool g_hold;
int g_pinned;                              // pinned allocations not given back
hipStreamCaptureMode g_mode = hipStreamCaptureModeGlobal;
std::vector<uint32_t> g_blob;              // the extra words of the launches, in order
std::vector<int32_t> g_rows;               // the rows they list, in grouped order
uint32_t g_generation;
dim3 g_grid, g_block;
hipError_t g_error = hipSuccess;

int failures = 0;
#define CHECK(cond, ...)                                   \
    do {                                                   \
        if (!(cond)) {                                     \
            std::fprintf(stderr, "FAIL %s:%d: ", __FILE__, __LINE__); \
            std::fprintf(stderr, __VA_ARGS__);             \
            std::fprintf(stderr, "\n");                    \
            ++failures;                                    \
        }                                                  \
    } while (0)

}  // namespace

hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
    if (g_mode != hipStreamCaptureModeRelaxed) return hipErrorStreamCaptureUnsupported;   // as beside a capture
    ++g_pinned;
    return hipMalloc(p, n);
}
hipError_t hipHostFree(void* p) {
    --g_pinned;
    return hipFree(p);
}
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) {
    std::swap(*m, g_mode);
    return hipSuccess;
}
// (g_hold: fills do not get through, as on a stream with earlier work)
hipError_t lora::launch_fill(uint32_t* p, uint32_t v, uint64_t n, hipStream_t) {
    if (!g_hold) std::fill(p, p + n, v);
    return hipSuccess;
}
hipError_t hipGetLastError() {
    const hipError_t e = g_error;
    g_error = hipSuccess;
    return e;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t) {
    g_grid = grid;
    g_block = block;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* s) {
    *grid = g_grid;
    *block = g_block;
    *lds = 0;
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3 grid, dim3, void** args, size_t, hipStream_t) {
    ++g_launches;
    if (g_fail_at > 0 && --g_fail_at == 0) return g_error = hipErrorOutOfMemory;
    const lora::PlanArgs& a = *(const lora::PlanArgs*)args[0];
    uint32_t v = 0;
    if (lora::header_word(a, 0, v)) g_generation = v;
    const uint32_t* data = a.staged ? a.staged : a.data;
    g_blob.insert(g_blob.end(), data + a.blob_at, data + a.blob_at + a.blob_words);
    for (int i = 0; i < a.n_rows; ++i) {
        const lora::PlanRow& r = ((const lora::PlanRow*)data)[i];
        const int32_t* listed = (const int32_t*)data + a.n_rows * lora::kRowWords + (-1 - r.row0);
        if (r.proj() == 0)
            for (int j = 0; j < r.nrows(); ++j) g_rows.push_back(r.row0 >= 0 ? r.row0 + j : listed[j]);
    }
    g_workgroups += (int)grid.x;
    return hipSuccess;
}

namespace {

alignas(16) unsigned char g_factor[16];    // stands for every factor: nothing reads it

lora_table_t table(int h_in, int h_out, const std::vector<int32_t>& ranks) {
    std::vector<const void*> p(ranks.size(), g_factor);
    std::vector<float> s(ranks.size(), 1.f);
    lora_table_t t = nullptr;
    const int rc = lora_register_adapters(&t, 0, h_in, h_out, LORA_BF16, (int)ranks.size(), p.data(), p.data(),
                                          ranks.data(), s.data(), nullptr);
    CHECK(rc == LORA_OK, "register: %d %s", rc, lora_last_error());
    return t;
}

// A plan made for a batch whose K ranges are cut by bytes holds a part of that
// batch whose ranges are not, and says so beforehand.
void check_parts_fit() {
    const int wide = 7, narrow = 60;
    std::vector<int32_t> ranks(wide, 128);
    ranks.insert(ranks.end(), narrow, 16);
    std::vector<int32_t> off(ranks.size() + 1), ad(ranks.size());
    std::iota(off.begin(), off.end(), 0);
    std::iota(ad.begin(), ad.end(), 0);
    const lora_table_t t = table(8192, 264, ranks);
    const lora_batch_t whole{wide + narrow, wide + narrow, off.data(), ad.data()};
    lora_plan_t p = nullptr;
    CHECK(lora_plan_create(&p, t, &whole, nullptr) == LORA_OK, "create: %s", lora_last_error());
    size_t ws = 0, pb = 0;
    CHECK(lora_workspace_bytes(t, &whole, &ws) == LORA_OK && lora_plan_bytes(t, &whole, &pb) == LORA_OK, "sizes");
    for (int n : {1, 3, wide, 30, wide + narrow}) {
        const lora_batch_t part{n, n, off.data(), ad.data()};
        size_t ws1 = 0, pb1 = 0;
        CHECK(lora_workspace_bytes(t, &part, &ws1) == LORA_OK && lora_plan_bytes(t, &part, &pb1) == LORA_OK, "sizes");
        CHECK(ws1 <= ws && pb1 <= pb, "%d of %d tokens: %zu of %zu, %zu of %zu bytes", n, wide + narrow, ws1, ws, pb1, pb);
        const int rc = lora_plan_update(p, nullptr, &part, nullptr);
        CHECK(rc == LORA_OK, "update to %d tokens: %d %s", n, rc, lora_last_error());
    }
    lora_plan_destroy(p);
    lora_release_adapters(t);
}

// An update arms the step buffers with the whole device: no workgroup writes more
// than 64 KiB of them while there are fewer than 1024.
void check_arming_is_spread() {
    for (int rows : {1, 16, 32, 64}) {
        for (int rank : {8, 64, 128, 256}) {
            const lora_table_t t = table(28672, 8192, {rank});
            std::vector<int32_t> off = {0, rows}, ad = {0};
            const lora_batch_t b{rows, 1, off.data(), ad.data()};
            lora_plan_t p = nullptr;
            CHECK(lora_plan_create(&p, t, &b, nullptr) == LORA_OK, "create: %s", lora_last_error());
            size_t ws = 0, pb = 0;                 // a plan's bytes are a workspace's and the step buffers'
            CHECK(lora_workspace_bytes(t, &b, &ws) == LORA_OK && lora_plan_bytes(t, &b, &pb) == LORA_OK, "sizes");
            g_launches = g_workgroups = 0;
            CHECK(lora_plan_update(p, nullptr, &b, nullptr) == LORA_OK, "update: %s", lora_last_error());
            CHECK(g_launches == 1, "%d launches", g_launches);
            CHECK(g_workgroups >= 1024 || (pb - ws) / g_workgroups <= 65536, "rank %d, %d rows: %zu bytes by %d workgroups",
                  rank, rows, pb - ws, g_workgroups);
            lora_plan_destroy(p);
            lora_release_adapters(t);
        }
    }
}

// A list written by several launches is no plan's until the last of them: when one
// fails, neither launches recorded for the batch before nor those of the new one run it.
void check_failed_update() {
    std::vector<int32_t> ranks(4, 16), off(1025), ad(1024);
    std::iota(off.begin(), off.end(), 0);
    for (int i = 0; i < 1024; ++i) ad[i] = i % 4;                // 16 row blocks of rows four apart
    const lora_table_t t = table(256, 264, ranks);
    const lora_batch_t b{1024, 1024, off.data(), ad.data()};
    lora_plan_t p = nullptr;
    CHECK(lora_plan_create(&p, t, &b, nullptr) == LORA_OK, "create: %s", lora_last_error());
    const uint32_t made = g_generation;
    g_launches = 0;
    CHECK(lora_plan_update(p, nullptr, &b, nullptr) == LORA_OK, "update: %s", lora_last_error());
    const int n = g_launches;
    CHECK(n >= 2 && g_generation == made + 1, "%d launches, generation %u after %u", n, g_generation, made);
    for (int at = 1; at <= n; ++at) {
        const uint32_t before = g_generation;
        g_fail_at = at;
        CHECK(lora_plan_update(p, nullptr, &b, nullptr) == LORA_E_HIP, "launch %d fails", at);
        CHECK(at == 1 ? g_generation == before : g_generation == 0, "launch %d failed: generation %u", at, g_generation);
        CHECK(lora_plan_update(p, nullptr, &b, nullptr) == LORA_OK && g_generation == before + 2, "update after a failure");
    }
    lora_plan_destroy(p);
    lora_release_adapters(t);
}

// Lists of more data than a few launches' arguments hold are written by one launch
// that reads pinned memory, as long as a slot of it is free, and by a chain of launches
// when none is; the row order and the base projection's tile list come out the same.
void check_staged_lists() {
    const int n = 8192;
    std::vector<int32_t> ranks(128, 16), off(n + 1), ad(n);
    std::iota(off.begin(), off.end(), 0);
    for (int i = 0; i < n; ++i) ad[i] = i % 128;
    const lora_table_t t = table(256, 264, ranks);
    const lora_table_t t2 = table(256, 520, ranks);
    const lora_batch_t b{n, n, off.data(), ad.data()};
    std::vector<int32_t> perm(n), goff(n + 1), gad(n);
    int32_t G = 0;
    CHECK(g_pinned == 0, "pinned memory before the first large list");
    CHECK(lora_group_rows(&b, 128, perm.data(), goff.data(), gad.data(), &G) == LORA_OK, "group");
    lora_plan_t p = nullptr;
    CHECK(lora_plan_create(&p, t, &b, nullptr) == LORA_OK, "create: %s", lora_last_error());
    for (const bool hold : {false, true}) {
        g_hold = hold;
        for (int k = 0; k < 12; ++k) {                           // more than there are slots
            g_launches = 0;
            g_rows.clear();
            CHECK(lora_plan_update(p, nullptr, &b, nullptr) == LORA_OK, "update: %s", lora_last_error());
            CHECK(g_rows == perm, "row order");
            CHECK(!hold || k < 8 ? g_launches == 1 : g_launches > 4, "held %d, call %d: %d launches", hold, k, g_launches);
        }
    }
    lora_plan_destroy(p);
    CHECK(g_pinned == 1 && g_mode == hipStreamCaptureModeGlobal, "%d pinned", g_pinned);
    lora_release_adapters(t);
    CHECK(g_pinned == 1, "another table is left");
    lora_release_adapters(t2);                                   // the ring goes, with what was held
    CHECK(g_pinned == 0, "pinned memory after the last table");
    g_hold = false;
    const lora_table_t t3 = table(256, 264, ranks), t4 = table(256, 520, ranks);
    // the call that allocates nothing
    std::vector<unsigned char> xy(2 * (size_t)n * (256 + 264) + 32);
    unsigned char* x = (unsigned char*)(((uintptr_t)xy.data() + 15) & ~(uintptr_t)15);
    g_launches = 0;
    CHECK(lora_apply_fused_static(t3, &b, x, 256, x + 2 * (size_t)n * 256, 264, nullptr) == LORA_OK, "static: %s", lora_last_error());
    CHECK(g_pinned == 0 && g_launches > 4, "%d pinned, %d launches", g_pinned, g_launches);
    // two projections list their scattered rows once: 16 blocks of 64 rows take two launches'
    // arguments, and 14 words more per block of the second
    const lora_table_t both[] = {t3, t4};
    const lora_batch_t few{1024, 1024, off.data(), ad.data()};
    for (int i = 0; i < 1024; ++i) ad[i] = i % 16;
    for (int m : {1, 2}) {
        g_launches = 0;
        CHECK(lora_plan_create_multi(&p, m, both, &few, nullptr) == LORA_OK, "multi: %s", lora_last_error());
        CHECK(g_launches == 2, "%d projections: %d launches", m, g_launches);
        lora_plan_destroy(p);
    }
    // the base projection's tile list
    for (int i = 0; i < n; ++i) ad[i] = i % 128;
    lora_base_plan_t bp = nullptr;
    g_blob.clear();
    g_launches = 0;
    CHECK(lora_base_plan_create(&bp, t3, &b, nullptr) == LORA_OK, "base: %s", lora_last_error());
    CHECK(g_launches == 1, "%d launches", g_launches);
    const std::vector<uint32_t> staged = g_blob;
    lora_base_plan_destroy(bp);
    g_hold = true;
    for (int k = 0; k < 9; ++k) {
        g_blob.clear();
        CHECK(lora_base_plan_create(&bp, t3, &b, nullptr) == LORA_OK, "base: %s", lora_last_error());
        CHECK(g_blob == staged && staged.size() >= 4 * (size_t)n, "tile list, call %d: %zu words", k, g_blob.size());
        lora_base_plan_destroy(bp);
    }
    g_hold = false;
    lora_release_adapters(t3);
    lora_release_adapters(t4);
}

}  // namespace

int main() {
    check_staged_lists();
    check_failed_update();
    check_arming_is_spread();
    check_parts_fit();
    if (failures) {
        std::fprintf(stderr, "%d checks failed\n", failures);
        return 1;
    }
    std::printf("plan_calls: all checks passed\n");
    return 0;
}
