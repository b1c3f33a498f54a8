// Host side of the C ABI declared in include/lora.h: adapter registry,
// argument validation, the rank-bucketed planner and the launches.
//
// Everything a call needs is checked here before anything is enqueued, so a
// bad argument never reaches a kernel.  The planner turns the step's segments
// into (a) the rows grouped by adapter and (b) flat lists of work items sized
// by bytes.  A plan depends on the batch, the ranks and the shapes only; each
// launch carries the weight pointers and scales of the table it is applied
// to, so one plan serves every compatible table.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "lora.h"
#include "lora_internal.h"
#include "lora_plan.h"

namespace lora {
hipError_t launch_shrink(const KernelArgs& a, const uint32_t* hdr, int dtype, hipStream_t s);
hipError_t launch_expand(const KernelArgs& a, const uint32_t* hdr, int dtype, hipStream_t s);
hipError_t launch_reduce(const KernelArgs& a, const uint32_t* hdr, hipStream_t s);
hipError_t launch_step(const KernelArgs& a, const uint32_t* hdr, int dtype, hipStream_t s);
hipError_t launch_fill(uint32_t* p, uint32_t v, uint64_t n_words, hipStream_t s);
hipError_t launch_base(const BaseArgs& a, int dtype, hipStream_t s);
int set_error(int code, const std::string& msg);
}  // namespace lora

using namespace lora;

namespace lora {

template <bool kStaged>
__global__ void __launch_bounds__(kThreads) lora_plan_kernel(PlanArgs a) {
    // read through the argument segment: a lane-dependent index into the
    // parameter would copy it to private memory
    const unsigned char* args = (const unsigned char*)__builtin_amdgcn_kernarg_segment_ptr();
    const uint32_t* data = kStaged ? a.staged : (const uint32_t*)(args + offsetof(PlanArgs, data));
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const int t = threadIdx.x;
    const int n_item_blocks = a.n_rows * a.slices;
    if ((int)blockIdx.x >= n_item_blocks) {   // (in one block, behind the items' branch: three branches in front of it cost 0.5 us)
        if ((int)blockIdx.x > n_item_blocks + a.arm_blocks) {
            const int at = ((int)blockIdx.x - n_item_blocks - a.arm_blocks - 1) * kBlobWords;
            uint32_t* dst = (uint32_t*)(a.w + a.off_blob);
            for (int q = at + t; q < min_i(at + kBlobWords, a.blob_words); q += kThreads) dst[q] = data[a.blob_at + q];
            return;
        }
        if ((int)blockIdx.x > n_item_blocks) {
            // the partial and v blocks in both step buffers: the sentinel
            u32x4* p0 = (u32x4*)(a.w + a.off_step_partials);
            u32x4* p1 = p0 + a.pbuf / 4;
            const u32x4 s4 = {0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu};
            const int64_t stride = (int64_t)a.arm_blocks * kThreads;
            for (int64_t q = (int64_t)(blockIdx.x - n_item_blocks - 1) * kThreads + t; q < a.arm_quads; q += stride) {
                p0[q] = s4;
                p1[q] = s4;
            }
            return;
        }
        uint32_t word;
        if (t < kHeaderBytes / 4 && header_word(a, t, word)) ((uint32_t*)a.w)[t] = word;
        if (a.first) {
            const uint16_t* count = (const uint16_t*)(args + offsetof(PlanArgs, step_count));
            u32x4* step = (u32x4*)(a.w + a.off_step);
            for (int q = t; q < 8 * a.step_len * a.n_xcd; q += kThreads)
                if ((q >> 3) / a.n_xcd >= (int)count[(q >> 3) % a.n_xcd]) step[q] = u32x4{0u, 0u, 0u, 0u};
        }
        return;
    }
    int slice = 0, block = blockIdx.x;        // (no division: few slices, most often one)
    for (; block >= a.n_rows; block -= a.n_rows) ++slice;
    const PlanRow r = ((const PlanRow*)data)[block];
    const int32_t* rows = (const int32_t*)data + a.n_rows * kRowWords + (r.row0 >= 0 ? 0 : -1 - r.row0);
    const PlanDims d = *(const PlanDims*)(args + offsetof(PlanArgs, dims) + r.proj() * sizeof(PlanDims));
    const RowGeom g = row_geom(d, r);
    const DevItem base = row_item(r, g, a.row_first + block, rows);
    const int n_reduce = g.direct ? 0 : g.nslice;
    const int total = g.nsplit + n_reduce + g.ntiles + g.nslice;
    const int part = t & 7;                   // this thread's 16 bytes of an item
    for (int q = slice * (kThreads / 8) + (t >> 3); q < total; q += a.slices * (kThreads / 8)) {
        DevItem it = base;
        int c = q, at, queue = -1;            // place in its list, and in its XCD's queue
        uint64_t list;
        if (c < g.nsplit) {
            to_shrink(it, d, g, c);
            list = a.off_shrink;
            at = r.shrink_at + c;
            queue = r.step_shrink + c;
        } else if ((c -= g.nsplit) < n_reduce) {
            to_reduce(it, g, c);
            list = a.off_reduce;
            at = r.reduce_at + c;
            queue = r.step_reduce + c;
        } else if ((c -= n_reduce) < g.ntiles) {
            to_expand(it, d, g, c);
            list = a.off_expand;
            at = r.expand_at + c;
            queue = r.step_expand + c;
        } else {
            c -= g.ntiles;
            to_reduce(it, g, c);
            list = a.off_all;
            at = r.all_at + c;
        }
        const uint64_t fp = (uint64_t)it.part;
        u32x4 v = {(uint32_t)fp, (uint32_t)(fp >> 32), (uint32_t)it.kind, (uint32_t)it.group};
        if (part == 1) v = u32x4{(uint32_t)it.adapter, (uint32_t)it.rank, (uint32_t)it.nrows, (uint32_t)it.lo};
        if (part == 2) v = u32x4{(uint32_t)it.len, (uint32_t)it.sub, (uint32_t)it.nsplit, (uint32_t)it.p0};
        if (part == 3) v = u32x4{(uint32_t)it.pstride, (uint32_t)it.rb, (uint32_t)it.nexp, (uint32_t)it.row0};
#pragma unroll
        for (int h = 0; h < 4; ++h)
            if (part == 4 + h)
                v = u32x4{(uint32_t)it.rows[4 * h], (uint32_t)it.rows[4 * h + 1], (uint32_t)it.rows[4 * h + 2],
                          (uint32_t)it.rows[4 * h + 3]};
        ((u32x4*)(a.w + list))[8 * (int64_t)at + part] = v;
        if (a.step_len && queue >= 0) ((u32x4*)(a.w + a.off_step))[8 * ((int64_t)queue * a.n_xcd + r.home()) + part] = v;
    }
    if (slice) return;
    int32_t* perm = (int32_t*)(a.w + a.off_perm) + r.p0;
    if (r.proj() == 0 && t < r.nrows()) perm[t] = r.row0 >= 0 ? r.row0 + t : rows[t];
    if (a.arm && t == 0) ((uint32_t*)(a.w + a.off_sync))[(int64_t)(a.row_first + block) * kSyncStride] = 0u;
}

}  // namespace lora

namespace {

thread_local std::string g_err;

int fail(int code, const std::string& msg) {
    g_err = msg;
    return code;
}

}  // namespace

// the same thread-local message for the library's other host sources
int lora::set_error(int code, const std::string& msg) { return fail(code, msg); }

namespace {

#define LORA_HIP_TRY(expr)                                                                    \
    do {                                                                                      \
        hipError_t e_ = (expr);                                                               \
        if (e_ != hipSuccess)                                                                 \
            return fail(LORA_E_HIP, std::string(#expr) + ": " + hipGetErrorString(e_));       \
    } while (0)

constexpr size_t kAlign = 256;
inline size_t align_up(size_t v, size_t a = kAlign) { return (v + a - 1) / a * a; }
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Workgroups the planner aims for when it sizes the K ranges of prompt-sized
// row blocks (two per CU on a 256-CU device).
constexpr int kTargetItems = 512;

// Polling rounds a step launch's thread may spend waiting before it gives up
// (each round is a device-coherent load, about a microsecond under load), in
// all: a quarter of a second, against waits of microseconds.
constexpr int kSpinLimit = 1 << 18;

struct DeviceGuard {
    int prev = -1;
    bool ok = true;
    explicit DeviceGuard(int d) {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != d) ok = hipSetDevice(d) == hipSuccess;
    }
    ~DeviceGuard() {
        int cur = -1;
        if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
    }
};

}  // namespace

// ---------------------------------------------------------------------------
// adapter table
// ---------------------------------------------------------------------------
struct lora_table_s {
    int device = 0;
    int n_xcd = 1;                      // XCDs of the device (workgroup p of a launch runs on XCD p % n_xcd)
    int n_cu = 0;                       // compute units of the device
    int h_in = 0, h_out = 0, dtype = 0, n = 0;
    std::vector<DevAdapter> host;
    DevAdapter* dev = nullptr;
};

// ---------------------------------------------------------------------------
// plan
// ---------------------------------------------------------------------------
namespace {

struct HostPlan {
    int h_in = 0, h_out = 0, dtype = 0, n_adapters = 0;
    int n_active = 0;
    int n_groups = 0;
    int r_max = 0;
    int n_rb = 0;                       // row blocks
    int n_proj = 1;                     // projections sharing x that one launch runs (their lists one after the other)
    std::vector<int> proj_h_out;        // their h_out (n_proj > 1)
    std::vector<int64_t> rb_bytes;      // bytes each row block streams
    std::vector<int32_t> perm, group_off, group_adapter, group_rank;
    std::vector<PlanRow> rows;          // the row blocks (row0 -1: their rows are perm[p0 ..])
    PlanDims dims[kMaxProj];
    int n_shrink = 0, n_reduce = 0, n_expand = 0, n_all = 0;   // items of each list (n_all: lora_shrink's reduce items)
    int n_xcd = 1, step_len = 0;        // step grid laid out per XCD: slots per XCD (0: the lists' own order)
    uint16_t step_count[64];            // items in each XCD's queue
    int max_items = 0;                  // items of a row block (in its lists together), at most
    int n_rows = 0;
    int64_t n_partials = 0;
    // The same of the plan without ranges cut by bytes: what it is sized for.
    // A part of a batch may fall below the line from which they are cut, and
    // has to fit where the whole batch did.
    struct Counts {
        int64_t shrink = 0, reduce = 0, all = 0, partials = 0;
    } uncut;
    size_t uncut_bytes = 0, uncut_total_bytes = 0;   // total_bytes and plan_total_bytes of that plan
    size_t off_shrink = 0, off_expand = 0, off_reduce = 0, off_reduce_all = 0, off_step = 0, off_perm = 0;
    size_t plan_bytes = 0, off_partials = 0, off_sync = 0, sync_bytes = 0, total_bytes = 0;
    size_t off_step_partials = 0, step_partials_bytes = 0, plan_total_bytes = 0;
    uint32_t generation = 0;            // header word 0 of the uploaded work list
    int n_step() const { return step_len ? step_len * n_xcd : n_shrink + n_reduce + n_expand; }
};

int validate_batch(const lora_batch_t* b, int n_adapters) {
    if (!b) return fail(LORA_E_ARG, "batch is NULL");
    if (b->n_rows < 0 || b->n_segments < 0) return fail(LORA_E_ARG, "negative n_rows or n_segments");
    if (!b->seg_offset) return fail(LORA_E_ARG, "seg_offset is NULL");
    if (b->n_segments > 0 && !b->seg_adapter) return fail(LORA_E_ARG, "seg_adapter is NULL");
    if (b->seg_offset[0] != 0) return fail(LORA_E_SHAPE, "seg_offset[0] must be 0");
    for (int s = 0; s < b->n_segments; ++s) {
        if (b->seg_offset[s + 1] < b->seg_offset[s])
            return fail(LORA_E_SHAPE, "seg_offset decreases at segment " + std::to_string(s));
        const int a = b->seg_adapter[s];
        if (a < -1 || a >= n_adapters)
            return fail(LORA_E_INDEX, "segment " + std::to_string(s) + " has adapter index " +
                                          std::to_string(a) + " outside [-1, " +
                                          std::to_string(n_adapters) + ")");
    }
    if (b->seg_offset[b->n_segments] != b->n_rows)
        return fail(LORA_E_SHAPE, "seg_offset[n_segments] != n_rows");
    return LORA_OK;
}

// Stable grouping: groups in order of the first row that uses the adapter,
// rows ascending inside a group, adapter -1 dropped.  O(n_rows + n_adapters).
void group_rows(const lora_batch_t* b, int n_adapters, std::vector<int32_t>& perm,
                std::vector<int32_t>& group_off, std::vector<int32_t>& group_adapter) {
    std::vector<int32_t> gid(n_adapters, -1);
    std::vector<int32_t> count;
    group_adapter.clear();
    for (int s = 0; s < b->n_segments; ++s) {
        const int a = b->seg_adapter[s];
        const int len = b->seg_offset[s + 1] - b->seg_offset[s];
        if (a < 0 || len == 0) continue;
        if (gid[a] < 0) {
            gid[a] = (int32_t)group_adapter.size();
            group_adapter.push_back(a);
            count.push_back(0);
        }
        count[gid[a]] += len;
    }
    const int G = (int)group_adapter.size();
    group_off.assign(G + 1, 0);
    for (int g = 0; g < G; ++g) group_off[g + 1] = group_off[g] + count[g];
    perm.assign(group_off[G], 0);
    std::vector<int32_t> fill(group_off.begin(), group_off.end() - 1);
    for (int s = 0; s < b->n_segments; ++s) {
        const int a = b->seg_adapter[s];
        // an empty segment may name an adapter that no row uses (no group)
        if (a < 0 || b->seg_offset[s + 1] == b->seg_offset[s]) continue;
        int32_t& f = fill[gid[a]];
        for (int t = b->seg_offset[s]; t < b->seg_offset[s + 1]; ++t) perm[f++] = t;
    }
}

int plan_lists(const lora_table_s* t, const lora_batch_t* b, HostPlan& p) {
    int rc = validate_batch(b, t->n);
    if (rc) return rc;
    p.h_in = t->h_in;
    p.h_out = t->h_out;
    p.dtype = t->dtype;
    p.n_adapters = t->n;
    group_rows(b, t->n, p.perm, p.group_off, p.group_adapter);
    p.n_groups = (int)p.group_adapter.size();
    p.n_active = p.n_groups ? p.group_off[p.n_groups] : 0;
    p.group_rank.assign(p.n_groups, 0);
    p.r_max = 0;
    p.n_rows = b->n_rows;
    p.rows.clear();
    p.rb_bytes.clear();
    p.n_proj = 1;
    p.n_partials = 0;
    p.uncut = {};
    p.max_items = 0;
    p.n_shrink = p.n_reduce = p.n_expand = p.n_all = 0;

    // Row blocks of more than 16 rows (prompt segments, popular adapters) are
    // cut into about kTargetItems / (number of such blocks) K ranges: few
    // such blocks get one pass per item (as the small blocks do), many get
    // fewer, longer items that stream their range in several passes.
    //
    int big_blocks = 0, blocks = 0;
    int64_t units = 0, small_units = 0, small_items = 0, small_bytes = 0;   // small: decode blocks that can stream
    for (int g = 0; g < p.n_groups; ++g) {
        const int r = t->host[p.group_adapter[g]].rank;
        const int rb = row_block(r);
        const int n = p.group_off[g + 1] - p.group_off[g];
        for (int q0 = 0; q0 < n; q0 += rb) {
            const int nb = std::min(rb, n - q0);
            units += nb + r;
            ++blocks;
            if (nb > kInlineRows) {
                ++big_blocks;
            } else if (shrink_can_dma(r, nb)) {
                small_units += nb + r;
                small_items += (t->h_in + shrink_sub(r, nb) - 1) / shrink_sub(r, nb);
                small_bytes += (int64_t)r * t->h_in * 2;
            }
        }
    }
    PlanDims& d = p.dims[0];
    d.h_in = t->h_in;
    d.h_out = t->h_out;
    d.big_split = big_blocks ? std::max(1, (kTargetItems + big_blocks - 1) / big_blocks) : 1;
    d.units = d.items = 0;
    d.small_step = 0;
    // A step whose shrink and expand items fit one round of workgroups
    // (decode) lets expand items add small partial blocks themselves, one hop
    // fewer on its critical path; larger steps add them in reduce items,
    // which leaves each expand item one v block to read (measured: 13B layer
    // 115.5 -> 110 us, decode step +0.1 us had it done so too).
    int64_t step_items = 0;
    for (int g = 0; g < p.n_groups; ++g) {
        const int r = t->host[p.group_adapter[g]].rank;
        const int rb = row_block(r);
        const int n = p.group_off[g + 1] - p.group_off[g];
        for (int q0 = 0; q0 < n; q0 += rb) {
            const RowGeom q = row_geom(d, r, std::min(rb, n - q0));
            step_items += q.nsplit + q.ntiles;
            p.uncut.shrink += q.nsplit;
            p.uncut.reduce += q.nslice;
            p.uncut.partials += (int64_t)(q.nsplit + 1) * q.pstride;
        }
    }
    p.uncut.all = p.uncut.reduce;
    d.small_step = step_items <= kTargetItems;
    // Steps whose decode blocks alone would take a round or more of one-pass
    // shrink items of 16 KiB and up, and that prompt blocks do not dominate, have
    // all blocks cut by bytes into about one round, a decode block's range
    // streaming in several passes: an item's fixed part (launch, work item,
    // pointer: about half of its 7 us at one pass of 32 KiB) is then paid once per
    // range.  Measured per launch, one pass per decode item against ranges: 70B-
    // shaped q and gate (256 tokens, 4 prompts of 512) 283 -> 251 us, 65 adapters of
    // rank 16 at 5120 -> 2768 16.2 -> 13.8.  Where an item would pass 64 KiB it is one
    // round and a half: that costs the 70B-shaped step 2% (246 us in 512 items; 257
    // in 1024, 266 in 1536) and keeps the steps that gain nothing from it from
    // losing (57 tokens of rank 8-128 at 8192 -> 3872: one pass 28.1 us, 768 items
    // 28.2, 512 29.2).  Past the lines it turns: 131 tokens at 9264 -> 13824 (485
    // decode items, one round anyway) 29.0 -> 30.6, 43 tokens of rank 8 at 12120 11.9
    // -> 13.0, 25 adapters beside 12 prompts of up to 364 tokens 49.5 -> 55.4 us.
    // (The cut depends on one projection only: a launch of several equals one
    // launch each, bit for bit.)
    if (!d.small_step && small_items >= kTargetItems && small_bytes >= (small_items << 14) &&
        3 * small_units >= units && units <= INT32_MAX) {
        const bool wide = units * t->h_in * 2 >= (int64_t)kTargetItems << 16;
        d.units = (int32_t)units;
        d.items = std::max(wide ? 3 * kTargetItems / 2 : kTargetItems, blocks);
    }

    for (int g = 0; g < p.n_groups; ++g) {
        const int r = t->host[p.group_adapter[g]].rank;
        p.group_rank[g] = r;
        p.r_max = std::max(p.r_max, r);
        const int rb = row_block(r);
        for (int p0 = p.group_off[g]; p0 < p.group_off[g + 1]; p0 += rb) {
            const int nb = std::min(rb, p.group_off[g + 1] - p0);
            const RowGeom q = row_geom(d, r, nb);
            if (shrink_lds_bytes(r, q.sub, nb) > kShrinkLds || !expand_fits_lds(r, nb))
                return fail(LORA_E_SHAPE, "internal: a tile exceeds LDS");
            PlanRow row{};
            row.group = g;
            row.adapter = p.group_adapter[g];
            row.shape = (int32_t)((uint32_t)(r | nb << 16) | (uint32_t)(q.sub / 32) << 26);
            row.cut = q.krange / q.sub << 8;
            row.p0 = p0;
            // the last row is nb - 1 past the first only when all are consecutive (rows ascend)
            row.row0 = p.perm[p0 + nb - 1] == p.perm[p0] + nb - 1 ? p.perm[p0] : -1;
            if ((uint64_t)(p.n_partials + (int64_t)(q.nsplit + 1) * q.pstride) * 4 > kMaxSpan)
                return fail(LORA_E_SHAPE, "batch too large: its partial results exceed 2 GiB");
            row.part = (uint32_t)p.n_partials;
            row.shrink_at = p.n_shrink;
            row.reduce_at = p.n_reduce;
            row.expand_at = p.n_expand;
            row.all_at = p.n_all;
            p.n_shrink += q.nsplit;
            p.n_reduce += q.direct ? 0 : q.nslice;
            p.n_expand += q.ntiles;
            p.n_all += q.nslice;
            p.max_items = std::max(p.max_items, q.nsplit + (q.direct ? 1 : 2) * q.nslice + q.ntiles);
            // the row block's nsplit partial blocks, then its v block
            p.n_partials += (int64_t)(q.nsplit + 1) * q.pstride;
            p.rb_bytes.push_back((int64_t)(r + nb) * t->h_in * 2 + (int64_t)(r + 2 * nb) * t->h_out * 2);
            p.rows.push_back(row);
        }
    }
    p.n_rb = (int)p.rows.size();
    if (d.items == 0) p.uncut = {p.n_shrink, p.n_reduce, p.n_all, p.n_partials};
    return LORA_OK;
}

// The lists of n projections that share x, one after the other: projection c
// carries c in its kind, its own partial and v blocks and its own row block
// counters (offsets past the projections before it).  Each projection's
// items wait only on items of the same projection.
int append_lists(HostPlan& p, const HostPlan& q, int c) {
    if ((uint64_t)(p.n_partials + q.n_partials) * 4 > kMaxSpan)
        return fail(LORA_E_SHAPE, "batch too large: its partial results exceed 2 GiB");
    for (PlanRow r : q.rows) {
        r.shape |= c << 24;
        r.part += (uint32_t)p.n_partials;
        r.shrink_at += p.n_shrink;
        r.reduce_at += p.n_reduce;
        r.expand_at += p.n_expand;
        r.all_at += p.n_all;
        p.rows.push_back(r);
    }
    p.dims[c] = q.dims[0];
    p.n_shrink += q.n_shrink;
    p.n_reduce += q.n_reduce;
    p.n_expand += q.n_expand;
    p.n_all += q.n_all;
    p.rb_bytes.insert(p.rb_bytes.end(), q.rb_bytes.begin(), q.rb_bytes.end());
    p.n_partials += q.n_partials;
    p.n_rb += q.n_rb;
    p.max_items = std::max(p.max_items, q.max_items);
    p.uncut.shrink += q.uncut.shrink;
    p.uncut.reduce += q.uncut.reduce;
    p.uncut.all += q.uncut.all;
    p.uncut.partials += q.uncut.partials;
    return LORA_OK;
}

// The grid layout and the device layout of the lists.
int plan_layout(const lora_table_s* t, HostPlan& p) {
    const std::vector<int64_t>& rb_bytes = p.rb_bytes;
    // A step small enough to run in one round of workgroups (decode) gets a
    // grid laid out per XCD: workgroup p of a launch runs on XCD p % n_xcd (the
    // order in which the hardware hands workgroups to the XCDs), every row
    // block gets one XCD (largest first, each to the XCD with the fewest bytes
    // so far), and on each XCD its shrink, reduce and expand items follow in
    // that order, slots it does not need holding items of no kind.  A row
    // block's partial and v blocks then stay in one L2 and one fabric path.
    // Larger steps keep the list order: there the balance of the whole grid
    // matters more (measured: the decode step 12.9 -> 12.2 us, the 13B-layer,
    // 70B and prompt steps 2-5% slower with the layout), and so do steps whose
    // row blocks cannot be spread evenly (the busiest XCD above 1.25 times the
    // average).  Every item still waits only on items earlier in the grid,
    // whatever the hardware does.
    p.step_len = 0;
    p.n_xcd = t->n_xcd;
    if (t->n_xcd > 1 && p.uncut.shrink + p.uncut.reduce + p.n_expand <= kTargetItems) {
        const int nx = t->n_xcd;
        std::vector<int> home(p.n_rb, 0), order(p.n_rb);
        for (int i = 0; i < p.n_rb; ++i) order[i] = i;
        std::stable_sort(order.begin(), order.end(), [&](int u, int v) { return rb_bytes[u] > rb_bytes[v]; });
        std::vector<int64_t> load(nx, 0);
        for (int i : order) {
            const int x = (int)(std::min_element(load.begin(), load.end()) - load.begin());
            home[i] = x;
            load[x] += rb_bytes[i];
        }
        // only when the XCDs come out balanced: a step of few row blocks
        // (few adapters) would otherwise leave XCDs idle
        int64_t total = 0, most = 0;
        for (int64_t v : load) {
            total += v;
            most = std::max(most, v);
        }
        if (4 * most * nx <= 5 * total) {
            // every XCD's queue: its shrink, then its reduce, then its expand items
            std::vector<int> at(nx, 0);
            for (int kind = 0; kind < 3; ++kind)
                for (int i = 0; i < p.n_rb; ++i) {
                    PlanRow& r = p.rows[i];
                    const RowGeom q = row_geom(p.dims[r.proj()], r);
                    int& u = at[home[i]];
                    r.cut |= kind == 0 ? home[i] : 0;
                    (kind == 0 ? r.step_shrink : (kind == 1 ? r.step_reduce : r.step_expand)) = u;
                    u += kind == 0 ? q.nsplit : (kind == 1 ? (q.direct ? 0 : q.nslice) : q.ntiles);
                }
            for (int x = 0; x < nx; ++x) {
                p.step_count[x] = (uint16_t)at[x];
                p.step_len = std::max(p.step_len, at[x]);
            }
        }
    }

    // device layout: [header][shrink items][reduce items][expand items][all reduce
    // items][step grid laid out per XCD, small steps only][perm] | [partial and v blocks][row block counters, status] (a
    // workspace ends here) | [step partial and v blocks x 2] (plans only: the
    // step launch's blocks in two buffers used by alternate launches, each
    // armed with the sentinel before the launch that reads it).  The first
    // three lists are contiguous: the step launch runs them as one grid (or the
    // fifth, the same items laid out per XCD); the separate launches run one
    // each, lora_shrink the fourth.
    size_t off = kHeaderBytes;                // the header (generation, status) comes first
    p.off_shrink = off;
    off += (size_t)p.n_shrink * sizeof(DevItem);
    p.off_reduce = off;
    off += (size_t)p.n_reduce * sizeof(DevItem);
    p.off_expand = off;
    off += (size_t)p.n_expand * sizeof(DevItem);
    p.off_reduce_all = off;
    off += (size_t)p.n_all * sizeof(DevItem);
    p.off_step = off;
    off = align_up(off + (size_t)p.step_len * p.n_xcd * sizeof(DevItem));
    p.off_perm = off;
    off = align_up(off + p.perm.size() * sizeof(int32_t));
    p.plan_bytes = off;
    p.off_partials = off;
    off = align_up(off + (size_t)p.n_partials * sizeof(float));
    p.off_sync = off;
    p.sync_bytes = align_up(std::max<size_t>(1, (size_t)p.n_rb) * kSyncStride * sizeof(uint32_t));
    off += p.sync_bytes;
    p.total_bytes = std::max<size_t>(off, kAlign);
    p.off_step_partials = off;
    p.step_partials_bytes = 2 * align_up((size_t)p.n_partials * sizeof(float));   // two buffers
    p.plan_total_bytes = std::max<size_t>(off + p.step_partials_bytes, kAlign);

    // the same sizes without ranges cut by bytes
    const size_t items = (size_t)(p.uncut.shrink + p.uncut.reduce + p.n_expand + p.uncut.all) + (size_t)p.step_len * p.n_xcd;
    off = align_up(kHeaderBytes + items * sizeof(DevItem));
    off = align_up(off + p.perm.size() * sizeof(int32_t));
    off = align_up(off + (size_t)p.uncut.partials * sizeof(float)) + p.sync_bytes;
    p.uncut_bytes = std::max<size_t>(off, kAlign);
    p.uncut_total_bytes = std::max<size_t>(off + 2 * align_up((size_t)p.uncut.partials * sizeof(float)), kAlign);
    return LORA_OK;
}

// The items of the single launch in grid order, and lora_shrink's reduce items,
// as lora_plan_kernel writes them.
void list_items(const HostPlan& p, std::vector<DevItem>& grid, std::vector<DevItem>& all) {
    grid.assign(p.n_step(), DevItem{});
    all.assign(p.n_all, DevItem{});
    for (int i = 0; i < p.n_rb; ++i) {
        const PlanRow& r = p.rows[i];
        const PlanDims& d = p.dims[r.proj()];
        const RowGeom g = row_geom(d, r);
        const DevItem base = row_item(r, g, i, p.perm.data() + r.p0);
        auto slot = [&](int queue, int list) -> DevItem& {
            return grid[p.step_len ? (size_t)queue * p.n_xcd + r.home() : (size_t)list];
        };
        for (int c = 0; c < g.nsplit; ++c) {
            DevItem it = base;
            to_shrink(it, d, g, c);
            slot(r.step_shrink + c, r.shrink_at + c) = it;
        }
        for (int c = 0; c < g.nslice; ++c) {
            DevItem it = base;
            to_reduce(it, g, c);
            all[r.all_at + c] = it;
            if (!g.direct) slot(r.step_reduce + c, p.n_shrink + r.reduce_at + c) = it;
        }
        for (int c = 0; c < g.ntiles; ++c) {
            DevItem it = base;
            to_expand(it, d, g, c);
            slot(r.step_expand + c, p.n_shrink + p.n_reduce + r.expand_at + c) = it;
        }
    }
}

int build_plan(const lora_table_s* t, const lora_batch_t* b, HostPlan& p) {
    if (int rc = plan_lists(t, b, p)) return rc;
    return plan_layout(t, p);
}

// One plan for n projections that share x (the same h_in and dtype, the
// batch's adapters of the same ranks in every table; h_out may differ).
int build_plan_multi(const lora_table_s* const* t, int n, const lora_batch_t* b, HostPlan& p) {
    if (int rc = plan_lists(t[0], b, p)) return rc;
    p.proj_h_out.assign(1, t[0]->h_out);
    for (int c = 1; c < n; ++c) {
        if (t[c]->h_in != t[0]->h_in || t[c]->dtype != t[0]->dtype)
            return fail(LORA_E_SHAPE, "the projections differ in h_in or dtype");
        HostPlan q;
        if (int rc = plan_lists(t[c], b, q)) return rc;
        if (int rc = append_lists(p, q, c)) return rc;
        p.proj_h_out.push_back(t[c]->h_out);
    }
    p.n_proj = n;
    return plan_layout(t[0], p);
}

int check_compatible(const HostPlan& p, const lora_table_s* t);

// Projection i of a plan of several projections: its table must agree with
// the plan in h_in, dtype, its projection's h_out and the referenced ranks.
int check_compatible_proj(const HostPlan& p, const lora_table_s* t, int i) {
    if (!t || !t->dev) return fail(LORA_E_ARG, "table is NULL or released");
    if (p.n_proj > 1 && t->h_out != p.proj_h_out[i])
        return fail(LORA_E_SHAPE, "table " + std::to_string(i) + " has another h_out than its projection in the plan");
    if (p.n_proj <= 1) return check_compatible(p, t);
    if (t->h_in != p.h_in || t->dtype != p.dtype) return fail(LORA_E_SHAPE, "table shape or dtype differs from the plan's");
    for (int g = 0; g < p.n_groups; ++g) {
        const int a = p.group_adapter[g];
        if (a >= t->n) return fail(LORA_E_INDEX, "table has fewer adapters than the plan references");
        if (t->host[a].rank != p.group_rank[g])
            return fail(LORA_E_RANK, "adapter " + std::to_string(a) + " has another rank than in the plan");
    }
    return LORA_OK;
}

// A table may run a plan made with another table when shapes, dtype and the
// ranks of every adapter the plan references agree.
int check_compatible(const HostPlan& p, const lora_table_s* t) {
    if (!t || !t->dev) return fail(LORA_E_ARG, "table is NULL or released");
    if (t->h_in != p.h_in || t->h_out != p.h_out || t->dtype != p.dtype)
        return fail(LORA_E_SHAPE, "table shape or dtype differs from the plan's");
    for (int g = 0; g < p.n_groups; ++g) {
        const int a = p.group_adapter[g];
        if (a >= t->n) return fail(LORA_E_INDEX, "table has fewer adapters than the plan references");
        if (t->host[a].rank != p.group_rank[g])
            return fail(LORA_E_RANK, "adapter " + std::to_string(a) + " has another rank than in the plan");
    }
    return LORA_OK;
}

// The calls that write a work list into device memory are not recorded in
// graphs: a replay would write the recorded batch's again, under launches made
// for another.  They refuse a capturing stream before enqueuing anything.
int check_not_capturing(hipStream_t s, const char* what) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    LORA_HIP_TRY(hipStreamIsCapturing(s, &cs));
    if (cs != hipStreamCaptureStatusNone)
        return fail(LORA_E_CAPTURE, std::string(what) +
                                        " cannot be recorded in a graph (it writes the work list that other "
                                        "launches run); record lora_plan_apply / _shrink / _expand instead");
    return LORA_OK;
}

// Pinned host memory for lists too large for kernel arguments: kStageSlots slots per
// device, allocated by the first such list and given back with the device's last table
// (taken with the first table instead, they cost every program 35 us and more).  A
// launch behind the one that reads a slot writes the slot's use number back; a slot is
// taken again once its last use has come back, and the host never waits for one (no
// event either: asking for one would break a capture on another stream).
struct StageRing {
    std::mutex mu;
    int tables = 0;
    bool tried = false;                       // allocated, or not to be had
    uint32_t* host = nullptr;                 // kStageSlots times kStagedWords, then the use numbers
    uint32_t* dev = nullptr;                  // the same as the device addresses it
    uint32_t uses[kStageSlots] = {};          // last use of each slot
    unsigned next = 0;
    static constexpr size_t kWords = (size_t)kStageSlots * (kStagedWords + kSyncStride);
    static size_t use_at(int slot) { return (size_t)kStageSlots * kStagedWords + (size_t)slot * kSyncStride; }
};
constexpr int kMaxDevices = 64;
StageRing g_stage[kMaxDevices];

void stage_retain(int device) {
    if (device >= kMaxDevices) return;
    std::lock_guard<std::mutex> lk(g_stage[device].mu);
    ++g_stage[device].tables;
}
void stage_release(int device) {
    if (device >= kMaxDevices) return;
    StageRing& r = g_stage[device];
    std::lock_guard<std::mutex> lk(r.mu);
    if (--r.tables) return;
    if (r.host) (void)hipHostFree(r.host);
    r.host = nullptr;
    r.dev = nullptr;
    r.tried = false;
}
// (the ring's mutex held, its device current; without the memory every list goes in
// arguments)
void stage_allocate(StageRing& r) {
    r.tried = true;
    // a thread that captures another stream meanwhile is not disturbed
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    if (hipThreadExchangeStreamCaptureMode(&mode) != hipSuccess) return (void)hipGetLastError();
    if (hipHostMalloc((void**)&r.host, sizeof(uint32_t) * StageRing::kWords, hipHostMallocMapped | hipHostMallocCoherent) !=
        hipSuccess)
        r.host = nullptr;
    if (!r.host || hipHostGetDevicePointer((void**)&r.dev, r.host, 0) != hipSuccess) {
        r.dev = nullptr;
        (void)hipGetLastError();
    }
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    for (int i = 0; i < kStageSlots; ++i) {
        r.uses[i] = 0;
        if (r.host) r.host[StageRing::use_at(i)] = 0;
    }
}
// A free slot, or -1 (the ring's mutex held).
int stage_take(StageRing& r, bool may_allocate) {
    if (!r.tried && may_allocate) stage_allocate(r);
    if (!r.dev) return -1;
    const int i = (int)(r.next % kStageSlots);
    if (__atomic_load_n(r.host + StageRing::use_at(i), __ATOMIC_ACQUIRE) != r.uses[i]) return -1;
    ++r.next;
    return i;
}

// Row blocks of p from the i-th on, then their listed rows, into the room words at dst:
// as many as fit.  Moves i past them and returns the words.
size_t pack_rows(const HostPlan& p, size_t& i, size_t room, uint32_t* dst) {
    const size_t i0 = i;
    size_t words = 0;
    for (; i < p.rows.size(); ++i) {
        const size_t need = kRowWords + p.rows[i].listed();
        if (words + need > room) break;
        words += need;
    }
    const size_t lists = (i - i0) * kRowWords;
    size_t at = lists;
    for (size_t j = i0; j < i; ++j) {
        PlanRow r = p.rows[j];
        if (const int n = r.listed()) {
            r.row0 = -1 - (int32_t)(at - lists);
            std::memcpy(dst + at, p.perm.data() + r.p0, sizeof(int32_t) * n);
            at += n;
        }
        std::memcpy(dst + (j - i0) * kRowWords, &r, sizeof r);
    }
    return words;
}

// Write plan p's header, work list and grouped row order into the memory at w
// (and, for a plan, clear its counters and arm its step buffers), and blob_bytes
// (a multiple of 4) from blob to w + off_blob.  The data ride in the arguments of up to
// kArgLaunches launches (64 row blocks of consecutive rows each, 11 of 64 listed rows);
// more of them, some thousand scattered rows or runs, in pinned memory that one launch
// reads.  No device allocation, no copy engine, nothing that the host or a later call
// waits for.
int write_plan(const HostPlan& p, unsigned char* w, bool arm, int device, hipStream_t s, const void* blob = nullptr,
               size_t blob_bytes = 0, size_t off_blob = 0, bool may_allocate = true) {
    PlanArgs a{};
    a.w = w;
    a.off_shrink = p.off_shrink;
    a.off_reduce = p.off_reduce;
    a.off_expand = p.off_expand;
    a.off_all = p.off_reduce_all;
    a.off_step = p.off_step;
    a.off_perm = p.off_perm;
    a.off_sync = p.off_sync;
    a.off_step_partials = p.off_step_partials;
    a.pbuf = (int64_t)(p.step_partials_bytes / 2 / sizeof(float));
    a.generation = p.generation;
    a.arm = arm;
    a.n_xcd = p.n_xcd;
    a.step_len = p.step_len;
    a.slices = std::max(1, std::min(kMaxSlices, (p.max_items + kSliceItems - 1) / kSliceItems));
    for (int c = 0; c < p.n_proj; ++c) a.dims[c] = p.dims[c];
    if (p.step_len) std::memcpy(a.step_count, p.step_count, sizeof(uint16_t) * p.n_xcd);
    const size_t blob_words = blob_bytes / 4;
    size_t left = blob_words;                 // words not yet on their way
    for (const PlanRow& r : p.rows) left += kRowWords + r.listed();
    size_t i = 0, blob_at = 0;
    a.first = 1;
    do {
        StageRing* ring = left > (size_t)kArgLaunches * kPlanWords && device < kMaxDevices ? &g_stage[device] : nullptr;
        std::unique_lock<std::mutex> lk;
        if (ring) lk = std::unique_lock<std::mutex>(ring->mu);
        const int slot = ring ? stage_take(*ring, may_allocate) : -1;
        const size_t room = slot >= 0 ? kStagedWords : kPlanWords;
        uint32_t* data = slot >= 0 ? ring->host + (size_t)slot * kStagedWords : a.data;
        a.staged = slot >= 0 ? ring->dev + (size_t)slot * kStagedWords : nullptr;
        a.row_first = (int32_t)i;
        const size_t words = pack_rows(p, i, room, data);
        a.n_rows = (int32_t)(i - a.row_first);
        a.blob_words = i == p.rows.size() ? (int32_t)std::min(room - words, blob_words - blob_at) : 0;
        a.blob_at = (int32_t)words;
        a.off_blob = off_blob + 4 * blob_at;
        if (a.blob_words) std::memcpy(data + words, (const unsigned char*)blob + 4 * blob_at, 4 * (size_t)a.blob_words);
        blob_at += a.blob_words;
        left -= words + a.blob_words;
        a.last = left == 0;
        a.arm_quads = a.first && arm ? (int32_t)(p.n_partials / 4) : 0;
        a.arm_blocks = std::min(kArmBlocks, (a.arm_quads + kArmQuads - 1) / kArmQuads);
        const dim3 grid(a.n_rows * a.slices + 1 + a.arm_blocks + (a.blob_words + kBlobWords - 1) / kBlobWords);
        if (slot >= 0) hipLaunchKernelGGL(lora_plan_kernel<true>, grid, dim3(kThreads), 0, s, a);
        else hipLaunchKernelGGL(lora_plan_kernel<false>, grid, dim3(kThreads), 0, s, a);
        LORA_HIP_TRY(hipGetLastError());
        if (slot >= 0) LORA_HIP_TRY(launch_fill(ring->dev + StageRing::use_at(slot), ++ring->uses[slot], 1, s));
        a.first = 0;
    } while (left);
    return LORA_OK;
}

// The allocation-free entry point's workspace: one array per device, set up
// by the HIP runtime when the library's code object is loaded there and kept
// until the process ends.  Host code never takes its address directly (that
// would be a host-side stand-in, not device memory): the first call on each
// device looks the device address up and keeps it.
constexpr size_t kScratchBytes = size_t(16) << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
std::mutex g_scratch_mu;
unsigned char* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on `device` (which must be current).
int scratch_address(int device, unsigned char** out) {
    if (device < 0 || device >= kMaxDevices) return fail(LORA_E_ARG, "device index beyond the static scratch table");
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[device]) {
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr)
            return fail(LORA_E_HIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        g_scratch_ptr[device] = (unsigned char*)ptr;
    }
    *out = g_scratch_ptr[device];
    return LORA_OK;
}

// Launch arguments of one plan on one table: the plan's buffers in workspace
// w and the factor pointers and scales of its groups.
KernelArgs make_args(const lora_table_s* t, const HostPlan& p, unsigned char* w, int spin_limit) {
    KernelArgs a{};
    a.perm = (const int32_t*)(w + p.off_perm);
    a.table = t->dev;
    a.partials = (float*)(w + p.off_partials);
    a.sync = (uint32_t*)(w + p.off_sync);
    a.status = (int32_t*)(w + sizeof(uint32_t));   // header word 1
    a.generation = p.generation;
    a.pbuf = (int64_t)(p.step_partials_bytes / 2 / sizeof(float));
    a.spin_limit = spin_limit;
    a.h_in = t->h_in;
    a.h_out = t->h_out;
    a.n_groups = p.n_groups;
    for (int c = 0; c < p.n_proj; ++c) a.streams |= p.dims[c].items > 0;
    const int ng = std::min(p.n_groups, kKargGroups);
    for (int g = 0; g < ng; ++g) {
        const DevAdapter& ad = t->host[p.group_adapter[g]];
        a.gfac[2 * g] = ad.A;
        a.gfac[2 * g + 1] = ad.B;
        a.gscale[g] = ad.scale;
    }
    return a;
}

int check_table(const lora_table_s* t) {
    if (!t || !t->dev) return fail(LORA_E_ARG, "table is NULL or released");
    return LORA_OK;
}

int check_ld(const char* name, int64_t ld, int h) {
    if (ld < h || ld % 8 != 0)
        return fail(LORA_E_SHAPE, std::string(name) + " must be a multiple of 8 and >= " +
                                      std::to_string(h));
    return LORA_OK;
}

int check_overlap(const void* x, int64_t ldx, int h_in, const void* y, int64_t ldy, int h_out,
                  int n_rows) {
    if (n_rows <= 0) return LORA_OK;
    const uintptr_t xs = (uintptr_t)x, ys = (uintptr_t)y;
    const uintptr_t xe = xs + ((uintptr_t)(n_rows - 1) * ldx + h_in) * 2;
    const uintptr_t ye = ys + ((uintptr_t)(n_rows - 1) * ldy + h_out) * 2;
    if (xs < ye && ys < xe) return fail(LORA_E_OVERLAP, "x and y overlap");
    return LORA_OK;
}

int check_ws(const HostPlan& p, const void* ws, size_t ws_bytes) {
    if (!ws) return fail(LORA_E_ARG, "workspace is NULL");
    if (!aligned16(ws)) return fail(LORA_E_ALIGN, "workspace not 16-byte aligned");
    if (ws_bytes < p.total_bytes)
        return fail(LORA_E_WORKSPACE, "workspace has " + std::to_string(ws_bytes) +
                                          " bytes, needs " + std::to_string(p.total_bytes));
    return LORA_OK;
}

// Bytes from the first element of a [n_rows, ld] matrix to the end of its
// last row of h elements.
uint64_t span_bytes(int n_rows, int64_t ld, int h) {
    return n_rows > 0 ? ((uint64_t)(n_rows - 1) * (uint64_t)ld + (uint64_t)h) * 2 : 0;
}

int check_x(const lora_table_s* t, const void* x, int64_t ldx, int n_rows) {
    if (!x) return fail(LORA_E_ARG, "x is NULL");
    if (!aligned16(x)) return fail(LORA_E_ALIGN, "x not 16-byte aligned");
    if (int rc = check_ld("ldx", ldx, t->h_in)) return rc;
    if (span_bytes(n_rows, ldx, t->h_in) > kMaxSpan) return fail(LORA_E_SHAPE, "x spans more than 2 GiB");
    return LORA_OK;
}

int check_y(const lora_table_s* t, const void* y, int64_t ldy, int n_rows) {
    if (!y) return fail(LORA_E_ARG, "y is NULL");
    if (!aligned16(y)) return fail(LORA_E_ALIGN, "y not 16-byte aligned");
    if (int rc = check_ld("ldy", ldy, t->h_out)) return rc;
    if (span_bytes(n_rows, ldy, t->h_out) > kMaxSpan) return fail(LORA_E_SHAPE, "y spans more than 2 GiB");
    return LORA_OK;
}

int check_v(const HostPlan& p, const void* v, int64_t ldv) {
    if (!v) return fail(LORA_E_ARG, "v is NULL");
    if (!aligned16(v)) return fail(LORA_E_ALIGN, "v not 16-byte aligned");
    if (ldv < p.r_max || ldv % 4)
        return fail(LORA_E_SHAPE, "ldv must be a multiple of 4 and >= the largest rank used");
    return LORA_OK;
}

// Enqueue the shrink (x != NULL) and/or the expand (y != NULL) of plan p on
// table t with its workspace at w, as separate launches: shrink, then (unless
// the caller reduces into its own v) reduce into the v blocks; expand.
int enqueue(const lora_table_s* t, const HostPlan& p, unsigned char* w, const void* x, int64_t ldx,
            void* y, int64_t ldy, hipStream_t s, bool v_out = false) {
    if (x) {
        KernelArgs a = make_args(t, p, w, kSpinLimit);
        a.items = (const DevItem*)(w + p.off_shrink);
        a.n_items = p.n_shrink;
        a.x = x;
        a.ldx = ldx;
        a.x_bytes = (uint32_t)span_bytes(p.n_rows, ldx, t->h_in);
        LORA_HIP_TRY(launch_shrink(a, (const uint32_t*)w, t->dtype, s));
        if (!v_out) {
            a.items = (const DevItem*)(w + p.off_reduce);
            a.n_items = p.n_reduce;
            LORA_HIP_TRY(launch_reduce(a, (const uint32_t*)w, s));
        }
    }
    if (y) {
        KernelArgs a = make_args(t, p, w, kSpinLimit);
        a.items = (const DevItem*)(w + p.off_expand);
        a.n_items = p.n_expand;
        a.y = y;
        a.ldy = ldy;
        a.y_bytes = (uint32_t)span_bytes(p.n_rows, ldy, t->h_out);
        LORA_HIP_TRY(launch_expand(a, (const uint32_t*)w, t->dtype, s));
    }
    return LORA_OK;
}

// Enqueue the whole step of plan p as one launch (shrink and expand items in
// one grid).  The row block counters at w + off_sync must be zero and the
// step partial blocks armed.
// The arguments of the step launch of plan p (one projection).
int step_args(const lora_table_s* t, const HostPlan& p, unsigned char* w, const void* x, int64_t ldx, void* y,
              int64_t ldy, int spin_limit, KernelArgs& out) {
    KernelArgs a = make_args(t, p, w, spin_limit);
    a.partials = (float*)(w + p.off_step_partials);
    if (p.step_len) {                         // the grid laid out per XCD
        a.items = (const DevItem*)(w + p.off_step);
        a.n_items = p.n_step();
    } else {
        a.items = (const DevItem*)(w + p.off_shrink);
        a.n_items = p.n_step();
    }
    a.x = x;
    a.ldx = ldx;
    a.x_bytes = (uint32_t)span_bytes(p.n_rows, ldx, t->h_in);
    a.y = y;
    a.ldy = ldy;
    a.y_bytes = (uint32_t)span_bytes(p.n_rows, ldy, t->h_out);
    out = a;
    return LORA_OK;
}

int enqueue_step(const lora_table_s* t, const HostPlan& p, unsigned char* w, const void* x,
                 int64_t ldx, void* y, int64_t ldy, int spin_limit, hipStream_t s) {
    KernelArgs a;
    if (int rc = step_args(t, p, w, x, ldx, y, ldy, spin_limit, a)) return rc;
    LORA_HIP_TRY(launch_step(a, (const uint32_t*)w, t->dtype, s));
    return LORA_OK;
}

// Status and row block counters to zero, both step partial buffers to the
// sentinel (all-ones words): fill kernels, no memset.  The status reset.
hipError_t arm_step(const HostPlan& p, unsigned char* w, hipStream_t s) {
    hipError_t e = launch_fill((uint32_t*)(w + sizeof(uint32_t)), 0u, 1, s);
    if (e == hipSuccess) e = launch_fill((uint32_t*)(w + p.off_sync), 0u, p.sync_bytes / sizeof(uint32_t), s);
    if (e == hipSuccess && p.step_partials_bytes)
        e = launch_fill((uint32_t*)(w + p.off_step_partials), 0xffffffffu, p.step_partials_bytes / sizeof(uint32_t), s);
    return e;
}

}  // namespace

// ---------------------------------------------------------------------------
// plan handle
// ---------------------------------------------------------------------------
struct lora_plan_s {
    const lora_table_s* table = nullptr;
    int device = 0;
    int n_rows = 0;
    int spin_limit = kSpinLimit;
    HostPlan plan;
    unsigned char* dmem = nullptr;
    size_t capacity = 0;                // device bytes at dmem, fixed at creation
    uint32_t generation = 0;            // of the work list last uploaded
};

namespace {

void plan_free(lora_plan_s* pl) {
    DeviceGuard dg(pl->device);
    if (pl->dmem) (void)hipFree(pl->dmem);
    pl->dmem = nullptr;
    delete pl;
}

// Write the plan's work list (header with a new generation, item lists, grouped
// row order) and arm its step buffers, on stream s.
int plan_upload(lora_plan_s* pl, hipStream_t s) {
    if (++pl->generation == 0) pl->generation = 1;
    pl->plan.generation = pl->generation;
    return write_plan(pl->plan, pl->dmem, true, pl->device, s);
}

}  // namespace

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
extern "C" {

int lora_abi_version(void) { return LORA_ABI_VERSION; }

const char* lora_last_error(void) { return g_err.c_str(); }

int lora_register_adapters(lora_table_t* out, int device, int h_in, int h_out, int dtype,
                           int n_adapters, const void* const* A_ptrs, const void* const* B_ptrs,
                           const int32_t* ranks, const float* scales, void* stream) {
    if (!out) return fail(LORA_E_ARG, "out is NULL");
    *out = nullptr;
    if (dtype != LORA_F16 && dtype != LORA_BF16) return fail(LORA_E_ARG, "dtype must be LORA_F16 or LORA_BF16");
    if (device < 0) return fail(LORA_E_ARG, "negative device");
    if (n_adapters < 0) return fail(LORA_E_ARG, "negative n_adapters");
    if (h_in <= 0 || h_out <= 0 || h_in % 8 || h_out % 8)
        return fail(LORA_E_SHAPE, "h_in and h_out must be positive multiples of 8");
    if ((uint64_t)std::max(h_in, h_out) * kMaxRank * 2 > kMaxSpan)
        return fail(LORA_E_SHAPE, "h_in and h_out must be at most 4 Mi elements (factors below 2 GiB)");
    if (n_adapters > 0 && (!A_ptrs || !B_ptrs || !ranks || !scales))
        return fail(LORA_E_ARG, "adapter arrays must not be NULL");
    std::vector<DevAdapter> host(n_adapters);
    for (int i = 0; i < n_adapters; ++i) {
        if (ranks[i] < 1 || ranks[i] > kMaxRank)
            return fail(LORA_E_RANK, "adapter " + std::to_string(i) + " has rank " +
                                         std::to_string(ranks[i]) + " outside [1, 256]");
        if (!A_ptrs[i] || !B_ptrs[i])
            return fail(LORA_E_ARG, "adapter " + std::to_string(i) + " has a NULL factor");
        if (!aligned16(A_ptrs[i]) || !aligned16(B_ptrs[i]))
            return fail(LORA_E_ALIGN, "adapter " + std::to_string(i) + " factor not 16-byte aligned");
        host[i].A = A_ptrs[i];
        host[i].B = B_ptrs[i];
        host[i].rank = ranks[i];
        host[i].scale = scales[i];
    }
    DeviceGuard dg(device);
    if (!dg.ok) return fail(LORA_E_HIP, "hipSetDevice failed");
    auto* t = new (std::nothrow) lora_table_s();
    if (!t) return fail(LORA_E_NOMEM, "table allocation failed");
    t->device = device;
    {
        int nx = 1;
        if (hipDeviceGetAttribute(&nx, hipDeviceAttributeNumberOfXccs, device) != hipSuccess || nx < 1) nx = 1;
        t->n_xcd = std::min(nx, 64);
        int nc = 0;
        if (hipDeviceGetAttribute(&nc, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess) nc = 0;
        t->n_cu = std::max(nc, 0);
    }
    t->h_in = h_in;
    t->h_out = h_out;
    t->dtype = dtype;
    t->n = n_adapters;
    t->host = std::move(host);
    const size_t bytes = std::max<size_t>(1, (size_t)n_adapters) * sizeof(DevAdapter);
    hipError_t e = hipMalloc((void**)&t->dev, bytes);
    if (e != hipSuccess) {
        delete t;
        return fail(LORA_E_NOMEM, std::string("hipMalloc of the adapter table: ") + hipGetErrorString(e));
    }
    if (n_adapters > 0) {
        hipStream_t s = (hipStream_t)stream;
        e = hipMemcpyAsync(t->dev, t->host.data(), n_adapters * sizeof(DevAdapter),
                           hipMemcpyHostToDevice, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) {
            (void)hipFree(t->dev);
            delete t;
            return fail(LORA_E_HIP, std::string("adapter table upload: ") + hipGetErrorString(e));
        }
    }
    stage_retain(device);
    *out = t;
    return LORA_OK;
}

int lora_release_adapters(lora_table_t t) {
    if (!t) return fail(LORA_E_ARG, "table is NULL");
    if (t->dev) {
        DeviceGuard dg(t->device);
        (void)hipFree(t->dev);
        stage_release(t->device);
    }
    delete t;
    return LORA_OK;
}

int lora_workspace_bytes(lora_table_t t, const lora_batch_t* b, size_t* bytes) {
    if (int rc = check_table(t)) return rc;
    if (!bytes) return fail(LORA_E_ARG, "bytes is NULL");
    HostPlan p;
    if (int rc = build_plan(t, b, p)) return rc;
    *bytes = p.uncut_bytes;
    return LORA_OK;
}

int lora_group_rows(const lora_batch_t* b, int32_t n_adapters, int32_t* perm, int32_t* group_off,
                    int32_t* group_adapter, int32_t* n_groups) {
    if (!perm || !group_off || !group_adapter || !n_groups) return fail(LORA_E_ARG, "output is NULL");
    if (n_adapters < 0) return fail(LORA_E_ARG, "negative n_adapters");
    if (int rc = validate_batch(b, n_adapters)) return rc;
    std::vector<int32_t> pv, go, ga;
    group_rows(b, n_adapters, pv, go, ga);
    std::copy(pv.begin(), pv.end(), perm);
    std::copy(go.begin(), go.end(), group_off);
    std::copy(ga.begin(), ga.end(), group_adapter);
    *n_groups = (int32_t)ga.size();
    return LORA_OK;
}

int lora_plan_inspect(const lora_batch_t* b, int32_t h_in, int32_t h_out, int32_t n_adapters,
                      const int32_t* ranks, int32_t n_xcd, lora_item_info_t* items, int32_t capacity,
                      int32_t* n_items) {
    if (!n_items) return fail(LORA_E_ARG, "n_items is NULL");
    *n_items = 0;
    if (h_in <= 0 || h_out <= 0 || h_in % 8 || h_out % 8)
        return fail(LORA_E_SHAPE, "h_in and h_out must be positive multiples of 8");
    if ((uint64_t)std::max(h_in, h_out) * kMaxRank * 2 > kMaxSpan)
        return fail(LORA_E_SHAPE, "h_in and h_out must be at most 4 Mi elements (factors below 2 GiB)");
    if (n_adapters < 0 || (n_adapters > 0 && !ranks)) return fail(LORA_E_ARG, "bad adapter ranks");
    if (capacity < 0) return fail(LORA_E_ARG, "negative capacity");
    lora_table_s t;                           // host-side table: ranks and shapes only
    t.h_in = h_in;
    t.h_out = h_out;
    t.n = n_adapters;
    t.n_xcd = std::max(1, std::min(n_xcd, 64));
    t.host.assign(n_adapters, DevAdapter{});
    for (int i = 0; i < n_adapters; ++i) {
        if (ranks[i] < 1 || ranks[i] > kMaxRank)
            return fail(LORA_E_RANK, "adapter " + std::to_string(i) + " has rank " + std::to_string(ranks[i]) +
                                         " outside [1, 256]");
        t.host[i].rank = ranks[i];
        t.host[i].scale = 1.f;
    }
    HostPlan p;
    if (int rc = build_plan(&t, b, p)) return rc;
    std::vector<DevItem> grid, all;
    list_items(p, grid, all);
    const size_t total = grid.size() + all.size();
    if (total > (size_t)INT32_MAX) return fail(LORA_E_SHAPE, "plan too large to list");
    *n_items = (int32_t)total;
    if (!items) return LORA_OK;               // size query
    if ((size_t)capacity < total) return fail(LORA_E_ARG, "capacity smaller than the plan's item count (see n_items)");
    auto put = [&](int32_t at, const DevItem& it, int32_t pos) {
        lora_item_info_t& o = items[at];
        o.kind = it.kind;
        o.row_block = it.rb;
        o.rank = it.rank;
        o.nrows = it.nrows;
        o.lo = it.lo;
        o.len = it.len;
        o.sub = it.sub & (kSubDma - 1);
        o.nsplit = it.nsplit;
        o.pstride = it.pstride;
        o.grid_pos = pos;
    };
    int32_t k = 0;
    for (size_t i = 0; i < grid.size(); ++i, ++k) put(k, grid[i], (int32_t)i);
    for (const DevItem& it : all) put(k++, it, -1);
    return LORA_OK;
}

int lora_shrink(lora_table_t t, const lora_batch_t* b, const void* x, int64_t ldx, float* v,
                int64_t ldv, void* ws, size_t ws_bytes, void* stream) {
    if (int rc = check_table(t)) return rc;
    HostPlan p;
    if (int rc = build_plan(t, b, p)) return rc;
    if (p.n_active == 0) return LORA_OK;
    if (int rc = check_x(t, x, ldx, b->n_rows)) return rc;
    if (int rc = check_v(p, v, ldv)) return rc;
    if (int rc = check_ws(p, ws, ws_bytes)) return rc;
    DeviceGuard dg(t->device);
    hipStream_t s = (hipStream_t)stream;
    if (int rc = check_not_capturing(s, "lora_shrink")) return rc;
    unsigned char* w = (unsigned char*)ws;
    if (int rc = write_plan(p, w, false, t->device, s)) return rc;
    if (int rc = enqueue(t, p, w, x, ldx, nullptr, 0, s, true)) return rc;
    KernelArgs a = make_args(t, p, w, kSpinLimit);
    a.items = (const DevItem*)(w + p.off_reduce_all);
    a.n_items = p.n_all;
    a.v = v;
    a.ldv = ldv;
    LORA_HIP_TRY(launch_reduce(a, (const uint32_t*)w, s));
    return LORA_OK;
}

int lora_expand(lora_table_t t, const lora_batch_t* b, const float* v, int64_t ldv, void* y,
                int64_t ldy, void* ws, size_t ws_bytes, void* stream) {
    if (int rc = check_table(t)) return rc;
    HostPlan p;
    if (int rc = build_plan(t, b, p)) return rc;
    if (p.n_active == 0) return LORA_OK;
    if (int rc = check_v(p, v, ldv)) return rc;
    if (int rc = check_y(t, y, ldy, b->n_rows)) return rc;
    if (int rc = check_ws(p, ws, ws_bytes)) return rc;
    DeviceGuard dg(t->device);
    hipStream_t s = (hipStream_t)stream;
    if (int rc = check_not_capturing(s, "lora_expand")) return rc;
    unsigned char* w = (unsigned char*)ws;
    if (int rc = write_plan(p, w, false, t->device, s)) return rc;
    KernelArgs a = make_args(t, p, w, kSpinLimit);
    a.items = (const DevItem*)(w + p.off_expand);
    a.n_items = p.n_expand;
    a.v = const_cast<float*>(v);
    a.ldv = ldv;
    a.y = y;
    a.ldy = ldy;
    a.y_bytes = (uint32_t)span_bytes(p.n_rows, ldy, t->h_out);
    LORA_HIP_TRY(launch_expand(a, (const uint32_t*)w, t->dtype, s));
    return LORA_OK;
}

int lora_apply_fused(lora_table_t t, const lora_batch_t* b, const void* x, int64_t ldx, void* y,
                     int64_t ldy, void* ws, size_t ws_bytes, void* stream) {
    if (int rc = check_table(t)) return rc;
    HostPlan p;
    if (int rc = build_plan(t, b, p)) return rc;
    if (p.n_active == 0) return LORA_OK;
    if (int rc = check_x(t, x, ldx, b->n_rows)) return rc;
    if (int rc = check_y(t, y, ldy, b->n_rows)) return rc;
    if (int rc = check_overlap(x, ldx, t->h_in, y, ldy, t->h_out, b->n_rows)) return rc;
    if (int rc = check_ws(p, ws, ws_bytes)) return rc;
    DeviceGuard dg(t->device);
    hipStream_t s = (hipStream_t)stream;
    if (int rc = check_not_capturing(s, "lora_apply_fused")) return rc;
    unsigned char* w = (unsigned char*)ws;
    if (int rc = write_plan(p, w, false, t->device, s)) return rc;
    return enqueue(t, p, w, x, ldx, y, ldy, s);
}

// ---------------------------------------------------------------------------
// fused base projection (Eq. 1 whole)
// ---------------------------------------------------------------------------
namespace {

// Workspace of lora_base_apply: [plan (header, items, grouped rows) | partial
// and v blocks | counters] [dense float32 v: n_rows x ldv] [per row tile:
// offsets into the runs, then the runs of rows that share an adapter]
// [float32 partial tiles of the split tiles].
struct BaseLayout {
    HostPlan p;
    int ldv = 8;
    int tile = kBaseBig;
    int n_mt = 0, n_nt = 0;
    int n_whole = 0, split = 1, chunk = 0;
    size_t off_v = 0, v_bytes = 0, off_pieces = 0, off_part = 0, part_bytes = 0, total = 0;
    std::vector<unsigned char> pieces_blob;
    size_t off_piece_list = 0;           // within pieces_blob
};

// Work of one launch: whole rounds of tiles over the compute units run whole;
// the tiles of a last, partial round are split along K into ranges of at
// least kBaseMinSplitStages stages (an even number of them), as many as fill
// the compute units, their partial tiles added by a second kernel.
void choose_split(int n_tiles, int h_in, int n_cu, BaseLayout& L) {
    const int bk = base_bk(L.tile);
    const int nk = ((h_in + 2 * bk - 1) / (2 * bk)) * 2;
    L.n_whole = n_tiles;
    L.split = 1;
    L.chunk = nk;
    if (n_cu <= 0 || n_tiles == 0) return;
    const int rounds = n_tiles / n_cu;
    const int rem = n_tiles - rounds * n_cu;
    if (rem == 0) return;
    const int s = std::min(n_cu / rem, nk / kBaseMinSplitStages);
    if (s < 2) return;
    const int chunk = round_up_i((nk + s - 1) / s, 2);
    const int split = (nk + chunk - 1) / chunk;
    if (split < 2) return;
    L.n_whole = rounds * n_cu;
    L.split = split;
    L.chunk = chunk;
}

int build_base(const lora_table_s* t, const lora_batch_t* b, BaseLayout& L) {
    if (int rc = build_plan(t, b, L.p)) return rc;
    L.ldv = round_up_i(std::max(L.p.r_max, 1), 8);
    L.off_v = align_up(L.p.uncut_bytes);
    L.v_bytes = (size_t)b->n_rows * L.ldv * sizeof(float);
    if (L.v_bytes > kMaxSpan) return fail(LORA_E_SHAPE, "batch too large: its float32 intermediate exceeds 2 GiB");
    // the big tile while its whole tiles fill the compute units; else the
    // small one, which has four times as many tiles to spread (a 1024-token
    // prompt at 4096 columns: 256 whole tiles instead of 64 split four ways)
    const int64_t big_tiles = (int64_t)((b->n_rows + kBaseBig - 1) / kBaseBig) * ((t->h_out + kBaseBig - 1) / kBaseBig);
    L.tile = big_tiles >= t->n_cu ? kBaseBig : kBaseSmall;
    L.n_mt = (b->n_rows + L.tile - 1) / L.tile;
    L.n_nt = (t->h_out + L.tile - 1) / L.tile;
    // runs of rows sharing an adapter, per row tile; neighbouring segments of
    // one adapter inside a tile make one run
    std::vector<std::vector<BasePiece>> per(L.n_mt);
    for (int sgi = 0; sgi < b->n_segments; ++sgi) {
        const int g = b->seg_adapter[sgi];
        int lo = b->seg_offset[sgi];
        const int hi = b->seg_offset[sgi + 1];
        if (g < 0) continue;
        while (lo < hi) {
            const int mt = lo / L.tile;
            const int e = std::min(hi, (mt + 1) * L.tile);
            auto& v = per[mt];
            if (!v.empty() && v.back().adapter == g && v.back().hi == lo) v.back().hi = e;
            else v.push_back(BasePiece{lo, e, g, 0});
            lo = e;
        }
    }
    std::vector<int32_t> off(L.n_mt + 1, 0);
    for (int m = 0; m < L.n_mt; ++m) off[m + 1] = off[m] + (int32_t)per[m].size();
    L.off_piece_list = align_up((size_t)(L.n_mt + 1) * sizeof(int32_t), 16);
    L.pieces_blob.assign(L.off_piece_list + (size_t)off[L.n_mt] * sizeof(BasePiece), 0);
    std::memcpy(L.pieces_blob.data(), off.data(), off.size() * sizeof(int32_t));
    size_t at = L.off_piece_list;
    for (const auto& v : per)
        for (const BasePiece& pc : v) {
            std::memcpy(L.pieces_blob.data() + at, &pc, sizeof pc);
            at += sizeof pc;
        }
    L.off_pieces = align_up(L.off_v + L.v_bytes);
    L.off_part = align_up(L.off_pieces + std::max<size_t>(L.pieces_blob.size(), 16));
    choose_split(L.n_mt * L.n_nt, t->h_in, t->n_cu, L);
    L.part_bytes = (size_t)(L.n_mt * L.n_nt - L.n_whole) * L.split * ((size_t)L.tile * L.tile * sizeof(float));
    if (L.split < 2) L.part_bytes = 0;
    L.total = L.off_part + L.part_bytes;
    return LORA_OK;
}

}  // namespace

int lora_base_workspace_bytes(lora_table_t t, const lora_batch_t* b, size_t* bytes) {
    if (int rc = check_table(t)) return rc;
    if (!bytes) return fail(LORA_E_ARG, "bytes is NULL");
    BaseLayout L;
    if (int rc = build_base(t, b, L)) return rc;
    *bytes = L.total;
    return LORA_OK;
}

int lora_base_inspect(const lora_batch_t* b, int32_t h_in, int32_t h_out, int32_t n_adapters, const int32_t* ranks,
                      int32_t n_cu, int32_t n_xcd, lora_base_info_t* out) {
    if (!out) return fail(LORA_E_ARG, "out is NULL");
    if (h_in <= 0 || h_out <= 0 || h_in % 8 || h_out % 8)
        return fail(LORA_E_SHAPE, "h_in and h_out must be positive multiples of 8");
    if ((uint64_t)std::max(h_in, h_out) * kMaxRank * 2 > kMaxSpan)
        return fail(LORA_E_SHAPE, "h_in and h_out must be at most 4 Mi elements (factors below 2 GiB)");
    if (n_adapters < 0 || (n_adapters > 0 && !ranks)) return fail(LORA_E_ARG, "bad adapter ranks");
    if (n_cu < 0) return fail(LORA_E_ARG, "negative n_cu");
    lora_table_s t;                           // host-side table: ranks and shapes only
    t.h_in = h_in;
    t.h_out = h_out;
    t.n = n_adapters;
    t.n_cu = n_cu;
    t.n_xcd = std::max(1, std::min(n_xcd, 64));
    t.host.assign(n_adapters, DevAdapter{});
    for (int i = 0; i < n_adapters; ++i) {
        if (ranks[i] < 1 || ranks[i] > kMaxRank)
            return fail(LORA_E_RANK, "adapter " + std::to_string(i) + " has rank " + std::to_string(ranks[i]) +
                                         " outside [1, 256]");
        t.host[i].rank = ranks[i];
        t.host[i].scale = 1.f;
    }
    BaseLayout L;
    if (int rc = build_base(&t, b, L)) return rc;
    const int bk = base_bk(L.tile);
    const int n_tiles = L.n_mt * L.n_nt;
    const int per_xcd = (L.n_whole + t.n_xcd - 1) / t.n_xcd;
    const int n_split = L.split > 1 ? n_tiles - L.n_whole : 0;
    out->tile = L.tile;
    out->n_mt = L.n_mt;
    out->n_nt = L.n_nt;
    out->n_whole = L.n_whole;
    out->split = L.split;
    out->chunk = L.chunk;
    out->n_stages = ((h_in + 2 * bk - 1) / (2 * bk)) * 2;
    out->stage_k = bk;
    out->per_xcd = per_xcd;
    out->grid = t.n_xcd * per_xcd + n_split * L.split;
    out->panel = kBasePanel;
    out->workspace_bytes = L.total;
    return LORA_OK;
}

}  // extern "C"

namespace {

// The operand checks of lora_base_apply and lora_base_plan_apply.
int check_base_operands(const lora_table_s* t, int n_rows, const void* x, int64_t ldx, const void* wt, int64_t ldw,
                        void* y, int64_t ldy, uint64_t* w_span_out) {
    if (int rc = check_x(t, x, ldx, n_rows)) return rc;
    if (int rc = check_y(t, y, ldy, n_rows)) return rc;
    if (!wt) return fail(LORA_E_ARG, "wt is NULL");
    if (!aligned16(wt)) return fail(LORA_E_ALIGN, "wt not 16-byte aligned");
    if (int rc = check_ld("ldw", ldw, t->h_in)) return rc;
    const uint64_t w_span = span_bytes(t->h_out, ldw, t->h_in);
    if (w_span > kMaxSpan) return fail(LORA_E_SHAPE, "wt spans more than 2 GiB");
    if (int rc = check_overlap(x, ldx, t->h_in, y, ldy, t->h_out, n_rows)) return rc;
    const uintptr_t ws0 = (uintptr_t)wt, we = ws0 + w_span;
    const uintptr_t ys = (uintptr_t)y, ye = ys + span_bytes(n_rows, ldy, t->h_out);
    if (ws0 < ye && ys < we) return fail(LORA_E_OVERLAP, "wt and y overlap");
    *w_span_out = w_span;
    return LORA_OK;
}

// Everything after the upload: the shrink of every adapted row into the dense
// float32 v, then the GEMM with the delta in its epilogue.  The work list and
// the tile pieces are at their layout offsets in w.  Kernels only (a graph
// may record it).
int base_run(const lora_table_s* t, const BaseLayout& L, int n_rows, unsigned char* w, const void* x, int64_t ldx,
             const void* wt, int64_t ldw, uint64_t w_span, void* y, int64_t ldy, hipStream_t s) {
    float* v = (float*)(w + L.off_v);
    const HostPlan& p = L.p;
    if (p.n_active > 0) {
        // v = x . A_g for every adapted row, into the dense float32 buffer
        if (int rc = enqueue(t, p, w, x, ldx, nullptr, 0, s, true)) return rc;
        KernelArgs ra = make_args(t, p, w, kSpinLimit);
        ra.items = (const DevItem*)(w + p.off_reduce_all);
        ra.n_items = p.n_all;
        ra.v = v;
        ra.ldv = L.ldv;
        LORA_HIP_TRY(launch_reduce(ra, (const uint32_t*)w, s));
    }
    BaseArgs a{};
    a.x = x;
    a.wt = wt;
    a.y = y;
    a.v = v;
    a.table = t->dev;
    a.piece_off = (const int32_t*)(w + L.off_pieces);
    a.pieces = (const BasePiece*)(w + L.off_pieces + L.off_piece_list);
    a.ldx = ldx;
    a.ldw = ldw;
    a.ldy = ldy;
    a.ldv = L.ldv;
    a.M = n_rows;
    a.N = t->h_out;
    a.K = t->h_in;
    a.tile = L.tile;
    a.n_mt = L.n_mt;
    a.n_nt = L.n_nt;
    a.n_xcd = std::max(1, t->n_xcd);
    a.n_whole = L.n_whole;
    a.per_xcd = (L.n_whole + a.n_xcd - 1) / a.n_xcd;
    a.split = L.split;
    a.chunk = L.chunk;
    a.part = L.split > 1 ? (float*)(w + L.off_part) : nullptr;
    a.x_bytes = (uint32_t)span_bytes(n_rows, ldx, t->h_in);
    a.w_bytes = (uint32_t)w_span;
    a.y_bytes = (uint32_t)span_bytes(n_rows, ldy, t->h_out);
    a.v_bytes = (uint32_t)L.v_bytes;
    a.b_span_ok = 1;
    LORA_HIP_TRY(launch_base(a, t->dtype, s));
    return LORA_OK;
}

}  // namespace

struct lora_base_plan_s {
    const lora_table_s* table = nullptr;
    int device = 0;
    int n_rows = 0;
    BaseLayout L;
    unsigned char* dmem = nullptr;
};

extern "C" {

int lora_base_apply(lora_table_t t, const lora_batch_t* b, const void* x, int64_t ldx, const void* wt,
                    int64_t ldw, void* y, int64_t ldy, void* ws, size_t ws_bytes, void* stream) {
    if (int rc = check_table(t)) return rc;
    BaseLayout L;
    if (int rc = build_base(t, b, L)) return rc;
    const int n_rows = b->n_rows;
    if (n_rows == 0) return LORA_OK;
    uint64_t w_span = 0;
    if (int rc = check_base_operands(t, n_rows, x, ldx, wt, ldw, y, ldy, &w_span)) return rc;
    if (!ws) return fail(LORA_E_ARG, "workspace is NULL");
    if (!aligned16(ws)) return fail(LORA_E_ALIGN, "workspace not 16-byte aligned");
    if (ws_bytes < L.total)
        return fail(LORA_E_WORKSPACE, "workspace has " + std::to_string(ws_bytes) + " bytes, needs " +
                                          std::to_string(L.total));
    DeviceGuard dg(t->device);
    hipStream_t s = (hipStream_t)stream;
    if (int rc = check_not_capturing(s, "lora_base_apply")) return rc;
    unsigned char* w = (unsigned char*)ws;
    if (int rc = write_plan(L.p, w, false, t->device, s, L.pieces_blob.data(), L.pieces_blob.size(), L.off_pieces)) return rc;
    return base_run(t, L, n_rows, w, x, ldx, wt, ldw, w_span, y, ldy, s);
}

int lora_base_plan_create(lora_base_plan_t* out, lora_table_t t, const lora_batch_t* b, void* stream) {
    if (!out) return fail(LORA_E_ARG, "out is NULL");
    *out = nullptr;
    if (int rc = check_table(t)) return rc;
    auto* pl = new (std::nothrow) lora_base_plan_s();
    if (!pl) return fail(LORA_E_NOMEM, "plan allocation failed");
    if (int rc = build_base(t, b, pl->L)) {
        delete pl;
        return rc;
    }
    DeviceGuard dg(t->device);
    hipStream_t s = (hipStream_t)stream;
    if (int rc = check_not_capturing(s, "lora_base_plan_create")) {
        delete pl;
        return rc;
    }
    pl->table = t;
    pl->device = t->device;
    pl->n_rows = b->n_rows;
    hipError_t e = hipMalloc((void**)&pl->dmem, std::max<size_t>(pl->L.total, 256));
    if (e != hipSuccess) {
        delete pl;
        return fail(LORA_E_NOMEM, std::string("hipMalloc of the base plan: ") + hipGetErrorString(e));
    }
    const BaseLayout& L = pl->L;
    if (int rc = write_plan(L.p, pl->dmem, false, t->device, s, L.pieces_blob.data(), L.pieces_blob.size(), L.off_pieces)) {
        (void)hipFree(pl->dmem);
        delete pl;
        return rc;
    }
    e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
        (void)hipFree(pl->dmem);
        delete pl;
        return fail(LORA_E_HIP, std::string("base plan upload: ") + hipGetErrorString(e));
    }
    *out = pl;
    return LORA_OK;
}

int lora_base_plan_apply(lora_base_plan_t pl, lora_table_t t, const void* x, int64_t ldx, const void* wt, int64_t ldw,
                         void* y, int64_t ldy, void* stream) {
    if (!pl || !pl->dmem) return fail(LORA_E_ARG, "plan is NULL");
    const lora_table_s* tt = t ? t : pl->table;
    if (int rc = check_compatible(pl->L.p, tt)) return rc;
    if (tt->device != pl->device) return fail(LORA_E_ARG, "table is on another device than the plan");
    if (pl->n_rows == 0) return LORA_OK;
    uint64_t w_span = 0;
    if (int rc = check_base_operands(tt, pl->n_rows, x, ldx, wt, ldw, y, ldy, &w_span)) return rc;
    DeviceGuard dg(tt->device);
    return base_run(tt, pl->L, pl->n_rows, pl->dmem, x, ldx, wt, ldw, w_span, y, ldy, (hipStream_t)stream);
}

int lora_base_plan_destroy(lora_base_plan_t pl) {
    if (!pl) return fail(LORA_E_ARG, "plan is NULL");
    if (pl->dmem) {
        DeviceGuard dg(pl->device);
        (void)hipFree(pl->dmem);
    }
    delete pl;
    return LORA_OK;
}

int lora_apply_fused_static(lora_table_t t, const lora_batch_t* b, const void* x, int64_t ldx, void* y,
                            int64_t ldy, void* stream) {
    if (int rc = check_table(t)) return rc;
    HostPlan p;
    if (int rc = build_plan(t, b, p)) return rc;
    if (p.n_active == 0) return LORA_OK;
    if (int rc = check_x(t, x, ldx, b->n_rows)) return rc;
    if (int rc = check_y(t, y, ldy, b->n_rows)) return rc;
    if (int rc = check_overlap(x, ldx, t->h_in, y, ldy, t->h_out, b->n_rows)) return rc;
    if (p.total_bytes > kScratchBytes)
        return fail(LORA_E_WORKSPACE, "the batch needs " + std::to_string(p.total_bytes) +
                                          " bytes of workspace; the static scratch holds " +
                                          std::to_string(kScratchBytes) + " (use lora_apply_fused)");
    DeviceGuard dg(t->device);
    if (!dg.ok) return fail(LORA_E_HIP, "hipSetDevice failed");
    hipStream_t s = (hipStream_t)stream;
    if (int rc = check_not_capturing(s, "lora_apply_fused_static")) return rc;
    unsigned char* w = nullptr;
    if (int rc = scratch_address(t->device, &w)) return rc;
    if (int rc = write_plan(p, w, false, t->device, s, nullptr, 0, 0, false)) return rc;   // allocates nothing
    return enqueue(t, p, w, x, ldx, y, ldy, s);
}

int lora_plan_bytes(lora_table_t t, const lora_batch_t* b, size_t* bytes) {
    if (int rc = check_table(t)) return rc;
    if (!bytes) return fail(LORA_E_ARG, "bytes is NULL");
    HostPlan p;
    if (int rc = build_plan(t, b, p)) return rc;
    *bytes = p.uncut_total_bytes;
    return LORA_OK;
}

}  // extern "C"

namespace {

// A plan of n projections sharing x (n = 1: an ordinary plan).
int plan_create(lora_plan_t* out, int n, const lora_table_t* tables, const lora_batch_t* b, size_t min_bytes,
                void* stream) {
    if (!out) return fail(LORA_E_ARG, "out is NULL");
    *out = nullptr;
    const lora_table_s* t = tables[0];
    if (int rc = check_table(t)) return rc;
    hipStream_t s = (hipStream_t)stream;
    if (int rc = check_not_capturing(s, "lora_plan_create")) return rc;
    auto* pl = new (std::nothrow) lora_plan_s();
    if (!pl) return fail(LORA_E_NOMEM, "plan allocation failed");
    pl->table = t;
    pl->device = t->device;
    for (int i = 1; i < n; ++i)
        if (tables[i]->device != t->device) {
            delete pl;
            return fail(LORA_E_ARG, "the projections' tables are on different devices");
        }
    if (int rc = n > 1 ? build_plan_multi(tables, n, b, pl->plan) : build_plan(t, b, pl->plan)) {
        delete pl;
        return rc;
    }
    for (int i = 1; i < n; ++i)
        if (int rc = check_compatible_proj(pl->plan, tables[i], i)) {
            delete pl;
            return rc;
        }
    pl->n_rows = b->n_rows;
    pl->capacity = align_up(std::max(pl->plan.uncut_total_bytes, min_bytes));
    DeviceGuard dg(t->device);
    hipError_t e = hipMalloc((void**)&pl->dmem, pl->capacity);
    if (e != hipSuccess) {
        plan_free(pl);
        return fail(LORA_E_NOMEM, std::string("plan memory: ") + hipGetErrorString(e));
    }
    int rc = plan_upload(pl, s);
    if (rc == LORA_OK && hipStreamSynchronize(s) != hipSuccess) rc = fail(LORA_E_HIP, "plan upload failed");
    if (rc != LORA_OK) {
        plan_free(pl);
        return rc;
    }
    *out = pl;
    return LORA_OK;
}

}  // namespace

extern "C" {

int lora_plan_create_reserved(lora_plan_t* out, lora_table_t t, const lora_batch_t* b, size_t min_bytes,
                              void* stream) {
    return plan_create(out, 1, &t, b, min_bytes, stream);
}

int lora_plan_create(lora_plan_t* out, lora_table_t t, const lora_batch_t* b, void* stream) {
    return lora_plan_create_reserved(out, t, b, 0, stream);
}

int lora_plan_create_multi(lora_plan_t* out, int32_t n, const lora_table_t* tables, const lora_batch_t* b,
                           void* stream) {
    if (!out) return fail(LORA_E_ARG, "out is NULL");
    *out = nullptr;
    if (n < 1 || n > kMaxProj) return fail(LORA_E_ARG, "n must be in [1, " + std::to_string(kMaxProj) + "]");
    if (!tables) return fail(LORA_E_ARG, "tables is NULL");
    for (int i = 0; i < n; ++i)
        if (int rc = check_table(tables[i])) return rc;
    return plan_create(out, n, tables, b, 0, stream);
}

int lora_plan_apply_multi(lora_plan_t pl, const lora_table_t* tables, const void* x, int64_t ldx, void* const* ys,
                          const int64_t* ldys, void* stream) {
    if (!pl || !pl->dmem) return fail(LORA_E_ARG, "plan is NULL");
    const int n = pl->plan.n_proj;
    if (!tables || !ys || !ldys || !x) return fail(LORA_E_ARG, "tables, ys, ldys or x is NULL");
    for (int i = 0; i < n; ++i) {
        const lora_table_s* tt = tables[i] ? tables[i] : (i == 0 ? pl->table : nullptr);
        if (!tt) return fail(LORA_E_ARG, "table " + std::to_string(i) + " is NULL");
        if (int rc = check_compatible_proj(pl->plan, tt, i)) return rc;
        if (tt->device != pl->device) return fail(LORA_E_ARG, "table is on another device than the plan");
        if (!ys[i]) return fail(LORA_E_ARG, "y " + std::to_string(i) + " is NULL");
        if (pl->plan.n_active == 0) continue;
        if (int rc = check_x(tt, x, ldx, pl->n_rows)) return rc;
        if (int rc = check_y(tt, ys[i], ldys[i], pl->n_rows)) return rc;
        if (int rc = check_overlap(x, ldx, tt->h_in, ys[i], ldys[i], tt->h_out, pl->n_rows)) return rc;
        for (int j = 0; j < i; ++j)
            if (int rc = check_overlap(ys[j], ldys[j], pl->plan.proj_h_out.empty() ? tt->h_out : pl->plan.proj_h_out[j],
                                       ys[i], ldys[i], tt->h_out, pl->n_rows))
                return rc;
    }
    if (pl->plan.n_active == 0) return LORA_OK;
    const lora_table_s* t0 = tables[0] ? tables[0] : pl->table;
    DeviceGuard dg(pl->device);
    KernelArgs a{};
    if (int rc = step_args(t0, pl->plan, pl->dmem, x, ldx, ys[0], ldys[0], pl->spin_limit, a)) return rc;
    a.n_proj = n;
    for (int i = 0; i < n; ++i) {
        const lora_table_s* tt = tables[i] ? tables[i] : pl->table;
        a.ptable[i] = tt->dev;
        a.py[i] = ys[i];
        a.pldy[i] = ldys[i];
        a.py_bytes[i] = (uint32_t)span_bytes(pl->n_rows, ldys[i], tt->h_out);
        a.ph_out[i] = tt->h_out;
    }
    LORA_HIP_TRY(launch_step(a, (const uint32_t*)pl->dmem, t0->dtype, (hipStream_t)stream));
    return LORA_OK;
}

int lora_plan_update(lora_plan_t pl, lora_table_t t, const lora_batch_t* b, void* stream) {
    if (!pl || !pl->dmem) return fail(LORA_E_ARG, "plan is NULL");
    const lora_table_s* tt = t ? t : pl->table;
    if (int rc = check_table(tt)) return rc;
    if (tt->device != pl->device) return fail(LORA_E_ARG, "table is on another device than the plan");
    hipStream_t s = (hipStream_t)stream;
    DeviceGuard dg(pl->device);
    if (int rc = check_not_capturing(s, "lora_plan_update")) return rc;
    if (pl->plan.n_proj > 1)
        return fail(LORA_E_ARG, "a plan of several projections is re-planned with lora_plan_create_multi");
    HostPlan np;
    if (int rc = build_plan(tt, b, np)) return rc;
    if (np.plan_total_bytes > pl->capacity)
        return fail(LORA_E_WORKSPACE, "the batch needs " + std::to_string(np.plan_total_bytes) +
                                          " bytes of plan memory; the plan holds " + std::to_string(pl->capacity) +
                                          " (lora_plan_create_reserved sets the capacity)");
    pl->plan = std::move(np);
    pl->table = tt;
    pl->n_rows = b->n_rows;
    return plan_upload(pl, s);
}

static int plan_run(lora_plan_t pl, lora_table_t t, const void* x, int64_t ldx, void* y, int64_t ldy,
                    void* stream) {
    if (!pl || !pl->dmem) return fail(LORA_E_ARG, "plan is NULL");
    if (pl->plan.n_proj > 1) return fail(LORA_E_ARG, "a plan of several projections runs through lora_plan_apply_multi");
    const lora_table_s* tt = t ? t : pl->table;
    if (int rc = check_compatible(pl->plan, tt)) return rc;
    if (tt->device != pl->device) return fail(LORA_E_ARG, "table is on another device than the plan");
    if (pl->plan.n_active == 0) return LORA_OK;
    if (x)
        if (int rc = check_x(tt, x, ldx, pl->n_rows)) return rc;
    if (y)
        if (int rc = check_y(tt, y, ldy, pl->n_rows)) return rc;
    if (x && y)
        if (int rc = check_overlap(x, ldx, tt->h_in, y, ldy, tt->h_out, pl->n_rows)) return rc;
    DeviceGuard dg(tt->device);
    if (x && y)
        return enqueue_step(tt, pl->plan, pl->dmem, x, ldx, y, ldy, pl->spin_limit, (hipStream_t)stream);
    return enqueue(tt, pl->plan, pl->dmem, x, ldx, y, ldy, (hipStream_t)stream);
}

int lora_plan_apply(lora_plan_t pl, lora_table_t t, const void* x, int64_t ldx, void* y, int64_t ldy,
                    void* stream) {
    if (!x || !y) return fail(LORA_E_ARG, "x or y is NULL");
    return plan_run(pl, t, x, ldx, y, ldy, stream);
}

int lora_plan_shrink(lora_plan_t pl, lora_table_t t, const void* x, int64_t ldx, void* stream) {
    if (!x) return fail(LORA_E_ARG, "x is NULL");
    return plan_run(pl, t, x, ldx, nullptr, 0, stream);
}

int lora_plan_expand(lora_plan_t pl, lora_table_t t, void* y, int64_t ldy, void* stream) {
    if (!y) return fail(LORA_E_ARG, "y is NULL");
    return plan_run(pl, t, nullptr, 0, y, ldy, stream);
}

int lora_plan_status(lora_plan_t pl, void* stream) {
    if (!pl || !pl->dmem) return fail(LORA_E_ARG, "plan is NULL");
    DeviceGuard dg(pl->device);
    hipStream_t s = (hipStream_t)stream;
    int32_t flag = 0;
    LORA_HIP_TRY(hipMemcpyAsync(&flag, pl->dmem + sizeof(uint32_t), sizeof(flag), hipMemcpyDeviceToHost, s));
    LORA_HIP_TRY(hipStreamSynchronize(s));
    if (flag == kStatusOk) return LORA_OK;
    LORA_HIP_TRY(arm_step(pl->plan, pl->dmem, s));
    LORA_HIP_TRY(hipStreamSynchronize(s));
    if (flag == kStatusStale)
        return fail(LORA_E_STALE, "a launch recorded for an earlier batch of this plan ran after lora_plan_update "
                                  "and did nothing");
    return fail(LORA_E_SYNC, "a step launch gave up waiting for its shrink items; its results are invalid");
}

int lora_plan_set_spin_limit(lora_plan_t pl, int32_t polls) {
    if (!pl) return fail(LORA_E_ARG, "plan is NULL");
    if (polls < 0) return fail(LORA_E_ARG, "negative spin limit");
    pl->spin_limit = polls;
    return LORA_OK;
}

int lora_plan_destroy(lora_plan_t pl) {
    if (!pl) return fail(LORA_E_ARG, "plan is NULL");
    plan_free(pl);
    return LORA_OK;
}

}  // extern "C"
