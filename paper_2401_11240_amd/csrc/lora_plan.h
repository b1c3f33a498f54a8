// The work list, item by item, from the row blocks: shared by the host (sizes,
// lora_plan_inspect) and the kernel that writes the list into device memory.
//
// A call hands the device its row blocks (56 bytes each, and the rows of those
// that are not consecutive) in the kernel arguments of lora_plan_kernel, which
// expands them into the items (128 bytes each; a few to some tens per block, over a
// thousand at h_in and h_out in the tens of thousands).
// Built on the host and copied from a pinned ring, the list bounded the one-shot
// calls: a shrink and an expand call on 1491 rows (40 blocks, 1200 items) took
// 86 us together against 39 us now, lora_apply_fused on 203 rows 39 against 20 us,
// an update of 48 decode rows and eight launches 128 against 103 us.
#pragma once
#include "lora_internal.h"

namespace lora {

// One projection of a plan: its shape and the two numbers that depend on the
// whole batch.
struct PlanDims {
    int32_t h_in, h_out;
    int32_t big_split;       // K ranges of row blocks of more than kInlineRows rows
    int32_t units, items;    // large decode steps (items > 0): all row blocks share so many shrink items by
                             // their bytes, rows + rank each (units: their sum)
    int32_t small_step;      // 1: the step's items fit one round of workgroups
};

// One row block, as the host passes it.
struct PlanRow {
    int32_t group, adapter;
    int32_t shape;           // rank | rows << 16 | projection << 24 | K per pass / 32 << 26
    int32_t p0;              // position of the first row in the grouped row order
    int32_t row0;            // the first row when they are consecutive; else -1 - (their place in the row
                             // list, where a projection past the first passes only inline rows)
    uint32_t part;           // float offset of its first partial block
    int32_t shrink_at, reduce_at, expand_at, all_at;   // its first item in each list
    int32_t cut;             // XCD (grid laid out per XCD) | passes per K range << 8
    int32_t step_shrink, step_reduce, step_expand;   // its first items in that XCD's queue
    LORA_HD int rank() const { return shape & 0xffff; }
    LORA_HD int nrows() const { return (shape >> 16) & 0xff; }
    LORA_HD int proj() const { return (shape >> 24) & 3; }
    LORA_HD int sub() const { return (int)((uint32_t)shape >> 26) * 32; }
    LORA_HD int home() const { return cut & 0xff; }
    LORA_HD int krange() const { return (cut >> 8) * sub(); }
    // rows in the row list: not the consecutive ones, and once for all projections where
    // only the grouped row order holds them
    LORA_HD int listed() const { return row0 < 0 && (proj() == 0 || nrows() <= kInlineRows) ? nrows() : 0; }
};
static_assert(sizeof(PlanRow) == 56, "PlanRow layout");
constexpr int kRowWords = sizeof(PlanRow) / 4;

// How a row block is cut into items.
struct RowGeom {
    int sub, krange, nsplit;      // shrink: K per pass, K per item, items
    int nlen, ntiles;             // expand: columns per item, items
    int pstride;                  // floats of one partial (or v) block
    bool direct;                  // the expand items add the partial blocks up themselves
    int slen, nslice;             // reduce: floats per item, items
};

// Its K ranges, `sub` K per pass (chosen on the host; a row block carries them).
inline void row_cut(const PlanDims& d, int rank, int nrows, int& sub, int& krange) {
    sub = shrink_sub(rank, nrows);
    krange = sub;
    if (nrows > kInlineRows) {
        const int per = (d.h_in + d.big_split - 1) / d.big_split;
        krange = round_up_i(max_i(per, sub), sub);
    }
    // (never more ranges than without the cut by bytes, so that a step it is taken
    // for needs no more memory: a plan or workspace that holds a batch holds its parts)
    if (d.items > 0 && (nrows > kInlineRows || shrink_can_dma(rank, nrows))) {
        const int n = (int)((int64_t)(nrows + rank) * d.items / d.units);
        const int per = n > 1 ? (d.h_in + n - 1) / n : d.h_in;
        krange = max_i(krange, round_up_i(per, sub));
    }
    // more ranges than the reduction can add up (h_in past 256 Ki at rank 256, 2 Mi at
    // rank 8): longer ones, of several passes
    if ((d.h_in - 1) / kMaxRanges >= krange) krange = round_up_i((d.h_in + kMaxRanges - 1) / kMaxRanges, sub);
}

LORA_HD inline RowGeom row_geom(const PlanDims& d, int rank, int nrows, int sub, int krange) {
    RowGeom g;
    g.sub = sub;
    g.krange = krange;
    g.nsplit = (d.h_in + g.krange - 1) / g.krange;
    g.nlen = expand_nlen(rank, nrows);
    g.ntiles = (d.h_out + g.nlen - 1) / g.nlen;
    g.pstride = nrows * rank_stride(rank);
    // small partial blocks of a small step are added up by the expand items themselves
    const int64_t pbytes = (int64_t)g.nsplit * g.pstride * 4;
    g.direct = d.small_step && g.nsplit <= kDirectSplits && pbytes <= kDirectBytes;
    // reduce slices: at most kReduceBytes of partial values each; split groups
    // share a float4 position (groups * positions <= threads), each thread adding
    // at most kMaxSplitLoads blocks (gmin <= kThreads, as nsplit <= kMaxRanges)
    int gmin = 1;
    while (gmin * kMaxSplitLoads < g.nsplit) gmin *= 2;
    const int64_t want = (pbytes + kReduceBytes - 1) / kReduceBytes;
    const int nslice = want > 1 ? (int)want : 1;
    g.slen = min_i(round_up_i((g.pstride + nslice - 1) / nslice, 4), 4 * (kThreads / gmin));
    g.nslice = (g.pstride + g.slen - 1) / g.slen;
    return g;
}
inline RowGeom row_geom(const PlanDims& d, int rank, int nrows) {
    int sub, krange;
    row_cut(d, rank, nrows, sub, krange);
    return row_geom(d, rank, nrows, sub, krange);
}
LORA_HD inline RowGeom row_geom(const PlanDims& d, const PlanRow& r) {
    return row_geom(d, r.rank(), r.nrows(), r.sub(), r.krange());
}

// What every item of the row block (number rb) carries; rows: its rows when they
// are not consecutive.
LORA_HD inline DevItem row_item(const PlanRow& r, const RowGeom& g, int rb, const int32_t* rows) {
    DevItem it{};
    it.part = r.part;
    it.kind = r.proj() << kProjShift;
    it.group = r.group;
    it.adapter = r.adapter;
    it.rank = r.rank();
    it.nrows = r.nrows();
    it.nsplit = g.nsplit;
    it.p0 = r.p0;
    it.pstride = g.pstride;
    it.rb = rb;
    it.nexp = g.ntiles;
    it.row0 = r.row0 >= 0 ? r.row0 : -1;
    if (it.nrows <= kInlineRows)
        for (int i = 0; i < kInlineRows; ++i) it.rows[i] = i < it.nrows ? (r.row0 >= 0 ? r.row0 + i : rows[i]) : 0;
    return it;
}
// Shrink item c: K range c of the row block.
LORA_HD inline void to_shrink(DevItem& it, const PlanDims& d, const RowGeom& g, int c) {
    it.kind |= kItemShrink;
    it.part += (int64_t)c * g.pstride;
    it.lo = c * g.krange;
    it.len = min_i(g.krange, d.h_in - c * g.krange);
    if (shrink_uses_dma(it.rank, it.nrows)) it.sub = shrink_stage_sub(it.rank, it.nrows);
    else if (d.items > 0 && it.len > g.sub && shrink_can_dma(it.rank, it.nrows))
        it.sub = shrink_stage_sub(it.rank, it.nrows) | kSubDma;
    else it.sub = g.sub;
}
// Reduce item c: slice c of the row block's v.  A row block whose expand items
// add the partial blocks up themselves adds them in order: one split group.
LORA_HD inline void to_reduce(DevItem& it, const RowGeom& g, int c) {
    it.kind |= kItemReduce;
    it.lo = c * g.slen;
    it.len = min_i(g.slen, g.pstride - c * g.slen);
    const int np = it.len / 4;
    int G = 1;
    while (!g.direct && 2 * G <= g.nsplit && 2 * G * np <= kThreads) G *= 2;
    it.sub = G;
}
// Expand item c: columns from c * nlen.
LORA_HD inline void to_expand(DevItem& it, const PlanDims& d, const RowGeom& g, int c) {
    it.kind |= kItemExpand;
    it.sub = g.direct ? 1 : 0;
    it.lo = c * g.nlen;
    it.len = min_i(g.nlen, d.h_out - c * g.nlen);
}

// Arguments of lora_plan_kernel: one launch carries some of the row blocks.
struct PlanArgs {
    unsigned char* w;            // the plan's or workspace's memory
    uint64_t off_shrink, off_reduce, off_expand, off_all, off_step, off_perm;
    uint64_t off_sync, off_step_partials;
    uint64_t off_blob;           // where the launch's extra words go
    int64_t pbuf;                // floats from the first step buffer to the second
    uint32_t generation;
    int32_t arm;                 // 1: also clear the counters (plans)
    int32_t arm_quads;           // 16-byte values of a step buffer to arm in this launch (both buffers; 0: none)
    int32_t first;               // 1: the launch that writes the header and the empty slots of the step grid
    int32_t last;                // 1: the launch that completes the list
    int32_t n_rows, row_first;   // row blocks in this launch, number of the first
    int32_t slices;              // workgroups that share a row block's items
    int32_t n_xcd, step_len;     // step grid laid out per XCD: slots per XCD (0: none)
    int32_t blob_at, blob_words; // extra words in data
    int32_t arm_blocks;          // workgroups that arm
    const uint32_t* staged;      // data in pinned host memory, instead of the one below
    PlanDims dims[kMaxProj];
    uint16_t step_count[64];     // items in each XCD's queue
    uint32_t data[896];          // row blocks, then the rows of those not consecutive, then the extra words
};
constexpr int kPlanWords = 896;
// A list whose data take more than this many launches' arguments is written by one
// launch that reads them from pinned host memory (256 KiB at a time), while one of the
// device's slots is free.  lora_apply_fused at 1024 x 1024 with listed rows, a chain of
// launches against pinned memory: 1 launch 25 and 31 us, 2 31 and 32, 3 40 and 35, 6 64
// and 36, 12 95 and 44.
constexpr int kArgLaunches = 2;
constexpr int kStagedWords = 64 * 1024, kStageSlots = 8;
constexpr int kBlobWords = 1024;   // extra words per workgroup
static_assert(sizeof(PlanArgs) <= 4096, "kernel arguments");

// Header word i after this launch, when it writes it: the generation only once the
// list is complete, 0 (no plan's) until then, so that nothing runs a list whose later
// launches failed.
LORA_HD inline bool header_word(const PlanArgs& a, int i, uint32_t& v) {
    v = i == 0 && a.last ? a.generation : 0u;
    return a.first || (a.last && i == 0);
}

// Eight lanes write an item (16 bytes each), `slices` workgroups the items of a row
// block, kSliceItems each; one workgroup writes the header and the empty slots, others the
// extra words, kBlobWords each, and the step buffers are armed by workgroups of their own, kArmQuads values
// of each buffer apiece, up to kArmBlocks of them.  A few KB of arguments in, some
// hundred KB of items out: about 3 us, the launch, where the step buffers are small.
// Armed by the workgroup of the row block, a single compute unit wrote all of a large
// block (29 MB at rank 256, h_in 28672): an update of 32 such rows
// took 214 us against 8.5, one of 64 rows of rank 128 at 8192 35 against 6.4.
constexpr int kSliceItems = 256, kMaxSlices = 16;
constexpr int kArmQuads = 1024, kArmBlocks = 1024;
template <bool kStaged>
__global__ void __launch_bounds__(kThreads) lora_plan_kernel(PlanArgs a);

}  // namespace lora
