// gfx950 kernel of Eq. 1 whole (Section 2.1): the base projection and the
// adapter delta of every row in one MFMA GEMM,
//
//     y[t, :] = round( x[t, :] . W  +  s_g (x[t, :] . A_g) . B_g ),
//
// where g is the adapter of row t's segment (rows of adapter -1 get x . W).
// The float32 v = x . A_g comes in beforehand (the shrink kernels); the
// delta s_g v . B_g is added in the epilogue of each output tile.  This is
// the shape of a prompt step of Section 4.1's GPU LoRA once the base
// projection is fused in: the base GEMM's arithmetic intensity is far above
// the MFMA ridge, so the tile runs at MFMA rate while the delta costs r_g/K of
// the base work.
//
// Tile: T rows of x (tokens) x T columns of y, T = 256 or 128, one
// workgroup: 2 x 4 waves of 128 x 64 for T = 256 (two per SIMD), 2 x 2 waves of
// 64 x 64 for T = 128, in MFMA blocks of 32 x 32.  The 128 tile serves
// launches whose big tiles would not fill the compute units (a 1024-token
// prompt), which it fills with whole tiles instead of K-split ones.  The contraction runs on
// v_mfma_f32_32x32x16 (measured here: about 34 cycles for its 32768 flop with
// four independent accumulators, against about 27 for the 16384 of a
// 16x16x32 even with sixteen) with the base weight as the A operand (rows =
// output columns) and x as the B operand, so each group of four accumulators
// holds four consecutive columns of one row of y.
//
// The base weight is taken transposed, W^T [h_out, h_in] (row n = column n of
// W, the layout of a linear layer's weight), so that both operands run along
// K in memory: every 16-byte chunk of 8 consecutive K is one MFMA operand
// slice, with no transpose.
//
// Pipeline: K advances in steps of 64 (a row's slice is one whole 128-byte
// line), brought into a ring of LDS buffers by buffer-to-LDS loads: no staging
// registers and no LDS write instructions.  A wave instruction moves 8 rows x
// 128 bytes; row r's 16-byte chunk c sits in slot c ^ (r / 2) % 8 of its row,
// so that the 16 rows x 16 bytes a quarter wave reads for an operand fragment
// fall in 16 different bank groups.  The fragments of the next K-16 slice are
// read while the current slice's MFMAs run, also across the step boundary: the
// wait for the next step's loads and the one barrier per step stand before the
// last slice, whose own fragments are already in registers, and the loads of
// the step that reuses the freed buffer start right behind it.  Rows past the
// batch, columns past h_out and K past h_in are loads out of the buffer's
// range, which write zeros.
//
// What bounds it (clock counters around bare loops of the same structure, 4096 x
// 4096 x 4096): the 256 tile takes 2254 cycles per step where its MFMAs alone take
// 2048 (91%), at a clock that the power limit holds near 1.5 GHz; MFMAs without any
// data movement reach 1.56-1.65 PFLOP/s on this card.  The 128 tile takes 766 cycles
// per step for 512 of MFMAs; its LDS reads (64 KiB) keep the LDS active for about 256
// of them by the counters, beside the 32 KiB that its loads write there.  Whole
// launches hold the MFMAs busy for 60% (256) and 33% (128) of their cycles.
// Kernel times against the earlier ring in registers (two steps loaded ahead,
// written to LDS by ds_write), traced on two boxes, 4096 columns of K 4096: 1024 rows
// 56-61 -> 41-44 us, 8437 rows 268-270 -> 256-258 us; 547 rows x 13824 of K 5120 in
// binary16 136-137 -> 120-126 us (a library product of that shape: 76 us).
//
// Epilogue: for every run of the tile's rows that share an adapter (at most
// a few for prompt segments), B_g's ranks and the tile's rows of v are staged
// in LDS 64 ranks at a time, and each wave adds s_g v . B_g for its rows into
// its base accumulators: s_g v is split into a high and a low 16-bit part that
// share one 32x32x16 MFMA (its 16 K slots hold 8 ranks twice), rows of other
// runs zero.  binary16 cannot hold a high part past 65504, so for it each
// wave first takes the largest |s_g v| it will use and, past 2^15, scales v
// and its accumulators by a power of two around those MFMAs and back after
// (exact).  The sum is rounded once to the storage dtype.
//
// Tiles go to XCDs in blocks: workgroup p runs on XCD p % n_xcd and takes the
// (p / n_xcd)-th tile of that XCD's contiguous share of the tile order.  The
// order runs over panels of kBasePanel row tiles, column by column inside a
// panel, so that an XCD's share, and the part of it that runs at a time, is a
// block of tiles a few row tiles high and a few column tiles wide: they share
// rows of x and columns of W in the XCD's L2 (a 1024-token prompt in tiles of
// 128: each XCD all 8 row tiles x 4 column tiles, 12 MiB of x and W, where
// one row tile x all 32 column tiles would be 33 MiB).  Every XCD gets
// per_xcd workgroups (the whole tiles over n_xcd, rounded up); those past the
// last tile end at once.
//
// A last round of tiles that would leave compute units idle is split along
// K: each of its tiles runs as `split` workgroups over consecutive K ranges,
// which store their float32 partial tiles (in accumulator order, the first
// range with the adapter delta added) to the workspace; the reduction kernel
// adds a tile's ranges in order 0, 1, ..., rounds once and stores y, so the
// result does not depend on timing.
#include <hip/hip_runtime.h>
#include <stddef.h>

#include "lora_device.h"
#include "lora_internal.h"

namespace lora {

namespace {

typedef __attribute__((address_space(3))) unsigned char lds_u8;
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kStepK = 64;                             // K per step of the pipeline
constexpr int kLdsBytes = 2 * kBaseStageBytes;         // the ring; the epilogue's staging afterwards

// Derived tiling of tile edge T.
template <int T>
struct BaseCfg {
    // waves over rows x columns of the tile: eight of 128 x 64 for the big tile
    // (two per SIMD, 128 accumulators per lane; four of 128 x 128 run its steps
    // as fast, 2244 against 2254 cycles, but spill in the epilogue), four of 64 x 64
    static constexpr int kWM = 2, kWN = T == 256 ? 4 : 2;
    static constexpr int kWaves = kWM * kWN, kThreads = 64 * kWaves;
    static constexpr int kWBM = T / kWM / 32, kWBN = T / kWN / 32;   // 32 x 32 blocks per wave
    static constexpr int kStepChunks = 2 * T * 8;            // 16-byte chunks of a step: T rows of x, T of W
    static constexpr int kRing = kLdsBytes / (16 * kStepChunks);   // steps in LDS: 2 (T = 256) or 4
    static constexpr int kLoads = T / 8 / kWaves;            // loads per wave and step of x (and of W)
    // K-16 slices over which a step's loads are spread, from the barrier on:
    // measured 2 and 4 against 1 (119.6 against 127.7 us, 36.7 against 38.9 us);
    // the ring of two buffers leaves no more than 2 without shortening the time
    // the last load has
    static constexpr int kSpread = kRing == 2 ? 2 : 4;
    static constexpr int kTileQuads = T * T / 4;
    static_assert(kRing >= 2 && 2 * kLoads * kRing < 64, "ring: loads in flight fit vmcnt");
    static_assert(kBaseLoraRanks * T * 2 <= kBaseStageBytes, "B_g staging fits one half of the LDS");
    static_assert(T * T * 2 <= kLdsBytes, "the rounded tile fits the LDS");
};

// s_waitcnt lgkmcnt(0), vmcnt and expcnt left free (gfx9 encoding).
__device__ __forceinline__ void wait_lgkm0() { __builtin_amdgcn_s_waitcnt(0xC07F); }
// s_waitcnt with lgkmcnt(0) and vmcnt(0).
__device__ __forceinline__ void wait_vm0_lgkm0() { __builtin_amdgcn_s_waitcnt(0x0070); }

// s_waitcnt vmcnt(N), the other counters left free.
template <int N>
__device__ __forceinline__ void wait_vm() {
    static_assert(N >= 0 && N < 64, "vmcnt");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// 16 bytes per lane from buffer r at byte offset off (zeros when out of range)
// into LDS at lds + 16 * lane; lds is the same in every lane.  Inline assembly,
// with no output: for the builtin the compiler waits for every such load in
// flight before each LDS read.  wait_vm() and a barrier order the reads after
// it.  The compiler looks for no hazards inside: the wait state after the write of m0
// is here, those of the resource in rsrc_words().
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // m0 is reserved: nothing to preserve, the clobber is what is said
__device__ __forceinline__ void lds_load16(const u32x4& r, uint32_t lds, int off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :: "s"(lds), "v"(off), "s"(r) : "memory", "m0");
}
#pragma clang diagnostic pop
// The resource of make_rsrc() as four scalar words, five wait states (gfx9) after the
// vector instructions that write them.  (In front of every load instead, the states cost
// 1 to 2% of a launch.  No base kernel spills a scalar register, whose reload would be
// another such write.)
__device__ __forceinline__ u32x4 rsrc_words(const void* base, uint32_t bytes) {
    const uint64_t b = (uint64_t)base;
    u32x4 r = {(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b),
               (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(b >> 32)) & 0xffffu,
               (uint32_t)__builtin_amdgcn_readfirstlane((int)bytes), (uint32_t)kRsrcWord3};
    asm volatile("s_nop 4" : "+s"(r));
    return r;
}

// v_mfma_f32_32x32x16: A [32 x 16] lane l holds A[l % 32][8 (l / 32) .. +7];
// B [16 x 32] lane l holds B[8 (l / 32) .. +7][l % 32]; accumulator r of
// lane l is D[8 (r / 4) + 4 (l / 32) + r % 4][l % 32].
template <class Fmt>
__device__ __forceinline__ f32x16 mma32x32(const u32x4& a, const u32x4& b, f32x16 c);
template <>
__device__ __forceinline__ f32x16 mma32x32<FmtF16>(const u32x4& a, const u32x4& b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c,
                                                  0, 0, 0);
}
template <>
__device__ __forceinline__ f32x16 mma32x32<FmtBF16>(const u32x4& a, const u32x4& b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                   c, 0, 0, 0);
}

// Row tile mt and column tile nt of tile index `tile` in the panel order.
__device__ __forceinline__ void tile_coords(const BaseArgs& a, int tile, int& mt, int& nt) {
    const int per_panel = kBasePanel * a.n_nt;
    const int panel = tile / per_panel;
    const int h = min_i(kBasePanel, a.n_mt - panel * kBasePanel);   // row tiles of this panel
    const int u = tile - panel * per_panel;
    nt = u / h;
    mt = panel * kBasePanel + (u - nt * h);
}

template <class Fmt, int TILE>
struct BaseTile {
    using C = BaseCfg<TILE>;
    static constexpr int WBM = C::kWBM, WBN = C::kWBN, NW = C::kWaves;
    static constexpr int NF = WBM + WBN;     // operand fragments of a slice: WBN of W, then WBM of x
    static constexpr int NL = 2 * C::kLoads; // loads of a step per wave: x, then W
    const BaseArgs& a;
    const int t, w, l, wm, wn;
    const int m0, n0;
    u32x4* lds;
    uint32_t lbase;                          // LDS address of the ring
    u32x4 xr, wr;                            // buffer resources of x and W
    // load i of a step brings rows 8 (NW i + w) .. + 7 of the tile, this lane chunk
    // c of row 8 (NW i + w) + l / 8
    int c;
    uint32_t xo[C::kLoads], wo[C::kLoads];   // byte offsets at K = 0; kOut for rows past the matrix
    int fo[4];                               // chunk of this lane's fragment of slice s in a 32-row block
    f32x16 acc[WBM][WBN];                    // [32-row block of x][32-column block of y]

    __device__ __forceinline__ BaseTile(const BaseArgs& args, u32x4* smem, int mt, int nt)
        : a(args), t(threadIdx.x), w(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)), l(threadIdx.x & 63),
          wm(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) / C::kWN),
          wn(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6) % C::kWN), m0(mt * TILE), n0(nt * TILE), lds(smem) {
        lbase = (uint32_t)(uintptr_t)(lds_u8*)(unsigned char*)smem;
        xr = rsrc_words(a.x, a.x_bytes);
        wr = rsrc_words(a.wt, a.w_bytes);
        // the slot of lane l is l % 8; its row's key is (row / 2) % 8
        c = (l & 7) ^ ((4 * (w & 1) + (l >> 4)) & 7);
#pragma unroll
        for (int i = 0; i < C::kLoads; ++i) {
            const int r = 8 * (NW * i + w) + (l >> 3);
            xo[i] = m0 + r < a.M ? (uint32_t)(((int64_t)(m0 + r) * a.ldx) * 2) + 16u * c : (uint32_t)kOut;
            wo[i] = n0 + r < a.N ? (uint32_t)(((int64_t)(n0 + r) * a.ldw) * 2) + 16u * c : (uint32_t)kOut;
        }
        // lane l reads chunk 2 s + l / 32 of row l % 32
#pragma unroll
        for (int s = 0; s < 4; ++s) fo[s] = (l & 31) * 8 + ((2 * s + (l >> 5)) ^ ((l >> 1) & 7));
#pragma unroll
        for (int i = 0; i < WBM; ++i)
#pragma unroll
            for (int j = 0; j < WBN; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    }

    // Load i of step k into ring buffer b.  Steps from kend on read zeros.
    __device__ __forceinline__ void load(int k, int kend, int b, int i) {
        // one select: K past the end moves the offset past the buffer (offsets
        // and kOut stay below 2^32 together, above its size)
        const uint32_t kb = k < kend && k * kStepK + 8 * c < a.K ? (uint32_t)k * (kStepK * 2) : (uint32_t)kOut;
        const uint32_t at = lbase + (uint32_t)(b * C::kStepChunks * 16);
        if (i < C::kLoads) lds_load16(xr, at + (uint32_t)(NW * i + w) * 1024u, (int)(xo[i] + kb));
        else lds_load16(wr, at + TILE * 128u + (uint32_t)(NW * (i - C::kLoads) + w) * 1024u, (int)(wo[i - C::kLoads] + kb));
    }

    // Fragment e of slice s of the step in buf.
    __device__ __forceinline__ u32x4 frag(const u32x4* buf, int s, int e) const {
        if (e < WBN) return buf[TILE * 8 + (wn * WBN + e) * 256 + fo[s]];
        return buf[(wm * WBM + e - WBN) * 256 + fo[s]];
    }

    // The product over steps [k0, k1), added into acc.  On return no load is in
    // flight and every wave's LDS reads are done.
    __device__ __forceinline__ void product(int k0, int k1) {
        constexpr int RB = C::kRing, SP = C::kSpread, NM = WBM * WBN;
        constexpr int kFirst = NL / SP;      // loads of a step issued in the slice of the barrier
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
            for (int i = 0; i < (b < RB - 1 ? NL : kFirst); ++i) load(k0 + b, k1, b, i);
        wait_vm<(RB - 2) * NL + kFirst>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        u32x4 f[2][NF];
#pragma unroll
        for (int e = 0; e < NF; ++e) f[0][e] = frag(lds, 0, e);
        int b = 0;
        for (int k = k0; k < k1; ++k) {
            const int bn = b + 1 == RB ? 0 : b + 1;      // the next step's buffer
            const int bp = b == 0 ? RB - 1 : b - 1;      // the last step's: being refilled
            const u32x4* cur = lds + b * C::kStepChunks;
            const u32x4* nxt = lds + bn * C::kStepChunks;
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                if (s == 3) {
                    // this wave's reads of cur are done and its loads of the next
                    // step have landed; past the barrier every wave's are and have
                    wait_lgkm0();
                    wait_vm<(RB - 2) * NL>();
                    __builtin_amdgcn_s_barrier();
                    __builtin_amdgcn_sched_barrier(0);
                }
                const int ph = (s + 1) & 3;              // 0 in the slice of the barrier
                int re = 0, ld = ph * kFirst;
#pragma unroll
                for (int m = 0; m < NM; ++m) {
                    acc[m / WBN][m % WBN] =
                        mma32x32<Fmt>(f[s & 1][m % WBN], f[s & 1][WBN + m / WBN], acc[m / WBN][m % WBN]);
                    // the next slice's fragments, early in the slice
                    const int want = min_i(NF, ((m + 1) * NF * 4 + NM * 3 - 1) / (NM * 3));
                    for (; re < want; ++re) f[(s + 1) & 1][re] = frag(s == 3 ? nxt : cur, (s + 1) & 3, re);
                    if (ph < SP)
                        for (; ld < ph * kFirst + ((m + 1) * kFirst) / NM; ++ld)
                            load(s == 3 ? k + RB : k - 1 + RB, k1, s == 3 ? b : bp, ld);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            b = bn;
        }
        wait_vm0_lgkm0();
        __builtin_amdgcn_s_barrier();
    }
};

// Transposing read: lane j of each 16 lanes gets element j % 4 of the 8-byte
// values that lanes j / 4, 4 + j / 4, 8 + j / 4 and 12 + j / 4 address.
typedef short s16x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ u32x2 lds_read_tr16(const unsigned char* p) {
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(lds_u8*)p));
}

// The adapter delta of one run of rows [lo, hi) with adapter g, ranks staged
// 64 at a time by buffer-to-LDS loads, all in flight together: B_g's rows as
// they are in the lower half of the LDS, the tile's rows of v in the upper.
// An operand slice of B_g (8 ranks of one column) comes out of LDS through two
// transposing reads.  (Staged through registers with B_g transposed by 2-byte
// LDS writes, whose lanes met in the same banks, the delta took about 10 us of
// a 256 tile at rank 64.)
template <class Fmt, int TILE>
__device__ __forceinline__ void tile_delta(BaseTile<Fmt, TILE>& T, const BasePiece& pc) {
    using C = BaseCfg<TILE>;
    constexpr int WBM = C::kWBM, WBN = C::kWBN, NW = C::kWaves;
    constexpr int TC = TILE / 8;                  // 16-byte chunks per staged row of B_g
    constexpr int BL = kBaseLoraRanks * TC / 64 / NW;  // B_g loads per wave (64 ranks)
    constexpr int VL = TILE * 16 / 64 / NW;       // v loads per wave (64 ranks)
    const BaseArgs& a = T.a;
    const DevAdapter ad = a.table[pc.adapter];
    const int R = ad.rank;
    const u32x4 br = rsrc_words(ad.B, (uint32_t)R * (uint32_t)a.N * 2u);
    const u32x4 vr = rsrc_words(a.v, a.v_bytes);
    const int l = T.l;
    const unsigned char* bt = (const unsigned char*)T.lds;
    f32x4* vt4 = (f32x4*)(T.lds + kBaseStageBytes / 16);
    for (int rc0 = 0; rc0 < R; rc0 += kBaseLoraRanks) {
        const int rr = min_i(kBaseLoraRanks, R - rc0);
        const int RC = (rr + 7) / 8;              // 8-rank chunks (one MFMA each)
        // B_g ranks [rc0, rc0 + 8 RC) of the tile's columns: chunk q of rank j at
        // slot q ^ 4 (j % 4) of row j (a transposing read's 4 rows x 32 bytes and
        // its neighbour's fall in different banks).  Ranks past R: zeros.
#pragma unroll
        for (int i = 0; i < BL; ++i) {
            const int first = (NW * i + T.w) * (64 / TC);      // the load's first rank (uniform)
            if (first < 8 * RC) {
                const int j = first + l / TC;
                const int col = T.n0 + 8 * ((l % TC) ^ (4 * (j & 3)));
                lds_load16(br, T.lbase + (uint32_t)(NW * i + T.w) * 1024u,
                           rc0 + j < R && col < a.N ? (int)((((int64_t)(rc0 + j) * a.N) + col) * 2) : kOut);
            }
        }
        // v of the tile's rows for ranks [rc0, rc0 + 64): float4 q (ranks
        // rc0 + 4 q .. + 3) of tile row r at 16 r + (q ^ (r % 16)), so that 16
        // lanes reading one chunk of 16 rows hit 16 bank groups.  Rows outside
        // [lo, hi) and float4s past R: zeros.
#pragma unroll
        for (int i = 0; i < VL; ++i) {
            const int r = 4 * (NW * i + T.w) + (l >> 4);
            const int m = T.m0 + r;
            const int j = rc0 + 4 * ((l & 15) ^ (r & 15));
            lds_load16(vr, T.lbase + (uint32_t)(kBaseStageBytes + (NW * i + T.w) * 1024),
                       m >= pc.lo && m < pc.hi && j < R ? (int)((((int64_t)m * a.ldv) + j) * 4) : kOut);
        }
        wait_vm<0>();
        __syncthreads();
        if (rr & 3) {                             // v past rank R, in the last float4, is whatever the buffer held
            for (int r = T.t; r < TILE; r += C::kThreads) {
                float* tail = (float*)(vt4 + 16 * r + ((rr >> 2) ^ (r & 15)));
                for (int e = rr & 3; e < 4; ++e) tail[e] = 0.f;
            }
            __syncthreads();
        }
        // v operand of block i, chunk c: lane l takes row 32 (WBM wm + i) + l % 32
        // of the tile, ranks rc0 + 8 c .. +7, the high part of s_g v for l < 32
        // and the low part for l >= 32 (the B_g operand holds the same ranks in
        // both halves of K).
        auto vload = [&](int i, int c, f32x4& v0, f32x4& v1) __attribute__((always_inline)) {
            const int r = 32 * WBM * T.wm + 32 * i + (l & 31);
            v0 = vt4[16 * r + ((2 * c) ^ (r & 15))];
            v1 = vt4[16 * r + ((2 * c + 1) ^ (r & 15))];
        };
        // v enters the MFMA pre-multiplied by s_g, so the delta adds straight
        // into the base accumulators.
        float vmul = ad.scale;
        const bool hi_half = l < 32;
        auto bload = [&](int c, int jn) __attribute__((always_inline)) -> u32x4 {
            const int col = 32 * (WBN * T.wn + jn) + 16 * ((l >> 4) & 1) + 4 * (l & 3);
            const int j = 8 * c + ((l >> 2) & 3);             // the two reads: ranks j and j + 4
            const unsigned char* p = bt + (j * TC + ((col >> 3) ^ (4 * (j & 3)))) * 16 + (l & 1) * 8;
            const u32x2 lo = lds_read_tr16(p), hi = lds_read_tr16(p + 4 * TC * 16);
            return u32x4{lo.x, lo.y, hi.x, hi.y};
        };
        auto vfrag = [&](const f32x4& v0, const f32x4& v1) __attribute__((always_inline)) -> u32x4 {
            u32x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const f32x4& v4 = e < 2 ? v0 : v1;
                const float p0 = v4[2 * (e & 1)] * vmul, p1 = v4[2 * (e & 1) + 1] * vmul;
                const uint32_t h = Fmt::pack2(p0, p1);
                // (p's own rounding is its high part)
                o[e] = Fmt::pack2(hi_half ? p0 : p0 - Fmt::to_f32(lo16(h)), hi_half ? p1 : p1 - Fmt::to_f32(hi16(h)));
            }
            return o;
        };
        // binary16 cannot hold a high part past 65504: past 2^15 the wave scales v
        // by 2^k (k < 0) and its accumulators by 2^k around these MFMAs, then
        // back by 2^-k; powers of two, exact for every accumulator at or above
        // 2^-126+|k| (far below the output's precision).
        float unscale = 1.f;
        if constexpr (Fmt::kNarrowRange) {
            float vabs = 0.f;
#pragma unroll 1
            for (int c = 0; c < RC; ++c)
#pragma unroll
                for (int i = 0; i < WBM; ++i) {
                    f32x4 v0, v1;
                    vload(i, c, v0, v1);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        vabs = fmaxf(vabs, fmaxf(fabsf(v0[e] * ad.scale), fabsf(v1[e] * ad.scale)));
                }
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) vabs = fmaxf(vabs, __shfl_xor(vabs, d, 64));
            if (vabs >= 32768.f) {
                const int E = (int)((__float_as_uint(vabs) >> 23) & 0xff) - 127;
                const int k = max_i(14 - E, -64);
                const float down = __uint_as_float((uint32_t)(127 + k) << 23);
                vmul = ad.scale * down;
                unscale = __uint_as_float((uint32_t)(127 - k) << 23);
#pragma unroll
                for (int i = 0; i < WBM; ++i)
#pragma unroll
                    for (int jn = 0; jn < WBN; ++jn) T.acc[i][jn] *= down;
            }
        }
        // In the small tile (one wave per SIMD) the next chunk's operands are
        // read while this one's MFMAs run; in the big one the SIMD's other wave
        // runs meanwhile and the registers are kept for the accumulators.
        constexpr bool kAhead = NW == 4;
        u32x4 bn[WBN];
        f32x4 vn[WBM][2];
        auto fetch = [&](int c) __attribute__((always_inline)) {
#pragma unroll
            for (int jn = 0; jn < WBN; ++jn) bn[jn] = bload(c, jn);
            if constexpr (kAhead)
#pragma unroll
                for (int i = 0; i < WBM; ++i) vload(i, c, vn[i][0], vn[i][1]);
        };
        if constexpr (kAhead) fetch(0);
#pragma unroll 1
        for (int c = 0; c < RC; ++c) {
            if constexpr (!kAhead) fetch(c);
            u32x4 bf[WBN];
#pragma unroll
            for (int jn = 0; jn < WBN; ++jn) bf[jn] = bn[jn];
            if constexpr (kAhead) {
                u32x4 vf[WBM];
#pragma unroll
                for (int i = 0; i < WBM; ++i) vf[i] = vfrag(vn[i][0], vn[i][1]);
                if (c + 1 < RC) fetch(c + 1);
#pragma unroll
                for (int i = 0; i < WBM; ++i)
#pragma unroll
                    for (int jn = 0; jn < WBN; ++jn) T.acc[i][jn] = mma32x32<Fmt>(bf[jn], vf[i], T.acc[i][jn]);
            } else {
#pragma unroll
                for (int i = 0; i < WBM; ++i) {
                    f32x4 v0, v1;
                    vload(i, c, v0, v1);
                    const u32x4 vf = vfrag(v0, v1);
#pragma unroll
                    for (int jn = 0; jn < WBN; ++jn) T.acc[i][jn] = mma32x32<Fmt>(bf[jn], vf, T.acc[i][jn]);
                }
            }
        }
        if constexpr (Fmt::kNarrowRange) {
            if (unscale != 1.f) {
#pragma unroll
                for (int i = 0; i < WBM; ++i)
#pragma unroll
                    for (int jn = 0; jn < WBN; ++jn) T.acc[i][jn] *= unscale;
            }
        }
        __syncthreads();                          // every wave's reads are done before the next staging
    }
}

template <class Fmt, int TILE>
__global__ void __launch_bounds__(BaseCfg<TILE>::kThreads) lora_base_kernel(BaseArgs a) {
    using C = BaseCfg<TILE>;
    constexpr int WBM = C::kWBM, WBN = C::kWBN;
    __shared__ __attribute__((aligned(1024))) u32x4 smem[kLdsBytes / 16];
    // K in stages of base_bk(TILE) (a range's unit) and in steps of kStepK
    constexpr int kStageSteps = base_bk(TILE) / kStepK;
    const int nk = (a.K + kStepK - 1) / kStepK;
    const int p = blockIdx.x;
    const int slots = a.n_xcd * a.per_xcd;   // workgroups of the whole tiles, per_xcd for every XCD
    int tile, k0 = 0, k1 = nk, range = -1;
    if (p < slots) {
        const int q = p / a.n_xcd;
        tile = (p - q * a.n_xcd) * a.per_xcd + q;
        if (tile >= a.n_whole) return;
    } else {
        const int u = p - slots;
        tile = a.n_whole + u / a.split;
        range = u - (tile - a.n_whole) * a.split;
        k0 = range * a.chunk * kStageSteps;
        k1 = min_i(nk, k0 + a.chunk * kStageSteps);
        if (tile >= a.n_mt * a.n_nt || k0 >= k1) return;
    }
    int mt, nt;
    tile_coords(a, tile, mt, nt);
    BaseTile<Fmt, TILE> T(a, smem, mt, nt);
    T.product(k0, k1);

    // the adapter delta of each run of rows that carries one (once per tile)
    if (range <= 0) {
        const int pe = a.piece_off[mt + 1];
        for (int pi = a.piece_off[mt]; pi < pe; ++pi) {
            const BasePiece pc = a.pieces[pi];
            tile_delta<Fmt, TILE>(T, pc);
        }
    }

    if (range >= 0) {
        // partial tile in accumulator order: float4 g of block (i, j) of wave
        // w, lane l at (((w WBM + i) WBN + j) 4 + g) 64 + l
        float4* dst = (float4*)a.part + (size_t)((tile - a.n_whole) * a.split + range) * C::kTileQuads;
#pragma unroll
        for (int i = 0; i < WBM; ++i)
#pragma unroll
            for (int j = 0; j < WBN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x16& c = T.acc[i][j];
                    dst[(((T.w * WBM + i) * WBN + j) * 4 + g) * 64 + T.l] =
                        float4{c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]};
                }
        return;
    }

    // y: accumulator r of block (i, j) is column 32 j + 8 (r / 4) + 4 (l / 32) + r % 4
    // of row 32 i + l % 32 of the wave's part of the tile.  Stored from there, a wave
    // instruction writes 8 bytes to each of 64 places (the tile's stores took
    // 13 us on 256 tiles of 256); so the rounded part goes through the wave's
    // own share of LDS (16-byte chunk q of row r at slot q ^ r % 16, its 8-byte
    // halves swapped for odd r / 16, so that writes and reads are free of bank
    // conflicts) and out by rows, 16 bytes per lane.
    const rsrc_t yr = make_rsrc(a.y, a.y_bytes);
    constexpr int QC = 4 * WBN;               // 16-byte chunks per row of the wave's part
    u32x2* q8 = (u32x2*)(smem + T.w * 32 * WBM * QC);
    const u32x4* q16 = (const u32x4*)q8;
    constexpr int kMask = QC < 16 ? QC - 1 : 15;
#pragma unroll
    for (int i = 0; i < WBM; ++i) {            // 32 rows at a time (registers)
        const int r = 32 * i + (T.l & 31);
#pragma unroll
        for (int j = 0; j < WBN; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int q = 4 * j + g, h = (T.l >> 5) ^ ((T.l >> 4) & 1);
                const f32x16& c = T.acc[i][j];
                q8[(r * QC + (q ^ (r & kMask))) * 2 + h] =
                    u32x2{Fmt::pack2(c[4 * g], c[4 * g + 1]), Fmt::pack2(c[4 * g + 2], c[4 * g + 3])};
            }
#pragma unroll
        for (int it = 0; it < QC / 2; ++it) {
            const int ro = 32 * i + it * (64 / QC) + T.l / QC, q = T.l % QC;
            const u32x4 v = q16[ro * QC + (q ^ (ro & kMask))];
            const int m = T.m0 + 32 * WBM * T.wm + ro, n = T.n0 + 32 * WBN * T.wn + 8 * q;
            bstore16((ro >> 4) & 1 ? u32x4{v.z, v.w, v.x, v.y} : v, yr,
                     m < a.M && n < a.N ? (int)((((int64_t)m * a.ldy) + n) * 2) : kOut);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// The split tiles: the float32 partials of ranges 0 .. split-1 added in that
// order, rounded once and stored.  One thread per four consecutive columns of
// one row (one float4 of every partial).
constexpr int kReduceThreads = 256;

template <class Fmt, int TILE>
__global__ void __launch_bounds__(kReduceThreads) lora_base_reduce_kernel(BaseArgs a) {
    using C = BaseCfg<TILE>;
    constexpr int WBM = C::kWBM, WBN = C::kWBN;
    static_assert(C::kTileQuads % kReduceThreads == 0, "reduce grid");
    const int gid = blockIdx.x * kReduceThreads + threadIdx.x;
    const int rt = gid / C::kTileQuads;
    const int e = gid - rt * C::kTileQuads;
    const int l = e & 63, g = (e >> 6) & 3, blk = e >> 8;
    const int j = blk % WBN, i = (blk / WBN) % WBM, w = blk / (WBN * WBM);
    const int tile = a.n_whole + rt;
    if (tile >= a.n_mt * a.n_nt) return;
    int mt, nt;
    tile_coords(a, tile, mt, nt);
    const int m = mt * TILE + 32 * (WBM * (w / C::kWN) + i) + (l & 31);
    const int n = nt * TILE + 32 * (WBN * (w % C::kWN) + j) + 8 * g + 4 * (l >> 5);
    const float4* src = (const float4*)a.part + (size_t)rt * a.split * C::kTileQuads + e;
    float4 sum = src[0];
    for (int r = 1; r < a.split; ++r) {
        const float4 v = src[(size_t)r * C::kTileQuads];
        sum.x += v.x;
        sum.y += v.y;
        sum.z += v.z;
        sum.w += v.w;
    }
    if (m < a.M && n < a.N) {
        const rsrc_t yr = make_rsrc(a.y, a.y_bytes);
        bstore8(u32x2{Fmt::pack2(sum.x, sum.y), Fmt::pack2(sum.z, sum.w)}, yr, (int)((((int64_t)m * a.ldy) + n) * 2));
    }
}

template <class Fmt, int TILE>
hipError_t launch_tiles(const BaseArgs& a, hipStream_t s) {
    const int n_split = a.split > 1 ? a.n_mt * a.n_nt - a.n_whole : 0;
    const int grid = a.n_xcd * a.per_xcd + n_split * a.split;
    if (grid <= 0) return hipSuccess;
    hipLaunchKernelGGL((lora_base_kernel<Fmt, TILE>), dim3(grid), dim3(BaseCfg<TILE>::kThreads), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n_split == 0) return e;
    const int rgrid = n_split * (BaseCfg<TILE>::kTileQuads / kReduceThreads);
    hipLaunchKernelGGL((lora_base_reduce_kernel<Fmt, TILE>), dim3(rgrid), dim3(kReduceThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_base(const BaseArgs& a, int dtype, hipStream_t s) {
    if (a.tile == kBaseBig)
        return dtype == 0 ? launch_tiles<FmtF16, kBaseBig>(a, s) : launch_tiles<FmtBF16, kBaseBig>(a, s);
    if (a.tile == kBaseSmall)
        return dtype == 0 ? launch_tiles<FmtF16, kBaseSmall>(a, s) : launch_tiles<FmtBF16, kBaseSmall>(a, s);
    return hipErrorInvalidValue;
}

}  // namespace lora
