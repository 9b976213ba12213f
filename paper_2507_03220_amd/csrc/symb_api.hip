// Host side of the C ABI declared in include/symb.h: argument checks, the segment
// planner, descriptor staging and the kernel launches.  Nothing here computes any part
// of the layer on the CPU; without a GPU every compute entry point fails with
// SYMB_ERR_DEVICE.
#include "../../include/symb.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <utility>
#include <vector>

#include "adapter_kernels.hpp"
#include "gemm16_kernel.hpp"
#include "narrow_kernel.hpp"
#include "shortk_kernel.hpp"
#include "small_kernels.hpp"
#include "symb_ring.hpp"

using namespace symb;

// Workspace of symb_base_linear_fwd_static: a file-scope array, so that entry point needs no device
// allocation at all.  In host code this name is only a stand-in for the symbol; the address
// of each device's copy is asked for once, in symb_create (hipGetSymbolAddress), and kept in the context.
static __device__ __align__(256) unsigned char symb_static_scratch[SYMB_STATIC_SCRATCH_BYTES];

// One workgroup per entry of `out`: the id of the XCD (hardware register XCC_ID) the workgroup runs on.
__global__ void symb_xcc_probe_kernel(int* out) {
    if (threadIdx.x == 0) {
        unsigned v;
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(v));
        out[blockIdx.x] = (int)(v & 0xfu);
    }
}

namespace {

thread_local std::string g_tls_error;

constexpr size_t kSlotBytes = (size_t)2 << 20;  // capacity of one descriptor blob
constexpr int kSkinnyRows = SKINNY_ROWS;        // rows per skinny / scale work item
constexpr int kMaxTimed = 4096;                 // GEMM launches recorded between two timing reads
constexpr int kTimedNarrow = 32, kTimedShortK = 33;      // symb_gemm_narrow_kernel, symb_gemm_shortk_kernel in the measurement hook
constexpr int kXccProbeGroups = 2048;           // workgroups of the XCD-rule measurement (8 rounds of 256)

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
inline int rpad_of(int r) { return (r + 15) / 16 * 16; }

struct HipRuntime {                             // what the descriptor ring asks of HIP
    using Stream = hipStream_t;
    using Event = hipEvent_t;
    using Status = hipError_t;
    static Status record(Event ev, Stream st) {
        const hipError_t e = hipEventRecord(ev, st);
        if (e != hipSuccess) (void)hipGetLastError();
        return e;
    }
    static Status wait(Event ev) { return hipEventSynchronize(ev); }
    static Status wait_all() { return hipDeviceSynchronize(); }
    static bool done(Event ev) {
        if (hipEventQuery(ev) == hipSuccess) return true;
        (void)hipGetLastError();                // (not ready yet is no error of this call)
        return false;
    }
    static StreamState state(Stream st, uint64_t* capture) {
        hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
        unsigned long long id = 0;
        const hipError_t e = hipStreamGetCaptureInfo(st, &s, &id);
        if (e == hipSuccess) {
            *capture = s == hipStreamCaptureStatusNone ? 0 : id + 1;
            return StreamState::Known;
        }
        (void)hipGetLastError();
        return e == hipErrorStreamCaptureImplicit ? StreamState::Unsure : StreamState::Gone;     // (HIP looks the handle up among its live streams)
    }
    static uint64_t thread(Stream st) {
        if (st != hipStreamPerThread) return 0;
        static std::atomic<uint64_t> threads{0};
        thread_local const uint64_t mine = ++threads;
        return mine;
    }
};
constexpr int kSlots = DescRing<HipRuntime>::kSlots;

}  // namespace

struct symb_context {
    int device = 0;
    unsigned char* host_ring = nullptr;   // pinned, kSlots * kSlotBytes
    unsigned char* dev_ring = nullptr;    // device, kSlots * kSlotBytes
    DescRing<HipRuntime> ring;
    HipRuntime rt;
    int64_t desc_sent = 0, desc_in_place = 0;
    int call_slot = -1;                   // the slot this call's descriptors went to (-1: none yet)
    std::string error;
    // measurement switches (symb_debug_set_option); all on by default
    bool opt_desc_reuse = true, opt_k_split = true, opt_small_rows = true, opt_skinny_deep = true;
    // Whether workgroup id mod 8 names the XCD a workgroup runs on, measured at creation: the K-split of
    // the GEMM keeps all parts of a tile on one XCD (behind one L2) and is used only if this holds.
    bool xcd_rule = false;
    int xcc_of_residue[8] = {-1, -1, -1, -1, -1, -1, -1, -1};
    unsigned char* static_scratch = nullptr;     // this device's copy of the file-scope scratch array
    std::vector<const void*> lds_attr_set;       // kernels whose dynamic-LDS limit was raised on this context's device
    // measurement hook: event pairs around GEMM launches
    bool timing = false;
    std::vector<hipEvent_t> tev;                 // 2 * kMaxTimed events, created on first enable
    struct Timed { int variant; double flops; };
    std::vector<Timed> timed;
};

namespace {

symb_status fail(symb_handle h, symb_status st, const char* fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (h) h->error = buf;
    g_tls_error = buf;
    return st;
}

#define SYMB_HIP(h, call)                                                                      \
    do {                                                                                       \
        hipError_t e_ = (call);                                                                \
        if (e_ != hipSuccess)                                                                  \
            return fail(h, SYMB_ERR_DEVICE, "%s failed: %s", #call, hipGetErrorString(e_));    \
    } while (0)

symb_status validate(symb_handle h, const symb_batch* b) {
    if (!b) return fail(h, SYMB_ERR_INVALID_ARG, "batch is null");
    if (b->d_in <= 0 || b->d_out <= 0) return fail(h, SYMB_ERR_INVALID_ARG, "d_in and d_out must be positive");
    if ((b->d_in % 8) || (b->d_out % 8)) return fail(h, SYMB_ERR_INVALID_ARG, "d_in and d_out must be multiples of 8");
    if (b->weight_layout != SYMB_WEIGHT_LINEAR && b->weight_layout != SYMB_WEIGHT_CONV1D)
        return fail(h, SYMB_ERR_INVALID_ARG, "unknown weight layout %d", b->weight_layout);
    if (b->num_segments < 0) return fail(h, SYMB_ERR_INVALID_ARG, "num_segments is negative");
    if (!b->seg_offsets) return fail(h, SYMB_ERR_INVALID_ARG, "seg_offsets is null");
    if (b->num_segments > 0 && !b->adapters) return fail(h, SYMB_ERR_INVALID_ARG, "adapters is null");
    if (b->seg_offsets[0] != 0) return fail(h, SYMB_ERR_BAD_SEGMENTS, "seg_offsets[0] must be 0");
    for (int i = 0; i < b->num_segments; ++i)
        if (b->seg_offsets[i + 1] < b->seg_offsets[i])
            return fail(h, SYMB_ERR_BAD_SEGMENTS, "seg_offsets decrease at segment %d", i);
    for (int i = 0; i < b->num_segments; ++i) {
        const symb_adapter& a = b->adapters[i];
        switch (a.kind) {
            case SYMB_ADAPTER_NONE: break;
            case SYMB_ADAPTER_LORA:
                if (a.rank < 1) return fail(h, SYMB_ERR_INVALID_ARG, "segment %d: LoRA rank must be >= 1", i);
                if (a.rank > SYMB_MAX_RANK)
                    return fail(h, SYMB_ERR_UNSUPPORTED, "segment %d: LoRA rank %d exceeds SYMB_MAX_RANK", i, a.rank);
                if (!a.A || !a.B) return fail(h, SYMB_ERR_INVALID_ARG, "segment %d: LoRA needs A and B", i);
                if (((uintptr_t)a.A & 15) || ((uintptr_t)a.dA & 15) || ((uintptr_t)a.dB & 3) || ((uintptr_t)a.B & 1))
                    return fail(h, SYMB_ERR_INVALID_ARG, "segment %d: adapter pointer misaligned", i);
                if ((a.rank % 8) == 0 && ((uintptr_t)a.B & 15))
                    return fail(h, SYMB_ERR_INVALID_ARG, "segment %d: B must be 16-byte aligned", i);
                break;
            case SYMB_ADAPTER_IA3:
                if (!a.A) return fail(h, SYMB_ERR_INVALID_ARG, "segment %d: IA3 needs its vector in A", i);
                if (((uintptr_t)a.A & 15) || ((uintptr_t)a.dA & 15))
                    return fail(h, SYMB_ERR_INVALID_ARG, "segment %d: adapter pointer misaligned", i);
                break;
            case SYMB_ADAPTER_IA3_IN:
                if (!a.A) return fail(h, SYMB_ERR_INVALID_ARG, "segment %d: IA3 input scaling needs its vector in A", i);
                if (((uintptr_t)a.A & 15) || ((uintptr_t)a.dA & 15))
                    return fail(h, SYMB_ERR_INVALID_ARG, "segment %d: adapter pointer misaligned", i);
                break;
            default: return fail(h, SYMB_ERR_INVALID_ARG, "segment %d: unknown adapter kind %d", i, a.kind);
        }
    }
    return SYMB_OK;
}

bool misaligned16(const void* p) { return ((uintptr_t)p & 15) != 0; }

// ---- planner (pure integer host work) ------------------------------------------------------
void plan_row_tiles(const symb_batch* b, int tile_m, std::vector<int32_t>& lo, std::vector<int32_t>& hi) {
    const int S = b->num_segments;
    const int32_t* off = b->seg_offsets;
    const int T = off[S];
    const int nt = (T + tile_m - 1) / tile_m;
    lo.assign(nt, 0);
    hi.assign(nt, -1);
    int s = 0;
    for (int u = 0; u < nt; ++u) {
        const int r0 = u * tile_m, r1 = std::min(T, r0 + tile_m);
        while (off[s + 1] <= r0) ++s;            // first segment that owns row r0 (non-empty by construction)
        int e = s;
        while (off[e + 1] < r1) ++e;             // segment that owns row r1 - 1
        lo[u] = s;
        hi[u] = e;
    }
}

// Per row tile: 1 if one of its segments is of `kind` (the tiles whose epilogue has rows to scale).
std::vector<int32_t> plan_tile_kind(const symb_batch* b, const std::vector<int32_t>& lo, const std::vector<int32_t>& hi, int kind) {
    std::vector<int32_t> v(lo.size(), 0);
    for (size_t u = 0; u < lo.size(); ++u)
        for (int i = lo[u]; i <= hi[u] && !v[u]; ++i) v[u] = b->adapters[i].kind == kind;
    return v;
}

// Row chunks of `rows` rows, never across a segment boundary; only_kind >= 0: of segments of that kind only.
void plan_chunks(const symb_batch* b, int rows, int only_kind, std::vector<RowChunk>& out) {
    out.clear();
    for (int i = 0; i < b->num_segments; ++i) {
        if (only_kind >= 0 && b->adapters[i].kind != only_kind) continue;
        for (int r = b->seg_offsets[i]; r < b->seg_offsets[i + 1]; r += rows)
            out.push_back(RowChunk{i, r, std::min(rows, b->seg_offsets[i + 1] - r), 0});
    }
}

struct BatchInfo {
    int S = 0, T = 0;
    int n_lora = 0, n_ia3 = 0, n_ia3in = 0;
    int max_rpad = 0;
    size_t packed_elems = 0;   // sum rpad_i * d_out over LoRA segments (packed B^T)
    size_t packed_at_elems = 0;// sum r_i * d_in over LoRA segments (packed A^T, input-major weight only)
};

BatchInfo inspect(const symb_batch* b) {
    BatchInfo bi;
    bi.S = b->num_segments;
    bi.T = b->seg_offsets[bi.S];
    for (int i = 0; i < bi.S; ++i) {
        const symb_adapter& a = b->adapters[i];
        if (a.kind == SYMB_ADAPTER_LORA) {
            ++bi.n_lora;
            bi.max_rpad = std::max(bi.max_rpad, rpad_of(a.rank));
            bi.packed_elems += (size_t)rpad_of(a.rank) * b->d_out;
            bi.packed_at_elems += align_up((size_t)a.rank * b->d_in, 8);
        } else if (a.kind == SYMB_ADAPTER_IA3) {
            ++bi.n_ia3;
        } else if (a.kind == SYMB_ADAPTER_IA3_IN) {
            ++bi.n_ia3in;
        }
    }
    return bi;
}

// Tile variants of the GEMM kernels (gemm16_kernel.hpp): 3 = 256x256 tile, taken when the problem has
// enough such tiles to fill the chip; 2 = 128x128 tile or, where gemm_plan says so, 4 = 256x128 or 5 = 32-row tile, for everything smaller.
constexpr int kTile128 = 2, kTile256 = 3, kTileTall = 4, kTileMid = 5;
int tile_rows(int variant) { return variant == kTileMid ? MID_ROWS : variant == kTile128 ? 128 : 256; }
int tile_cols(int variant) { return variant == kTile256 ? 256 : 128; }
int gemm_variant(int M, int N, int K) {
    const long big = (long)((M + 255) / 256) * ((N + 255) / 256), small = (long)((M + 127) / 128) * ((N + 127) / 128);
    if (big < 128) return 2;
    // From 128 tiles of 256x256 on, as long as the 128x128 ones are one round of two per CU, those fill the chip where the others leave up to half the CUs
    // idle, but they read twice the LDS bytes per flop, and lose on a long inner dimension, sooner the wider the output.  Weights from HBM, us in
    // small / big tiles: 2048 rows, 4096 wide, K = 4096 70 / 76, 4608 80 / 81, 5120 90 / 88, 8192 128 / 119; 8192 rows, 1024 wide, K = 4608 80 / 81; 1024 rows, 8192 wide,
    // K = 2048 42 / 55, 4096 77 / 77, 4608 87 / 81; 512 rows, 16384 wide, K = 2048 45 / 54, 4096 84 / 79; ragged: 1800 rows, 4096 wide, K = 4608 74 / 81;
    // 3700 rows, 2056 wide (135 big tiles, 493 small) K = 4096 65 / 79; 3840 rows, 2184 wide (135, 540) K = 2048 52 / 46.
    // (The 256x128 tile, which gemm_plan puts in the small one's place, has not been weighed against the big one.)
    return small <= 512 && K <= (N <= 4096 ? 4608 : N <= 8192 ? 4096 : 3072) ? 2 : 3;
}

// Row tiles per group of the tile walk (a group is walked column by column, so the 32 tiles an XCD runs
// at once are g row tiles x 32 / g column tiles).  Measured on the Gemma2-27B-shaped launches (80 row
// tiles), GEMM calls of a step summed: g = 5 32.7 ms, 4 32.9, 6 33.1, 8 33.3, 10 33.1, 7 33.6, 16 34+:
// small groups win (most on the long-K shapes, 2-3 %), and a g that does not divide the row tiles loses
// (ragged last group, groups straddling the XCDs' runs).  That holds for launches of many rounds whose
// tiles cost the same.  Where row tiles differ (a mixed batch: a row tile of dozens of one-token LoRA
// segments takes far longer than one inside a long segment) small groups put more column tiles of the
// slowest row tile side by side and lose (+6 % on the mixed workload's step), and launches of two or
// three rounds do not care.  So: 8 unless the launch has at least five rounds per XCD and at most two
// segments per row tile; then the divisor of the row-tile count nearest 5 among 3..8, else 4.
int gemm_group_m(int num_m_tiles, int num_n_tiles, const std::vector<int32_t>& seg_lo, const std::vector<int32_t>& seg_hi) {
    int most = 0;
    for (size_t u = 0; u < seg_lo.size(); ++u) most = std::max(most, seg_hi[u] - seg_lo[u] + 1);
    if (most > 2 || ((long)num_m_tiles * num_n_tiles + 7) / 8 < 160) return 8;
    for (int g : {5, 4, 6, 3, 8, 7})
        if (num_m_tiles % g == 0) return g;
    return 4;
}

// K-split.  Every XCD walks a contiguous run of per_xcd = ceil(tiles / 8) tiles; the tiles of that run
// from number `whole` on are computed by `parts` workgroups each, one per K range, which leave fp32
// partial tiles in the workspace; the last one to arrive adds them up in part order and writes the
// tile.  Two uses:
//  * 128x128 tiles, launches that leave most of the chip idle (batches of a few hundred rows on a
//    4096-wide layer: 96 tiles for 256 CUs, each workgroup walking the whole K extent alone, a chain
//    of load and LDS latencies of about 0.5 us per 64 k): all tiles split (whole = 0),
//    parts = 320 / tiles: three parts for 96 tiles, none from 161 tiles on; at least 12 stages per part
//    (96 rows of 4096 x 4096: 20.6 us in 5 parts, 23.4 in 8; 2000 rows of 1024 x 1024: 13.6 us whole, 17.4 in 2); up to four parts
//    from 8 stages on, where all of them together are at most 160 workgroups (2048 x 2048: 64 rows 13.9 us in 4 parts, 15.4 in 2,
//    256 rows 15.5 / 17.2; in 6 parts 14.6 / 16.3); twice
//    as many where a part would have 64 stages or more and a second workgroup per CU finds room (397 rows of
//    11008 -> 4096: 57.8 us in 4 parts, 73 in 2).
//  * 256x256 tiles, one workgroup per CU, 32 CUs per XCD: a run of per_xcd tiles ends in a round of
//    rem = per_xcd % 32 tiles that takes as long as a full one.  These last tiles are split into the
//    number of parts (at most 4) that makes the round shortest by a simple model of its time: e.g.
//    4 parts for 8 tiles (a quarter of a tile's time), 3 parts for 20 tiles of a long K (60
//    workgroups in two passes of a third each), none where the sum of the partial tiles (256 KiB
//    each) would cost what the split saves.
// parts is at most 8.  A pure function of the shape: the
// workspace figure does not depend on the process environment or on the handle.
struct SplitPlan {
    int parts = 1;        // K ranges per split tile (1: no split)
    int whole = 0;        // tiles per XCD that stay whole
    int slots = 0;        // split tiles of the launch (over all XCDs): arrival counters
    size_t bytes = 0;     // partial tiles: slots * parts * tile rows * tile columns * 4
    bool doubled = false; // half the parts would do as well (see above)
};
SplitPlan gemm_split_plan(int M, int N, int K) {
    SplitPlan s;
    constexpr int target = 320, tail_max = 4;
    if (M <= 0) return s;
    const int KF = K / 64;
    if (gemm_variant(M, N, K) == 2) {
        const long tiles = (long)((M + 127) / 128) * ((N + 127) / 128);
        int P = std::min({8, KF / 12, (int)(target / tiles)});
        if (KF >= 24) P = std::max(P, std::min({4, KF / 8, (int)(160 / tiles)}));
        if (P < 2) return s;
        if (P <= 4 && KF / P >= 64 && 2 * P * tiles <= 512) {
            P *= 2;
            s.doubled = true;
        }
        s.parts = P;
        s.slots = (int)tiles;                  // whole = 0: a tile's slot is its number in the walk
        s.bytes = (size_t)tiles * P * 128 * 128 * 4;
    } else {
        const long tiles = (long)((M + 255) / 256) * ((N + 255) / 256);
        const int per_xcd = (int)((tiles + 7) / 8), rem = per_xcd % 32;
        if (rem == 0) return s;
        // The last round takes ceil(rem * P / 32) / P of a tile's time (a tile: about 1.45 us per stage)
        // plus, when split, about 8 + 4 P us for storing and adding up the partial tiles.
        const double tile_us = 1.45 * KF;
        int P = 1;
        double best = tile_us;
        for (int q = 2; q <= std::min(tail_max, KF / 8); ++q) {
            const double us = (double)((rem * q + 31) / 32) / q * tile_us + 8.0 + 4.0 * q;
            if (us < best - 4.0) { best = us; P = q; }      // a gain of a few us is not worth the traffic
        }
        if (P < 2 || best > 0.85 * tile_us) return s;      // nor is a gain of less than 15 % of the round
        s.parts = P;
        s.whole = per_xcd - rem;
        s.slots = 8 * rem;
        s.bytes = (size_t)s.slots * P * 256 * 256 * 4;
    }
    return s;
}

struct DeltaPlan {
    std::vector<RowChunk> items;          // the segments (pad: first row of their terms)
    int rows = 0;                         // rows of terms
};
// The tile of a product, its K split and the terms of short segments that it adds from memory (gemm_plan).
struct GemmPlan {
    int variant = kTile128;
    SplitPlan split;
    bool unsplit_for_base = false;    // the shape would split, but the pre-adapter output is wanted
    DeltaPlan terms;
};

// Short LoRA segments (at most kDeltaRows rows) whose term the tiled kernels add from memory (symb_lora_delta_kernel) instead of running a chain of k-steps
// for each: all of them that meet a row tile with at least delta_steps() such steps.  The steps of the row tile with the most set what the
// chains cost (the K parts of a split tile share them), a launch and the traffic of the fp32 terms (8 bytes per row and output column) what they
// cost from memory.  Measured over clients of 1 to 16 rows and ranks 8 to 128, 96 to 2048 such rows alone or beside long segments, 1024 to 11008
// columns, both directions, us from memory / in steps: 4096 x 4096, 96 rows (five parts), 24 steps 40.8 / 37.4, 48 steps 42.3 / 43.4, 96 steps
// 53.7 / 61.8; 64 rows beside 1984 (whole), 16 steps 9 us less, 8 steps equal; 512 rows of 11008 -> 4096 (four parts) 32 steps 108 / 99, 64 steps equal; 2048
// rows of 4096 -> 11008 (256x256 tile) 16 steps 232 / 205, 64 steps 270 / 317.  By the lines below what is chosen is at most 3 %, what is not
// at most 5 % slower than the other way, over the whole sweep.  The 256x128 tile, whose parts share the steps too, has the 128x128 one's line: 400 calls of 129 to 4500 rows
// with 3 to 150 short clients, whole and in two or three parts, are at most 4.1 % slower than the faster way, 0.16 % on average; by the 256x256 tile's line 6.5 and
// 0.35 % (3894 rows of 9072 -> 544 in three parts, 16 steps, 101.1 from memory / 94.9 in steps; 252 of 7192 -> 16256 in two, 10 steps, 115.0 / 108.2).
// A launch whose shape would split, but whose pre-adapter output is wanted, has the line of two parts: 40 training steps with such calls, terms against steps, lost up to 4 % at 8
// to 15 steps (136 rows of 6144 -> 1416, 13 steps in both directions, 255.1 us in steps, 265.6 from memory) and gained up to 18 % from 17 on (348 of 4096 -> 1104, 58
// steps, 167.5 / 141.6).
// Batches of more than kDeltaSegments segments, or of more terms than kDeltaBytes, keep the steps, as does one whose descriptors have no
// room for the terms' (add_gemm_desc).
constexpr int kDeltaRows = 16, kDeltaSegments = 4096;
constexpr size_t kDeltaBytes = (size_t)160 << 20;
int delta_steps(const GemmPlan& plan, int rows, int N) {
    const double elems = 1e-6 * rows * N;
    const int parts = plan.unsplit_for_base ? 2 : plan.split.parts;
    return (int)(plan.variant == kTile256 ? 8 + 1.5 * elems : 8 * parts + 5 * elems);
}
DeltaPlan delta_plan(const symb_batch* b, const GemmPlan& plan, int N) {
    const int tile_m = tile_rows(plan.variant);
    DeltaPlan d;
    const int S = b->num_segments;
    auto steps = [&](int i) {
        const int n = b->seg_offsets[i + 1] - b->seg_offsets[i];
        return b->adapters[i].kind == SYMB_ADAPTER_LORA && n > 0 && n <= kDeltaRows ? rpad_of(b->adapters[i].rank) / 16 : 0;
    };
    if (S > kDeltaSegments) return d;
    int all = 0, rows = 0;
    for (int i = 0; i < S; ++i)
        if (const int k = steps(i)) {
            all += k;
            rows += b->seg_offsets[i + 1] - b->seg_offsets[i];
        }
    const int least = delta_steps(plan, rows, N);
    if (all < least || (size_t)rows * N * 4 > kDeltaBytes) return d;
    std::vector<int> tile((b->seg_offsets[S] + tile_m - 1) / tile_m, 0);
    for (int i = 0; i < S; ++i)
        if (const int k = steps(i)) {
            const int u = b->seg_offsets[i] / tile_m, v = (b->seg_offsets[i + 1] - 1) / tile_m;
            tile[u] += k;
            if (v != u) tile[v] += k;
        }
    for (int i = 0; i < S; ++i)
        if (steps(i)) {
            const int lo = b->seg_offsets[i], n = b->seg_offsets[i + 1] - lo;
            if (tile[lo / tile_m] < least && tile[(lo + n - 1) / tile_m] < least) continue;
            d.items.push_back(RowChunk{i, lo, n, d.rows});
            d.rows += n;
        }
    return d;
}

// The LoRA k-steps of the 256-row tile that has the most (a segment of rank r: 2 ceil16(r) / 32): those of long segments and of the short ones that
// the terms leave out; short ones, whichever way they go, as at least min(8, their steps).  few256: short ones alone, all of them.
struct LoraSteps {
    int most256 = 0, few256 = 0;
};
LoraSteps lora_steps(const symb_batch* b, const DeltaPlan& terms) {
    LoraSteps s;
    int tile = -1, sum = 0, few = 0, left = 0;       // the tile so far: steps of long and of short segments, and of the short ones that keep theirs
    size_t at = 0;                                   // the terms are in the segments' order
    for (int i = 0; i < b->num_segments; ++i) {
        const bool taken = at < terms.items.size() && terms.items[at].seg == i;
        at += taken;
        const int lo = b->seg_offsets[i], n = b->seg_offsets[i + 1] - lo;
        if (b->adapters[i].kind != SYMB_ADAPTER_LORA || !n) continue;
        const int k = rpad_of(b->adapters[i].rank) / 16, first = lo / 256, last = (lo + n - 1) / 256;
        for (int u : {first, last}) {                // (the tiles in between hold this segment alone)
            if (u != tile) { tile = u; sum = few = left = 0; }
            (n > kDeltaRows ? sum : few) += k;
            if (n <= kDeltaRows && !taken) left += k;
            s.most256 = std::max(s.most256, sum + std::max(left, std::min(few, 8)));
            s.few256 = std::max(s.few256, few);
            if (first == last) break;
        }
    }
    return s;
}

// The tile and the K split of a product.  Of the launches that gemm_variant gives to the 128x128 tile, those of more such tiles than CUs whose 256x128 tiles
// are at most one per CU, or fewer in two or three K parts, take that tile: it moves three quarters of the bytes per flop from L2 to LDS and waits out
// HBM latency with two stages in flight.  Time of the 128x128 tile over its, medians inside calls of one product, three sets of operands in turn, 260 of 129 to 4200 rows: more
// than 256 small tiles (some CUs run two) K = 3072 to 4100 1.05 to 1.2, to 6100 1.2 to 1.27, to 8200 1.19 to 1.4, above 1.1 to 1.3, also where up to two fifths of the 128-row halves are empty (600
// rows of 8192 -> 8192 and back 217 / 185 us) and from 129 tiles on (731 of 6144 -> 6144 and back 152 / 143); up to 256 small tiles, one per CU, 0.75 to 0.88 (in parts 0.62 to 0.85);
// K = 1000 to 3072 1.03 to 1.12, which calls with adapter passes lose again.  Whole calls of all flows whose tile this changed gained 9 % on average.  In two or three parts, 65 to 128 tiles, operands from HBM,
// 1.1 to 1.46 for K >= 3072 and 0.93 to 0.99 below; but inside calls, with their activations in cache and the partial tiles (up to 32 MiB) pushing weights out of it, 210 calls of all
// flows: two parts of K = 3072 to 6000 0.81 to 1.13, median 0.97 (457 rows of 4096 -> 6144 and back 106 / 131, 861 of 3312 -> 4096 40 / 45.6), from 6144 on 0.95 to 1.48, median 1.14; three parts 0.93 to 1.14
// up to 4700, 1.02 to 1.22 from there on; one row tile 0.95 to 1.05 below 4096, 0.95 to 1.21, median 1.09, from there on; fewer tiles 0.76 to 1.0 (and 1.15 in four parts of K > 5000).  Up to 128 rows half of every
// such tile would be empty.  The parts are as many as fit an XCD's 32 CUs: 81 to 85 tiles in three parts are 33 workgroups on most XCDs, a second
// round (84 tiles, us in two / three parts, 128x128 tile: 2993 rows of 4608 -> 856 42.2 / 59.4, 58.3; 2855 of 11192 -> 776 109.7 / 129.2, 130.3).  397 rows of 4096 -> 11008 with the adapters of
// eleven clients 85.5 / 78 us, 16384 rows of 6144 -> 256 80.6 / 59.3.  Inside calls, behind the adapter passes, the whole ones of K < 3072 only break even (6000 rows of
// 2032 -> 800 74.5 / 77.4, the call): from K = 3072 on.  In parts: at most an eighth of the 128-row halves empty.  Not with LoRA steps beyond a quarter of the K stages: a tile of twice the
// rows has up to twice as many, one after the other (batches whose terms do not come from memory, for want of room or by their number, count in full: 2000 one-token clients on
// 4096 x 4096 with room for nothing optional keep 128x128 tiles of 128 steps each).
// Where few columns stream many activation rows that do not lie on whole lines (K no multiple of 64), a launch has to fill the chip to keep as many
// loads on their way as the 128x128 tiles: 4500 to 20000 rows, M >= 3 N, 128x128 tile's time over its, whole, K < 4300 1.03 to 1.26, above 0.81 to 1.03 up to 216 tiles (8770 rows
// of 9176 -> 768 145 / 178 us, 4689 of 17872 -> 1216 255 / 300) and 1.02 to 1.28 from 220 on; in two parts 0.89 to 1.04 up to
// K = 7000, 0.95 to 1.05 up to 10000, 1.0 to 1.6 above; on whole lines 0.95 to 1.4.  Up to 160 tiles: M >= N, K = 12528 to 14872 0.88 to 0.94, to 11120 1.07 to 1.27; and on whole lines, M >= 18 N,
// 0.94 to 1.01 (8761 rows of 4864 -> 472).
// Small layers take the tiles of 32 rows (symb_gemm_mid_kernel) as long as these are one round of workgroups: time of the 128x128 tile over theirs, 13 300 products
// of 65 to 1500 rows, medians by K, K-contiguous weight: 1.2 (K = 256), 1.3 to 1.37 (512), 1.3 to 1.46 (768), 1.4 to 1.57 (1024), 1.55 to 1.74 (1536) up to 256
// workgroups, 0.9 to 1.0 with 257 to 512, 0.6 beyond; where the 128x128 tiles are split over K 1.23 to 1.34 up to K = 2048, 1.03 to 1.1 above;
// N-contiguous 1.07 to 1.25 up to 192 workgroups, 0.75 beyond 256, and 0.9 to 1.0 against split tiles.  (The workspace figure stays the split's.)  Not with
// a pre-adapter output or with steps enough to be computed beforehand.
// room: bytes behind the mandatory regions, for partial tiles (can_split) and, behind them, the terms.  Doubled parts that do not fit (397 rows of 11008 -> 4096 with an
// adapter in the 32 MiB static scratch) are halved again, any other plan runs unsplit.
GemmPlan gemm_plan(const symb_batch* b, int N, int K, bool nn, bool lora, bool with_base, bool can_split, size_t room) {
    GemmPlan p;
    const int M = b->seg_offsets[b->num_segments];
    const size_t split_room = can_split ? room : 0;
    auto with_terms = [&](GemmPlan& g) {
        if (lora) g.terms = delta_plan(b, g, N);
        if (!g.terms.items.empty() && align_up(g.split.bytes, 256) + (size_t)g.terms.rows * N * 4 > room) g.terms = DeltaPlan{};
    };
    p.variant = gemm_variant(M, N, K);
    p.split = gemm_split_plan(M, N, K);
    p.unsplit_for_base = with_base && p.variant == kTile128 && p.split.parts > 1;
    const long tall = (long)((M + 255) / 256) * ((N + 127) / 128);
    const long small = (long)((M + 127) / 128) * ((N + 127) / 128);
    if (p.variant == kTile128 && M > 128 && K >= 3072 && !p.split.doubled) {
        const int parts = (int)(32 / std::max((tall + 7) / 8, 1L));      // of an XCD's tiles, in its 32 CUs
        const size_t bytes = (size_t)tall * parts * 256 * 128 * 4;
        const bool streamed = M >= 3L * N && K % 64 != 0;
        const bool few_streamed = K % 64 != 0 && (tall <= 160 ? M >= N && K >= 11500 : M >= 3L * N && K >= 4500 && tall < 220);
        const bool whole = small > 256 && tall <= 256 && !few_streamed && !(tall <= 160 && M >= 12L * N);
        const bool split = 4 * small >= 7 * tall && tall > 64 && tall <= 128 && K >= (M <= 256 ? 4096 : parts == 3 ? 4700 : streamed ? 7168 : 6144) && bytes <= split_room;
        GemmPlan t;
        t.variant = kTileTall;
        if (split) t.split = SplitPlan{parts, 0, (int)tall, bytes, false};
        if (whole || split) {
            with_terms(t);
            if (!lora || 4 * lora_steps(b, t.terms).most256 <= K / 64) return t;
        }
    }
    if (p.split.bytes > split_room && p.split.doubled) {
        p.split.parts /= 2;
        p.split.bytes /= 2;
    }
    if (p.split.bytes > split_room) p.split = SplitPlan{};
    const long mid = (long)((M + MID_ROWS - 1) / MID_ROWS) * ((N + small_cols(nn) - 1) / small_cols(nn));
    if (p.variant == kTile128 && !with_base &&
        (p.split.parts == 1 ? K <= 1536 && mid <= (nn ? 192 : 256) : !nn && K <= 2048 && mid <= 192)) {
        const LoraSteps steps = lora ? lora_steps(b, DeltaPlan{}) : LoraSteps{};
        if (steps.most256 <= 16 && steps.few256 < 8) {
            p.variant = kTileMid;
            return p;
        }
    }
    with_terms(p);
    return p;
}

// One-pass dH + dB kernel: the number of workgroups along d_out, kDhDbBlocks blocks of 256 columns each (0: the layer is too narrow for it:
// with few column blocks the launch has too few workgroups, each walking its tokens alone, and the two
// separate passes are faster).
constexpr int kDhDbBlocks = 2;
int dhdb_groups(int d_out) { return d_out >= GRAD_WIDE ? ((d_out + 255) / 256 + kDhDbBlocks - 1) / kDhDbBlocks : 0; }

// LoRA gradients of long segments: a segment of more than GRAD_SPLIT_MIN tokens is walked in runs of
// GRAD_SPLIT tokens, each by workgroups of its own, which leave fp32 sums of the result's size in the
// workspace; a second kernel adds the runs up in order.  Number of runs of a segment of n tokens:
int grad_runs(int n) { return n > GRAD_SPLIT_MIN ? (n + GRAD_SPLIT - 1) / GRAD_SPLIT : 1; }
// Floats of workspace the runs of dB (of_b) or dA take for this batch.
size_t grad_split_floats(const symb_batch* b, bool of_b) {
    size_t n = 0;
    for (int i = 0; i < b->num_segments; ++i) {
        const symb_adapter& a = b->adapters[i];
        if (a.kind != SYMB_ADAPTER_LORA || !(of_b ? a.dB : a.dA)) continue;
        const int runs = grad_runs(b->seg_offsets[i + 1] - b->seg_offsets[i]);
        if (runs > 1) n += (size_t)runs * a.rank * (of_b ? b->d_out : b->d_in);
    }
    return n;
}

// Workspace layout (all regions 256-byte aligned, in this order; absent regions have size 0).
// Hs, dH and packed B^T sit at the same offsets for all three operations of one batch, so that a
// gradient call on the same workspace can take over what the forward call (Hs) and the
// input-gradient call (dH) left there (SYMB_GRAD_REUSE_HS / SYMB_GRAD_REUSE_DH).
struct WsLayout {
    size_t h_off = 0, h_bytes = 0;        // Hs  [T][2*max_rpad] bf16
    size_t dh_off = 0, dh_bytes = 0;      // dH  [T][2*max_rpad] bf16
    size_t pk_off = 0, pk_bytes = 0;      // packed B^T
    size_t sc_off = 0, sc_bytes = 0;      // IA3-scaled copy of dY [T][d_out] (input gradient) or of X [T][d_in] (forward, IA3_IN) bf16
    size_t pa_off = 0, pa_bytes = 0;      // packed A^T (input-major weight, input gradient only)
    size_t so_off = 0, so_bytes = 0;      // flat output [T][width] bf16 of a per-segment call whose outputs overlap its inputs
    size_t gr_off = 0, gr_bytes = 0;      // fp32 runs of the LoRA gradients of split segments (see grad_split)
    size_t dp_off = 0, dp_bytes = 0;      // fp32 partial sums of dH per group of column blocks (one-pass dH + dB, ranks up to 16)
    // optional regions (a workspace that ends before them makes the call take the tiled kernel, unsplit); those of the small-batch
    // kernels and those of the tiled ones share their place, a call uses one or the other:
    size_t sp_off = 0, sp_bytes = 0;      // calls of at most SMALL_MAX_ROWS rows: fp32 partial sums of the base product per K range
    size_t sh_off = 0, sh_bytes = 0;      // ... and of the LoRA shrink
    size_t tp_off = 0, tp_bytes = 0;      // tiled: fp32 partial tiles of a K-split GEMM (see gemm_split_plan)
    size_t de_off = 0, de_bytes = 0;      // ... fp32 LoRA terms of short segments of the batch (see DeltaPlan); after the partial tiles: a
                                          // workspace of a fixed size loses the terms before it loses the split
    bool small = false;                   // the call takes the small-batch kernels if their regions are there
    size_t mandatory = 0;                 // end of the regions a call cannot do without
    size_t total = 0;
};

// The grid of a call of at most SMALL_MAX_ROWS rows (small_kernels.hpp): column tiles x K ranges of the base product beside
// shrink pieces x K ranges, at most 16 ranges of either (the finish kernel reads them back).
struct SmallPlan {
    int tiles = 0, ranges = 0, items = 0, h_ranges = 0;
    bool direct = false;      // no LoRA term, one range: no partial sums, no finish kernel
    bool narrow = false;      // direct, in symb_small_narrow_kernel
    bool one_buffer = false;  // see small_base_nbuf
    bool wins = false;        // faster than the tiled kernels
    size_t base_bytes = 0, h_bytes = 0;
};
// Whether the small-batch kernels are faster than the tiled ones for T <= SMALL_MAX_ROWS rows: measured both ways over 22 layers of 256 to 36864
// columns, 1 to 64 rows, both weight layouts, without LoRA, with one or four clients, and a client per row.  With up to 16 rows, or more than a
// few LoRA clients, always (4096 x 4096, rank-16 clients of one row each, us per call, the weight read K- / N-contiguous: 14 / 28, 15 / 34, 20 / 54
// and 14 / 35, 15 / 38, 24 / 62 for 1, 16 and 64 rows).  Else the tiled kernels keep (us streamed / tiled):
//  * short inner dimensions, where there is little to stream: without LoRA, 32 rows of 256 -> 6144 N-contiguous 9.2 / 8.6; beyond 32 rows
//    256 -> 11008 11.4 / 8.7 and 9.8 / 8.7 (K-contiguous), 1024 -> 4096 N-contiguous 12.5 to 16 / 12.5, 2048 -> 4608 19.1 / 16.5 (4096 -> 1024 13.5 / 15.7);
//    with one LoRA client, 64 rows of 256 -> 11008 18.8 / 13.6 N-contiguous, 18.5 / 14 K-contiguous;
//  * wide outputs where the partial sums, written and read back, weigh more than a tenth of the weight (8 r T N bytes of 2 K N): 64 rows without LoRA of 4608 -> 36864 N-contiguous 107.5 / 98, of 4096 -> 16384 40 / 37.4, of 4096 -> 24576 K-contiguous 63.8 / 61 (but 6144 -> 24576 90 / 99, 8192 -> 28672
//    N-contiguous 103 / 111); with one LoRA client 4608 -> 36864 123 / 106;
//  * K-contiguous with one to four LoRA clients, N >= 24576: 64 rows of 4608 -> 36864 119 / 106, of 4096 -> 24576 74 / 69.
bool small_wins(bool base_nn, int K, int N, int T, int n_lora, int ranges) {
    if (T <= 16 || n_lora > 4) return true;
    const bool sums_weigh = 40LL * ranges * T > K;
    if (n_lora == 0) {
        if (K <= 512 && (base_nn || T > 32)) return false;
        if (base_nn && K <= 2048 && T > 32) return false;
        return !(sums_weigh && K >= 4096 && N >= (base_nn ? 16384 : 24576));
    }
    if (T <= 32) return true;
    if (N >= 8192 && K < 1024) return base_nn && T <= 40;
    return N < 24576 || (base_nn && !sums_weigh);
}
SmallPlan small_plan(const symb_batch* b, const BatchInfo& bi, int op, bool lora, bool staged) {
    SmallPlan s;
    // the contraction runs over d_in in the forward, over d_out in the input gradient; the weight is read N-contiguous by the
    // forward of an input-major weight and by the input gradient of an nn.Linear one
    const int K = op == SYMB_OP_FWD ? b->d_in : b->d_out, N = op == SYMB_OP_FWD ? b->d_out : b->d_in;
    const bool shrink_nn = op == SYMB_OP_BWD_INPUT, base_nn = (op == SYMB_OP_FWD) == (b->weight_layout == SYMB_WEIGHT_CONV1D);
    if (lora)
        for (int i = 0; i < bi.S; ++i)
            if (b->adapters[i].kind == SYMB_ADAPTER_LORA && b->seg_offsets[i + 1] > b->seg_offsets[i])
                s.items += shrink_nn ? 1 : rpad_of(b->adapters[i].rank) / 16;
    s.tiles = (N + small_cols(base_nn) - 1) / small_cols(base_nn);
    // Ranges per tile: the launch runs in rounds of 256 workgroups (one per CU), each of a 1 / ranges share of a tile's strip of the
    // weight plus what a round costs besides (first loads, the wavefronts' sums, partial sums): about a quarter of a strip.  Measured
    // over 1 to 16 ranges: a count just past a round loses (input gradient of 4608 -> 36864, 36 tiles, one row: 65.5 us at 6
    // ranges, 82.2 at 8, 66.5 at 12), and a second workgroup per CU gains nothing (4096 -> 11008, 172 tiles: 19.4 us at 1, 22.8 at 2).
    double best = 1e30;
    for (int r = 1; r <= std::max(1, std::min(K / 256, 16)); ++r) {
        double cost = (double)((s.tiles * r + 255) / 256) * (1.0 / r + 0.25);
        // More N-contiguous tiles than CUs: the CUs with a tile more than the others set a third of the time, against the traffic of the partial
        // sums (8 r T N bytes for 2 K N) and the finish kernel (about 4 us, the time of 19 MB).  4608 -> 36864, 288 tiles: one row 71.5 us at 2 ranges, 65.3 at 6; 16 rows 79.0 / 76.3; 32 rows
        // 85.5, 83.6 at 3; 2048 -> 36864, one row 39.1 at 1, 34.9 at 4; 4608 -> 49152, 384 tiles, stays at 2, 2048 -> 65536, 512 tiles, at 1.
        if (base_nn && s.tiles > 256)
            cost = 0.65 + 0.35 * ((s.tiles * r + 255) / 256) * 256.0 / ((double)s.tiles * r) + 4.0 * r * bi.T / K + (r > 1 ? 9.4e6 / ((double)K * N) : 0.0);
        if (cost < best) { best = cost; s.ranges = r; }
    }
    // One buffer: long strips, at most 16 rows, N-contiguous; less than a full round of workgroups is faster there (64 tiles of 28672 -> 8192, one row: 81.9 us
    // at 3 ranges, 86.4 at 4; 36 of 36864 -> 4608 62.7 at 6, with two buffers 64.7 at 7).
    if (base_nn && bi.T <= 16) {
        const int r = s.tiles <= 112 ? std::min(224 / s.tiles, 16) : s.ranges, n = s.tiles * r;
        s.one_buffer = K / r >= 2048 && n >= 160 && n <= 256;
        if (s.one_buffer) s.ranges = r;
    }
    // Without a LoRA term, in one kernel where what a second one costs outweighs the ranges (not where outputs overlap inputs: every row must be
    // read before any is written).  N-contiguous, us in one kernel / in 8 ranges: 1024 -> 4096 one row 9.8 / 10.0, 17 rows 11.8 / 10.5; 2048 x 2048 one row
    // 11.9 / 10.3, 64 rows 22.1 / 13.9.  K-contiguous in tiles of 32 columns: see symb_small_narrow_kernel.
    const bool can_direct = !s.items && !staged;
    s.narrow = can_direct && !base_nn && N <= 8192 && (long long)K * N <= 10 << 20 && K <= (bi.T <= 32 ? 4608 : 2048);
    if (s.narrow) s.tiles = (N + SMALL_NARROW_COLS - 1) / SMALL_NARROW_COLS;
    if (s.narrow || (can_direct && K <= (!base_nn ? 2048 : bi.T <= 16 ? 1024 : 768))) s.ranges = 1;
    s.direct = can_direct && s.ranges == 1;
    s.wins = small_wins(base_nn, K, N, bi.T, s.items ? bi.n_lora : 0, s.ranges);
    s.base_bytes = s.direct ? 0 : (size_t)s.ranges * bi.T * N * 4;
    if (!s.items) return s;
    s.h_ranges = std::max(1, std::min({256 / s.items, K / 512, 16}));      // at most a round of its own, two slices per wavefront
    s.h_bytes = (size_t)s.h_ranges * bi.T * bi.max_rpad * 4;
    return s;
}

std::vector<TileDelta> delta_tiles(const DeltaPlan& d, int num_m_tiles, int tile_m) {
    std::vector<TileDelta> v(d.items.empty() ? 0 : num_m_tiles, TileDelta{});
    for (const RowChunk& it : d.items)
        for (int t = it.row0; t < it.row0 + it.nrows; ++t) v[t / tile_m].mask[t % tile_m / 32] |= 1u << (t % 32);
    int at = 0;
    for (TileDelta& t : v) {
        t.first = at;
        for (uint32_t m : t.mask) at += __builtin_popcount(m);
    }
    return v;
}

WsLayout ws_layout(const symb_batch* b, const BatchInfo& bi, int op, bool full_bwd, bool any_lora_grad, bool staged_out = false) {
    WsLayout w;
    size_t cur = 0;
    auto take = [&](size_t& off, size_t& bytes, size_t n) {
        off = cur;
        bytes = n;
        cur += align_up(n, 256);
    };
    const size_t hb = (size_t)bi.T * (2 * bi.max_rpad) * 2;   // value + residual halves
    const bool conv1d = b->weight_layout == SYMB_WEIGHT_CONV1D;
    if (op == SYMB_OP_FWD) {
        if (bi.n_lora) take(w.h_off, w.h_bytes, hb);
        if (bi.n_lora && conv1d) {            // the N-contiguous GEMM wants B_i^T: same packing as the input gradient's
            take(w.dh_off, w.dh_bytes, hb);   // (gap: keeps packed B^T where the other operations have it)
            take(w.pk_off, w.pk_bytes, bi.packed_elems * 2);
        }
        if (bi.n_ia3in) take(w.sc_off, w.sc_bytes, (size_t)bi.T * b->d_in * 2);   // X with IA3_IN rows scaled
    } else if (op == SYMB_OP_BWD_INPUT) {
        if (full_bwd && bi.n_lora) {
            take(w.h_off, w.h_bytes, hb);     // not touched here: keeps the forward call's Hs intact
            take(w.dh_off, w.dh_bytes, hb);
            take(w.pk_off, w.pk_bytes, bi.packed_elems * 2);
        }
        if (full_bwd && bi.n_ia3) take(w.sc_off, w.sc_bytes, (size_t)bi.T * b->d_out * 2);
        if (full_bwd && bi.n_lora && conv1d) take(w.pa_off, w.pa_bytes, bi.packed_at_elems * 2);
    } else {
        if (any_lora_grad) {
            take(w.h_off, w.h_bytes, hb);
            take(w.dh_off, w.dh_bytes, hb);
            take(w.pk_off, w.pk_bytes, bi.packed_elems * 2);
            const size_t gr = std::max(grad_split_floats(b, true), grad_split_floats(b, false)) * 4;   // dB's runs, then dA's, in the same place
            if (gr) take(w.gr_off, w.gr_bytes, gr);
            if (bi.max_rpad == 16 && dhdb_groups(b->d_out)) take(w.dp_off, w.dp_bytes, (size_t)dhdb_groups(b->d_out) * bi.T * 16 * 4);
        }
    }
    if (staged_out && op != SYMB_OP_ADAPTER_GRAD)
        take(w.so_off, w.so_bytes, (size_t)bi.T * (op == SYMB_OP_FWD ? b->d_out : b->d_in) * 2);
    w.mandatory = cur;
    if (op != SYMB_OP_ADAPTER_GRAD && bi.T > 0 && bi.T <= SMALL_MAX_ROWS) {
        const SmallPlan sm = small_plan(b, bi, op, op == SYMB_OP_FWD || full_bwd, staged_out);
        if (sm.wins) {
            w.small = true;
            take(w.sp_off, w.sp_bytes, sm.base_bytes);
            take(w.sh_off, w.sh_bytes, sm.h_bytes);
        }
    }
    const size_t small_end = cur;
    cur = w.mandatory;
    if (op != SYMB_OP_ADAPTER_GRAD) {
        const int N = op == SYMB_OP_FWD ? b->d_out : b->d_in, K = op == SYMB_OP_FWD ? b->d_in : b->d_out;
        const bool lora = bi.n_lora && (op == SYMB_OP_FWD || full_bwd);
        const GemmPlan plan = gemm_plan(b, N, K, (op == SYMB_OP_FWD) == conv1d, lora, false, true, SIZE_MAX);
        take(w.tp_off, w.tp_bytes, plan.split.bytes);
        take(w.de_off, w.de_bytes, (size_t)plan.terms.rows * N * 4);
    }
    w.total = std::max(small_end, cur);
    return w;
}

// Where a call's terms of short segments start: right behind its own partial tiles.  A call that does not split (pre-adapter output wanted) may select
// more rows than the figure counts for a split call, and has the place of the figure's partial tiles for them, at least twice the whole output in fp32.
size_t terms_offset(const WsLayout& w, const GemmPlan& plan) { return w.tp_off + align_up(plan.split.bytes, 256); }

// ---- descriptor blob -------------------------------------------------------------------------
struct Blob {
    std::vector<unsigned char> bytes;
    template <class T>
    size_t add(const T* p, size_t n) {
        const size_t off = align_up(bytes.size(), 16);
        bytes.resize(off + std::max<size_t>(n, 1) * sizeof(T));
        if (n) memcpy(bytes.data() + off, p, n * sizeof(T));
        return off;
    }
};

// The last descriptors of a GEMM call: the segments as the GEMM reads them and, with a DeltaPlan, its items and the tiles' masks.  The
// masks are 36 bytes for every row tile: a plan whose descriptors do not fit beside the others is dropped (its segments keep their
// steps), so that a batch is refused or accepted as it would be without one.
struct DeltaBlob {
    size_t seg = 0, items = 0, tiles = 0;
};
DeltaBlob add_gemm_desc(Blob& blob, std::vector<SegDesc>& sd_gemm, DeltaPlan& delta, int num_m_tiles, int tile_m) {
    const size_t extra = sd_gemm.size() * sizeof(SegDesc) + delta.items.size() * sizeof(RowChunk) + (size_t)num_m_tiles * sizeof(TileDelta) + 3 * 16;
    if (blob.bytes.size() + extra > kSlotBytes) delta = DeltaPlan{};
    for (const RowChunk& it : delta.items) sd_gemm[it.seg].kind = KIND_DELTA;
    DeltaBlob d;
    d.seg = blob.add(sd_gemm.data(), sd_gemm.size());
    if (delta.items.empty()) return d;
    const std::vector<TileDelta> tiles = delta_tiles(delta, num_m_tiles, tile_m);
    d.items = blob.add(delta.items.data(), delta.items.size());
    d.tiles = blob.add(tiles.data(), tiles.size());
    return d;
}

symb_status upload(symb_handle h, const Blob& blob, hipStream_t st, unsigned char** dev_base) {
    if (blob.bytes.size() > kSlotBytes)
        return fail(h, SYMB_ERR_UNSUPPORTED, "batch descriptors need %zu bytes, capacity is %zu", blob.bytes.size(), kSlotBytes);
    // The kernels only read a slot's device copy (the K-split arrival counters are back at zero when
    // a launch ends), so a batch that comes again with the same offsets, adapters and buffers -- the
    // next decode step of the same clients, the same projection in the next training step -- finds
    // its descriptors in place.  The pinned copy of a slot is what its device copy holds.
    const size_t n = blob.bytes.size();
    uint64_t hash = 0x9E3779B97F4A7C15ull ^ n;
    {
        size_t i = 0;
        for (; i + 8 <= n; i += 8) {
            uint64_t w;
            memcpy(&w, blob.bytes.data() + i, 8);
            hash = (hash ^ w) * 0x100000001B3ull;
            hash ^= hash >> 29;
        }
        for (; i < n; ++i) hash = (hash ^ blob.bytes[i]) * 0x100000001B3ull;
    }
    h->ring.begin(h->rt, st);
    const int in_place = h->opt_desc_reuse ? h->ring.find(n, hash, [&](int j) { return memcmp(h->host_ring + (size_t)j * kSlotBytes, blob.bytes.data(), n) == 0; }) : -1;
    if (in_place >= 0) {
        h->call_slot = in_place;
        ++h->desc_in_place;
        *dev_base = h->dev_ring + (size_t)in_place * kSlotBytes;
        return SYMB_OK;
    }
    SYMB_HIP(h, h->ring.take(h->rt));
    const int slot = h->call_slot = h->ring.cur;
    unsigned char* hp = h->host_ring + (size_t)slot * kSlotBytes;
    unsigned char* dp = h->dev_ring + (size_t)slot * kSlotBytes;
    memcpy(hp, blob.bytes.data(), n);
    SYMB_HIP(h, hipMemcpyAsync(dp, hp, n, hipMemcpyHostToDevice, st));
    ++h->desc_sent;
    SYMB_HIP(h, h->ring.sent(h->rt, n, hash));
    *dev_base = dp;
    return SYMB_OK;
}

// A call that fails after its descriptors went to a slot may leave that slot's device copy in a state
// no later call should take over (a GEMM that never ran has not put its K-split counters back to zero, a
// launch may be half enqueued): unless the call completes, its slot is never matched again.
struct CallGuard {
    symb_handle h;
    bool completed = false;
    explicit CallGuard(symb_handle h_) : h(h_) { h->call_slot = -1; }
    ~CallGuard() {
        if (!completed && h->call_slot >= 0) h->ring.slot[h->call_slot].size = SIZE_MAX;
    }
};

symb_status seal_slot(symb_handle h) {
    SYMB_HIP(h, h->ring.seal(h->rt));
    return SYMB_OK;
}

std::vector<SegDesc> make_segdesc(const symb_batch* b) {
    std::vector<SegDesc> v(b->num_segments);
    for (int i = 0; i < b->num_segments; ++i) {
        const symb_adapter& a = b->adapters[i];
        SegDesc d{};
        d.kind = a.kind;
        d.rank = a.kind == SYMB_ADAPTER_LORA ? a.rank : 0;
        d.rpad = rpad_of(d.rank);
        d.scale = a.kind == SYMB_ADAPTER_LORA ? a.scale : 0.f;
        d.A = (const bf16*)a.A;
        d.B = (const bf16*)a.B;
        d.dA = (float*)a.dA;
        d.dB = (float*)a.dB;
        v[i] = d;
    }
    return v;
}

// ---- GEMM launch -----------------------------------------------------------------------------
template <class KFN>
symb_status launch_gemm_fn(symb_handle h, GemmParams gp, hipStream_t st, KFN kfn, int BM, int BN, int threads, int smem, int variant) {
    // once per context (= per device): the attribute belongs to the device the kernel is loaded on
    const void* kptr = reinterpret_cast<const void*>(kfn);
    if (std::find(h->lds_attr_set.begin(), h->lds_attr_set.end(), kptr) == h->lds_attr_set.end()) {
        SYMB_HIP(h, hipFuncSetAttribute(kptr, hipFuncAttributeMaxDynamicSharedMemorySize, smem));
        h->lds_attr_set.push_back(kptr);
    }
    gp.num_m_tiles = (gp.M + BM - 1) / BM;
    gp.num_n_tiles = (gp.N + BN - 1) / BN;
    if (gp.group_m <= 0) gp.group_m = 8;
    const int total = gp.num_m_tiles * gp.num_n_tiles;
    const int per_xcd = (total + 7) / 8;
    int grid = per_xcd * 8;
    if (gp.k_parts > 1) grid = 8 * (gp.k_whole + (per_xcd - gp.k_whole) * gp.k_parts);
    const bool timed = h->timing && (int)h->timed.size() < kMaxTimed;
    const size_t slot = h->timed.size();
    if (timed) SYMB_HIP(h, hipEventRecord(h->tev[2 * slot], st));
    hipLaunchKernelGGL(kfn, dim3(grid), dim3(threads), smem, st, gp);
    SYMB_HIP(h, hipGetLastError());
    if (timed) {
        SYMB_HIP(h, hipEventRecord(h->tev[2 * slot + 1], st));
        h->timed.push_back({variant, gp.timing_flops});
    }
    return SYMB_OK;
}

template <int MBLK, int NBLK, bool NN, bool PLAIN>
symb_status launch_gemm16_t(symb_handle h, const GemmParams& gp, hipStream_t st) {
    using TT = Gemm16Tile<MBLK, NBLK>;
    // instantiation number of the measurement hook: bit 0 = N-contiguous weight, bit 1 = tile of 128 columns, bit 2 = full epilogue, bit 3 = 256x128 tile
    constexpr int variant = (NN ? 1 : 0) | (NBLK == 4 ? 2 : 0) | (PLAIN ? 0 : 4) | (TT::TALL ? 8 : 0);
    return launch_gemm_fn(h, gp, st, symb_gemm16_kernel<NBLK, NN, PLAIN, MBLK>, TT::BM, TT::BN, TT::NT, TT::SMEM, variant);
}

// Algorithmic work of one GEMM launch: 2 M N K plus the LoRA term of the segments that have their steps in it.
double gemm_flops(const symb_batch* b, const std::vector<SegDesc>& sd_gemm, int N, int K, bool lora) {
    const int S = b->num_segments;
    double f = 2.0 * b->seg_offsets[S] * (double)N * K;
    if (lora)
        for (int i = 0; i < S; ++i)
            if (sd_gemm[i].kind == KIND_LORA)
                f += 2.0 * (b->seg_offsets[i + 1] - b->seg_offsets[i]) * (double)b->adapters[i].rank * N;
    return f;
}

template <bool NN>
symb_status launch_gemm(symb_handle h, const GemmParams& gp, hipStream_t st) {
    const bool plain = !gp.bias && !gp.epi_ia3 && !gp.Cbase && !gp.neff && !gp.delta;
    if (gp.variant == kTileMid) {
        GemmParams g = gp;
        g.num_m_tiles = (gp.M + MID_ROWS - 1) / MID_ROWS;
        const bool timed = h->timing && (int)h->timed.size() < kMaxTimed;
        const size_t slot = h->timed.size();
        if (timed) SYMB_HIP(h, hipEventRecord(h->tev[2 * slot], st));
        hipLaunchKernelGGL(symb_gemm_mid_kernel<NN>, dim3((unsigned)(g.num_m_tiles * ((gp.N + small_cols(NN) - 1) / small_cols(NN)))), dim3(256), 0, st, g);
        SYMB_HIP(h, hipGetLastError());
        if (timed) {
            SYMB_HIP(h, hipEventRecord(h->tev[2 * slot + 1], st));
            h->timed.push_back({(NN ? 1 : 0) | 2 | (plain ? 0 : 4) | 16, gp.timing_flops});
        }
        return SYMB_OK;
    }
    if (gp.variant == kTile256) return plain ? launch_gemm16_t<8, 8, NN, true>(h, gp, st) : launch_gemm16_t<8, 8, NN, false>(h, gp, st);
    if (gp.variant == kTileTall) return plain ? launch_gemm16_t<8, 4, NN, true>(h, gp, st) : launch_gemm16_t<8, 4, NN, false>(h, gp, st);
    return plain ? launch_gemm16_t<4, 4, NN, true>(h, gp, st) : launch_gemm16_t<4, 4, NN, false>(h, gp, st);
}

// Row chunks of a launch of the skinny kernel over `segs`, and the build that takes them (SkinnyBuild): chunks of 16, 32 or 48 rows where that is at most one
// workgroup per compute unit, for the eight-wavefront builds; else 32 rows.
struct SkinnyChunks {
    int build = 0;
    std::vector<RowChunk> items;
};
SkinnyChunks plan_skinny(symb_handle h, const symb_batch* b, const std::vector<int32_t>& segs, int max_rpad) {
    SkinnyChunks c;
    const int rb = max_rpad <= 16 ? 1 : max_rpad <= 32 ? 2 : max_rpad <= 64 ? 4 : 8;
    for (int blks = 1; h->opt_skinny_deep && b->num_segments <= 4096 && blks <= 3 && !c.build && skinny_has(rb, blks); ++blks) {
        long n = 0;
        for (int i : segs) n += (b->seg_offsets[i + 1] - b->seg_offsets[i] + 16 * blks - 1) / (16 * blks);
        if (n <= 256) c.build = blks;
    }
    const int rows = c.build ? 16 * c.build : kSkinnyRows;
    for (int i : segs)
        for (int r = b->seg_offsets[i]; r < b->seg_offsets[i + 1]; r += rows)
            c.items.push_back(RowChunk{i, r, std::min(rows, b->seg_offsets[i + 1] - r), 0});
    return c;
}
std::vector<int32_t> lora_segments(const symb_batch* b) {
    std::vector<int32_t> v;
    for (int i = 0; i < b->num_segments; ++i)
        if (b->adapters[i].kind == SYMB_ADAPTER_LORA) v.push_back(i);
    return v;
}
template <int RB, int BUILD, bool BT>
void launch_skinny_build(const SkinnyParams& sp, int nchunks, hipStream_t st) {
    if constexpr (skinny_has(RB, BUILD))
        hipLaunchKernelGGL((symb_skinny_kernel<RB, BUILD, BT>), dim3(nchunks), dim3(skinny_threads(BUILD)), 0, st, sp);
}
template <int RB, bool BT>
void launch_skinny_rb(const SkinnyParams& sp, const SkinnyChunks& c, hipStream_t st) {
    const int n = (int)c.items.size();
    if (c.build == 1) launch_skinny_build<RB, 1, BT>(sp, n, st);
    else if (c.build == 2) launch_skinny_build<RB, 2, BT>(sp, n, st);
    else if (c.build == 3) launch_skinny_build<RB, 3, BT>(sp, n, st);
    else launch_skinny_build<RB, 0, BT>(sp, n, st);
}
template <bool BT>
symb_status launch_skinny(symb_handle h, const SkinnyParams& sp, const SkinnyChunks& c, int max_rpad, hipStream_t st) {
    if (c.items.empty()) return SYMB_OK;
    if (max_rpad <= 16) launch_skinny_rb<1, BT>(sp, c, st);
    else if (max_rpad <= 32) launch_skinny_rb<2, BT>(sp, c, st);
    else if (max_rpad <= 64) launch_skinny_rb<4, BT>(sp, c, st);
    else launch_skinny_rb<8, BT>(sp, c, st);
    SYMB_HIP(h, hipGetLastError());
    return SYMB_OK;
}
// Whether the shrink of the backward reads every B_i [d_out][r] of these segments as it lies: 64 k of it must be whole 16-byte
// chunks at 8-byte aligned rows.  Otherwise one launch packs all of them first (4 us on a 4096-wide layer, 29 on a 36864-wide one).
bool reads_bt(const symb_batch* b) {
    for (int i = 0; i < b->num_segments; ++i) {
        const symb_adapter& a = b->adapters[i];
        if (a.kind == SYMB_ADAPTER_LORA && b->seg_offsets[i + 1] > b->seg_offsets[i] && ((a.rank & 3) || ((uintptr_t)a.B & 15))) return false;
    }
    return true;
}
// dH = s dY B of the rows in sp.chunks (sp: everything but the adapter side).
symb_status launch_skinny_dh(symb_handle h, const symb_batch* b, SkinnyParams sp, bf16* packed, const int64_t* packed_off, const SkinnyChunks& c, int max_rpad, hipStream_t st) {
    if (reads_bt(b)) return launch_skinny<true>(h, sp, c, max_rpad, st);
    PackParams pp{sp.seg, packed, packed_off, b->d_out};
    hipLaunchKernelGGL(symb_pack_bt_kernel, dim3((b->d_out + 255) / 256, b->num_segments), dim3(256), 0, st, pp);
    SYMB_HIP(h, hipGetLastError());
    sp.packed = packed;
    sp.packed_off = packed_off;
    sp.use_packed = 1;
    return launch_skinny<false>(h, sp, c, max_rpad, st);
}

template <int RB, bool CM>
void launch_grad_rb(const GradParams& gp, int nitems, hipStream_t st) {
    hipLaunchKernelGGL((symb_lora_grad_kernel<RB, CM>), dim3((gp.ncols + GRAD_CT<RB> - 1) / GRAD_CT<RB>, nitems), dim3(256), 0, st, gp);
}
template <int RB, bool CM>
void launch_grad_wave(const GradParams& gp, int nitems, hipStream_t st) {
    hipLaunchKernelGGL((symb_lora_grad_wave_kernel<RB, CM>), dim3((gp.ncols + GRAD_WAVE_CT - 1) / GRAD_WAVE_CT, nitems), dim3(256), 0, st, gp);
}
// Whether a launch takes the kernel that deals tokens out over the wavefronts.  `w` is about the launch's workgroups at its widest rank: with more than one
// per CU (two, for ranks to 16) the other kernel, which fits many of them on one, is faster unless the walks are long; and a workgroup of the
// widest kernel (128 KiB of LDS) needs a long walk to pay for its sums.  Measured on both gradients of 2 to 64 segments of 16 to 1024 tokens, 768, 4096 and 11008
// columns, time against the other kernel's: rank 8, 512 workgroups 1.05 (32 tokens) 0.94 (64 to 512), 1376 1.35 (16) 1.05 (192) 1.00 (512); rank 32, 256
// workgroups 0.82 to 1.04, 384 1.5 to 1.2, 688 1.36 (16) 1.13 (192) 0.93 (1024); rank 64, 64 workgroups 1.34 (16) 1.01 (256) 0.82 (1024), 512 1.7 to 1.2.
bool grad_wave(const symb_batch* b, const std::vector<GradItem>& items, int ncols) {
    int most = 0, least = INT32_MAX;
    long long tokens = 0, ranks = 0;
    for (const GradItem& it : items) {
        const int r = rpad_of(b->adapters[it.seg].rank);
        most = std::max(most, r);
        least = std::min(least, r);
        tokens += it.t_hi - it.t_lo;
        ranks += r;
    }
    if (items.empty() || least > GRAD_WAVE_RANK) return false;
    const double w = (double)((ncols + GRAD_WAVE_CT - 1) / GRAD_WAVE_CT) * (double)ranks / most, mean = (double)tokens / (double)items.size();
    if (most <= 16) return w <= 256 || mean >= 256 || (w <= 512 && mean >= 64);
    return w <= 256 && (most <= 32 || mean >= 384);
}
// wave_rpad: the items take the kernel that deals tokens out over the wavefronts, this is their widest rank (plan_items; 0: the other one).
template <bool CM>
symb_status launch_grad(symb_handle h, const GradParams& gp, int wave_rpad, int nitems, int max_rpad, hipStream_t st) {
    if (nitems == 0) return SYMB_OK;
    if (wave_rpad > 0) {
        if (wave_rpad <= 16) launch_grad_wave<1, CM>(gp, nitems, st);
        else if (wave_rpad <= 32) launch_grad_wave<2, CM>(gp, nitems, st);
        else if (wave_rpad <= 64) launch_grad_wave<4, CM>(gp, nitems, st);
        else launch_grad_wave<8, CM>(gp, nitems, st);
    } else {
        if (max_rpad <= 16) launch_grad_rb<1, CM>(gp, nitems, st);
        else if (max_rpad <= 32) launch_grad_rb<2, CM>(gp, nitems, st);
        else if (max_rpad <= 64) launch_grad_rb<4, CM>(gp, nitems, st);
        else launch_grad_rb<8, CM>(gp, nitems, st);
    }
    SYMB_HIP(h, hipGetLastError());
    return SYMB_OK;
}
// Stable sort of a list that mostly is sorted: calls of many small segments are bound by the host.
template <class LESS>
void sort_once(std::vector<int32_t>& v, LESS&& less) {
    if (!std::is_sorted(v.begin(), v.end(), less)) std::stable_sort(v.begin(), v.end(), less);
}

// IA3 gradients of the segments `want` (the list p.seg_list holds on the device).  The long shape of the kernel where the longest walk sets the
// time: from 1024 tokens on, or from 192 where the short shape would have at most 128 workgroups (2 segments of 256 tokens, 4096 wide: 0.84
// of the short shape's time, 8 segments 1.15; 768 wide, 16 segments 0.93).  Segments of both kinds share the long shape's launch unless the
// short ones would be more than 2048 workgroups of it.
symb_status launch_ia3_grad(symb_handle h, const symb_batch* b, Ia3GradParams p, const std::vector<int32_t>& want, hipStream_t st) {
    const auto tokens = [&](int i) { return b->seg_offsets[i + 1] - b->seg_offsets[i]; };
    const auto blocks = [&](bool lng) { return (unsigned)((p.d_out + ia3_grad_cols(lng) - 1) / ia3_grad_cols(lng)); };
    const int least = blocks(false) * want.size() <= 128 ? 192 : 1024;
    size_t n_long = 0;                                   // (the list is sorted by it)
    while (n_long < want.size() && tokens(want[n_long]) >= least) ++n_long;
    if (n_long && (want.size() - n_long) * blocks(true) <= 2048) n_long = want.size();
    if (n_long) {
        hipLaunchKernelGGL(symb_ia3_grad_kernel<true>, dim3(blocks(true), (unsigned)n_long), dim3(ia3_grad_threads(true)), 0, st, p);
        SYMB_HIP(h, hipGetLastError());
    }
    if (n_long < want.size()) {
        p.seg_list += n_long;
        hipLaunchKernelGGL(symb_ia3_grad_kernel<false>, dim3(blocks(false), (unsigned)(want.size() - n_long)), dim3(ia3_grad_threads(false)), 0, st, p);
        SYMB_HIP(h, hipGetLastError());
    }
    return SYMB_OK;
}

// Adds up the runs of the split segments (none: nothing to do).  At most 128 * 36864 floats per segment
// at 1024 per workgroup and pass.
symb_status launch_grad_reduce(symb_handle h, const GradReduceParams& rp, int nsplit, hipStream_t st) {
    if (nsplit == 0) return SYMB_OK;
    hipLaunchKernelGGL(symb_grad_reduce_kernel, dim3(1024, nsplit), dim3(256), 0, st, rp);
    SYMB_HIP(h, hipGetLastError());
    return SYMB_OK;
}

// An elementwise pass over the rows of a chunk list (adapter_kernels.hpp, ROWPASS_*).  A grid has at most 65535 chunks in
// y; longer lists take several launches, each from its own place in the list.
template <class P>
symb_status launch_row_pass(symb_handle h, void (*kfn)(P), P p, int width, size_t nchunks, hipStream_t st) {
    for (size_t at = 0; at < nchunks; at += 65535) {
        const unsigned n = (unsigned)std::min<size_t>(65535, nchunks - at);
        hipLaunchKernelGGL(kfn, dim3((width / 8 + ROWPASS_COLS - 1) / ROWPASS_COLS, n, SKINNY_ROWS / ROWPASS_ROWS), dim3(ROWPASS_COLS), 0, st, p);
        SYMB_HIP(h, hipGetLastError());
        p.chunks += n;
    }
    return SYMB_OK;
}

// The terms of a DeltaPlan, from the rows of H in the workspace.
symb_status launch_delta(symb_handle h, bool backward, const SegDesc* seg, const RowChunk* items, int nitems, int N, const bf16* h_rows, int h_pitch, float* out, hipStream_t st) {
    const LoraDeltaParams dp{h_rows, h_pitch, N, seg, items, out};
    hipLaunchKernelGGL(backward ? symb_lora_delta_kernel<true> : symb_lora_delta_kernel<false>, dim3((N + 255) / 256, nitems), dim3(256), 0, st, dp);
    SYMB_HIP(h, hipGetLastError());
    return SYMB_OK;
}

template <bool BASE_NN, bool SHRINK_NN>
void launch_small_stream(const SmallStreamParams& p, bool one_buffer, hipStream_t st) {
    const dim3 grid((unsigned)(p.num_items * p.h_ranges + p.tiles * p.ranges));
    if (one_buffer) {
        if constexpr (BASE_NN) hipLaunchKernelGGL((symb_small_stream_kernel<1, true, SHRINK_NN, true>), grid, dim3(256), 0, st, p);
    } else if (p.T <= 16) hipLaunchKernelGGL((symb_small_stream_kernel<1, BASE_NN, SHRINK_NN, false>), grid, dim3(256), 0, st, p);
    else if (p.T <= 32) hipLaunchKernelGGL((symb_small_stream_kernel<2, BASE_NN, SHRINK_NN, false>), grid, dim3(256), 0, st, p);
    else hipLaunchKernelGGL((symb_small_stream_kernel<4, BASE_NN, SHRINK_NN, false>), grid, dim3(256), 0, st, p);
}

// Whether a call takes the small-batch kernels: at most SMALL_MAX_ROWS rows, a shape on which they are the faster ones (small_wins), and a
// workspace with their regions.
bool small_path(symb_handle h, const BatchInfo& bi, const WsLayout& wl, const void* ws, size_t ws_bytes) {
    const size_t need = wl.sh_off + wl.sh_bytes;
    return h->opt_small_rows && bi.T <= SMALL_MAX_ROWS && wl.small && ws_bytes >= need && (ws || !need);
}

// One call of the small-batch kernels, forward or input gradient: what differs between the two comes in through the
// arguments.  x_flat: the rows to multiply (or null with x_seg); scale: those rows are first copied, rows of that kind scaled by their vector
// (0: no copy); h_rows: where H is left as value + residual; take_h: H is there already.
struct SmallCall {
    int op;
    const void *x_flat, *W, *bias, *out, *out_base;
    const void* const* x_seg;
    void* const* out_seg;
    const NoiseDesc* neff;    // HOST, S entries, or null
    int scale;
    bf16 *copy, *h_rows;
    bool lora, take_h, staged;
};
symb_status run_small(symb_handle h, const symb_batch* b, const BatchInfo& bi, const WsLayout& wl, unsigned char* wsb, const SmallCall& c, hipStream_t s) {
    symb_status st;
    const bool fwd = c.op == SYMB_OP_FWD;
    const int K = fwd ? b->d_in : b->d_out, N = fwd ? b->d_out : b->d_in;
    const SmallPlan plan = small_plan(b, bi, c.op, c.lora, c.staged);
    SmallRows rows{};
    for (int i = 0; i < bi.S; ++i)
        for (int t = b->seg_offsets[i]; t < b->seg_offsets[i + 1]; ++t) rows.at[t] = (uint32_t)i << 8 | (uint32_t)(t - b->seg_offsets[i]);
    const bool shrink = plan.items > 0 && !c.take_h;
    std::vector<SmallItem> items;
    if (shrink)
        for (int i = 0; i < bi.S; ++i) {
            const int n = b->seg_offsets[i + 1] - b->seg_offsets[i];
            if (b->adapters[i].kind != SYMB_ADAPTER_LORA || !n) continue;
            for (int p0 = 0; p0 < (fwd ? rpad_of(b->adapters[i].rank) : 1); p0 += 16) items.push_back(SmallItem{i, p0, b->seg_offsets[i], n});
        }
    std::vector<RowChunk> chunks;
    if (c.scale) plan_chunks(b, kSkinnyRows, -1, chunks);
    const std::vector<SegDesc> sd = make_segdesc(b);
    Blob blob;
    const size_t o_seg = blob.add(sd.data(), sd.size());
    const size_t o_it = blob.add(items.data(), items.size());
    const size_t o_nd = blob.add(c.neff, c.neff ? (size_t)bi.S : 0);
    const size_t o_xs = blob.add(c.x_seg, c.x_seg ? (size_t)bi.S : 0);
    const size_t o_cs = blob.add(c.out_seg, c.out_seg ? (size_t)bi.S : 0);
    const size_t o_off = blob.add(b->seg_offsets, c.scale ? (size_t)bi.S + 1 : 0);
    const size_t o_ch = blob.add(chunks.data(), chunks.size());
    // as many segments as the tiled kernels' descriptors have room for: a batch is refused or accepted whatever its row count
    const size_t tiled = (2 * sizeof(SegDesc) + sizeof(int32_t) + sizeof(int64_t) + (c.neff ? sizeof(NoiseDesc) : 0) + (c.x_seg ? 16 : 0)) * (size_t)bi.S;
    if (tiled > kSlotBytes) return fail(h, SYMB_ERR_UNSUPPORTED, "batch descriptors need %zu bytes, capacity is %zu", tiled, kSlotBytes);
    unsigned char* dev = nullptr;
    if ((st = upload(h, blob, s, &dev)) != SYMB_OK) return st;
    const SegDesc* const dseg = (const SegDesc*)(dev + o_seg);

    SmallStreamParams sp{};
    sp.W = (const bf16*)c.W;
    sp.X = (const bf16*)c.x_flat;
    sp.x_seg = c.x_seg ? (const bf16* const*)(dev + o_xs) : nullptr;
    if (c.scale) {
        ScaleParams sc{sp.X, c.copy, K, (const RowChunk*)(dev + o_ch), dseg, c.scale, sp.x_seg, (const int32_t*)(dev + o_off)};
        if ((st = launch_row_pass(h, symb_ia3_scale_rows_kernel, sc, K, chunks.size(), s)) != SYMB_OK) return st;
        sp.X = c.copy;
        sp.x_seg = nullptr;
    }
    sp.N = N;
    sp.K = K;
    sp.T = bi.T;
    sp.tiles = plan.tiles;
    sp.ranges = plan.ranges;
    sp.partial = (float*)(wsb + wl.sp_off);
    sp.items = (const SmallItem*)(dev + o_it);
    sp.num_items = (int)items.size();
    sp.h_ranges = plan.h_ranges;
    sp.seg = dseg;
    sp.h_partial = (float*)(wsb + wl.sh_off);
    sp.h_pitch = bi.max_rpad;
    sp.rows = rows;
    sp.direct = plan.direct;
    sp.out = SmallOut{(bf16*)c.out, (bf16*)c.out_base, c.out_seg ? (bf16* const*)(dev + o_cs) : nullptr, (const bf16*)c.bias,
                      c.neff ? (const NoiseDesc*)(dev + o_nd) : nullptr, fwd ? (bi.n_ia3 ? KIND_IA3 : 0) : c.lora && bi.n_ia3in ? KIND_IA3_IN : 0};
    const bool conv1d = b->weight_layout == SYMB_WEIGHT_CONV1D;
    if (plan.narrow) {
        if (bi.T <= 16) hipLaunchKernelGGL(symb_small_narrow_kernel<1>, dim3(plan.tiles), dim3(256), 0, s, sp);
        else if (bi.T <= 32) hipLaunchKernelGGL(symb_small_narrow_kernel<2>, dim3(plan.tiles), dim3(256), 0, s, sp);
        else hipLaunchKernelGGL(symb_small_narrow_kernel<4>, dim3(plan.tiles), dim3(256), 0, s, sp);
    } else if (fwd) conv1d ? launch_small_stream<true, false>(sp, plan.one_buffer, s) : launch_small_stream<false, false>(sp, false, s);
    else conv1d ? launch_small_stream<false, true>(sp, false, s) : launch_small_stream<true, true>(sp, plan.one_buffer, s);
    SYMB_HIP(h, hipGetLastError());
    if (plan.direct) return seal_slot(h);

    SmallFinishParams fp{};
    fp.partial = sp.partial;
    fp.h_partial = c.take_h ? nullptr : sp.h_partial;
    fp.ranges = plan.ranges;
    fp.h_ranges = plan.h_ranges;
    fp.h_pitch = bi.max_rpad;
    fp.h_rows = c.h_rows;
    fp.lora_term = plan.items > 0;
    fp.out = sp.out;
    fp.N = N;
    fp.T = bi.T;
    fp.seg = dseg;
    fp.rows = rows;
    hipLaunchKernelGGL(fwd ? symb_small_finish_kernel<false> : symb_small_finish_kernel<true>, dim3((N + 255) / 256, bi.T), dim3(128), 0, s, fp);
    SYMB_HIP(h, hipGetLastError());
    return seal_slot(h);
}

// The forward of a narrow layer in one launch, shrink included (narrow_kernel.hpp): its chunks of rows, none if the call is not one for it.  One column tile
// (N <= 256, above 128: half of it), stages of 64 k without a remainder, ranks to 16; one round of workgroups that is 60 % full, or more that are 85 %.  Two launches / this, us, 8 clients of ranks 8 and
// 16, 256 columns: 9900 rows (62 % of a round) of K = 512 17.9 / 13.0, 2048 36.6 / 29.6, 6144 90.9 / 81.2, 11008 143 / 137; 13000 rows 18.8 / 13.5, 36.5 / 30.9, 106 / 84, 174 / 140; 20000 (62 % of two)
// 23.9 / 23.7, 52.1 / 59.2, 146 / 160, 284 / 268; 136 to 248 columns of K = 64 to 6144 1.05 to 1.9 times as fast in one round.
// A chunk costs the whole weight whatever it holds, so beyond short inner dimensions, where the two launches' own latencies weigh more, its rows have to be there.  Two launches / this, segments of
// 1 to 1000 rows, 256 columns, rank 8.  One round: K <= 1536 1.0 to 3.5; above, seven eighths of the rows there or 9600 of them 0.97 to 1.5, else 0.37 to 0.97 (160, 200, 256 one-token clients of
// K = 6144 60.7 / 74.4, 58.5 / 76.4, 63.7 / 78.3).  More rounds: K <= 128 1.0 to 2.3; segments of one chunk each, K = 256 1.17 to 2.2, 512 up to 16 rows each 1.12 to 1.7, longer ones 0.9 to 1.1; K = 6144 and
// 11008, filled, up to three rounds 1.0 to 1.16, four 0.97; everything else 0.2 to 1.05 (500 one-token clients of K = 6144 71.8 / 147.4).
std::vector<RowChunk> narrow_chunks(const symb_batch* b, const BatchInfo& bi) {
    std::vector<RowChunk> v;
    if (b->weight_layout != SYMB_WEIGHT_LINEAR || !bi.n_lora || bi.n_ia3in || bi.max_rpad > 16 || b->d_out <= NARROW_COLS / 2 || b->d_out > NARROW_COLS || b->d_in % 64 || bi.S > 4096) return v;
    long n = 0, segments = 0;
    for (int i = 0; i < bi.S; ++i) {
        const int rows = b->seg_offsets[i + 1] - b->seg_offsets[i];
        n += (rows + NARROW_ROWS - 1) / NARROW_ROWS;
        segments += rows > 0;
    }
    if (n > 65536 || (n <= 256 ? 10 * n < 6 * 256 : 20 * n < 17 * 256 * ((n + 255) / 256))) return v;
    const bool filled = 8L * bi.T >= 7 * NARROW_ROWS * n;
    if (n <= 256 ? b->d_in > 1536 && !filled && bi.T < 9600
                 : b->d_in > 128 && !(n == segments && b->d_in <= (bi.T <= 16 * n ? 512 : 384)) && !(filled && b->d_in >= 6144 && n <= 768)) return v;
    plan_chunks(b, NARROW_ROWS, -1, v);
    return v;
}
symb_status run_narrow(symb_handle h, const symb_batch* b, const BatchInfo& bi, const std::vector<RowChunk>& chunks, const void* X, const void* W, const void* bias, void* Y, bf16* h_rows, hipStream_t s) {
    symb_status st;
    const std::vector<SegDesc> sd = make_segdesc(b);
    Blob blob;
    const size_t o_seg = blob.add(sd.data(), sd.size());
    const size_t o_ch = blob.add(chunks.data(), chunks.size());
    unsigned char* dev = nullptr;
    if ((st = upload(h, blob, s, &dev)) != SYMB_OK) return st;
    const NarrowParams np{(const bf16*)X, (const bf16*)W, (const bf16*)bias, (bf16*)Y, h_rows, b->d_out, b->d_in, 2 * bi.max_rpad, (const RowChunk*)(dev + o_ch), (const SegDesc*)(dev + o_seg)};
    const bool timed = h->timing && (int)h->timed.size() < kMaxTimed;
    const size_t slot = h->timed.size();
    if (timed) SYMB_HIP(h, hipEventRecord(h->tev[2 * slot], s));
    hipLaunchKernelGGL(symb_gemm_narrow_kernel, dim3((unsigned)chunks.size()), dim3(256), 0, s, np);
    SYMB_HIP(h, hipGetLastError());
    if (timed) {
        SYMB_HIP(h, hipEventRecord(h->tev[2 * slot + 1], s));
        h->timed.push_back({kTimedNarrow, gemm_flops(b, sd, b->d_out, b->d_in, true)});
    }
    return seal_slot(h);
}

// The input gradient of a layer of 64 to 256 outputs over many rows (shortk_kernel.hpp): its chunks of rows, none if the call is not one for it.  Enough of them that each of two workgroups per CU has four; up
// to 128 outputs not where many rows of a large output leave nothing but its stores (tiled kernel / this, without adapters, us, columns x rows: 64 outputs 1024 x 16384 13.5 / 11.8, 6144 x 3000 18.8 / 13.0, 11008 x 6000 44.5 / 44.3,
// 4096 x 16384 49.4 / 46.1, x 20480 49.8 / 55.3, 6144 x 20480 73.1 / 81.8; 256 outputs 2048 x 10000 25.4 / 17.8, 6144 x 6000 39.2 / 27.4, x 16384 85.3 / 74.3, 11008 x 10000 107.8 / 79.8, 24576 x 10000 205 / 164).
// A chunk costs as much whatever it holds.  Tiled kernels / this, with the dH launch that both make, LoRA segments of 1 to 64 rows, 64 to 256 outputs, 1024 to 24576 columns: under four rows a chunk 1.04 to 1.5 up to 2.1
// million chunks x columns, 0.94 to 1.2 to 3.2 million, 0.68 to 0.93 above (512 one-token clients of 11008 columns, 256 outputs, 96.8 / 141.6), but for 1.16 at 2048 of 24576; four rows and more 0.96 to 1.7,
// but where 1000 rows and more fill 512 to 1280 chunks in all strips of columns together 0.82 to 1.02 (4096 columns x 500 clients of 4 47.9 / 58.2).  Without adapters a chunk may cross segments.
std::vector<RowChunk> shortk_chunks(const symb_batch* b, const BatchInfo& bi, bool lora) {
    std::vector<RowChunk> v;
    if (b->weight_layout != SYMB_WEIGHT_LINEAR || b->d_out % 64 || b->d_out > 256 || (lora && bi.max_rpad > 16) || bi.S > 4096) return v;
    long n = 0;
    for (int i = 0; lora && i < bi.S; ++i) n += (b->seg_offsets[i + 1] - b->seg_offsets[i] + 31) / 32;
    if (!lora) n = (bi.T + 31) / 32;
    const long strips = (b->d_in + SHORTK_COLS - 1) / SHORTK_COLS;
    if (n * strips < 2048 || n > 16384) return v;       // (their list lies beside the others in the descriptors)
    if (bi.T < 4 * n ? n * b->d_in > 3200000 : bi.T >= 1000 && bi.T * strips > 512 * 32 && bi.T * strips < 1280 * 32) return v;
    if (b->d_out <= 128 && bi.T > 12000 && (long long)bi.T * b->d_in > 48000000) return v;
    if (lora) plan_chunks(b, 32, -1, v);
    else for (int r = 0; r < bi.T; r += 32) v.push_back(RowChunk{0, r, std::min(32, bi.T - r), 0});
    return v;
}
symb_status launch_shortk(symb_handle h, ShortKParams p, int K, double flops, hipStream_t s) {
    const int strips = (p.N + SHORTK_COLS - 1) / SHORTK_COLS, most = std::max(1, std::min(p.num_chunks, 512 / strips));      // two workgroups per CU
    p.per_group = (p.num_chunks + most - 1) / most;
    p.groups = (p.num_chunks + p.per_group - 1) / p.per_group;
    const dim3 grid((unsigned)((strips * p.groups + 7) / 8 * 8));
    const bool timed = h->timing && (int)h->timed.size() < kMaxTimed;
    const size_t slot = h->timed.size();
    if (timed) SYMB_HIP(h, hipEventRecord(h->tev[2 * slot], s));
    switch (K / 64) {
        case 1: hipLaunchKernelGGL(symb_gemm_shortk_kernel<2>, grid, dim3(256), 0, s, p); break;
        case 2: hipLaunchKernelGGL(symb_gemm_shortk_kernel<4>, grid, dim3(256), 0, s, p); break;
        case 3: hipLaunchKernelGGL(symb_gemm_shortk_kernel<6>, grid, dim3(256), 0, s, p); break;
        default: hipLaunchKernelGGL(symb_gemm_shortk_kernel<8>, grid, dim3(256), 0, s, p); break;
    }
    SYMB_HIP(h, hipGetLastError());
    if (timed) {
        SYMB_HIP(h, hipEventRecord(h->tev[2 * slot + 1], s));
        h->timed.push_back({kTimedShortK, flops});
    }
    return SYMB_OK;
}

symb_status check_handle(symb_handle h) {
    if (!h) return fail(nullptr, SYMB_ERR_INVALID_ARG, "handle is null");
    if (hipSetDevice(h->device) != hipSuccess) return fail(h, SYMB_ERR_DEVICE, "hipSetDevice(%d) failed", h->device);
    return SYMB_OK;
}

}  // namespace

// =============================================================================================
extern "C" {

const char* symb_status_string(symb_status s) {
    switch (s) {
        case SYMB_OK: return "SYMB_OK";
        case SYMB_ERR_INVALID_ARG: return "SYMB_ERR_INVALID_ARG";
        case SYMB_ERR_BAD_SEGMENTS: return "SYMB_ERR_BAD_SEGMENTS";
        case SYMB_ERR_UNSUPPORTED: return "SYMB_ERR_UNSUPPORTED";
        case SYMB_ERR_WORKSPACE_TOO_SMALL: return "SYMB_ERR_WORKSPACE_TOO_SMALL";
        case SYMB_ERR_DEVICE: return "SYMB_ERR_DEVICE";
    }
    return "SYMB_ERR_UNKNOWN";
}

const char* symb_last_error(symb_handle h) { return h ? h->error.c_str() : g_tls_error.c_str(); }

symb_status symb_create(symb_handle* out, int device) {
    if (!out) return fail(nullptr, SYMB_ERR_INVALID_ARG, "out is null");
    *out = nullptr;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0) return fail(nullptr, SYMB_ERR_DEVICE, "no HIP device available");
    if (device < 0 || device >= ndev) return fail(nullptr, SYMB_ERR_INVALID_ARG, "device %d out of range (%d devices)", device, ndev);
    SYMB_HIP(nullptr, hipSetDevice(device));
    symb_context* c = new symb_context();
    c->device = device;
    if (hipHostMalloc((void**)&c->host_ring, kSlots * kSlotBytes, hipHostMallocDefault) != hipSuccess ||
        hipMalloc((void**)&c->dev_ring, kSlots * kSlotBytes) != hipSuccess) {
        if (c->host_ring) (void)hipHostFree(c->host_ring);
        delete c;
        return fail(nullptr, SYMB_ERR_DEVICE, "descriptor staging allocation failed");
    }
    for (auto& r : c->ring.slot)
        if (hipEventCreateWithFlags(&r.done, hipEventDisableTiming) != hipSuccess) {
            symb_destroy(c);
            return fail(nullptr, SYMB_ERR_DEVICE, "hipEventCreate failed");
        }
    for (auto& u : c->ring.uses)
        if (hipEventCreateWithFlags(&u.ev, hipEventDisableTiming) != hipSuccess) {
            symb_destroy(c);
            return fail(nullptr, SYMB_ERR_DEVICE, "hipEventCreate failed");
        }
    // The K-split of the GEMM assumes that workgroup id mod 8 names the XCD: measure it.  Every
    // workgroup of a probe launch records the XCD it ran on; the rule holds if all workgroups of a
    // residue class report the same one.  (A device with a single XCD passes trivially.)
    {
        int* probe = reinterpret_cast<int*>(c->dev_ring);          // the ring is idle: borrow its first 8 KiB
        std::vector<int> xcc(kXccProbeGroups, -1);
        hipLaunchKernelGGL(symb_xcc_probe_kernel, dim3(kXccProbeGroups), dim3(64), 0, nullptr, probe);
        if (hipGetLastError() != hipSuccess ||
            hipMemcpy(xcc.data(), probe, sizeof(int) * kXccProbeGroups, hipMemcpyDeviceToHost) != hipSuccess) {
            symb_destroy(c);
            return fail(nullptr, SYMB_ERR_DEVICE, "XCD probe launch failed");
        }
        bool ok = true;
        for (int i = 0; i < kXccProbeGroups; ++i) ok = ok && xcc[i] == xcc[i & 7];
        c->xcd_rule = ok;
        for (int r = 0; r < 8; ++r) c->xcc_of_residue[r] = xcc[r];
    }
    {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(symb_static_scratch)) != hipSuccess || !p) {
            symb_destroy(c);
            return fail(nullptr, SYMB_ERR_DEVICE, "hipGetSymbolAddress(symb_static_scratch) failed");
        }
        c->static_scratch = static_cast<unsigned char*>(p);
    }
    *out = c;
    return SYMB_OK;
}

symb_status symb_debug_set_option(symb_handle h, int32_t option, int32_t value) {
    symb_status st = check_handle(h);
    if (st != SYMB_OK) return st;
    switch (option) {
        case SYMB_OPT_DESCRIPTOR_REUSE: h->opt_desc_reuse = value != 0; break;
        case SYMB_OPT_K_SPLIT: h->opt_k_split = value != 0; break;
        case SYMB_OPT_SMALL_BATCH_KERNELS: h->opt_small_rows = value != 0; break;
        case SYMB_OPT_SKINNY_DEEP: h->opt_skinny_deep = value != 0; break;
        default: return fail(h, SYMB_ERR_INVALID_ARG, "unknown option %d", option);
    }
    return SYMB_OK;
}

symb_status symb_debug_xcd_rule(symb_handle h, int32_t* holds, int32_t* xcc_of_residue) {
    symb_status st = check_handle(h);
    if (st != SYMB_OK) return st;
    if (holds) *holds = h->xcd_rule ? 1 : 0;
    if (xcc_of_residue)
        for (int r = 0; r < 8; ++r) xcc_of_residue[r] = h->xcc_of_residue[r];
    return SYMB_OK;
}

symb_status symb_debug_descriptor_stats(symb_handle h, int64_t* sent, int64_t* in_place) {
    symb_status st = check_handle(h);
    if (st != SYMB_OK) return st;
    if (sent) *sent = h->desc_sent;
    if (in_place) *in_place = h->desc_in_place;
    return SYMB_OK;
}

symb_status symb_debug_gemm_timing_enable(symb_handle h, int32_t on) {
    symb_status st = check_handle(h);
    if (st != SYMB_OK) return st;
    if (on && h->tev.empty()) {
        h->tev.resize(2 * kMaxTimed);
        for (auto& e : h->tev) SYMB_HIP(h, hipEventCreate(&e));
        h->timed.reserve(kMaxTimed);
    }
    h->timing = on != 0;
    h->timed.clear();
    return SYMB_OK;
}

symb_status symb_debug_gemm_timing_read(symb_handle h, int32_t variant, double* ms_total, int64_t* launches,
                                        double* flops_total) {
    symb_status st = check_handle(h);
    if (st != SYMB_OK) return st;
    if (!ms_total || !launches || !flops_total) return fail(h, SYMB_ERR_INVALID_ARG, "null output pointer");
    *ms_total = 0.0;
    *launches = 0;
    *flops_total = 0.0;
    for (size_t i = 0; i < h->timed.size(); ++i) {
        const int v = h->timed[i].variant;
        if ((variant >= 8 || v >= kTimedNarrow ? v : v & 7) != variant) continue;
        SYMB_HIP(h, hipEventSynchronize(h->tev[2 * i + 1]));
        float ms = 0.f;
        SYMB_HIP(h, hipEventElapsedTime(&ms, h->tev[2 * i], h->tev[2 * i + 1]));
        *ms_total += ms;
        *launches += 1;
        *flops_total += h->timed[i].flops;
    }
    return SYMB_OK;
}

symb_status symb_destroy(symb_handle h) {
    if (!h) return SYMB_OK;
    (void)hipSetDevice(h->device);
    for (auto& e : h->tev) (void)hipEventDestroy(e);
    for (auto& r : h->ring.slot) {
        if (r.used) (void)hipEventSynchronize(r.done);
        if (r.done) (void)hipEventDestroy(r.done);
    }
    (void)hipDeviceSynchronize();                        // calls without an event of their own
    for (auto& u : h->ring.uses)
        if (u.ev) (void)hipEventDestroy(u.ev);
    if (h->dev_ring) (void)hipFree(h->dev_ring);
    if (h->host_ring) (void)hipHostFree(h->host_ring);
    delete h;
    return SYMB_OK;
}

symb_status symb_validate_batch(const symb_batch* b) { return validate(nullptr, b); }

symb_status symb_debug_row_segment_map(const symb_batch* b, int32_t* host_out) {
    symb_status st = validate(nullptr, b);
    if (st != SYMB_OK) return st;
    if (!host_out && b->seg_offsets[b->num_segments] > 0) return fail(nullptr, SYMB_ERR_INVALID_ARG, "host_out is null");
    for (int i = 0; i < b->num_segments; ++i)
        for (int t = b->seg_offsets[i]; t < b->seg_offsets[i + 1]; ++t) host_out[t] = i;
    return SYMB_OK;
}

symb_status symb_plan_row_tiles(const symb_batch* b, int32_t tile_m, int32_t* seg_lo, int32_t* seg_hi, int32_t* num_tiles) {
    symb_status st = validate(nullptr, b);
    if (st != SYMB_OK) return st;
    if (tile_m <= 0 || !num_tiles) return fail(nullptr, SYMB_ERR_INVALID_ARG, "tile_m must be positive and num_tiles non-null");
    std::vector<int32_t> lo, hi;
    plan_row_tiles(b, tile_m, lo, hi);
    *num_tiles = (int32_t)lo.size();
    if (!lo.empty() && (!seg_lo || !seg_hi)) return fail(nullptr, SYMB_ERR_INVALID_ARG, "seg_lo / seg_hi is null");
    for (size_t u = 0; u < lo.size(); ++u) {
        seg_lo[u] = lo[u];
        seg_hi[u] = hi[u];
    }
    return SYMB_OK;
}

static bool wants_lora_grad(const symb_batch* b) {
    for (int i = 0; i < b->num_segments; ++i)
        if (b->adapters[i].kind == SYMB_ADAPTER_LORA && (b->adapters[i].dA || b->adapters[i].dB) &&
            b->seg_offsets[i + 1] > b->seg_offsets[i])
            return true;
    return false;
}

symb_status symb_workspace_bytes(const symb_batch* b, int32_t op, size_t* out) {
    symb_status st = validate(nullptr, b);
    if (st != SYMB_OK) return st;
    if (!out) return fail(nullptr, SYMB_ERR_INVALID_ARG, "out is null");
    if (op < SYMB_OP_FWD || op > SYMB_OP_BWD_INPUT_INPLACE) return fail(nullptr, SYMB_ERR_INVALID_ARG, "unknown op %d", op);
    const BatchInfo bi = inspect(b);
    const bool staged = op == SYMB_OP_FWD_INPLACE || op == SYMB_OP_BWD_INPUT_INPLACE;
    const int base_op = op == SYMB_OP_FWD_INPLACE ? SYMB_OP_FWD : op == SYMB_OP_BWD_INPUT_INPLACE ? SYMB_OP_BWD_INPUT : op;
    *out = ws_layout(b, bi, base_op, true, wants_lora_grad(b), staged).total;
    return SYMB_OK;
}

// ---------------------------------------------------------------------------------------------
// Checks a per-segment noise array (width = row length in elements) and turns it into device descriptors.
symb_status make_noisedesc(symb_handle h, const symb_batch* b, const symb_noise* noise, const char* what,
                           std::vector<NoiseDesc>& out) {
    out.assign(b->num_segments, NoiseDesc{nullptr, 0, 0});
    for (int i = 0; i < b->num_segments; ++i) {
        const symb_noise& n = noise[i];
        if (!n.ptr) continue;
        const int len = b->seg_offsets[i + 1] - b->seg_offsets[i];
        if (n.rows != 1 && n.rows != len)
            return fail(h, SYMB_ERR_INVALID_ARG, "%s of segment %d has %d rows: must be 1 or the segment's %d tokens", what, i, n.rows, len);
        if (misaligned16(n.ptr)) return fail(h, SYMB_ERR_INVALID_ARG, "%s of segment %d is not 16-byte aligned", what, i);
        out[i] = NoiseDesc{(const bf16*)n.ptr, n.rows, 0};
    }
    return SYMB_OK;
}

// Per-segment buffers (one DEVICE pointer per segment, HOST array): alignment, presence for
// non-empty segments, and, for the GEMM's activation operand, that they all lie inside one 4 GiB
// window (lane offsets are 32 bits wide).  *base receives the lowest address.
symb_status check_seg_ptrs(symb_handle h, const symb_batch* b, const void* const* seg, size_t row_bytes, const char* what,
                           bool need_window, const void** base) {
    uintptr_t lo = UINTPTR_MAX, hi = 0;
    for (int i = 0; i < b->num_segments; ++i) {
        const size_t n = (size_t)(b->seg_offsets[i + 1] - b->seg_offsets[i]);
        if (!n) continue;
        if (!seg[i]) return fail(h, SYMB_ERR_INVALID_ARG, "%s of segment %d is null", what, i);
        if (misaligned16(seg[i])) return fail(h, SYMB_ERR_INVALID_ARG, "%s of segment %d is not 16-byte aligned", what, i);
        lo = std::min(lo, (uintptr_t)seg[i]);
        hi = std::max(hi, (uintptr_t)seg[i] + n * row_bytes);
    }
    if (need_window && hi > lo && hi - lo > ((uint64_t)1 << 32) - 65536)
        return fail(h, SYMB_ERR_UNSUPPORTED, "%s buffers span %zu bytes: they must lie within one 4 GiB window", what, (size_t)(hi - lo));
    if (base) *base = (const void*)(lo == UINTPTR_MAX ? 0 : lo);
    return SYMB_OK;
}

// Whether any output buffer of a per-segment call shares bytes with any of its input buffers.
static bool seg_buffers_overlap(const symb_batch* b, const void* const* in_seg, size_t in_row_bytes, void* const* out_seg,
                                size_t out_row_bytes) {
    std::vector<std::pair<uintptr_t, uintptr_t>> in;
    for (int i = 0; i < b->num_segments; ++i) {
        const size_t n = (size_t)(b->seg_offsets[i + 1] - b->seg_offsets[i]);
        if (n) in.emplace_back((uintptr_t)in_seg[i], (uintptr_t)in_seg[i] + n * in_row_bytes);
    }
    std::sort(in.begin(), in.end());
    for (size_t k = 1; k < in.size(); ++k) in[k].second = std::max(in[k].second, in[k - 1].second);   // running end: sorted by start
    for (int i = 0; i < b->num_segments; ++i) {
        const size_t n = (size_t)(b->seg_offsets[i + 1] - b->seg_offsets[i]);
        if (!n) continue;
        const uintptr_t lo = (uintptr_t)out_seg[i], hi = lo + n * out_row_bytes;
        // the last input interval that starts before hi: with the running end it tells whether any reaches past lo
        auto it = std::lower_bound(in.begin(), in.end(), std::make_pair(hi, (uintptr_t)0));
        if (it != in.begin() && std::prev(it)->second > lo) return true;
    }
    return false;
}

static symb_status forward_impl(symb_handle h, const symb_batch* b, const void* X, const void* W, const void* bias,
                                const symb_noise* noise_effect, void* Y, void* Ybase, void* ws, size_t ws_bytes, void* stream,
                                const void* const* X_seg = nullptr, void* const* Y_seg = nullptr) {
    symb_status st = check_handle(h);
    if (st != SYMB_OK) return st;
    CallGuard guard(h);
    if ((st = validate(h, b)) != SYMB_OK) return st;
    const BatchInfo bi = inspect(b);
    if (bi.T == 0) return SYMB_OK;
    const bool seg_io = X_seg != nullptr;
    const void* x_base = nullptr;
    if (seg_io) {
        if (!Y_seg || !W) return fail(h, SYMB_ERR_INVALID_ARG, "X_seg, Y_seg and W are required");
        // with an IA3_IN segment the GEMM reads a flat, scaled copy of the rows: no window needed then
        if ((st = check_seg_ptrs(h, b, X_seg, (size_t)b->d_in * 2, "X", bi.n_ia3in == 0, &x_base)) != SYMB_OK) return st;
        if ((st = check_seg_ptrs(h, b, (const void* const*)Y_seg, (size_t)b->d_out * 2, "Y", false, nullptr)) != SYMB_OK) return st;
    } else if (!X || !W || !Y) return fail(h, SYMB_ERR_INVALID_ARG, "X, W and Y are required");
    std::vector<NoiseDesc> nd;
    if (noise_effect && (st = make_noisedesc(h, b, noise_effect, "noise effect", nd)) != SYMB_OK) return st;
    if (misaligned16(X) || misaligned16(W) || misaligned16(Y) || misaligned16(Ybase) || misaligned16(bias) || misaligned16(ws))
        return fail(h, SYMB_ERR_INVALID_ARG, "device pointers must be 16-byte aligned");
    // Per-segment buffers whose outputs overlap inputs (a client's one buffer used for both, Sec. 3.5):
    // column tiles of a row tile run at different times, so the GEMM writes a flat copy in the
    // workspace and a row scatter, after it on the stream, fills the clients' buffers.
    const bool staged = seg_io && seg_buffers_overlap(b, X_seg, (size_t)b->d_in * 2, Y_seg, (size_t)b->d_out * 2);
    const WsLayout wl = ws_layout(b, bi, SYMB_OP_FWD, true, false, staged);
    const size_t ws_need = wl.mandatory;     // the regions after it are optional
    if (ws_need > ws_bytes || (ws_need && !ws))
        return fail(h, SYMB_ERR_WORKSPACE_TOO_SMALL, "forward needs %zu workspace bytes, got %zu%s", ws_need, ws_bytes,
                    staged ? " (output buffers overlap input buffers: size the workspace with SYMB_OP_FWD_INPLACE)" : "");
    hipStream_t s = (hipStream_t)stream;
    if (small_path(h, bi, wl, ws, ws_bytes)) {     // (partial sums between: overlapping buffers need no flat copy)
        unsigned char* const base = (unsigned char*)ws;
        const SmallCall c{SYMB_OP_FWD, X, W, bias, Y, Ybase, X_seg, Y_seg, nd.empty() ? nullptr : nd.data(), bi.n_ia3in ? (int)KIND_IA3_IN : 0,
                          (bf16*)(base + wl.sc_off), (bf16*)(base + wl.h_off), true, false, staged};
        if ((st = run_small(h, b, bi, wl, base, c, s)) != SYMB_OK) return st;
        guard.completed = true;
        return SYMB_OK;
    }

    if (!seg_io && nd.empty() && !Ybase) {
        const std::vector<RowChunk> chunks = narrow_chunks(b, bi);
        if (!chunks.empty()) {
            if ((st = run_narrow(h, b, bi, chunks, X, W, bias, Y, (bf16*)((unsigned char*)ws + wl.h_off), s)) != SYMB_OK) return st;
            guard.completed = true;
            return SYMB_OK;
        }
    }
    GemmPlan plan = gemm_plan(b, b->d_out, b->d_in, b->weight_layout == SYMB_WEIGHT_CONV1D, bi.n_lora > 0, Ybase != nullptr, !Ybase && h->opt_k_split && h->xcd_rule,
                              ws && ws_bytes > wl.tp_off ? ws_bytes - wl.tp_off : 0);
    const bool k_split = plan.split.parts > 1 && plan.variant != kTileMid;
    const int bm = tile_rows(plan.variant), bn = tile_cols(plan.variant);
    std::vector<int32_t> lo, hi;
    plan_row_tiles(b, bm, lo, hi);
    const SkinnyChunks chunks = plan_skinny(h, b, lora_segments(b), bi.max_rpad);
    std::vector<RowChunk> all_chunks;
    // Input-major weight: the forward is the N-contiguous GEMM, whose LoRA steps read the adapter
    // side as [rank][d_out] rows: B_i^T, packed into the workspace; a second descriptor set points there.
    const bool conv1d = b->weight_layout == SYMB_WEIGHT_CONV1D;
    const bool copy_rows = bi.n_ia3in > 0;      // the product reads a flat copy of X (IA3_IN rows scaled)
    if (copy_rows || staged) plan_chunks(b, kSkinnyRows, -1, all_chunks);
    const std::vector<SegDesc> sd = make_segdesc(b);
    unsigned char* wsb = (unsigned char*)ws;
    std::vector<SegDesc> sd_gemm = sd;
    std::vector<int64_t> pk_off(bi.S, 0);
    DeltaPlan& delta = plan.terms;
    const size_t de_off = terms_offset(wl, plan);
    if (conv1d && bi.n_lora) {
        int64_t cur = 0;
        for (int i = 0; i < bi.S; ++i)
            if (sd[i].kind == KIND_LORA) {
                pk_off[i] = cur;
                sd_gemm[i].A = (const bf16*)(wsb + wl.pk_off) + cur;
                cur += (int64_t)sd[i].rpad * b->d_out;
            }
    }
    Blob blob;
    const size_t o_seg = blob.add(sd.data(), sd.size());
    const size_t o_off = blob.add(b->seg_offsets, (size_t)bi.S + 1);
    const size_t o_lo = blob.add(lo.data(), lo.size());
    const size_t o_hi = blob.add(hi.data(), hi.size());
    const std::vector<int32_t> tile_epi = plan_tile_kind(b, lo, hi, SYMB_ADAPTER_IA3);
    const size_t o_te = blob.add(tile_epi.data(), tile_epi.size());
    const size_t o_ch = blob.add(chunks.items.data(), chunks.items.size());
    const size_t o_nd = blob.add(nd.data(), nd.size());
    const size_t o_pk = blob.add(pk_off.data(), pk_off.size());
    const size_t o_all = blob.add(all_chunks.data(), all_chunks.size());
    const size_t o_xs = blob.add(X_seg, seg_io ? (size_t)bi.S : 0);
    const size_t o_ys = blob.add(Y_seg, seg_io ? (size_t)bi.S : 0);
    const std::vector<int32_t> k_zero(k_split ? plan.split.slots : 0, 0);
    const size_t o_kc = blob.add(k_zero.data(), k_zero.size());   // arrival counters of the K-split tiles
    const DeltaBlob db = add_gemm_desc(blob, sd_gemm, delta, (int)lo.size(), bm);
    unsigned char* dev = nullptr;
    if ((st = upload(h, blob, s, &dev)) != SYMB_OK) return st;

    // IA3 input scaling: the GEMM multiplies a copy of X whose IA3_IN rows are scaled by l_i
    // (LoRA segments, if any, still shrink the caller's X: their rows are not touched by the copy)
    const bf16* x_op = (const bf16*)X;
    if (copy_rows) {
        bf16* const copy = (bf16*)(wsb + wl.sc_off);
        ScaleParams sc{(const bf16*)X, copy, b->d_in, (const RowChunk*)(dev + o_all),
                       (const SegDesc*)(dev + o_seg), KIND_IA3_IN, seg_io ? (const bf16* const*)(dev + o_xs) : nullptr,
                       (const int32_t*)(dev + o_off)};
        if ((st = launch_row_pass(h, symb_ia3_scale_rows_kernel, sc, sc.d_out, all_chunks.size(), s)) != SYMB_OK) return st;
        x_op = copy;
    }
    bf16* Hs = bi.n_lora ? (bf16*)(wsb + wl.h_off) : nullptr;
    if (conv1d && bi.n_lora) {
        PackParams pp{(const SegDesc*)(dev + o_seg), (bf16*)(wsb + wl.pk_off), (const int64_t*)(dev + o_pk), b->d_out};
        hipLaunchKernelGGL(symb_pack_bt_kernel, dim3((b->d_out + 255) / 256, bi.S), dim3(256), 0, s, pp);
        SYMB_HIP(h, hipGetLastError());
    }
    if (bi.n_lora) {
        SkinnyParams sp{};
        sp.L = (const bf16*)X;
        sp.out = Hs;
        sp.K = b->d_in;
        sp.out_pitch = 2 * bi.max_rpad;
        sp.chunks = (const RowChunk*)(dev + o_ch);
        sp.seg = (const SegDesc*)(dev + o_seg);
        sp.use_packed = 0;
        if (seg_io) {
            sp.L_seg = (const bf16* const*)(dev + o_xs);
            sp.off = (const int32_t*)(dev + o_off);
        }
        if ((st = launch_skinny<false>(h, sp, chunks, bi.max_rpad, s)) != SYMB_OK) return st;
    }
    if (!delta.items.empty() && (st = launch_delta(h, false, (const SegDesc*)(dev + o_seg), (const RowChunk*)(dev + db.items), (int)delta.items.size(), b->d_out,
                                                   Hs, bi.max_rpad, (float*)(wsb + de_off), s)) != SYMB_OK) return st;
    GemmParams gp{};
    if (!delta.items.empty()) {
        gp.delta = (const float*)(wsb + de_off);
        gp.tile_delta = (const TileDelta*)(dev + db.tiles);
    }
    gp.Aop = x_op;
    if (seg_io) {
        if (!copy_rows) {          // (a flat copy of the rows, scaled for IA3_IN, is read as one tensor)
            gp.Aop = nullptr;
            gp.a_seg = (const bf16* const*)(dev + o_xs);
            gp.a_base = (const bf16*)x_base;
        }
        if (!staged) gp.c_seg = (bf16* const*)(dev + o_ys);
    }
    gp.Bop = (const bf16*)W;
    gp.C = staged ? (bf16*)(wsb + wl.so_off) : (bf16*)Y;
    gp.Cbase = (bf16*)Ybase;
    gp.bias = (const bf16*)bias;
    gp.M = bi.T;
    gp.N = b->d_out;
    gp.K = b->d_in;
    gp.off = (const int32_t*)(dev + o_off);
    gp.seg = (const SegDesc*)(dev + db.seg);
    gp.tile_seg_lo = (const int32_t*)(dev + o_lo);
    gp.tile_seg_hi = (const int32_t*)(dev + o_hi);
    gp.ext = Hs;
    gp.ext_pitch = 2 * bi.max_rpad;
    gp.epi_ia3 = bi.n_ia3 > 0 ? KIND_IA3 : 0;
    gp.tile_epi = (const int32_t*)(dev + o_te);
    gp.neff = nd.empty() ? nullptr : (const NoiseDesc*)(dev + o_nd);
    gp.timing_flops = gemm_flops(b, sd_gemm, b->d_out, b->d_in, bi.n_lora > 0);
    gp.variant = plan.variant;
    gp.group_m = gemm_group_m((bi.T + bm - 1) / bm, (b->d_out + bn - 1) / bn, lo, hi);
    if (k_split) {
        gp.k_parts = plan.split.parts;
        gp.k_whole = plan.split.whole;
        gp.partial = (float*)(wsb + wl.tp_off);
        gp.k_count = (int*)(dev + o_kc);
    }
    // W [d_out][d_in]: K-contiguous weight rows.  W [d_in][d_out]: the weight is the [K][N] operand.
    st = conv1d ? launch_gemm<true>(h, gp, s) : launch_gemm<false>(h, gp, s);
    if (st != SYMB_OK) return st;
    if (staged) {
        ScatterParams sc{(const bf16*)(wsb + wl.so_off), b->d_out, (const RowChunk*)(dev + o_all), (bf16* const*)(dev + o_ys),
                         (const int32_t*)(dev + o_off)};
        hipLaunchKernelGGL(symb_scatter_rows_kernel, dim3((unsigned)all_chunks.size()), dim3(256), 0, s, sc);
        SYMB_HIP(h, hipGetLastError());
    }
    { guard.completed = true; return seal_slot(h); }
}

symb_status symb_base_linear_fwd(symb_handle h, const symb_batch* b, const void* X, const void* W, const void* bias,
                                 void* Y, void* Ybase, void* ws, size_t ws_bytes, void* stream) {
    return forward_impl(h, b, X, W, bias, nullptr, Y, Ybase, ws, ws_bytes, stream);
}

// The forward with its workspace in the file-scope scratch array of this device: no device allocation
// by the library or the caller.  Same kernels and launches as symb_base_linear_fwd.
symb_status symb_base_linear_fwd_static(symb_handle h, const symb_batch* b, const void* X, const void* W, const void* bias,
                                        void* Y, void* Ybase, void* stream) {
    symb_status st = check_handle(h);
    if (st != SYMB_OK) return st;
    if ((st = validate(h, b)) != SYMB_OK) return st;
    const BatchInfo bi = inspect(b);
    const WsLayout wl = ws_layout(b, bi, SYMB_OP_FWD, true, false);
    const size_t need = wl.mandatory;        // the optional regions (small-batch kernels, K-split partial tiles) are used only if they fit too
    if (need > (size_t)SYMB_STATIC_SCRATCH_BYTES)
        return fail(h, SYMB_ERR_WORKSPACE_TOO_SMALL, "this batch needs %zu bytes of workspace; the static scratch array holds %zu "
                    "(use symb_base_linear_fwd with a workspace of the caller's)", need, (size_t)SYMB_STATIC_SCRATCH_BYTES);
    return forward_impl(h, b, X, W, bias, nullptr, Y, Ybase, h->static_scratch, (size_t)SYMB_STATIC_SCRATCH_BYTES, stream);
}

symb_status symb_base_linear_fwd_seg(symb_handle h, const symb_batch* b, const void* const* X_seg, const void* W,
                                     const void* bias, void* const* Y_seg, void* ws, size_t ws_bytes, void* stream) {
    symb_status st = check_handle(h);
    if (st != SYMB_OK) return st;
    if (!X_seg || !Y_seg) return fail(h, SYMB_ERR_INVALID_ARG, "X_seg and Y_seg are required");
    return forward_impl(h, b, nullptr, W, bias, nullptr, nullptr, nullptr, ws, ws_bytes, stream, X_seg, Y_seg);
}

symb_status symb_base_linear_fwd_denoise(symb_handle h, const symb_batch* b, const void* Xn, const void* W, const void* bias,
                                         const symb_noise* noise_effect, void* Y, void* ws, size_t ws_bytes, void* stream) {
    symb_status st = check_handle(h);
    if (st != SYMB_OK) return st;
    if (!noise_effect) return fail(h, SYMB_ERR_INVALID_ARG, "noise_effect is required");
    return forward_impl(h, b, Xn, W, bias, noise_effect, Y, nullptr, ws, ws_bytes, stream);
}

symb_status symb_noise_add(symb_handle h, const symb_batch* b, const void* X, const symb_noise* noise, void* Xn, void* stream) {
    symb_status st = check_handle(h);
    if (st != SYMB_OK) return st;
    CallGuard guard(h);
    if ((st = validate(h, b)) != SYMB_OK) return st;
    if (!noise) return fail(h, SYMB_ERR_INVALID_ARG, "noise is required");
    const BatchInfo bi = inspect(b);
    if (bi.T == 0) return SYMB_OK;
    if (!X || !Xn) return fail(h, SYMB_ERR_INVALID_ARG, "X and Xn are required");
    if (misaligned16(X) || misaligned16(Xn)) return fail(h, SYMB_ERR_INVALID_ARG, "device pointers must be 16-byte aligned");
    std::vector<NoiseDesc> nd;
    if ((st = make_noisedesc(h, b, noise, "noise", nd)) != SYMB_OK) return st;
    hipStream_t s = (hipStream_t)stream;
    std::vector<RowChunk> chunks;
    plan_chunks(b, kSkinnyRows, -1, chunks);
    Blob blob;
    const size_t o_off = blob.add(b->seg_offsets, (size_t)bi.S + 1);
    const size_t o_ch = blob.add(chunks.data(), chunks.size());
    const size_t o_nd = blob.add(nd.data(), nd.size());
    unsigned char* dev = nullptr;
    if ((st = upload(h, blob, s, &dev)) != SYMB_OK) return st;
    NoiseAddParams np{(const bf16*)X, (bf16*)Xn, b->d_in, (const RowChunk*)(dev + o_ch), (const int32_t*)(dev + o_off),
                      (const NoiseDesc*)(dev + o_nd)};
    if ((st = launch_row_pass(h, symb_noise_add_kernel, np, b->d_in, chunks.size(), s)) != SYMB_OK) return st;
    { guard.completed = true; return seal_slot(h); }
}

// ---------------------------------------------------------------------------------------------
static symb_status backward_input_impl(symb_handle h, const symb_batch* b, const void* dY, const void* W, void* dX,
                                       void* dXbase, uint32_t flags, void* ws, size_t ws_bytes, void* stream,
                                       const void* const* dY_seg, void* const* dX_seg);

symb_status symb_base_linear_bwd_input(symb_handle h, const symb_batch* b, const void* dY, const void* W, void* dX,
                                       uint32_t flags, void* ws, size_t ws_bytes, void* stream) {
    return backward_input_impl(h, b, dY, W, dX, nullptr, flags, ws, ws_bytes, stream, nullptr, nullptr);
}

symb_status symb_base_linear_bwd_input_ex(symb_handle h, const symb_batch* b, const void* dY, const void* W, void* dX,
                                          void* dXbase, uint32_t flags, void* ws, size_t ws_bytes, void* stream) {
    return backward_input_impl(h, b, dY, W, dX, dXbase, flags, ws, ws_bytes, stream, nullptr, nullptr);
}

symb_status symb_base_linear_bwd_input_seg(symb_handle h, const symb_batch* b, const void* const* dY_seg, const void* W,
                                           void* const* dX_seg, uint32_t flags, void* ws, size_t ws_bytes, void* stream) {
    symb_status st = check_handle(h);
    if (st != SYMB_OK) return st;
    if (!dY_seg || !dX_seg) return fail(h, SYMB_ERR_INVALID_ARG, "dY_seg and dX_seg are required");
    return backward_input_impl(h, b, nullptr, W, nullptr, nullptr, flags, ws, ws_bytes, stream, dY_seg, dX_seg);
}

static symb_status backward_input_impl(symb_handle h, const symb_batch* b, const void* dY, const void* W, void* dX,
                                       void* dXbase, uint32_t flags, void* ws, size_t ws_bytes, void* stream,
                                       const void* const* dY_seg, void* const* dX_seg) {
    symb_status st = check_handle(h);
    if (st != SYMB_OK) return st;
    CallGuard guard(h);
    if ((st = validate(h, b)) != SYMB_OK) return st;
    if (flags & ~(uint32_t)(SYMB_BWD_BASE_ONLY | SYMB_BWD_REUSE_DH)) return fail(h, SYMB_ERR_INVALID_ARG, "unknown backward flag %u", flags);
    if ((flags & SYMB_BWD_BASE_ONLY) && (flags & SYMB_BWD_REUSE_DH))
        return fail(h, SYMB_ERR_INVALID_ARG, "SYMB_BWD_REUSE_DH makes no sense with SYMB_BWD_BASE_ONLY");
    const bool take_dh = (flags & SYMB_BWD_REUSE_DH) != 0;      // dH is in the workspace already (a gradient call on this batch left it)
    const BatchInfo bi = inspect(b);
    if (bi.T == 0) return SYMB_OK;
    const bool seg_io = dY_seg != nullptr;
    const void* g_base = nullptr;
    if (seg_io) {
        if (!W) return fail(h, SYMB_ERR_INVALID_ARG, "W is required");
        const bool copy_first = !(flags & SYMB_BWD_BASE_ONLY) && bi.n_ia3 > 0;     // then the GEMM reads the scaled copy, not the buffers
        if ((st = check_seg_ptrs(h, b, dY_seg, (size_t)b->d_out * 2, "dY", !copy_first, &g_base)) != SYMB_OK) return st;
        if ((st = check_seg_ptrs(h, b, (const void* const*)dX_seg, (size_t)b->d_in * 2, "dX", false, nullptr)) != SYMB_OK) return st;
    } else if (!dY || !W || !dX) return fail(h, SYMB_ERR_INVALID_ARG, "dY, W and dX are required");
    if (misaligned16(dY) || misaligned16(W) || misaligned16(dX) || misaligned16(dXbase) || misaligned16(ws))
        return fail(h, SYMB_ERR_INVALID_ARG, "device pointers must be 16-byte aligned");
    const bool full = !(flags & SYMB_BWD_BASE_ONLY);
    const bool staged = seg_io && seg_buffers_overlap(b, dY_seg, (size_t)b->d_out * 2, dX_seg, (size_t)b->d_in * 2);   // see the forward
    const WsLayout wl = ws_layout(b, bi, SYMB_OP_BWD_INPUT, full, false, staged);
    const size_t ws_need = wl.mandatory;     // the regions after it are optional
    if (ws_need > ws_bytes || (ws_need && !ws))
        return fail(h, SYMB_ERR_WORKSPACE_TOO_SMALL, "backward needs %zu workspace bytes, got %zu%s", ws_need, ws_bytes,
                    staged ? " (output buffers overlap input buffers: size the workspace with SYMB_OP_BWD_INPUT_INPLACE)" : "");
    hipStream_t s = (hipStream_t)stream;
    const bool lora = full && bi.n_lora > 0, ia3 = full && bi.n_ia3 > 0;
    if (small_path(h, bi, wl, ws, ws_bytes)) {     // (partial sums between: overlapping buffers need no flat copy)
        unsigned char* const base = (unsigned char*)ws;
        const SmallCall c{SYMB_OP_BWD_INPUT, dY, W, nullptr, dX, dXbase, dY_seg, dX_seg, nullptr, ia3 ? (int)KIND_IA3 : 0,
                          (bf16*)(base + wl.sc_off), (bf16*)(base + wl.dh_off), full, take_dh, staged};
        if ((st = run_small(h, b, bi, wl, base, c, s)) != SYMB_OK) return st;
        guard.completed = true;
        return SYMB_OK;
    }

    GemmPlan plan = gemm_plan(b, b->d_in, b->d_out, b->weight_layout != SYMB_WEIGHT_CONV1D, lora, dXbase != nullptr, !dXbase && h->opt_k_split && h->xcd_rule,
                              ws && ws_bytes > wl.tp_off ? ws_bytes - wl.tp_off : 0);
    std::vector<RowChunk> sk_chunks;
    if (!seg_io && !dXbase && !ia3 && !(full && bi.n_ia3in)) sk_chunks = shortk_chunks(b, bi, lora);
    if (!sk_chunks.empty()) plan = GemmPlan{};
    const bool k_split = plan.split.parts > 1 && plan.variant != kTileMid;
    const int bm = tile_rows(plan.variant), bn = tile_cols(plan.variant);
    std::vector<int32_t> lo, hi;
    plan_row_tiles(b, bm, lo, hi);
    SkinnyChunks chunks;
    if (lora && !take_dh) chunks = plan_skinny(h, b, lora_segments(b), bi.max_rpad);
    std::vector<RowChunk> all_chunks;
    // Rows of IA3 segments enter the GEMM scaled by l_i: a scaled copy of those rows goes to the
    // workspace, and the GEMM takes every row from where it lies (per-row base pointers: the copy for
    // IA3 rows, the caller's dY for the others).  Lane offsets are 32 bits wide, so this needs all those
    // rows within one 4 GiB window; failing that, all rows are copied and the GEMM reads the copy alone.
    unsigned char* const wsb0 = (unsigned char*)ws;
    std::vector<const void*> mix;           // per segment: where the GEMM reads its rows
    bool ia3_mixed = false;
    if (ia3) {
        mix.assign(bi.S, nullptr);
        uintptr_t lo_a = UINTPTR_MAX, hi_a = 0;
        for (int i = 0; i < bi.S; ++i) {
            const size_t n = (size_t)(b->seg_offsets[i + 1] - b->seg_offsets[i]), row_bytes = (size_t)b->d_out * 2;
            if (!n) continue;
            const unsigned char* src = b->adapters[i].kind == SYMB_ADAPTER_IA3
                                           ? wsb0 + wl.sc_off + (size_t)b->seg_offsets[i] * row_bytes
                                           : (seg_io ? (const unsigned char*)dY_seg[i] : (const unsigned char*)dY + (size_t)b->seg_offsets[i] * row_bytes);
            mix[i] = src;
            lo_a = std::min(lo_a, (uintptr_t)src);
            hi_a = std::max(hi_a, (uintptr_t)src + n * row_bytes);
        }
        ia3_mixed = hi_a > lo_a && hi_a - lo_a <= ((uint64_t)1 << 32) - 65536;
        if (ia3_mixed) g_base = (const void*)lo_a;
        plan_chunks(b, kSkinnyRows, ia3_mixed ? (int)SYMB_ADAPTER_IA3 : -1, all_chunks);
    }
    const std::vector<SegDesc> sd = make_segdesc(b);
    unsigned char* wsb = (unsigned char*)ws;
    // Input-major weight: the input gradient is the K-contiguous GEMM (W rows are d_out long),
    // whose LoRA steps read the adapter side as [d_in][rank] rows: A_i^T, packed into the workspace.
    const bool conv1d = b->weight_layout == SYMB_WEIGHT_CONV1D;
    std::vector<SegDesc> sd_gemm = sd;
    DeltaPlan& delta = plan.terms;
    const size_t de_off = terms_offset(wl, plan);
    std::vector<int64_t> pk_off(bi.S, 0), pa_off(bi.S, 0);
    {
        int64_t cur = 0, cura = 0;
        for (int i = 0; i < bi.S; ++i)
            if (sd[i].kind == KIND_LORA) {
                pk_off[i] = cur;
                cur += (int64_t)sd[i].rpad * b->d_out;
                if (conv1d && lora) {
                    pa_off[i] = cura;
                    sd_gemm[i].B = (const bf16*)(wsb + wl.pa_off) + cura;
                    cura += (int64_t)align_up((size_t)sd[i].rank * b->d_in, 8);
                }
            }
    }
    Blob blob;
    const size_t o_seg = blob.add(sd.data(), sd.size());
    const size_t o_off = blob.add(b->seg_offsets, (size_t)bi.S + 1);
    const size_t o_lo = blob.add(lo.data(), lo.size());
    const size_t o_hi = blob.add(hi.data(), hi.size());
    const std::vector<int32_t> tile_epi = plan_tile_kind(b, lo, hi, SYMB_ADAPTER_IA3_IN);
    const size_t o_te = blob.add(tile_epi.data(), tile_epi.size());
    const size_t o_ch = blob.add(chunks.items.data(), chunks.items.size());
    const size_t o_all = blob.add(all_chunks.data(), all_chunks.size());
    const size_t o_pk = blob.add(pk_off.data(), pk_off.size());
    const size_t o_pa = blob.add(pa_off.data(), pa_off.size());
    const size_t o_gs = blob.add(dY_seg, seg_io ? (size_t)bi.S : 0);
    const size_t o_xs = blob.add(dX_seg, seg_io ? (size_t)bi.S : 0);
    const size_t o_mix = blob.add(mix.data(), ia3_mixed ? mix.size() : 0);
    std::vector<RowChunk> row_chunks;
    if (staged) plan_chunks(b, kSkinnyRows, -1, row_chunks);
    const size_t o_rows = blob.add(row_chunks.data(), row_chunks.size());
    const size_t o_sk = blob.add(sk_chunks.data(), sk_chunks.size());
    const std::vector<int32_t> k_zero(k_split ? plan.split.slots : 0, 0);
    const size_t o_kc = blob.add(k_zero.data(), k_zero.size());   // arrival counters of the K-split tiles
    const DeltaBlob db = add_gemm_desc(blob, sd_gemm, delta, (int)lo.size(), bm);
    unsigned char* dev = nullptr;
    if ((st = upload(h, blob, s, &dev)) != SYMB_OK) return st;

    const bf16* a_op = (const bf16*)dY;
    bf16* dH = nullptr;
    if (lora && conv1d) {
        PackAtParams pa{(const SegDesc*)(dev + o_seg), (bf16*)(wsb + wl.pa_off), (const int64_t*)(dev + o_pa), b->d_in};
        hipLaunchKernelGGL(symb_pack_at_kernel, dim3((b->d_in + 255) / 256, bi.S), dim3(256), 0, s, pa);
        SYMB_HIP(h, hipGetLastError());
    }
    if (lora) dH = (bf16*)(wsb + wl.dh_off);
    if (lora && !take_dh) {
        SkinnyParams sp{};
        sp.L = (const bf16*)dY;
        sp.out = dH;
        sp.K = b->d_out;
        sp.out_pitch = 2 * bi.max_rpad;
        sp.chunks = (const RowChunk*)(dev + o_ch);
        sp.seg = (const SegDesc*)(dev + o_seg);
        if (seg_io) {
            sp.L_seg = (const bf16* const*)(dev + o_gs);
            sp.off = (const int32_t*)(dev + o_off);
        }
        if ((st = launch_skinny_dh(h, b, sp, (bf16*)(wsb + wl.pk_off), (const int64_t*)(dev + o_pk), chunks, bi.max_rpad, s)) != SYMB_OK) return st;
    }
    bool a_from_seg = seg_io;
    if (ia3) {
        a_from_seg = ia3_mixed;
        bf16* const copy = (bf16*)(wsb + wl.sc_off);
        ScaleParams sc{(const bf16*)dY, copy, b->d_out, (const RowChunk*)(dev + o_all), (const SegDesc*)(dev + o_seg),
                       KIND_IA3, seg_io ? (const bf16* const*)(dev + o_gs) : nullptr, (const int32_t*)(dev + o_off)};
        // (every IA3 segment of the batch may be empty: nothing to scale then)
        if ((st = launch_row_pass(h, symb_ia3_scale_rows_kernel, sc, sc.d_out, all_chunks.size(), s)) != SYMB_OK) return st;
        a_op = copy;
    }
    if (!sk_chunks.empty()) {
        const ShortKParams kp{(const bf16*)dY, (const bf16*)W, (bf16*)dX, dH, b->d_in, (int)sk_chunks.size(), 0, 0, (const RowChunk*)(dev + o_sk), (const SegDesc*)(dev + o_seg)};
        if ((st = launch_shortk(h, kp, b->d_out, gemm_flops(b, sd, b->d_in, b->d_out, lora), s)) != SYMB_OK) return st;
        guard.completed = true;
        return seal_slot(h);
    }
    if (!delta.items.empty() && (st = launch_delta(h, true, (const SegDesc*)(dev + o_seg), (const RowChunk*)(dev + db.items), (int)delta.items.size(), b->d_in,
                                                   dH, bi.max_rpad, (float*)(wsb + de_off), s)) != SYMB_OK) return st;
    GemmParams gp{};
    if (!delta.items.empty()) {
        gp.delta = (const float*)(wsb + de_off);
        gp.tile_delta = (const TileDelta*)(dev + db.tiles);
    }
    gp.Aop = a_op;
    gp.Bop = (const bf16*)W;
    gp.C = (bf16*)dX;
    gp.Cbase = (bf16*)dXbase;
    if (a_from_seg) {
        gp.Aop = nullptr;
        gp.a_seg = (const bf16* const*)(dev + (ia3_mixed ? o_mix : o_gs));
        gp.a_base = (const bf16*)g_base;
    }
    if (seg_io && !staged) gp.c_seg = (bf16* const*)(dev + o_xs);
    if (staged) gp.C = (bf16*)(wsb + wl.so_off);
    gp.M = bi.T;
    gp.N = b->d_in;
    gp.K = b->d_out;
    gp.off = (const int32_t*)(dev + o_off);
    gp.seg = (const SegDesc*)(dev + db.seg);
    gp.tile_seg_lo = (const int32_t*)(dev + o_lo);
    gp.tile_seg_hi = (const int32_t*)(dev + o_hi);
    gp.ext = dH;
    gp.ext_pitch = 2 * bi.max_rpad;
    gp.epi_ia3 = (full && bi.n_ia3in > 0) ? KIND_IA3_IN : 0;      // dX rows of IA3_IN segments: l_i * (dY W)
    gp.tile_epi = (const int32_t*)(dev + o_te);
    gp.timing_flops = gemm_flops(b, sd_gemm, b->d_in, b->d_out, lora);
    gp.variant = plan.variant;
    gp.group_m = gemm_group_m((bi.T + bm - 1) / bm, (b->d_in + bn - 1) / bn, lo, hi);
    if (k_split) {
        gp.k_parts = plan.split.parts;
        gp.k_whole = plan.split.whole;
        gp.partial = (float*)(wsb + wl.tp_off);
        gp.k_count = (int*)(dev + o_kc);
    }
    // W [d_out][d_in] is the [K][N] operand of dX = dY W; W [d_in][d_out] gives K-contiguous rows.
    st = conv1d ? launch_gemm<false>(h, gp, s) : launch_gemm<true>(h, gp, s);
    if (st != SYMB_OK) return st;
    if (staged) {
        ScatterParams sc{(const bf16*)(wsb + wl.so_off), b->d_in, (const RowChunk*)(dev + o_rows), (bf16* const*)(dev + o_xs),
                         (const int32_t*)(dev + o_off)};
        hipLaunchKernelGGL(symb_scatter_rows_kernel, dim3((unsigned)row_chunks.size()), dim3(256), 0, s, sc);
        SYMB_HIP(h, hipGetLastError());
    }
    { guard.completed = true; return seal_slot(h); }
}

// ---------------------------------------------------------------------------------------------
static symb_status adapter_grad_impl(symb_handle h, const symb_batch* b, const void* X, const void* dY, const void* Ybase,
                                     const void* dXbase, uint32_t flags, void* ws, size_t ws_bytes, void* stream,
                                     const void* const* X_seg, const void* const* dY_seg, const void* const* Ybase_seg);

symb_status symb_adapter_grad(symb_handle h, const symb_batch* b, const void* X, const void* dY, const void* Ybase,
                              uint32_t flags, void* ws, size_t ws_bytes, void* stream) {
    return adapter_grad_impl(h, b, X, dY, Ybase, nullptr, flags, ws, ws_bytes, stream, nullptr, nullptr, nullptr);
}

symb_status symb_adapter_grad_ex(symb_handle h, const symb_batch* b, const void* X, const void* dY, const void* Ybase,
                                 const void* dXbase, uint32_t flags, void* ws, size_t ws_bytes, void* stream) {
    return adapter_grad_impl(h, b, X, dY, Ybase, dXbase, flags, ws, ws_bytes, stream, nullptr, nullptr, nullptr);
}

symb_status symb_adapter_grad_seg(symb_handle h, const symb_batch* b, const void* const* X_seg, const void* const* dY_seg,
                                  const void* const* Ybase_seg, uint32_t flags, void* ws, size_t ws_bytes, void* stream) {
    symb_status st = check_handle(h);
    if (st != SYMB_OK) return st;
    if (!X_seg || !dY_seg) return fail(h, SYMB_ERR_INVALID_ARG, "X_seg and dY_seg are required");
    return adapter_grad_impl(h, b, nullptr, nullptr, nullptr, nullptr, flags, ws, ws_bytes, stream, X_seg, dY_seg, Ybase_seg);
}

static symb_status adapter_grad_impl(symb_handle h, const symb_batch* b, const void* X, const void* dY, const void* Ybase,
                                     const void* dXbase, uint32_t flags, void* ws, size_t ws_bytes, void* stream,
                                     const void* const* X_seg, const void* const* dY_seg, const void* const* Ybase_seg) {
    symb_status st = check_handle(h);
    if (st != SYMB_OK) return st;
    CallGuard guard(h);
    if ((st = validate(h, b)) != SYMB_OK) return st;
    if (flags & ~(uint32_t)(SYMB_GRAD_ACCUMULATE | SYMB_GRAD_REUSE_DH | SYMB_GRAD_REUSE_HS))
        return fail(h, SYMB_ERR_INVALID_ARG, "unknown gradient flag %u", flags);
    const bool reuse_dh = (flags & SYMB_GRAD_REUSE_DH) != 0, reuse_hs = (flags & SYMB_GRAD_REUSE_HS) != 0;
    const BatchInfo bi = inspect(b);
    const bool seg_io = X_seg != nullptr;
    if (seg_io) {
        if ((st = check_seg_ptrs(h, b, X_seg, (size_t)b->d_in * 2, "X", false, nullptr)) != SYMB_OK) return st;
        if ((st = check_seg_ptrs(h, b, dY_seg, (size_t)b->d_out * 2, "dY", false, nullptr)) != SYMB_OK) return st;
        if (Ybase_seg) {
            // what the client kept for dl: the pre-adapter output rows (IA3), the input gradient before the input scale (IA3_IN)
            for (int i = 0; i < bi.S; ++i) {
                const int k = b->adapters[i].kind;
                if ((k == SYMB_ADAPTER_IA3 || k == SYMB_ADAPTER_IA3_IN) && b->adapters[i].dA && b->seg_offsets[i + 1] > b->seg_offsets[i] &&
                    (!Ybase_seg[i] || misaligned16(Ybase_seg[i])))
                    return fail(h, SYMB_ERR_INVALID_ARG, "the saved rows of IA3 segment %d are null or misaligned", i);
            }
        }
    } else if (!X || !dY) {
        if (bi.T > 0) return fail(h, SYMB_ERR_INVALID_ARG, "X and dY are required");
    }
    if (misaligned16(X) || misaligned16(dY) || misaligned16(Ybase) || misaligned16(dXbase) || misaligned16(ws))
        return fail(h, SYMB_ERR_INVALID_ARG, "device pointers must be 16-byte aligned");
    const bool acc = (flags & SYMB_GRAD_ACCUMULATE) != 0;
    hipStream_t s = (hipStream_t)stream;

    // Which segments want which gradient.  Empty segments: zeros when overwriting, nothing otherwise.
    std::vector<int32_t> want_a, want_b, want_l, want_lin;
    std::vector<std::pair<float*, size_t>> zero_fill;
    int grad_max_rpad = 0;
    for (int i = 0; i < bi.S; ++i) {
        const symb_adapter& a = b->adapters[i];
        const bool empty = b->seg_offsets[i + 1] == b->seg_offsets[i];
        if (a.kind == SYMB_ADAPTER_LORA) {
            if (empty) {
                if (!acc && a.dA) zero_fill.emplace_back((float*)a.dA, (size_t)a.rank * b->d_in);
                if (!acc && a.dB) zero_fill.emplace_back((float*)a.dB, (size_t)a.rank * b->d_out);
                continue;
            }
            if (a.dA) want_a.push_back(i);
            if (a.dB) want_b.push_back(i);
            if (a.dA || a.dB) grad_max_rpad = std::max(grad_max_rpad, rpad_of(a.rank));
        } else if (a.kind == SYMB_ADAPTER_IA3 && a.dA) {
            if (empty) {
                if (!acc) zero_fill.emplace_back((float*)a.dA, (size_t)b->d_out);
                continue;
            }
            want_l.push_back(i);
        } else if (a.kind == SYMB_ADAPTER_IA3_IN && a.dA) {
            if (empty) {
                if (!acc) zero_fill.emplace_back((float*)a.dA, (size_t)b->d_in);
                continue;
            }
            want_lin.push_back(i);
        }
    }
    if (!want_lin.empty() && !(seg_io ? (const void*)Ybase_seg : dXbase))
        return fail(h, SYMB_ERR_INVALID_ARG, "an IA3_IN segment wants dl but dXbase (the input gradient before the input scale) is null");
    if (!want_l.empty() && !(seg_io ? (const void*)Ybase_seg : Ybase))
        return fail(h, SYMB_ERR_INVALID_ARG, "an IA3 segment wants dl but Ybase (the pre-adapter output) is null");
    for (auto* w : {&want_l, &want_lin})                 // longest first (launch_ia3_grad)
        sort_once(*w, [&](int x, int y) { return b->seg_offsets[x + 1] - b->seg_offsets[x] > b->seg_offsets[y + 1] - b->seg_offsets[y]; });
    const bool any_lora = !want_a.empty() || !want_b.empty();
    const WsLayout wl = ws_layout(b, bi, SYMB_OP_ADAPTER_GRAD, true, any_lora);
    if (wl.total > ws_bytes || (wl.total && !ws))
        return fail(h, SYMB_ERR_WORKSPACE_TOO_SMALL, "adapter_grad needs %zu workspace bytes, got %zu", wl.total, ws_bytes);
    // zeros of the empty segments: fill kernels, not memset nodes (safe under graph capture); enqueued
    // only once nothing before the launches can fail any more
    auto fill_zeros = [&]() -> symb_status {
        for (const auto& z : zero_fill) {
            hipLaunchKernelGGL(symb_fill_zero_kernel, dim3((unsigned)std::min<size_t>((z.second + 255) / 256, 1024)), dim3(256), 0, s, z.first, z.second);
            SYMB_HIP(h, hipGetLastError());
        }
        return SYMB_OK;
    };
    if (!any_lora && want_l.empty() && want_lin.empty()) return fill_zeros();

    const std::vector<SegDesc> sd = make_segdesc(b);
    std::vector<int64_t> pk_off(bi.S, 0);
    {
        int64_t cur = 0;
        for (int i = 0; i < bi.S; ++i)
            if (sd[i].kind == KIND_LORA) {
                pk_off[i] = cur;
                cur += (int64_t)sd[i].rpad * b->d_out;
            }
    }
    // Work items of the two gradient launches: whole segments, or the runs of long ones (see grad_runs).
    // Widest ranks (the longest walks) first.  Returns the widest rank (padded) if the items take the kernel that deals tokens out over the
    // wavefronts (grad_wave); 0, for the other one, also in a wide layer's dB.
    auto plan_items = [&](std::vector<int32_t> want, int ncols, bool of_b, std::vector<GradItem>& items, std::vector<GradReduceItem>& red) {
        const auto rpad = [&](int i) { return rpad_of(b->adapters[i].rank); };
        sort_once(want, [&](int x, int y) { return rpad(x) > rpad(y); });
        int64_t cur = 0;
        for (int i : want) {
            const int lo = b->seg_offsets[i], hi = b->seg_offsets[i + 1], runs = grad_runs(hi - lo);
            if (runs == 1) {
                items.push_back(GradItem{i, lo, hi, 1, 0});
                continue;
            }
            const int64_t n = (int64_t)b->adapters[i].rank * ncols;
            red.push_back(GradReduceItem{i, runs, cur});
            for (int q = 0; q < runs; ++q, cur += n)
                items.push_back(GradItem{i, lo + q * GRAD_SPLIT, std::min(hi, lo + (q + 1) * GRAD_SPLIT), 0, cur});
        }
        return want.empty() || (of_b && ncols >= GRAD_WIDE) || !grad_wave(b, items, ncols) ? 0 : rpad(want[0]);
    };
    std::vector<GradItem> it_a, it_b;
    std::vector<GradReduceItem> red_a, red_b;
    const int wave_rpad_b = plan_items(want_b, b->d_out, true, it_b, red_b), wave_rpad_a = plan_items(want_a, b->d_in, false, it_a, red_a);
    // One pass over dY for dB and dH: when both gradients are wanted of the same segments, dH has to be
    // computed here anyway, and the ranks fit one rank block.  The pass leaves dH in the workspace where an
    // input-gradient call with SYMB_BWD_REUSE_DH (same batch, same dY, same workspace) takes it.
    const bool one_pass = !reuse_dh && want_a == want_b && !want_b.empty() && bi.max_rpad == 16 && wl.dp_bytes;
    // Small calls: dH beside dB in one launch (at most one workgroup per CU).
    const int col_blocks = (b->d_out + GRAD_WAVE_CT - 1) / GRAD_WAVE_CT;
    long long pair_groups = (long long)col_blocks * (long long)it_b.size();
    for (int i : want_a) pair_groups += (b->seg_offsets[i + 1] - b->seg_offsets[i] + kSkinnyRows - 1) / kSkinnyRows;
    const bool pair = !one_pass && !reuse_dh && !want_b.empty() && !want_a.empty() && b->d_out < GRAD_WIDE && (wave_rpad_b > 0 || grad_max_rpad > 32) &&
                      grad_max_rpad <= GRAD_WAVE_RANK && h->opt_skinny_deep && reads_bt(b) && pair_groups <= 256;
    // Short segments: dA, dB and dH in one launch, every workgroup of dA with a dH of its own; as long as what each reads for it (a CU takes in
    // 64 bytes per clock: 512 KiB 4 us) is less than another launch and its chain, and all of them are one per CU.
    const int a_blocks = (b->d_in + GRAD_SHORT_CT - 1) / GRAD_SHORT_CT, b_blocks = (b->d_out + GRAD_SHORT_CT - 1) / GRAD_SHORT_CT;
    int longest = 0;
    for (int i : want_a) longest = std::max(longest, b->seg_offsets[i + 1] - b->seg_offsets[i]);
    const bool short_grads = !one_pass && !reuse_dh && !want_a.empty() && want_a == want_b && grad_max_rpad <= 16 && longest <= GRAD_SHORT_TOKENS && b->d_out < GRAD_WIDE &&
                             (longest + 16) * (long long)b->d_out * 2 <= 512 << 10 && (a_blocks + b_blocks) * (long long)want_a.size() <= 256 && h->opt_skinny_deep && reads_bt(b);
    // Row chunks of the LoRA segments that want a gradient (Hs for dB, dH for dA).
    SkinnyChunks ch_h, ch_dh;
    if (!reuse_hs) ch_h = plan_skinny(h, b, want_b, grad_max_rpad);
    if (short_grads) {
    } else if (one_pass || pair) {
        for (int i : want_a)
            for (int r = b->seg_offsets[i]; r < b->seg_offsets[i + 1]; r += kSkinnyRows)
                ch_dh.items.push_back(RowChunk{i, r, std::min(kSkinnyRows, b->seg_offsets[i + 1] - r), 0});
    } else if (!reuse_dh) ch_dh = plan_skinny(h, b, want_a, grad_max_rpad);
    Blob blob;
    const size_t o_seg = blob.add(sd.data(), sd.size());
    const size_t o_off = blob.add(b->seg_offsets, (size_t)bi.S + 1);
    const size_t o_ita = blob.add(it_a.data(), it_a.size());
    const size_t o_itb = blob.add(it_b.data(), it_b.size());
    const size_t o_rda = blob.add(red_a.data(), red_a.size());
    const size_t o_rdb = blob.add(red_b.data(), red_b.size());
    const size_t o_chh = blob.add(ch_h.items.data(), ch_h.items.size());
    const size_t o_chd = blob.add(ch_dh.items.data(), ch_dh.items.size());
    const size_t o_pk = blob.add(pk_off.data(), pk_off.size());
    const size_t o_wl = blob.add(want_l.data(), want_l.size());
    const size_t o_wli = blob.add(want_lin.data(), want_lin.size());
    const size_t o_xs = blob.add(X_seg, seg_io ? (size_t)bi.S : 0);
    const size_t o_gs = blob.add(dY_seg, seg_io ? (size_t)bi.S : 0);
    const size_t o_ys = blob.add(Ybase_seg, (seg_io && Ybase_seg) ? (size_t)bi.S : 0);
    unsigned char* dev = nullptr;
    if ((st = upload(h, blob, s, &dev)) != SYMB_OK) return st;
    if ((st = fill_zeros()) != SYMB_OK) return st;
    unsigned char* wsb = (unsigned char*)ws;
    const SegDesc* dseg = (const SegDesc*)(dev + o_seg);
    const int32_t* doff = (const int32_t*)(dev + o_off);

    auto run_skinny_h = [&]() -> symb_status {          // Hs = s X A^T of the segments that want dB
        SkinnyParams sp{};
        sp.L = (const bf16*)X;
        sp.out = (bf16*)(wsb + wl.h_off);
        sp.K = b->d_in;
        sp.out_pitch = 2 * bi.max_rpad;
        sp.chunks = (const RowChunk*)(dev + o_chh);
        sp.seg = dseg;
        sp.use_packed = 0;
        if (seg_io) {
            sp.L_seg = (const bf16* const*)(dev + o_xs);
            sp.off = doff;
        }
        return launch_skinny<false>(h, sp, ch_h, grad_max_rpad, s);
    };
    auto skinny_dh = [&]() {                            // dH = s dY B of the segments that want dA
        SkinnyParams sp{};
        sp.L = (const bf16*)dY;
        sp.out = (bf16*)(wsb + wl.dh_off);
        sp.K = b->d_out;
        sp.out_pitch = 2 * bi.max_rpad;
        sp.chunks = (const RowChunk*)(dev + o_chd);
        sp.seg = dseg;
        if (seg_io) {
            sp.L_seg = (const bf16* const*)(dev + o_gs);
            sp.off = doff;
        }
        return sp;
    };
    bool have_dh = reuse_dh;
    if (one_pass) {
        if (!reuse_hs && (st = run_skinny_h()) != SYMB_OK) return st;
        DhDbParams dp{(const bf16*)dY, (const bf16*)(wsb + wl.h_off), b->d_out, 2 * bi.max_rpad, doff, dseg, (const GradItem*)(dev + o_itb), acc ? 1 : 0,
                      seg_io ? (const bf16* const*)(dev + o_gs) : nullptr, (float*)(wsb + wl.gr_off), (float*)(wsb + wl.dp_off), bi.T};
        const int groups = dhdb_groups(b->d_out);
        hipLaunchKernelGGL(symb_lora_dhdb_kernel<kDhDbBlocks>, dim3(groups, (unsigned)it_b.size()), dim3(256), 0, s, dp);
        SYMB_HIP(h, hipGetLastError());
        if ((st = launch_grad_reduce(h, GradReduceParams{dseg, (const GradReduceItem*)(dev + o_rdb), (const float*)(wsb + wl.gr_off), b->d_out, 1, acc ? 1 : 0},
                                     (int)red_b.size(), s)) != SYMB_OK) return st;
        DhFinishParams fp{(const float*)(wsb + wl.dp_off), groups, bi.T, (bf16*)(wsb + wl.dh_off), 2 * bi.max_rpad,
                          (const RowChunk*)(dev + o_chd), dseg};
        hipLaunchKernelGGL(symb_dh_finish_kernel, dim3((unsigned)ch_dh.items.size()), dim3(128), 0, s, fp);
        SYMB_HIP(h, hipGetLastError());
        have_dh = true;
    } else if (short_grads) {
        if (!reuse_hs && (st = run_skinny_h()) != SYMB_OK) return st;
        const GradParams ga{(const bf16*)X, nullptr, b->d_in, 2 * bi.max_rpad, doff, dseg, (const GradItem*)(dev + o_ita), acc ? 1 : 0, seg_io ? (const bf16* const*)(dev + o_xs) : nullptr, nullptr};
        const GradParams gb{(const bf16*)dY, (const bf16*)(wsb + wl.h_off), b->d_out, 2 * bi.max_rpad, doff, dseg, (const GradItem*)(dev + o_itb), acc ? 1 : 0,
                            seg_io ? (const bf16* const*)(dev + o_gs) : nullptr, nullptr};
        const int a_groups = a_blocks * (int)it_a.size();
        hipLaunchKernelGGL(symb_lora_grad_short_kernel, dim3((unsigned)(a_groups + b_blocks * (int)it_b.size())), dim3(512), 0, s, skinny_dh(), ga, a_blocks, a_groups, gb, b_blocks);
        SYMB_HIP(h, hipGetLastError());
    } else if (!want_b.empty()) {       // dB_i = s_i * dY_i^T H_i  ==  dY_i^T Hs_i
        if (!reuse_hs && (st = run_skinny_h()) != SYMB_OK) return st;
        GradParams gp{(const bf16*)dY, (const bf16*)(wsb + wl.h_off), b->d_out, 2 * bi.max_rpad, doff, dseg,
                      (const GradItem*)(dev + o_itb), acc ? 1 : 0, seg_io ? (const bf16* const*)(dev + o_gs) : nullptr,
                      (float*)(wsb + wl.gr_off)};
        if (pair) {
            const dim3 grid((unsigned)pair_groups);
            const SkinnyParams sp = skinny_dh();
            auto launch = [&](auto kfn) { hipLaunchKernelGGL(kfn, grid, dim3(256), 0, s, sp, (int)ch_dh.items.size(), gp, col_blocks, wave_rpad_b > 0 ? 1 : 0); };
            if (grad_max_rpad <= 16) launch(symb_lora_grad_pair_kernel<1>);
            else if (grad_max_rpad <= 32) launch(symb_lora_grad_pair_kernel<2>);
            else launch(symb_lora_grad_pair_kernel<4>);
            SYMB_HIP(h, hipGetLastError());
            have_dh = true;
        } else if ((st = launch_grad<true>(h, gp, wave_rpad_b, (int)it_b.size(), grad_max_rpad, s)) != SYMB_OK) return st;
        if ((st = launch_grad_reduce(h, GradReduceParams{dseg, (const GradReduceItem*)(dev + o_rdb), (const float*)(wsb + wl.gr_off), b->d_out, 1, acc ? 1 : 0},
                                     (int)red_b.size(), s)) != SYMB_OK) return st;
    }
    if (!want_a.empty() && !short_grads) {       // dA_i = dH_i^T X_i
        if (!have_dh) {
            if ((st = launch_skinny_dh(h, b, skinny_dh(), (bf16*)(wsb + wl.pk_off), (const int64_t*)(dev + o_pk), ch_dh, grad_max_rpad, s)) != SYMB_OK) return st;
        }
        GradParams gp{(const bf16*)X, (const bf16*)(wsb + wl.dh_off), b->d_in, 2 * bi.max_rpad, doff, dseg,
                      (const GradItem*)(dev + o_ita), acc ? 1 : 0, seg_io ? (const bf16* const*)(dev + o_xs) : nullptr,
                      (float*)(wsb + wl.gr_off)};
        if ((st = launch_grad<false>(h, gp, wave_rpad_a, (int)it_a.size(), grad_max_rpad, s)) != SYMB_OK) return st;
        if ((st = launch_grad_reduce(h, GradReduceParams{dseg, (const GradReduceItem*)(dev + o_rda), (const float*)(wsb + wl.gr_off), b->d_in, 0, acc ? 1 : 0},
                                     (int)red_a.size(), s)) != SYMB_OK) return st;
    }
    if (!want_l.empty()) {
        Ia3GradParams ip{(const bf16*)dY, (const bf16*)Ybase, b->d_out, doff, dseg, (const int32_t*)(dev + o_wl), acc ? 1 : 0,
                         seg_io ? (const bf16* const*)(dev + o_gs) : nullptr, seg_io ? (const bf16* const*)(dev + o_ys) : nullptr};
        if ((st = launch_ia3_grad(h, b, ip, want_l, s)) != SYMB_OK) return st;
    }
    if (!want_lin.empty()) {     // dl_i[k] = sum_t X[t][k] * (dY W)[t][k]: the same reduction over the input width
        Ia3GradParams ip{(const bf16*)X, (const bf16*)dXbase, b->d_in, doff, dseg, (const int32_t*)(dev + o_wli), acc ? 1 : 0,
                         seg_io ? (const bf16* const*)(dev + o_xs) : nullptr, seg_io ? (const bf16* const*)(dev + o_ys) : nullptr};
        if ((st = launch_ia3_grad(h, b, ip, want_lin, s)) != SYMB_OK) return st;
    }
    { guard.completed = true; return seal_slot(h); }
}

}  // extern "C"
