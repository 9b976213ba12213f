// Calls of at most 64 rows (decode steps of inference clients, short fine-tuning segments; Sec. 3.6 / 3.7: such
// requests interleave with the large ones layer by layer).  A tiled GEMM launches too few workgroups for so few rows
// to stream the weight at HBM speed, and the adapters of many short segments are a chain of small steps there, so
// these calls take two kernels of their own, in every call form:
//
//   symb_small_stream_kernel   reads the weight and all adapter matrices of the shrink side (forward A_i, backward
//                              B_i) exactly once, side by side in one grid, over K ranges, and leaves fp32 partial sums
//                                C0[range][t][n] = sum_{k in range} X[t][k] Wop(n, k)
//                                H [range][t][p] = sum_{k in range} X[t][k] A_i[p][k]      (rows t of segment i)
//   symb_small_finish_kernel   adds the ranges up in order and finishes every (row, column): bias, pre-adapter
//                              output, the row's own adapter (H stays fp32 here), noise effect, one rounding to bf16;
//                              it also leaves H in the workspace as value + residual, as the skinny kernel does, for
//                              a gradient call that takes it from there.
//
// A call without a LoRA term whose tiles need no K ranges is finished by the first kernel alone, or, on a K-contiguous weight of at most 8192
// columns and 10 M elements, by symb_small_narrow_kernel, whose tiles are narrower.  Which of these calls stay in the tiled kernels: small_wins.
//
// Bound by HBM: 2 K N bytes of weight plus 2 r (K + N) of each LoRA client.  What these calls spent their time on
// before was one launch after the other (shrink, weight, for the input gradient also a transposed copy of B_i),
// each a chain of memory latencies on a part of the chip, and from 17 rows on, in the tiled kernel, a chain of small steps for each
// client's adapter.  Measured per call, in the tiled kernels / now: one client on 4096 x 4096 21.6 / 11.3 us (8.3 us the first kernel, 4.1 TB/s; 3.7 the
// second), 16 mixed clients on 4096 -> 11008 69.0 / 26.1, 48 clients of ranks to 128 on 11008 -> 4096 134.9 / 38.0 (of the difference 2.8 us are the event that every call ended with; the figures
// in the rules below have it on both sides).
#pragma once
#include "adapter_kernels.hpp"
#include "gemm16_kernel.hpp"

namespace symb {

constexpr int SMALL_MAX_ROWS = 64;
constexpr int small_cols(bool nn) { return nn ? 128 : 64; }     // columns of a tile of the base product (weight read N-contiguous, K-contiguous)

constexpr int SMALL_NARROW_COLS = 32;    // ... of symb_small_narrow_kernel

// The segment of each row and the row's index inside it, carried in the launch arguments (a search on the device is a chain
// of dependent loads).
struct SmallRows {
    uint32_t at[SMALL_MAX_ROWS];          // segment << 8 | row inside it
};
// A piece of shrink work: ranks [p0, p0 + 16) (weight read K-contiguous) or all ranks (N-contiguous) of segment seg.
struct SmallItem {
    int32_t seg, p0, row0, nrows;
};

// Where finished rows go and what is done to them besides the LoRA term.
struct SmallOut {
    bf16* C;                  // [T][N], or null with c_seg
    bf16* Cbase;              // [T][N] or null: the value (+ bias) before the adapter term
    bf16* const* c_seg;       // device [S] or null: row t of segment i goes to c_seg[i] + (row inside i) * N
    const bf16* bias;         // [N] or null
    const NoiseDesc* neff;    // device [S] or null: noise effect, subtracted last
    int scale_kind;           // rows of this kind are scaled by their vector (0: none)
};

struct SmallStreamParams {
    const bf16* W;            // [N][K], or [K][N] (BASE_NN)
    const bf16* X;            // [T][K]
    const bf16* const* x_seg; // device [S] or null: rows of segment i start at x_seg[i]
    int N, K, T;
    int tiles, ranges;        // column tiles of the base product, K ranges
    float* partial;           // [ranges][T][N]
    const SmallItem* items;   // device: shrink work (may be empty)
    int num_items, h_ranges;
    const SegDesc* seg;
    float* h_partial;         // [h_ranges][T][h_pitch]
    int h_pitch;
    int direct;               // no LoRA term and one range: the tiles are finished here, no partial sums
    SmallOut out;
    SmallRows rows;
};

// Row t of the activations.
__device__ __forceinline__ const bf16* small_row(const SmallStreamParams& p, int t) {
    const uint32_t at = p.rows.at[t];
    return p.x_seg ? p.x_seg[at >> 8] + (size_t)(at & 255) * p.K : p.X + (size_t)t * p.K;
}

// ---- 16 CB columns of the product against 16 MB activation rows, in slices of the K range.  The wavefronts take every
// fourth slice and bring operand and activation rows in by LDS DMA into NBUF buffers of their own: no workgroup barrier in the
// loop, and NBUF slices per wavefront are in flight from the start.
//   NN = false: the operand is K-contiguous, a slice is 16 CB rows of 64 k (128-byte lines); chunk c (16 bytes) of row r lies at c ^ (r / 2) % 8.
//   NN = true (CB = 8): N-contiguous, a slice is 32 k-rows of 128 columns, read back through the transposing LDS read; a 16-lane
//   group of that read fetches 4 k-rows x 32 bytes, so the pairs of chunks of row k are stored at pair ^ f(k), f(k) = bits 3, 1 and 0
//   of k: the 32 lanes the LDS serves at a time then meet all banks once.  (64 k-rows of 64 columns, the
//   same bytes in 128-byte pieces, stream 4096 -> 24576 in 47 us where these take 41.5, 4.9 TB/s.)
// Activation rows: a slice's 64 (32) k of 16 rows are 2 (1) KiB, chunk c of row r at c ^ (r / 2) % 8 (c ^ (r / 4) % 4).
template <int CB, int MB, int NBUF_, bool NN>
struct SmallTile {
    static constexpr int SK = NN ? 32 : 64, NBUF = NBUF_;
    static constexpr int WREQ = NN ? 8 : 2 * CB, XREQ = MB * SK / 32, REQ = WREQ + XREQ;     // DMA requests of 1 KiB
    static constexpr int SLICE = REQ * 1024, WAVE = NBUF * SLICE, BYTES = 4 * WAVE;
    static_assert(4 * CB * MB * 1024 <= BYTES, "the partial sums of the wavefronts fit the slice buffers");
};
// Buffers of a base tile, and of a piece of shrink work (little per slice, so more of them).  ONE: a single buffer, for long N-contiguous strips of at most
// 16 rows with about one workgroup per CU: there fewer requests in flight stream faster (one row, us with 2 buffers / 1: 8192 -> 28672 84.5 / 79.3,
// 28672 -> 8192 91.3 / 81.9, 4096 -> 16384 30.7 / 29.7), while short strips need both (4608 -> 2048 12.2 / 13.0).
constexpr int small_base_nbuf(int mb, bool nn, bool one = false) { return one ? 1 : nn && mb == 4 ? 3 : 2; }
constexpr int small_shrink_nbuf(int mb) { return mb == 1 ? 4 : 2; }
__device__ __forceinline__ int small_nn_swz(int k) { return (((k >> 3) & 1) << 2) | (k & 3); }

// The wavefronts' sums meet in LDS; block b is added up in wavefront order and stored by wavefront b % 4.  beside(at): what else a wavefront leaves there, behind the sums.
struct NothingBeside {
    __device__ __forceinline__ void operator()(floatx4*) const {}
};
template <int CB, int MB, class STORE, class BESIDE = NothingBeside>
__device__ __forceinline__ void small_sum(const floatx4 (&acc)[CB][MB], unsigned char* smem, STORE&& store, BESIDE&& beside = {}) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    floatx4* const red = reinterpret_cast<floatx4*>(smem);
    __syncthreads();                                     // every wavefront is done with what it had in LDS
#pragma unroll
    for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int m = 0; m < MB; ++m) red[((wave * CB + c) * MB + m) * 64 + lane] = acc[c][m];
    beside(red + 4 * CB * MB * 64);
    __syncthreads();
#pragma unroll
    for (int b = 0; b < CB * MB; ++b) {
        if ((b & 3) != wave) continue;
        const int c = b / MB, m = b % MB;
        floatx4 v = red[b * 64 + lane];
#pragma unroll
        for (int w = 1; w < 4; ++w) v += red[(w * CB * MB + b) * 64 + lane];
        store(m * 16 + (lane & 15), c * 16 + ((lane >> 4) << 2), v);        // C[t][n .. n + 3]
    }
}
// ... to rows row0 .. of partial sums.
template <int CB, int MB>
__device__ __forceinline__ void small_store(const floatx4 (&acc)[CB][MB], unsigned char* smem, int row0, int nrows, float* out, int out_pitch, int out_cols) {
    small_sum<CB, MB>(acc, smem, [&](int t, int n, const floatx4& v) __attribute__((always_inline)) {
        if (t < nrows && n < out_cols) *reinterpret_cast<floatx4*>(out + (size_t)(row0 + t) * out_pitch + n) = v;
    });
}

// The accumulators of a tile over slices [KF range / ranges, ..).  w: the operand's first row (column, NN) of the tile; ld: its row
// pitch; wvalid: its valid rows (columns, NN).
// xrow(t): row t of the activations; meanwhile(acc): adds to the zeroed accumulators while the first slices are on their way.
template <int CB, int MB, int NBUF, bool NN, class XROW, class MEANWHILE>
__device__ __forceinline__ void small_tile_of(int K, XROW&& xrow, const bf16* w, int ld, int wvalid, int row0, int nrows, int range,
                                              int ranges, unsigned char* smem, floatx4 (&acc)[CB][MB], MEANWHILE&& meanwhile) {
    static_assert(!NN || CB == 8, "an N-contiguous tile is 128 columns wide");
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    using ST = SmallTile<CB, MB, NBUF, NN>;
    constexpr int NH = ST::SK / 32;                      // 32-k steps per slice
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l15 = lane & 15, kq = lane >> 4;
    unsigned char* const wbuf = smem + wave * ST::WAVE;
    // this lane's 16 bytes of every DMA request of a slice, at k = 0; what lies past the last valid row or column repeats it
    const bf16* src[ST::REQ];
    const size_t wstep = NN ? (size_t)ld : 1;            // operand elements from one k to the next
#pragma unroll
    for (int i = 0; i < ST::WREQ; ++i) {
        if constexpr (NN) {                              // 4 k-rows of 256 bytes
            const int k = i * 4 + (lane >> 4), slot = lane & 15;
            src[i] = w + (size_t)k * ld + min(((((slot >> 1) ^ small_nn_swz(k)) << 1) | (slot & 1)) * 8, wvalid - 8);
        } else {                                         // 8 rows of 128 bytes
            const int r = i * 8 + (lane >> 3);
            src[i] = w + (size_t)min(r, wvalid - 1) * ld + (((lane & 7) ^ ((r >> 1) & 7)) * 8);
        }
    }
#pragma unroll
    for (int i = 0; i < ST::XREQ; ++i) {
        const int r = NN ? i * 16 + (lane >> 2) : i * 8 + (lane >> 3);
        src[ST::WREQ + i] = xrow(row0 + min(r, nrows - 1)) + (NN ? (lane & 3) ^ ((r >> 2) & 3) : (lane & 7) ^ ((r >> 1) & 7)) * 8;
    }
    unsigned woff[CB][NH], xoff[MB][NH];                 // fragment of block b, 32-k step h
#pragma unroll
    for (int h = 0; h < NH; ++h) {
#pragma unroll
        for (int b = 0; b < CB; ++b) {
            if constexpr (NN) {
                const int k = kq * 8 + (l15 >> 2);       // first of the two transposing reads; the second is 4 k-rows further (same f)
                woff[b][h] = (unsigned)(size_t)wbuf + (unsigned)(k * 256 + ((b ^ small_nn_swz(k)) * 32) + (l15 & 3) * 8);
            } else {
                woff[b][h] = (unsigned)(size_t)wbuf + (unsigned)((b * 16 + l15) * 128 + (((h * 4 + kq) ^ ((l15 >> 1) & 7)) * 16));
            }
        }
#pragma unroll
        for (int b = 0; b < MB; ++b)
            xoff[b][h] = (unsigned)(size_t)wbuf + (unsigned)(ST::WREQ * 1024 + (b * 16 + l15) * (ST::SK * 2) +
                                                             (NN ? kq ^ ((l15 >> 2) & 3) : (h * 4 + kq) ^ ((l15 >> 1) & 7)) * 16);
    }
#pragma unroll
    for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int m = 0; m < MB; ++m) acc[c][m] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto dma = [&](int buf, int k) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < ST::REQ; ++i)
            __builtin_amdgcn_global_load_lds((glb_void_t*)(src[i] + (i < ST::WREQ ? (size_t)k * wstep : (size_t)k)),
                                             (lds_void_t*)(wbuf + buf * ST::SLICE + i * 1024), 16, 0, 0);
    };
    // fragment reads with a wait of their own (see the skinny kernel); returns with the buffer free again
    auto mul = [&](int buf) __attribute__((always_inline)) {
        u32x4 wv[NN ? 1 : CB][NH], xv[MB][NH];
        u32x2 wt[NN ? CB : 1][2];
        const unsigned at = (unsigned)(buf * ST::SLICE);
#pragma unroll
        for (int h = 0; h < NH; ++h) {
#pragma unroll
            for (int b = 0; b < CB; ++b) {
                if constexpr (NN) {
                    asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(wt[b][0]) : "v"(woff[b][h] + at));
                    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:1024" : "=v"(wt[b][1]) : "v"(woff[b][h] + at));
                } else {
                    asm volatile("ds_read_b128 %0, %1" : "=v"(wv[b][h]) : "v"(woff[b][h] + at));
                }
            }
#pragma unroll
            for (int b = 0; b < MB; ++b) asm volatile("ds_read_b128 %0, %1" : "=v"(xv[b][h]) : "v"(xoff[b][h] + at));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
#pragma unroll
        for (int h = 0; h < NH; ++h) {
#pragma unroll
            for (int b = 0; b < CB; ++b) {
                if constexpr (NN) { asm volatile("" : "+v"(wt[b][0])); asm volatile("" : "+v"(wt[b][1])); }
                else asm volatile("" : "+v"(wv[b][h]));
            }
#pragma unroll
            for (int b = 0; b < MB; ++b) asm volatile("" : "+v"(xv[b][h]));
        }
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                u32x4 f;
                if constexpr (NN) f = __builtin_shufflevector(wt[c][0], wt[c][1], 0, 1, 2, 3);
                else f = wv[c][h];
#pragma unroll
                for (int m = 0; m < MB; ++m)
                    acc[c][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f), __builtin_bit_cast(bf16x8, xv[m][h]), acc[c][m], 0, 0, 0);
            }
    };
    const int KF = K / ST::SK;                           // full slices; the range's own: [lo, hi)
    const int lo = KF * range / ranges, hi = KF * (range + 1) / ranges;
    const int ns = hi - lo > wave ? (hi - lo - wave + 3) >> 2 : 0;
    int k = (lo + wave) * ST::SK;                        // the next slice to request
    for (int d = 0; d < min(ns, NBUF); ++d, k += 4 * ST::SK) dma(d, k);
    meanwhile(acc);
    int buf = 0, s = 0;
    for (; s + NBUF <= ns; ++s) {                        // NBUF slices requested and not yet used: all but the oldest may stay in flight
        asm volatile("s_waitcnt vmcnt(%0)" : : "n"((NBUF - 1) * ST::REQ) : "memory");
        mul(buf);
        if (s + NBUF < ns) { dma(buf, k); k += 4 * ST::SK; }
        buf = buf + 1 == NBUF ? 0 : buf + 1;
    }
    if (s < ns) {
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        for (; s < ns; ++s) {
            mul(buf);
            buf = buf + 1 == NBUF ? 0 : buf + 1;
        }
    }
    // the part of K past the last full slice: masked fragments straight from global memory, one wavefront of the last range
    if (K % ST::SK && range == ranges - 1 && wave == 3) {
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const int kk = KF * ST::SK + h * 32 + kq * 8;
            const bool ok = kk < K;
            u32x4 xv[MB];
#pragma unroll
            for (int m = 0; m < MB; ++m) xv[m] = ok ? ld_glb16(xrow(row0 + min(m * 16 + l15, nrows - 1)) + kk) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                u32x4 f = u32x4{0u, 0u, 0u, 0u};
                if (ok) {
                    if constexpr (NN) {
                        const unsigned short* const e = reinterpret_cast<const unsigned short*>(w) + (size_t)kk * ld + min(c * 16 + l15, wvalid - 1);
#pragma unroll
                        for (int q = 0; q < 4; ++q) f[q] = e[(size_t)(2 * q) * ld] | ((unsigned)e[(size_t)(2 * q + 1) * ld] << 16);
                    } else {
                        f = ld_glb16(w + (size_t)min(c * 16 + l15, wvalid - 1) * ld + kk);
                    }
                }
#pragma unroll
                for (int m = 0; m < MB; ++m)
                    acc[c][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f), __builtin_bit_cast(bf16x8, xv[m]), acc[c][m], 0, 0, 0);
            }
        }
    }
}

template <int CB, int MB, int NBUF, bool NN>
__device__ __forceinline__ void small_tile(const SmallStreamParams& p, const bf16* w, int ld, int wvalid, int row0, int nrows, int range,
                                           int ranges, unsigned char* smem, floatx4 (&acc)[CB][MB]) {
    small_tile_of<CB, MB, NBUF, NN>(p.K, [&](int t) __attribute__((always_inline)) { return small_row(p, t); }, w, ld, wvalid, row0, nrows, range, ranges, smem, acc,
                                    [](floatx4 (&)[CB][MB]) {});
}

// ---- shrink against an adapter matrix stored [K][r] (B_i in the input gradient): all r columns against 16 MB activation rows.  64 k of
// it are one contiguous run of 128 r bytes, which a wavefront brings in by LDS DMA as it lies, with its 64-k slice of the
// activation rows, as many slices at once as its share of the LDS holds; fragments come back through the transposing LDS read
// (columns past r hold the next rows' bytes: their results are never read).  Needs 16-byte alignment and r a multiple of 4
// (8-byte aligned rows in LDS); NB = rank blocks of 16 in use at most.
template <int NB, int MB>
__device__ __forceinline__ void small_bt(const SmallStreamParams& p, const bf16* w, int r, int row0, int nrows, int range, int ranges,
                                         unsigned char* smem, int smem_bytes, float* out, int out_pitch) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l15 = lane & 15, kq = lane >> 4, K = p.K;
    const int nreq = (r + 7) >> 3, xat = nreq * 1024, slice = xat + MB * 2048, nb = (r + 15) >> 4;
    const int share = (smem_bytes / 4) & ~1023, nbuf = share / slice;
    unsigned char* const wbuf = smem + wave * share;
    const bf16* xsrc[2 * MB];
#pragma unroll
    for (int i = 0; i < 2 * MB; ++i) {
        const int t = i * 8 + (lane >> 3);
        xsrc[i] = small_row(p, row0 + min(t, nrows - 1)) + (((lane & 7) ^ ((t >> 1) & 7)) * 8);
    }
    unsigned woff[2], xoff[MB][2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        woff[h] = (unsigned)(size_t)wbuf + (unsigned)((h * 32 + kq * 8 + (l15 >> 2)) * r * 2 + (l15 & 3) * 8);
#pragma unroll
        for (int b = 0; b < MB; ++b) xoff[b][h] = (unsigned)(size_t)wbuf + (unsigned)(xat + (b * 16 + l15) * 128 + (((h * 4 + kq) ^ ((l15 >> 1) & 7)) * 16));
    }
    floatx4 acc[NB][MB];
#pragma unroll
    for (int c = 0; c < NB; ++c)
#pragma unroll
        for (int m = 0; m < MB; ++m) acc[c][m] = floatx4{0.f, 0.f, 0.f, 0.f};
    const int KF = K >> 6, lo = KF * range / ranges, hi = KF * (range + 1) / ranges;
    for (int s0 = lo + wave; s0 < hi; s0 += 4 * nbuf) {
        for (int d = 0; d < nbuf && s0 + 4 * d < hi; ++d) {
            const int k = (s0 + 4 * d) << 6;
            const unsigned char* const run = reinterpret_cast<const unsigned char*>(w + (size_t)k * r);
            for (int i = 0; i < nreq; ++i)
                __builtin_amdgcn_global_load_lds((glb_void_t*)(run + min(i * 1024 + lane * 16, 128 * r - 16)), (lds_void_t*)(wbuf + d * slice + i * 1024), 16, 0, 0);
#pragma unroll
            for (int i = 0; i < 2 * MB; ++i)
                __builtin_amdgcn_global_load_lds((glb_void_t*)(xsrc[i] + k), (lds_void_t*)(wbuf + d * slice + xat + i * 1024), 16, 0, 0);
        }
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        for (int d = 0; d < nbuf && s0 + 4 * d < hi; ++d) {
            const unsigned at = (unsigned)(d * slice);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                u32x2 wt[NB][2];
                u32x4 xv[MB];
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    const unsigned o = woff[h] + at + (unsigned)(min(b, nb - 1) * 32);
                    asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(wt[b][0]) : "v"(o));
                    asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(wt[b][1]) : "v"(o + 8 * r));
                }
#pragma unroll
                for (int b = 0; b < MB; ++b) asm volatile("ds_read_b128 %0, %1" : "=v"(xv[b]) : "v"(xoff[b][h] + at));
                asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
#pragma unroll
                for (int b = 0; b < NB; ++b) { asm volatile("" : "+v"(wt[b][0])); asm volatile("" : "+v"(wt[b][1])); }
#pragma unroll
                for (int b = 0; b < MB; ++b) asm volatile("" : "+v"(xv[b]));
#pragma unroll
                for (int c = 0; c < NB; ++c) {
                    const u32x4 f = __builtin_shufflevector(wt[c][0], wt[c][1], 0, 1, 2, 3);
#pragma unroll
                    for (int m = 0; m < MB; ++m)
                        acc[c][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f), __builtin_bit_cast(bf16x8, xv[m]), acc[c][m], 0, 0, 0);
                }
            }
        }
    }
    if ((K & 63) && range == ranges - 1 && wave == 3) {                     // see small_tile
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int kk = (KF << 6) + h * 32 + kq * 8;
            const bool ok = kk < K;
            u32x4 xv[MB];
#pragma unroll
            for (int m = 0; m < MB; ++m) xv[m] = ok ? ld_glb16(small_row(p, row0 + min(m * 16 + l15, nrows - 1)) + kk) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int c = 0; c < NB; ++c) {
                u32x4 f = u32x4{0u, 0u, 0u, 0u};
                if (ok) {
                    const unsigned short* const e = reinterpret_cast<const unsigned short*>(w) + (size_t)kk * r + min(c * 16 + l15, r - 1);
#pragma unroll
                    for (int q = 0; q < 4; ++q) f[q] = e[(size_t)(2 * q) * r] | ((unsigned)e[(size_t)(2 * q + 1) * r] << 16);
                }
#pragma unroll
                for (int m = 0; m < MB; ++m)
                    acc[c][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f), __builtin_bit_cast(bf16x8, xv[m]), acc[c][m], 0, 0, 0);
            }
        }
    }
    small_store<NB, MB>(acc, smem, row0, nrows, out, out_pitch, nb * 16);
}

// ---- the same for any rank and alignment: element loads, no LDS staging.  Lane l15 of a fragment holds rank l15 of a block.
template <int MB>
__device__ __forceinline__ void small_bt_any(const SmallStreamParams& p, const bf16* w, int r, int row0, int nrows, int range, int ranges,
                                             unsigned char* smem, float* out, int out_pitch) {
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l15 = lane & 15, kq = lane >> 4, K = p.K;
    const int k32 = (K + 31) >> 5, lo = k32 * range / ranges, hi = k32 * (range + 1) / ranges;
    for (int p0 = 0; p0 < r; p0 += 16) {
        floatx4 acc[1][MB];
#pragma unroll
        for (int m = 0; m < MB; ++m) acc[0][m] = floatx4{0.f, 0.f, 0.f, 0.f};
        for (int s = lo + wave; s < hi; s += 4) {
            const int kk = s * 32 + kq * 8;
            const bool ok = kk < K;
            const unsigned short* const e = reinterpret_cast<const unsigned short*>(w) + (size_t)(ok ? kk : 0) * r + min(p0 + l15, r - 1);
            u32x4 f;
#pragma unroll
            for (int q = 0; q < 4; ++q) f[q] = e[(size_t)(2 * q) * r] | ((unsigned)e[(size_t)(2 * q + 1) * r] << 16);
            if (!ok) f = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                u32x4 xv = ld_glb16(small_row(p, row0 + min(m * 16 + l15, nrows - 1)) + (ok ? kk : 0));
                if (!ok) xv = u32x4{0u, 0u, 0u, 0u};
                acc[0][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f), __builtin_bit_cast(bf16x8, xv), acc[0][m], 0, 0, 0);
            }
        }
        small_store<1, MB>(acc, smem, row0, nrows, out + p0, out_pitch, 16);
    }
}

// Finishes four columns of row t without a LoRA term (the same steps as symb_small_finish_kernel).
__device__ __forceinline__ void small_direct(const SmallStreamParams& p, int t, int n, floatx4 v) {
    const uint32_t at = p.rows.at[t];
    auto quad = [&](const bf16* q) __attribute__((always_inline)) {
        const uint2 b = *reinterpret_cast<const uint2*>(q);
        return floatx4{bf16_bits_to_f32((unsigned short)(b.x & 0xffffu)), bf16_bits_to_f32((unsigned short)(b.x >> 16)),
                       bf16_bits_to_f32((unsigned short)(b.y & 0xffffu)), bf16_bits_to_f32((unsigned short)(b.y >> 16))};
    };
    auto put = [&](bf16* q) __attribute__((always_inline)) {
        *reinterpret_cast<uint2*>(q) = make_uint2(pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3]));
    };
    if (p.out.bias) v += quad(p.out.bias + n);
    if (p.out.Cbase) put(p.out.Cbase + (size_t)t * p.N + n);
    if (p.out.scale_kind) {
        const SegDesc sd = p.seg[at >> 8];
        if (sd.kind == p.out.scale_kind) v *= quad(sd.A + n);
    }
    if (p.out.neff) {
        const NoiseDesc nd = p.out.neff[at >> 8];
        if (nd.ptr) v -= quad(nd.ptr + (size_t)(nd.rows == 1 ? 0 : at & 255) * p.N + n);
    }
    put((p.out.c_seg ? p.out.c_seg[at >> 8] + (size_t)(at & 255) * p.N : p.out.C + (size_t)t * p.N) + n);
}

// grid = num_items * h_ranges + tiles * ranges workgroups.  MB: row blocks of 16 (T <= 16 MB).  BASE_NN / SHRINK_NN: the weight / the
// adapter matrix is read N-contiguous (forward: the weight of a Conv1D layer, never A_i; input gradient: the weight of an
// nn.Linear layer, always B_i).
template <int MB, bool BASE_NN, bool SHRINK_NN, bool ONE>
SYMB_KERNEL void __launch_bounds__(256)
symb_small_stream_kernel(const SmallStreamParams p) {
    static_assert(!ONE || (MB == 1 && BASE_NN), "one buffer: see small_base_nbuf");
    constexpr int CB = small_cols(BASE_NN) / 16, NB = small_base_nbuf(MB, BASE_NN, ONE), SNB1 = small_shrink_nbuf(1), SNB = small_shrink_nbuf(MB);
    constexpr int BASE_BYTES = SmallTile<CB, MB, NB, BASE_NN>::BYTES, ROWS16 = SmallTile<1, 1, SNB1, false>::BYTES, ALL = SmallTile<1, MB, SNB, false>::BYTES;
    // SHRINK_NN: one slice of rank 128 per wavefront at least, 16 KiB and the activation rows; the partial sums fit there too
    constexpr int SHRINK_BYTES = SHRINK_NN ? 4 * (16 + 2 * MB) * 1024 : ROWS16 > ALL ? ROWS16 : ALL;
    __shared__ __attribute__((aligned(16))) unsigned char smem[BASE_BYTES > SHRINK_BYTES ? BASE_BYTES : SHRINK_BYTES];
    const int nshrink = p.num_items * p.h_ranges;
    if ((int)blockIdx.x < nshrink) {
        const int item = blockIdx.x % p.num_items, range = blockIdx.x / p.num_items;
        const SmallItem it = p.items[item];
        const SegDesc sd = p.seg[it.seg];
        float* const out = p.h_partial + (size_t)range * p.T * p.h_pitch + it.p0;
        auto go = [&](auto MBC) __attribute__((always_inline)) {
            constexpr int MBI = decltype(MBC)::value;
            if constexpr (!SHRINK_NN) {
                floatx4 acc[1][MBI];
                small_tile<1, MBI, small_shrink_nbuf(MBI), false>(p, sd.A + (size_t)it.p0 * p.K, p.K, min(sd.rank - it.p0, 16), it.row0, it.nrows,
                                                                  range, p.h_ranges, smem, acc);
                small_store<1, MBI>(acc, smem, it.row0, it.nrows, out, p.h_pitch, 16);
            } else if ((sd.rank & 3) || ((size_t)sd.B & 15)) {
                small_bt_any<MBI>(p, sd.B, sd.rank, it.row0, it.nrows, range, p.h_ranges, smem, out, p.h_pitch);
            } else if (sd.rank <= 32) {
                small_bt<2, MBI>(p, sd.B, sd.rank, it.row0, it.nrows, range, p.h_ranges, smem, (int)sizeof smem, out, p.h_pitch);
            } else {
                small_bt<8, MBI>(p, sd.B, sd.rank, it.row0, it.nrows, range, p.h_ranges, smem, (int)sizeof smem, out, p.h_pitch);
            }
        };
        if (it.nrows <= 16) go(std::integral_constant<int, 1>{});
        else if constexpr (MB > 1) go(std::integral_constant<int, MB>{});
        return;
    }
    const int g = blockIdx.x - nshrink, tile = g % p.tiles, range = g / p.tiles, n0 = tile * small_cols(BASE_NN);
    floatx4 acc[CB][MB];
    small_tile<CB, MB, NB, BASE_NN>(p, p.W + (BASE_NN ? (size_t)n0 : (size_t)n0 * p.K), BASE_NN ? p.N : p.K, p.N - n0, 0, p.T, range, p.ranges, smem, acc);
    if (p.direct) {
        small_sum<CB, MB>(acc, smem, [&](int t, int n, const floatx4& v) __attribute__((always_inline)) {
            if (t < p.T && n0 + n < p.N) small_direct(p, t, n0 + n, v);
        });
    } else {
        small_store<CB, MB>(acc, smem, 0, p.T, p.partial + (size_t)range * p.T * p.N + n0, p.N, p.N - n0);
    }
}

// Calls without a LoRA term on a small layer whose weight is read K-contiguous: tiles of 32 columns over the whole inner dimension, finished
// here.  Such a call is one chain of latencies; half the columns per workgroup are twice the workgroups, with up to four slices in flight
// per wavefront.  One row, us with 64 columns / 32: 2048 x 2048 9.1 / 8.0, 3072 -> 768 10.3 / 8.5 (in K ranges), 4608 -> 2048 11.7 / 9.9, 1024 -> 8192 8.3 / 8.0,
// but 4096 x 4096 12.5 / 14.9 and 16 rows of 256 -> 11008 7.6 / 8.2; 64 rows of 2048 x 2048 14.3 / 11.1.  grid = tiles; ranges, items and partial sums of p are not used.
template <int MB>
SYMB_KERNEL void __launch_bounds__(256)
symb_small_narrow_kernel(const SmallStreamParams p) {
    constexpr int CB = SMALL_NARROW_COLS / 16, NBUF = MB == 4 ? 3 : 4;
    __shared__ __attribute__((aligned(16))) unsigned char smem[SmallTile<CB, MB, NBUF, false>::BYTES];
    const int n0 = blockIdx.x * SMALL_NARROW_COLS;
    floatx4 acc[CB][MB];
    small_tile<CB, MB, NBUF, false>(p, p.W + (size_t)n0 * p.K, p.K, p.N - n0, 0, p.T, 0, 1, smem, acc);
    small_sum<CB, MB>(acc, smem, [&](int t, int n, const floatx4& v) __attribute__((always_inline)) {
        if (t < p.T && n0 + n < p.N) small_direct(p, t, n0 + n, v);
    });
}

// ---- The tiled product of small layers: tiles of 32 rows and 64 (weight read K-contiguous) or 128 columns, the four wavefronts of a workgroup
// splitting K.  Such a launch is one chain of latencies (launch, first loads, K, epilogue); the 128x128 tile walks its K stages one behind the other and
// leaves the chip to a dozen workgroups.  Here up to 768 of K (the weight read N-contiguous: 512) are in flight at once, in the four wavefronts together, and the loads of the
// LoRA steps (H and the adapter straight from memory, dealt out over the wavefronts) go out behind them: their latency is hidden, their matrix instructions
// wait, as loads return in order, for the slices requested before.  256 rows of 768 x 768 with one rank-8 step
// per tile, us: K-contiguous 11.7 -> 6.9, N-contiguous 11.5 -> 8.9 (11.4 with the element loads of A_i under a condition).  gemm_plan has the rule.  No pre-adapter
// output, no terms computed beforehand.
constexpr int MID_ROWS = 32;
template <bool NN>
SYMB_KERNEL void __launch_bounds__(256)
symb_gemm_mid_kernel(const GemmParams p) {
    constexpr int MB = MID_ROWS / 16, CB = small_cols(NN) / 16, NBUF = NN ? 4 : 3;
    __shared__ __attribute__((aligned(16))) unsigned char smem[SmallTile<CB, MB, NBUF, NN>::BYTES];
    const int tm = blockIdx.x % p.num_m_tiles, tn = blockIdx.x / p.num_m_tiles, m0 = tm * MID_ROWS, n0 = tn * small_cols(NN);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l15 = lane & 15, kq = lane >> 4;
    const int seg_lo = p.tile_seg_lo[tm], seg_hi = p.tile_seg_hi[tm];
    auto xrow = [&](int m) __attribute__((always_inline)) -> const bf16* {
        if (!p.a_seg) return p.Aop + (size_t)m * p.K;
        const int s = seg_of_row(p.off, seg_lo, seg_hi, m);
        return p.a_seg[s] + (size_t)(m - p.off[s]) * p.K;
    };
    // LoRA steps, 32 of a segment's extended columns each, dealt out over the wavefronts so that a sum hangs on its own segment alone.  A segment of several goes by their number inside it.
    // Segments of one step go by their number inside the tile, up to two to a wavefront; their operands wait in registers until the wavefronts' sums meet, and their terms, formed
    // then, are added to the total, which does not depend on whose they were.  All by their number inside the segment, every one-step segment's first and only step is the first wavefront's, us: forward of 150 rows of
    // 1024 -> 1536 in six such clients 13.0 -> 11.4, the training step 38.0 -> 33.9, of 200 rows of 768 x 768 in eight of ranks 8 to 32 34.4 -> 32.7; tiles with one client each pay
    // for the second sum, 256 rows of 768 x 768 in four 25.4 -> 25.9.  (All by their number inside the tile, as fast, let a row's last bit hang on the tile's other segments.)
    int end = min(m0 + MID_ROWS, p.M);
    asm volatile("" : "+s"(end));                        // (a minimum of three is a vector instruction)
    struct Seg {
        const bf16* w;                                   // A_i [rank][N] (NN) or B_i [N][rank]
        int rank, rpad, lo, hi;                          // rows of the tile; rpad 0: no adapter, or no rows
    };
    auto segment = [&](int s) __attribute__((always_inline)) {       // (scalar loads, all at once: vector loads would be waited for with the slices requested before them)
        const __attribute__((address_space(4))) SegDesc* const sd = (const __attribute__((address_space(4))) SegDesc*)reinterpret_cast<const SegDesc*>(p.seg + s);
        const __attribute__((address_space(4))) int* const off = (const __attribute__((address_space(4))) int*)reinterpret_cast<const int*>(p.off + s);
        int kind = sd->kind, rank = sd->rank, rpad = sd->rpad, lo = off[0], hi = off[1];
        const bf16* w = NN ? sd->A : sd->B;
        asm volatile("" : "+s"(kind), "+s"(rank), "+s"(rpad), "+s"(lo), "+s"(hi), "+s"(w));
        lo = max(lo, m0);
        hi = min(hi, end);
        return Seg{w, rank, kind == KIND_LORA && hi > lo ? rpad : 0, lo, hi};
    };
    struct Operands { u32x4 x[MB], w[CB]; };
    // every load unconditional and in bounds, what does not belong to the step zeroed afterwards (under a condition each would be waited for)
    auto fetch = [&](const Seg& sd, int e, Operands& o) __attribute__((always_inline)) {
        const int rank = sd.rank, pk = e + kq * 8, pp = pk >= sd.rpad ? pk - sd.rpad : pk;         // both halves of the extended columns meet the same adapter matrix
#pragma unroll
        for (int m = 0; m < MB; ++m) o.x[m] = ld_glb16(p.ext + (size_t)min(max(m0 + m * 16 + l15, sd.lo), sd.hi - 1) * p.ext_pitch + pk);
        if (!NN && (rank & 7) == 0) {
#pragma unroll
            for (int c = 0; c < CB; ++c) o.w[c] = ld_glb16(sd.w + (size_t)min(n0 + c * 16 + l15, p.N - 1) * rank + min(pp, rank - 8));
        } else {                                         // A_i [rank][N] or B_i [N][rank], element by element
            const __attribute__((address_space(1))) unsigned short* const w = (const __attribute__((address_space(1))) unsigned short*)reinterpret_cast<const unsigned short*>(sd.w);
            unsigned el[CB][8];
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                const int n = min(n0 + c * 16 + l15, p.N - 1);
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int r = min(pp + q, rank - 1);
                    el[c][q] = w[NN ? (size_t)r * p.N + n : (size_t)n * rank + r];
                }
            }
#pragma unroll
            for (int c = 0; c < CB; ++c) {
                __builtin_amdgcn_sched_barrier(0);       // (every load before the first wait, then as they come)
#pragma unroll
                for (int q = 0; q < 8; ++q) el[c][q] = pp + q < rank ? el[c][q] : 0u;
                o.w[c] = u32x4{el[c][0] | el[c][1] << 16, el[c][2] | el[c][3] << 16, el[c][4] | el[c][5] << 16, el[c][6] | el[c][7] << 16};
            }
        }
#pragma unroll
        for (int c = 0; c < CB; ++c) o.w[c] = pp < rank ? o.w[c] : u32x4{0u, 0u, 0u, 0u};
    };
    unsigned singles = 0, mine[2] = {0, 0};              // rows of segments of one step, of this wavefront's
    Operands single[2];
    auto lora = [&](floatx4 (&acc)[CB][MB]) __attribute__((always_inline)) {
        if (!p.ext) return;
        int no = 0, several = seg_hi + 1;                // the first segment of several steps
        Seg own[2] = {}, sd_several = {};
        for (int s = seg_lo; s <= seg_hi; ++s) {
            const Seg sd = segment(s);
            if (!sd.rpad) continue;
            if (sd.rpad > 16 || no == 8) {
                if (several > seg_hi) { several = s; sd_several = sd; }
                continue;
            }
            singles |= (unsigned)((1ull << (sd.hi - m0)) - (1ull << (sd.lo - m0)));
            // (from the last wavefront down, as the others start with the first)
            if (no == 3 - wave) own[0] = sd;
            if (no == 7 - wave) own[1] = sd;
            ++no;
        }
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (own[k].rpad) {
                mine[k] = (unsigned)((1ull << (own[k].hi - m0)) - (1ull << (own[k].lo - m0)));
                fetch(own[k], 0, single[k]);
            }
        Seg sd = sd_several;
        for (int s = several; s <= seg_hi;) {
            const int lo = sd.lo, hi = sd.hi, steps = sd.rpad && !(singles >> (lo - m0) & 1) ? 2 * sd.rpad : 0;
            for (int e = wave * 32; e < steps; e += 128) {
                Operands o;
                fetch(sd, e, o);
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    const int t = m0 + m * 16 + l15;
                    asm volatile("" : "+v"(o.x[m]));     // (its load not under the condition below)
                    o.x[m] = t >= lo && t < hi ? o.x[m] : u32x4{0u, 0u, 0u, 0u};
                }
#pragma unroll
                for (int m = 0; m < MB; ++m) {
                    if (lo >= m0 + m * 16 + 16 || hi <= m0 + m * 16) continue;      // 16 rows of other segments
#pragma unroll
                    for (int c = 0; c < CB; ++c)
                        acc[c][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, o.w[c]), __builtin_bit_cast(bf16x8, o.x[m]), acc[c][m], 0, 0, 0);
                }
            }
            if (++s <= seg_hi) sd = segment(s);
        }
    };
    floatx4 acc[CB][MB];
    small_tile_of<CB, MB, NBUF, NN>(p.K, xrow, p.Bop + (NN ? (size_t)n0 : (size_t)n0 * p.K), NN ? p.N : p.K, p.N - n0, m0, min(MID_ROWS, p.M - m0), 0, 1, smem, acc, lora);
    const bool scale = p.epi_ia3 != 0 && p.tile_epi[tm] != 0;
    static_assert(5 * CB * MB * 1024 <= SmallTile<CB, MB, NBUF, NN>::BYTES, "the wavefronts' sums and the terms fit the slice buffers");
    const floatx4* const terms = reinterpret_cast<const floatx4*>(smem) + 4 * CB * MB * 64;
    small_sum<CB, MB>(acc, smem, [&](int r, int c, floatx4 v) __attribute__((always_inline)) {
        const int t = m0 + r, n = n0 + c;
        if (singles >> r & 1) v += terms[((c >> 4) * MB + (r >> 4)) * 64 + lane];
        if (t >= p.M || n >= p.N) return;
        auto quad = [&](const bf16* q) __attribute__((always_inline)) {
            const uint2 b = *reinterpret_cast<const uint2*>(q);
            return floatx4{bf16_bits_to_f32((unsigned short)(b.x & 0xffffu)), bf16_bits_to_f32((unsigned short)(b.x >> 16)),
                           bf16_bits_to_f32((unsigned short)(b.y & 0xffffu)), bf16_bits_to_f32((unsigned short)(b.y >> 16))};
        };
        bf16* out = p.C + (size_t)t * p.N;
        if (p.bias) v += quad(p.bias + n);
        if (scale || p.neff || p.c_seg) {
            const int s = seg_of_row(p.off, seg_lo, seg_hi, t);
            if (scale && p.seg[s].kind == p.epi_ia3) v *= quad(p.seg[s].A + n);
            if (p.neff && p.neff[s].ptr) v -= quad(p.neff[s].ptr + (size_t)(p.neff[s].rows == 1 ? 0 : t - p.off[s]) * p.N + n);
            if (p.c_seg) out = p.c_seg[s] + (size_t)(t - p.off[s]) * p.N;
        }
        *reinterpret_cast<uint2*>(out + n) = make_uint2(pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3]));
    }, [&](floatx4* at) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (!mine[k]) continue;
#pragma unroll
            for (int m = 0; m < MB; ++m) {
                if (!(mine[k] >> (m * 16) & 0xffffu)) continue;
#pragma unroll
                for (int c = 0; c < CB; ++c) {
                    const floatx4 v = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, single[k].w[c]), __builtin_bit_cast(bf16x8, single[k].x[m]), floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    if (mine[k] >> (m * 16 + l15) & 1) at[(c * MB + m) * 64 + lane] = v;
                }
            }
        }
    });
}

struct SmallFinishParams {
    const float* partial;     // [ranges][T][N]
    const float* h_partial;   // [h_ranges][T][h_pitch], or null: H comes from h_rows (value + residual, left there by an earlier call)
    int ranges, h_ranges, h_pitch;
    bf16* h_rows;             // [T][2 * h_pitch]: per row rpad values then rpad residuals of the row's own segment
    int lora_term;            // + H B_i[n][.] (forward) / + H A_i[.][n] (input gradient); 0: none in this batch, or base only
    SmallOut out;
    int N, T;
    const SegDesc* seg;
    SmallRows rows;
};
// What a workgroup (128 threads, 256 columns of one row) adds to its columns' sums v0, v1: the partial sums of the K ranges, bias, and
// the row's LoRA term.  The partial sums of the first eight ranges, the call's and H's, are requested before the row's descriptor is there (SmallFirst); what hangs on
// that one, the adapter matrix, goes out next; the workgroup reads it together, 16 bytes per lane and NCH chunks per thread, unconditionally.
// (A thread per column would read B_i in 64 lines per load and A_i two bytes at a time, a chain of dozens of
// loads at rank 128.)  NCH: 0 = no LoRA term; else 4, 8, 16, 32 for ranks to 16, 32, 64, 128; -1 = forward at a rank that is no multiple of 8.
struct SmallFirst {
    float2 c[8];
    float h[8];
};
template <bool BACKWARD, int NCH>
__device__ __forceinline__ void small_finish_sums(const SmallFinishParams& p, const SegDesc& sd, int t, int c0, const SmallFirst& first, float* hs, float* us, float& v0, float& v1) {
    constexpr int NC = NCH > 0 ? NCH : 1;
    const int tid = threadIdx.x, n = c0 + 2 * tid, nc = min(n, p.N - 2);
    // Forward: the 256 columns' rows of B_i are one contiguous run, L chunks per column, chunk number x = 128 i + tid.  Input gradient:
    // chunk i of a thread is 8 columns of rank row 4 i + tid / 32 of A_i.
    const int L = sd.rank >> 3, g = tid >> 5;
    const unsigned inv = NCH > 0 && !BACKWARD ? 65536u / (unsigned)L + 1u : 0u;       // x / L == x inv >> 16 for x < 4096, L <= 16
    auto col_of = [&](int x) __attribute__((always_inline)) { return (int)(((unsigned)x * inv) >> 16); };
    u32x4 bw[NC];
    if constexpr (NCH > 0) {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const int x = i * 128 + tid, c = col_of(x);
            bw[i] = BACKWARD ? ld_glb16(sd.A + (size_t)min(i * 4 + g, sd.rank - 1) * p.N + min(c0 + (tid & 31) * 8, p.N - 8))
                             : ld_glb16(sd.B + (size_t)min(c0 + c, p.N - 1) * sd.rank + (x - c * L) * 8);
        }
    }
    float hv = 0.f;
    unsigned short* const row = reinterpret_cast<unsigned short*>(p.h_rows) + (size_t)t * 2 * p.h_pitch;
    if constexpr (NCH != 0) {
        if (!p.h_partial) {
            if (tid < sd.rpad) hv = bf16_bits_to_f32(row[tid]) + bf16_bits_to_f32(row[sd.rpad + tid]);
        } else {
            const float* const src = p.h_partial + (size_t)t * p.h_pitch + min(tid, sd.rank - 1);
#pragma unroll
            for (int q = 0; q < 8; ++q) hv += q < p.h_ranges ? first.h[q] : 0.f;
            for (int r = 8; r < p.h_ranges; r += 8) {    // eight loads in flight, the ones past the last range discarded
                float a[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) a[q] = src[(size_t)min(r + q, p.h_ranges - 1) * p.T * p.h_pitch];
#pragma unroll
                for (int q = 0; q < 8; ++q) hv += r + q < p.h_ranges ? a[q] : 0.f;
            }
            hv = tid < sd.rank ? hv * sd.scale : 0.f;    // (past the rank h_partial holds anything)
        }
    }
    {
        const float* const src = p.partial + (size_t)t * p.N + nc;
        const size_t stride = (size_t)p.T * p.N;
#pragma unroll
        for (int q = 0; q < 8; ++q) { v0 += q < p.ranges ? first.c[q].x : 0.f; v1 += q < p.ranges ? first.c[q].y : 0.f; }
        for (int r = 8; r < p.ranges; r += 8) {
            float2 a[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) a[q] = *reinterpret_cast<const float2*>(src + (size_t)min(r + q, p.ranges - 1) * stride);
#pragma unroll
            for (int q = 0; q < 8; ++q) { v0 += r + q < p.ranges ? a[q].x : 0.f; v1 += r + q < p.ranges ? a[q].y : 0.f; }
        }
    }
    if (p.out.bias) {
        const unsigned b = *reinterpret_cast<const unsigned*>(p.out.bias + nc);
        v0 += bf16_bits_to_f32((unsigned short)(b & 0xffffu));
        v1 += bf16_bits_to_f32((unsigned short)(b >> 16));
    }
    if (p.out.Cbase && n < p.N) *reinterpret_cast<unsigned*>(p.out.Cbase + (size_t)t * p.N + n) = pack2_bf16(v0, v1);
    if constexpr (NCH == 0) return;
    if (p.h_partial && blockIdx.x == 0 && tid < sd.rpad) {
        const unsigned short hi = f32_to_bf16_bits(hv);
        row[tid] = hi;
        row[sd.rpad + tid] = f32_to_bf16_bits(hv - bf16_bits_to_f32(hi));
    }
    hs[tid] = hv;                                        // zero past the rank
    __syncthreads();
    float u0 = 0.f, u1 = 0.f;
    if constexpr (NCH < 0) {
        const unsigned short* const b = reinterpret_cast<const unsigned short*>(sd.B) + (size_t)nc * sd.rank;
#pragma unroll 8
        for (int q = 0; q < sd.rank; ++q) {
            u0 += hs[q] * bf16_bits_to_f32(b[q]);
            u1 += hs[q] * bf16_bits_to_f32(b[sd.rank + q]);
        }
    } else if constexpr (!BACKWARD) {
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const int x = i * 128 + tid, c = col_of(x), q = (x - c * L) * 8;
            const float4 h0 = *reinterpret_cast<const float4*>(hs + q), h1 = *reinterpret_cast<const float4*>(hs + q + 4);
            const float he[8] = {h0.x, h0.y, h0.z, h0.w, h1.x, h1.y, h1.z, h1.w};
            float d = 0.f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                d += he[2 * e] * bf16_bits_to_f32((unsigned short)(bw[i][e] & 0xffffu));
                d += he[2 * e + 1] * bf16_bits_to_f32((unsigned short)(bw[i][e] >> 16));
            }
            us[x + (x >> 5)] = d;                        // (chunks past the last column land past the ones read below)
        }
        __syncthreads();
        for (int j = 0; j < L; ++j) {
            const int x = 2 * tid * L + j, y = x + L;
            u0 += us[x + (x >> 5)];
            u1 += us[y + (y >> 5)];
        }
    } else {
        float d[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const float hq = hs[i * 4 + g];
            const unsigned keep = i * 4 + g < sd.rank ? 0xffffffffu : 0u;        // rank rows past the last repeated it: zero (an infinity times hq = 0 is none)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned w = bw[i][e] & keep;
                d[2 * e] += hq * bf16_bits_to_f32((unsigned short)(w & 0xffffu));
                d[2 * e + 1] += hq * bf16_bits_to_f32((unsigned short)(w >> 16));
            }
        }
        // row groups 264 floats apart: the stores and the column reads stay off each other's banks
        *reinterpret_cast<float4*>(us + g * 264 + (tid & 31) * 8) = make_float4(d[0], d[1], d[2], d[3]);
        *reinterpret_cast<float4*>(us + g * 264 + (tid & 31) * 8 + 4) = make_float4(d[4], d[5], d[6], d[7]);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float2 a = *reinterpret_cast<const float2*>(us + j * 264 + 2 * tid);
            u0 += a.x;
            u1 += a.y;
        }
    }
    v0 += u0;
    v1 += u1;
}

// grid = (blocks of 256 columns, rows); a thread finishes two columns of one row.
template <bool BACKWARD>
SYMB_KERNEL void __launch_bounds__(128)
symb_small_finish_kernel(const SmallFinishParams p) {
    __shared__ __attribute__((aligned(16))) float hs[128], us[4096 + 128];
    const int t = blockIdx.y, c0 = blockIdx.x * 256, n = c0 + 2 * (int)threadIdx.x;
    SmallFirst first;
    {
        const float* const c = p.partial + (size_t)t * p.N + min(n, p.N - 2);
#pragma unroll
        for (int q = 0; q < 8; ++q) first.c[q] = *reinterpret_cast<const float2*>(c + (size_t)min(q, p.ranges - 1) * ((size_t)p.T * p.N));
        // (without a LoRA term or with H there already: some floats of the call's sums)
        const bool h = p.lora_term && p.h_partial;
        const float* const src = h ? p.h_partial + (size_t)t * p.h_pitch + min((int)threadIdx.x, p.h_pitch - 1) : c;
#pragma unroll
        for (int q = 0; q < 8; ++q) first.h[q] = src[h ? (size_t)min(q, p.h_ranges - 1) * ((size_t)p.T * p.h_pitch) : 0];
    }
    const uint32_t at = p.rows.at[t];
    const int s = at >> 8, in_seg = at & 255;
    const SegDesc sd = p.seg[s];
    float v0 = 0.f, v1 = 0.f;
    auto sums = [&](auto NCH) __attribute__((always_inline)) { small_finish_sums<BACKWARD, decltype(NCH)::value>(p, sd, t, c0, first, hs, us, v0, v1); };
    // uniform over the workgroup (one row, one segment)
    if (!p.lora_term || sd.kind != KIND_LORA) sums(std::integral_constant<int, 0>{});
    else if (!BACKWARD && (sd.rank & 7)) sums(std::integral_constant<int, -1>{});
    else if (sd.rank <= 16) sums(std::integral_constant<int, 4>{});
    else if (sd.rank <= 32) sums(std::integral_constant<int, 8>{});
    else if (sd.rank <= 64) sums(std::integral_constant<int, 16>{});
    else sums(std::integral_constant<int, 32>{});
    if (n >= p.N) return;
    if (p.out.scale_kind && sd.kind == p.out.scale_kind) {
        const unsigned l = *reinterpret_cast<const unsigned*>(sd.A + n);
        v0 *= bf16_bits_to_f32((unsigned short)(l & 0xffffu));
        v1 *= bf16_bits_to_f32((unsigned short)(l >> 16));
    }
    if (!BACKWARD && p.out.neff) {
        const NoiseDesc nd = p.out.neff[s];
        if (nd.ptr) {
            const unsigned e = *reinterpret_cast<const unsigned*>(nd.ptr + (size_t)(nd.rows == 1 ? 0 : in_seg) * p.N + n);
            v0 -= bf16_bits_to_f32((unsigned short)(e & 0xffffu));
            v1 -= bf16_bits_to_f32((unsigned short)(e >> 16));
        }
    }
    bf16* const out = p.out.c_seg ? p.out.c_seg[s] + (size_t)in_seg * p.N : p.out.C + (size_t)t * p.N;
    *reinterpret_cast<unsigned*>(out + n) = pack2_bf16(v0, v1);
}

// LoRA terms of short segments (at most 16 rows) of a larger batch, in fp32, for the tiled kernel to add: out[d][n] = sum_q H[t][q] B_i[n][q]
// (forward) or A_i[q][n] (input gradient), H from the rows the skinny kernel left.  Inside the tiled kernel every LoRA segment that meets
// a row tile is a chain of 2 rpad / 32 register-staged steps of 1 to 1.6 us, whatever few rows it has, and the launch waits for the
// row tile that holds the most of them; here the segments run side by side.  All rows of a segment are one block of 16 for the
// matrix cores, against value and residual of H as in the tiled kernel's steps: the adapter is read once per segment, and a wavefront needs neither
// LDS nor a barrier.  A wavefront owns 64 columns: lane l15 holds columns 4 l15 .. + 3 as fragments of four products, so that the
// result of a row is one 16-byte store per lane.  Bound by the fp32 terms it writes.
// grid = (blocks of 256 columns, segments).  NS: 32-wide steps over the ranks (padded rank <= 32 NS).
struct LoraDeltaParams {
    const bf16* h_rows;       // [T][2 * h_pitch]
    int h_pitch, N;
    const SegDesc* seg;
    const RowChunk* items;    // device: segment, first row, rows, pad = first row of out
    float* out;               // [.][N]
};
template <bool BACKWARD, int NS>
__device__ __forceinline__ void lora_delta(const LoraDeltaParams& p, const RowChunk& it, const SegDesc& sd) {
    const int tid = threadIdx.x, lane = tid & 63, l15 = lane & 15, kq = lane >> 4;
    const int n = blockIdx.x * 256 + (tid >> 6) * 64 + l15 * 4;           // this lane's columns n .. n + 3 (N is a multiple of 8)
    if (n - l15 * 4 >= p.N) return;
    u32x4 h[NS][2];
    const bf16* const hrow = p.h_rows + (size_t)(it.row0 + min(l15, it.nrows - 1)) * 2 * p.h_pitch;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int q0 = s * 32 + kq * 8, at = min(q0, sd.rpad - 8);        // ranks past the padded one count as zero, in both operands
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            h[s][half] = ld_glb16(hrow + half * sd.rpad + at);
            if (q0 >= sd.rpad) h[s][half] = u32x4{0u, 0u, 0u, 0u};
        }
    }
    u32x4 w[NS][4];                                      // column n + j, ranks q0 .. q0 + 7
    if constexpr (BACKWARD) {
        uint2 x[NS][8];
        const bf16* const col = sd.A + min(n, p.N - 4);
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int e = 0; e < 8; ++e) x[s][e] = *reinterpret_cast<const uint2*>(col + (size_t)min(s * 32 + kq * 8 + e, sd.rank - 1) * p.N);
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint2 a = x[s][2 * e], b = x[s][2 * e + 1];
                const int q = s * 32 + kq * 8 + 2 * e;
                if (q >= sd.rank) a = make_uint2(0u, 0u);
                if (q + 1 >= sd.rank) b = make_uint2(0u, 0u);
                w[s][0][e] = (a.x & 0xffffu) | (b.x << 16);
                w[s][1][e] = (a.x >> 16) | (b.x & 0xffff0000u);
                w[s][2][e] = (a.y & 0xffffu) | (b.y << 16);
                w[s][3][e] = (a.y >> 16) | (b.y & 0xffff0000u);
            }
    } else if ((sd.rank & 7) == 0) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int q0 = s * 32 + kq * 8;
                w[s][j] = ld_glb16(sd.B + (size_t)min(n + j, p.N - 1) * sd.rank + min(q0, sd.rank - 8));
                if (q0 >= sd.rank) w[s][j] = u32x4{0u, 0u, 0u, 0u};
            }
    } else {
        // rows of B_i that are no whole 16-byte chunks: element loads
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned short* const b = reinterpret_cast<const unsigned short*>(sd.B) + (size_t)min(n + j, p.N - 1) * sd.rank;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int q = s * 32 + kq * 8 + 2 * e;
                    const unsigned a = b[min(q, sd.rank - 1)], c = b[min(q + 1, sd.rank - 1)];
                    w[s][j][e] = (q < sd.rank ? a : 0u) | (q + 1 < sd.rank ? c << 16 : 0u);
                }
            }
    }
    floatx4 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, h[s][half]), __builtin_bit_cast(bf16x8, w[s][j]), acc[j], 0, 0, 0);
    if (n >= p.N) return;
    float* const out = p.out + (size_t)(it.pad + kq * 4) * p.N + n;        // rows 4 kq .. + 3 of the block
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (kq * 4 + q < it.nrows) *reinterpret_cast<float4*>(out + (size_t)q * p.N) = make_float4(acc[0][q], acc[1][q], acc[2][q], acc[3][q]);
}
template <bool BACKWARD>
SYMB_KERNEL void __launch_bounds__(256)
symb_lora_delta_kernel(const LoraDeltaParams p) {
    const RowChunk it = p.items[blockIdx.y];
    const SegDesc sd = p.seg[it.seg];
    if (sd.rpad <= 32) lora_delta<BACKWARD, 1>(p, it, sd);                 // uniform over the workgroup
    else if (sd.rpad <= 64) lora_delta<BACKWARD, 2>(p, it, sd);
    else lora_delta<BACKWARD, 4>(p, it, sd);
}

}  // namespace symb
