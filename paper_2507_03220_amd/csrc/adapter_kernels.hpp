// HBM-bound kernels around the base GEMM: LoRA shrink (Hs = s X A^T), its backward twin
// (dH = s dY B), the per-segment parameter gradients (dA, dB, dl) and the IA3 row scale
// of dY.  All of them walk segment-aligned row chunks from a host-built work list, so a
// chunk never mixes two clients.
#pragma once
#include <type_traits>

#include "symb_device.hpp"

namespace symb {

// One unit of row work: rows [row0, row0 + nrows) of segment `seg` (nrows <= chunk size).
struct RowChunk {
    int32_t seg, row0, nrows, pad;
};

// -------------------------------------------------------------------------------------------
// Skinny projection:  out[t][p] = s_i * sum_k L[t][k] * R_i[p][k],  p < rpad_i, stored as a bf16
// value plus a bf16 residual (out[t][rpad_i + p])
//   forward shrink : L = X  [T][K=d_in],  R_i = A_i  [r][d_in]
//   backward dH    : L = dY [T][K=d_out], R_i = B_i^T: read from B_i [d_out][r] as it lies (BT), or, where a rank is no multiple
//                    of 4 or a B_i not 16-byte aligned, from a packed copy [rpad][d_out] (see pack kernel)
// A workgroup owns 32 rows (16 to 48 in launches of few rows); its 4 (8) wavefronts split K in interleaved slices, bring the rows in
// through LDS (see SkinnyStage below), take the adapter rows from L2, and meet in LDS for the
// final sum.  RB = max rank blocks of 16.
// -------------------------------------------------------------------------------------------
struct SkinnyParams {
    const bf16* L;            // [T][K]
    bf16* out;                // [T][out_pitch], out_pitch >= 2 * rpad_i
    int K, out_pitch;
    const RowChunk* chunks;   // device
    const SegDesc* seg;       // device
    const bf16* packed;       // backward through a packed copy: base of packed B^T area, else null
    const int64_t* packed_off;// backward: element offset of segment i's [rpad][K] block
    int use_packed;
    const bf16* const* L_seg; // device [S] or null: rows of segment i start at L_seg[i] instead of L + off[i] * K
    const int32_t* off;       // device [S+1] (read only with L_seg)
};

constexpr int SKINNY_ROWS = 32;                        // rows per workgroup, unless launch_skinny chooses others

// The skinny kernel's row stream.  A lane of an MFMA operand holds 16 bytes of one row, so fragment
// loads straight from global memory touch 16 cache lines per 16 lanes, 16 bytes of each; the
// memory pipeline then runs at a fraction of what whole-line requests reach.  Here every wavefront
// brings its K slices (the workgroup's rows x SK elements) in through LDS DMA, whole rows of the slice
// per request, into NBUF buffers of its own (no workgroup barrier in the loop), and reads the
// fragments from LDS.  The 16-byte chunks of a row are stored at chunk ^ f(row), so the 16 rows a
// fragment read touches fall on different banks.  The adapter rows of a slice (from L2) come the same
// way, into one more buffer.  Measured on 1.5 GB inputs: 4.0 -> 5.0 TB/s; 128-element slices are best
// at rank <= 16, 64-element ones above (LDS for the adapter rows); a third buffer or a third workgroup
// per CU changes nothing.
template <int RB, int NBUF_, bool RDEEP_, int BLKS_, int NW_>
struct SkinnyStage {
    static constexpr int BLKS = BLKS_, ROWS = 16 * BLKS;  // 16-row MFMA blocks
    static constexpr int NW = NW_;                        // wavefronts
    static constexpr int SK = RB >= 2 || NW > 4 ? 64 : 128;         // K elements per slice
    static constexpr int NBUF = NBUF_;                    // slices a wavefront keeps in LDS
    static constexpr bool RDEEP = RDEEP_;                 // the adapter rows are requested with their slice, NBUF deep as well
    static constexpr int ROW_BYTES = SK * 2;
    static constexpr int LPR = ROW_BYTES / 16;            // lanes (16-byte chunks) per row
    static constexpr int RPI = 64 / LPR;                  // rows per DMA request of one wavefront
    static constexpr int DPS = ROWS / RPI;         // DMA requests per slice
    static constexpr int SLICE = ROWS * ROW_BYTES;
    static constexpr int RSLICE = RB * 16 * ROW_BYTES;    // the adapter rows of one slice (one buffer)
    static constexpr int WAVE_BYTES = NBUF * SLICE + (RDEEP ? NBUF : 1) * RSLICE;
    static constexpr int BYTES = NW * WAVE_BYTES;
    static_assert(SK == 64 || SK == 128, "a row of a slice is one or two 128-byte lines");
    __device__ static constexpr int swz(int r) { return (r / (16 / LPR)) & (LPR - 1); }
};
typedef __attribute__((address_space(1))) void glb_void_t;
typedef __attribute__((address_space(3))) void lds_void_t;
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
// 16 bytes from global memory.  Said explicitly: a pointer that was itself loaded from memory (an
// adapter's address in its descriptor) is generic to the compiler, and a generic load counts on both
// memory counters, which forces full waits around it.
__device__ __forceinline__ u32x4 ld_glb16(const bf16* p) {
    return *reinterpret_cast<const __attribute__((address_space(1))) u32x4*>((const __attribute__((address_space(1))) bf16*)p);
}

// One wavefront's share of K for a chunk whose segment uses NB rank blocks (compile time, so that the
// loop holds no conditional load: the compiler's wait counts for the adapter rows are then exact).
// lrow / rrow point at the lane's first 8 elements (row start + kq*8); src[i] at the 16 bytes this
// lane brings in with DMA request i of a slice (at k = 0); wbuf = this wavefront's slice buffers.
// BT: rbase is B_i [K][rrows].  The SK k-rows of a slice are one contiguous run of it, brought in as it lies and read back
// through the transposing LDS read.  Rows of 128 or 256 bytes (ranks 64, 128) would put the 8 k-rows such a read serves at a time
// on the same banks: their 32-byte pieces are stored at piece ^ skinny_bt_swz.
__device__ __forceinline__ int skinny_bt_swz(int r, int k) {
    return r == 128 ? ((((k >> 3) & 1) << 2) | (k & 3)) : r == 64 ? ((((k >> 3) & 1) << 1) | ((k >> 1) & 1)) : 0;
}
template <int RB, int NB, bool BT, class ST>
__device__ __forceinline__ void skinny_stream(const bf16* (&lrow)[ST::BLKS], const bf16* (&rrow)[RB], const bool (&r_ok)[RB],
                                              const bf16* (&src)[ST::DPS], const bf16* rbase, int rrows,
                                              unsigned char* wbuf, int K, int wave, int lane, floatx4 (&acc)[ST::BLKS][RB]) {
    constexpr int BLKS = ST::BLKS, KSTEP = ST::NW * ST::SK;        // (K from one slice of a wavefront to its next)
    constexpr int NH = ST::SK / 32;                      // MFMA k-steps per slice
    constexpr int NRD = NB * 16 / ST::RPI;               // DMA requests for the adapter rows of a slice
    const int trow = lane & 15, kq = lane >> 4;
    unsigned char* const rbuf = wbuf + ST::NBUF * ST::SLICE;
    unsigned foff[BLKS][NH], roff[NB][NH];        // fragment (b, h) / (j, h) of this lane within a slice buffer
#pragma unroll
    for (int h = 0; h < NH; ++h) {
#pragma unroll
        for (int b = 0; b < BLKS; ++b) {
            const int r = b * 16 + trow;
            foff[b][h] = (unsigned)(size_t)wbuf + (unsigned)(r * ST::ROW_BYTES + (((h * 4 + kq) ^ ST::swz(r)) * 16));
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int r = j * 16 + trow, k = h * 32 + kq * 8 + (trow >> 2);      // BT: first of the two reads; the second is 4 k-rows further
            roff[j][h] = (unsigned)(size_t)rbuf + (BT ? (unsigned)(k * rrows * 2 + ((j ^ skinny_bt_swz(rrows, k)) * 32) + (trow & 3) * 8)
                                                      : (unsigned)(r * ST::ROW_BYTES + (((h * 4 + kq) ^ ST::swz(r)) * 16)));
        }
    }
    // The adapter rows (from L2) come in by LDS DMA as well, whole row pieces per request: fragment loads
    // straight from global memory are 64-byte pieces of 16 rows each, twice the requests for the bytes.
    // Rows past the adapter's last are read from row 0 and count as zero (r_ok).
    const bf16* rsrc[NRD];
    const size_t rstep = BT ? (size_t)rrows : 1;         // adapter elements from one k to the next
#pragma unroll
    for (int i = 0; i < NRD; ++i) {
        if constexpr (BT) {                              // (past the run's end: its last 16 bytes again)
            const int c = min(i * 64 + lane, ST::SK * rrows / 8 - 1), per = rrows >> 3;        // 16-byte chunk of the run
            const int f = rrows == 64 || rrows == 128 ? skinny_bt_swz(rrows, c / per) : 0;
            rsrc[i] = rbase + (c ^ (f << 1)) * 8;
            continue;
        }
        const int r = i * ST::RPI + lane / ST::LPR;
        rsrc[i] = rbase + (size_t)(r < rrows ? r : 0) * K + (((lane % ST::LPR) ^ ST::swz(r)) * 8);
    }
    auto dma = [&](int buf, int k) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < ST::DPS; ++i)
            __builtin_amdgcn_global_load_lds((glb_void_t*)(src[i] + k), (lds_void_t*)(wbuf + buf * ST::SLICE + i * 1024), 16, 0, 0);
    };
    auto dma_r = [&](int buf, int k) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NRD; ++i)
            __builtin_amdgcn_global_load_lds((glb_void_t*)(rsrc[i] + k * rstep), (lds_void_t*)(rbuf + (ST::RDEEP ? buf * ST::RSLICE : 0) + i * 1024), 16, 0, 0);
    };
    // The fragment reads are assembly statements with a wait of their own: while an LDS DMA request is in
    // flight the compiler makes every load result it can see wait for all memory traffic of the
    // wavefront, the slice requested ahead included.  Each result is tied ("+v") to the wait that
    // covers it, so no use can move in front of that wait.  mul() returns with its LDS reads
    // complete: both buffers it read may be requested again.
    auto mul = [&](int buf) __attribute__((always_inline)) {
        typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
        u32x4 lv[BLKS][NH], rv[BT ? 1 : NB][NH];
        u32x2 rt[BT ? NB : 1][NH][2];
#pragma unroll
        for (int h = 0; h < NH; ++h) {
#pragma unroll
            for (int b = 0; b < BLKS; ++b) asm volatile("ds_read_b128 %0, %1" : "=v"(lv[b][h]) : "v"(foff[b][h] + buf * ST::SLICE));
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const unsigned at = roff[j][h] + (ST::RDEEP ? buf * ST::RSLICE : 0);
                if constexpr (BT) {
                    asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(rt[j][h][0]) : "v"(at));
                    asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(rt[j][h][1]) : "v"(at + 8 * rrows));
                } else {
                    asm volatile("ds_read_b128 %0, %1" : "=v"(rv[j][h]) : "v"(at));
                }
            }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
#pragma unroll
        for (int h = 0; h < NH; ++h) {
#pragma unroll
            for (int b = 0; b < BLKS; ++b) asm volatile("" : "+v"(lv[b][h]));
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                if constexpr (BT) { asm volatile("" : "+v"(rt[j][h][0])); asm volatile("" : "+v"(rt[j][h][1])); }
                else asm volatile("" : "+v"(rv[j][h]));
            }
        }
#pragma unroll
        for (int h = 0; h < NH; ++h)
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                u32x4 raw;
                if constexpr (BT) raw = __builtin_shufflevector(rt[j][h][0], rt[j][h][1], 0, 1, 2, 3);
                else raw = rv[j][h];
                const bf16x8 rf = __builtin_bit_cast(bf16x8, r_ok[j] ? raw : u32x4{0u, 0u, 0u, 0u});
#pragma unroll
                for (int b = 0; b < BLKS; ++b)
                    acc[b][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(rf, __builtin_bit_cast(bf16x8, lv[b][h]), acc[b][j], 0, 0, 0);
            }
    };
    // ---- full slices of this wavefront: k = wave * SK + 4 (8) SK s, s < ns, through LDS.  Slices 0 .. np-1
    // are requested up front; iteration s requests slice s + np (while there is one) into the buffer
    // iteration s - 1 has finished reading, after the adapter rows of slice s: the memory counter
    // retires in order, so the wait for slice s and its adapter rows leaves exactly the newest slice's
    // DPS requests in flight.
    int k0 = wave * ST::SK;
    const int ns = K >= k0 + ST::SK ? (K - k0 - ST::SK) / (KSTEP) + 1 : 0;
    const int np = ns < ST::NBUF - 1 ? ns : ST::NBUF - 1;
    for (int d = 0; d < np; ++d) {
        dma(d, k0 + d * KSTEP);
        if constexpr (ST::RDEEP) dma_r(d, k0 + d * KSTEP);
    }
    int cur = 0, nxt = np;                               // buffer of slice s, of slice s + np
    int s = 0;
    for (; s + np < ns; ++s) {
        if constexpr (ST::RDEEP) {                       // slice and adapter rows together, NBUF - 1 of them in flight
            dma(nxt, k0 + np * KSTEP);
            dma_r(nxt, k0 + np * KSTEP);
            asm volatile("s_waitcnt vmcnt(%0)" : : "n"((ST::NBUF - 1) * (ST::DPS + NRD)) : "memory");
        } else {
            dma_r(0, k0);
            dma(nxt, k0 + np * KSTEP);
            asm volatile("s_waitcnt vmcnt(%0)" : : "n"(ST::DPS) : "memory");
        }
        mul(cur);
        cur = cur + 1 == ST::NBUF ? 0 : cur + 1;
        nxt = nxt + 1 == ST::NBUF ? 0 : nxt + 1;
        k0 += KSTEP;
    }
    for (; s < ns; ++s) {                                // the last np slices: nothing left to request
        if constexpr (!ST::RDEEP) dma_r(0, k0);
        asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        mul(cur);
        cur = cur + 1 == ST::NBUF ? 0 : cur + 1;
        k0 += KSTEP;
    }
    // ---- the slice that crosses the end of K: masked fragments straight from global memory
    if (k0 < K) {
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const bool kok = (k0 + h * 32 + kq * 8) < K;
            u32x4 lv[BLKS];
#pragma unroll
            for (int b = 0; b < BLKS; ++b) lv[b] = kok ? ld_glb16(lrow[b] + k0 + h * 32) : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                u32x4 rv = u32x4{0u, 0u, 0u, 0u};
                if (kok && r_ok[j]) {
                    if constexpr (BT) {                  // column j*16 + trow of 8 k-rows
                        const unsigned short* const e = reinterpret_cast<const unsigned short*>(rbase) + (size_t)(k0 + h * 32 + kq * 8) * rrows + j * 16 + trow;
#pragma unroll
                        for (int q = 0; q < 4; ++q) rv[q] = e[(size_t)(2 * q) * rrows] | ((unsigned)e[(size_t)(2 * q + 1) * rrows] << 16);
                    } else {
                        rv = ld_glb16(rrow[j] + k0 + h * 32);
                    }
                }
#pragma unroll
                for (int b = 0; b < BLKS; ++b)
                    acc[b][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, rv), __builtin_bit_cast(bf16x8, lv[b]), acc[b][j], 0, 0, 0);
            }
        }
    }
}

// Calls skinny_stream<RB, nb> for the run-time nb in 1..RB.
template <int RB, bool BT, class ST, int NB = 1, typename... Args>
__device__ __forceinline__ void skinny_stream_dispatch(int nb, Args&&... args) {
    if (nb == NB) skinny_stream<RB, NB, BT, ST>(args...);
    else if constexpr (NB < RB) skinny_stream_dispatch<RB, BT, ST, NB + 1>(nb, args...);
}

// Slice buffers and wavefronts by the build of the kernel.  0: four wavefronts, two buffers.  4: three buffers with the adapter rows beside each slice,
// two slices in flight per wavefront (dH beside dB in one launch).  Launches of at most one workgroup per CU take eight wavefronts and
// BUILD = 1, 2 or 3 blocks of 16 rows, as few as that needs: such a launch is one chain of memory latencies along K, not bandwidth, and half of K per wavefront
// and fewer rows shorten it.  As many slices in flight as 160 KiB hold; where the adapter rows leave no room for two of theirs they are requested with the slice that is
// multiplied next.  At rank 128 only 16 rows fit that way.  Four wavefronts on 32 rows / this, us: 381 rows of ranks to 64, K = 4096 9.8 / 8.5; 2000 of rank 16, K = 4608 10.4 / 8.6;
// 10240 of ranks to 64, K = 4096 31.8 / 27.5, against B_i 25.2 / 20.6; 1000 of ranks to 32, K = 11008, against B_i 24.0 / 17.7; 1300 of ranks to 128, K = 4096 27.4 / 24.1.  The rest is what a CU takes in
// (64 bytes per clock: 1 MiB of a rank-128 adapter 8 us) and, before it, launch, descriptors and first lines.
constexpr int SKINNY_DEEP = 4;
constexpr int skinny_threads(int build) { return build >= 1 && build <= 3 ? 512 : 256; }
constexpr bool skinny_has(int rb, int build) { return rb <= 4 || build <= 1; }
template <int RB, int BUILD>
struct SkinnyBuild {
    static constexpr bool WIDE = BUILD >= 1 && BUILD <= 3;
    static constexpr int BLKS = WIDE ? BUILD : 2, NW = WIDE ? 8 : 4;
    static constexpr int KIB = WIDE ? 20 : 64, X = BLKS * 2, R = RB * 2;          // KiB of a wavefront, of its slice, of the adapter rows of it (SK = 64)
    static constexpr bool RDEEP = BUILD == SKINNY_DEEP || (WIDE && 2 * (X + R) <= KIB);
    static constexpr int NBUF = BUILD == SKINNY_DEEP ? 3 : !WIDE ? 2 : !RDEEP ? 2 : KIB / (X + R) < 4 ? KIB / (X + R) : 4;
    using ST = SkinnyStage<RB, NBUF, RDEEP, BLKS, NW>;
    static constexpr int RED = NW * ST::ROWS * (RB * 16 + 4) * 4;                 // the wavefronts' sums, afterwards
    static constexpr int BYTES = ST::BYTES > RED ? ST::BYTES : RED;
    static_assert(BYTES <= 160 << 10, "LDS of a CU");
};
// The rows of one chunk: store(t, pp, value) gets ranks pp .. pp + 3 of its row t, as a bf16 value and its bf16 rounding residual, four of each packed.
template <int RB, class ST, bool BT, class STORE>
__device__ __forceinline__ void skinny_rows(const SkinnyParams& p, const RowChunk ch, const SegDesc sd, unsigned char* smem, STORE&& store) {
    constexpr int BLKS = ST::BLKS, ROWS = ST::ROWS;
    float (*red)[ROWS][RB * 16 + 4] = reinterpret_cast<float (*)[ROWS][RB * 16 + 4]>(smem);
    const int nb = sd.rpad >> 4;                         // rank blocks in use (uniform), 1..RB
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int trow = lane & 15, kq = lane >> 4;
    // rows past the chunk are clamped onto its last row; their results are never stored
    const bf16* lrow[BLKS];
    const bf16* const lbase = p.L_seg ? p.L_seg[ch.seg] - (size_t)p.off[ch.seg] * p.K : p.L;
#pragma unroll
    for (int b = 0; b < BLKS; ++b) lrow[b] = lbase + (size_t)(ch.row0 + min(b * 16 + trow, ch.nrows - 1)) * p.K + kq * 8;
    const bf16* src[ST::DPS];
#pragma unroll
    for (int i = 0; i < ST::DPS; ++i) {
        const int r = i * ST::RPI + lane / ST::LPR;
        src[i] = lbase + (size_t)(ch.row0 + min(r, ch.nrows - 1)) * p.K + (((lane % ST::LPR) ^ ST::swz(r)) * 8);
    }
    const bf16* rbase = BT ? sd.B : p.use_packed ? (p.packed + p.packed_off[ch.seg]) : sd.A;
    const int rrows = !BT && p.use_packed ? sd.rpad : sd.rank;     // valid adapter rows; the rest count as zero
    const bf16* rrow[RB];
    bool r_ok[RB];
#pragma unroll
    for (int j = 0; j < RB; ++j) {
        r_ok[j] = (j * 16 + trow) < rrows;
        rrow[j] = rbase + (size_t)(r_ok[j] ? (j * 16 + trow) : 0) * p.K + kq * 8;
    }

    floatx4 acc[BLKS][RB];
#pragma unroll
    for (int b = 0; b < BLKS; ++b)
#pragma unroll
        for (int j = 0; j < RB; ++j) acc[b][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    skinny_stream_dispatch<RB, BT, ST>(nb, lrow, rrow, r_ok, src, rbase, rrows, smem + wave * ST::WAVE_BYTES, p.K, wave, lane, acc);
    __syncthreads();                                     // every wavefront is done with its slice buffers
    // lane holds out[t = b*16 + trow][p = j*16 + 4*kq + q]
#pragma unroll
    for (int b = 0; b < BLKS; ++b)
#pragma unroll
        for (int j = 0; j < RB; ++j)
            if (j < nb) *reinterpret_cast<floatx4*>(&red[wave][b * 16 + trow][j * 16 + kq * 4]) = acc[b][j];
    __syncthreads();
    // One row of `out` holds, for its own segment, rpad values rounded to bf16 followed by the
    // rpad rounding residuals (also bf16): value + residual carries ~16 significand bits on.
    const int per = sd.rpad >> 2;                        // quads of ranks per row, dealt out over the threads; the wavefronts' sums in order
    for (int e = tid; e < ch.nrows * per; e += 64 * ST::NW) {
        const int t = e / per, pp = (e - t * per) * 4;
        floatx4 v = *reinterpret_cast<const floatx4*>(&red[0][t][pp]);
#pragma unroll
        for (int w = 1; w < ST::NW; ++w) v += *reinterpret_cast<const floatx4*>(&red[w][t][pp]);
        v *= sd.scale;
        const unsigned h01 = pack2_bf16(v[0], v[1]), h23 = pack2_bf16(v[2], v[3]);
        uint2 hi2, lo2;
        hi2.x = h01;
        hi2.y = h23;
        lo2.x = pack2_bf16(v[0] - bf16_bits_to_f32((unsigned short)(h01 & 0xffffu)), v[1] - bf16_bits_to_f32((unsigned short)(h01 >> 16)));
        lo2.y = pack2_bf16(v[2] - bf16_bits_to_f32((unsigned short)(h23 & 0xffffu)), v[3] - bf16_bits_to_f32((unsigned short)(h23 >> 16)));
        store(t, pp, hi2, lo2);
    }
}
template <int RB, int BUILD, bool BT>
__device__ __forceinline__ void skinny_chunk(const SkinnyParams& p, int chunk, unsigned char* smem) {
    const RowChunk ch = p.chunks[chunk];
    const SegDesc sd = p.seg[ch.seg];
    bf16* const out = p.out + (size_t)ch.row0 * p.out_pitch;
    const int pitch = p.out_pitch, rpad = sd.rpad;
    skinny_rows<RB, typename SkinnyBuild<RB, BUILD>::ST, BT>(p, ch, sd, smem, [=](int t, int pp, uint2 hi, uint2 lo) __attribute__((always_inline)) {
        bf16* const row = out + (size_t)t * pitch + pp;
        *reinterpret_cast<uint2*>(row) = hi;
        *reinterpret_cast<uint2*>(row + rpad) = lo;
    });
}

template <int RB, int BUILD, bool BT>
SYMB_KERNEL void __launch_bounds__(skinny_threads(BUILD))
symb_skinny_kernel(const SkinnyParams p) {
    __shared__ __align__(16) unsigned char smem[SkinnyBuild<RB, BUILD>::BYTES];
    skinny_chunk<RB, BUILD, BT>(p, blockIdx.x, smem);
}

// Transposing LDS read of an MFMA fragment whose k axis runs down the rows of a column-contiguous tile.
__device__ __forceinline__ bf16x8 lds_read_tr_16x32(const unsigned char* base, int pitch_bytes, int col0, int lane) {
    // tile [32 t][cols] (column-contiguous); returns for lane l: column col0 + (l & 15), t = 8*(l >> 4) + 0..7
    const int g = lane >> 4, jj = lane & 15;
    const unsigned char* p0 = base + (g * 8 + (jj >> 2)) * pitch_bytes + (col0 + ((jj & 3) << 2)) * 2;
    typedef __attribute__((address_space(3))) shortx4 lds_s4;
    shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(p0));
    shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4*)(p0 + 4 * pitch_bytes));
    typedef __attribute__((__vector_size__(8 * sizeof(short)))) short shortx8;
    shortx8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

// Packs B_i [d_out][r] into B_i^T [rpad][d_out] (zero rows beyond r) so the backward
// projection reads K-contiguous adapter rows.  grid.y = segment, grid.x covers d_out.
struct PackParams {
    const SegDesc* seg;
    bf16* packed;
    const int64_t* packed_off;
    int d_out;
};
SYMB_KERNEL void __launch_bounds__(256) symb_pack_bt_kernel(const PackParams p) {
    const SegDesc sd = p.seg[blockIdx.y];
    if (sd.kind != KIND_LORA) return;
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= p.d_out) return;
    unsigned short* dst = reinterpret_cast<unsigned short*>(p.packed + p.packed_off[blockIdx.y]);
    const unsigned short* src = reinterpret_cast<const unsigned short*>(sd.B) + (size_t)j * sd.rank;
    for (int q = 0; q < sd.rpad; ++q) dst[(size_t)q * p.d_out + j] = (q < sd.rank) ? src[q] : (unsigned short)0;
}

// Packs A_i [r][d_in] into A_i^T [d_in][r] (exactly r columns): the adapter-side operand of the
// input gradient when the base weight is stored input-major (the K-contiguous GEMM then wants the
// adapter rows rank-contiguous per input column).  grid.y = segment, grid.x covers d_in.
struct PackAtParams {
    const SegDesc* seg;
    bf16* packed;
    const int64_t* packed_off;
    int d_in;
};
SYMB_KERNEL void __launch_bounds__(256) symb_pack_at_kernel(const PackAtParams p) {
    const SegDesc sd = p.seg[blockIdx.y];
    if (sd.kind != KIND_LORA) return;
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k >= p.d_in) return;
    unsigned short* dst = reinterpret_cast<unsigned short*>(p.packed + p.packed_off[blockIdx.y]) + (size_t)k * sd.rank;
    const unsigned short* src = reinterpret_cast<const unsigned short*>(sd.A);
    for (int q = 0; q < sd.rank; ++q) dst[q] = src[(size_t)q * p.d_in + k];
}

// -------------------------------------------------------------------------------------------
// LoRA parameter gradients of one segment, contraction over its tokens:
//   G[c][pp] = sum_t R[t][c] * L[t][pp]
//   dB_i (CMAJOR = true ): R = dY, L = Hs -> out[c * rank + pp]      ([d_out][r])
//   dA_i (CMAJOR = false): R = X,  L = dH -> out[pp * ncols + c]     ([r][d_in])
// A workgroup owns 256 columns (128 at ranks above 32) of one work item and walks its tokens 32 at a time through
// LDS; both MFMA operands are token-strided in memory and are read with the transposing
// LDS load.  A work item is a whole segment, or, for a segment of more than GRAD_SPLIT_MIN
// tokens, one of its runs of GRAD_SPLIT tokens: a long segment walked by one workgroup per
// column block would set the time of the whole launch.  Such a run leaves its sum in the
// workspace (same layout as the result) and symb_grad_reduce_kernel adds the runs up in
// order.  Fixed summation order within this kernel, a function of the segment's length alone.
// -------------------------------------------------------------------------------------------
constexpr int GRAD_SPLIT = 1024;       // tokens per run of a split segment (a multiple of GRAD_TT)
constexpr int GRAD_SPLIT_MIN = 1536;   // segments up to this length stay whole
struct GradItem {
    int32_t seg, t_lo, t_hi;  // tokens [t_lo, t_hi) of segment seg
    int32_t direct;           // 1: the result goes to the segment's dA / dB; 0: to partial + partial_off
    int64_t partial_off;      // in floats
};
struct GradParams {
    const bf16* R;            // [T][ncols]
    const bf16* L;            // [T][l_pitch]: per row rpad_i values then rpad_i residuals (see skinny kernel)
    int ncols, l_pitch;
    const int32_t* off;
    const SegDesc* seg;
    const GradItem* items;    // device: the work of this launch (grid.y indexes it)
    int accumulate;
    const bf16* const* R_seg; // device [S] or null: rows of segment i of R start at R_seg[i]
    float* partial;           // workspace region of the split segments' runs
};

template <int RB> constexpr int GRAD_CT = RB <= 2 ? 256 : 128;   // columns per workgroup (512-byte row pieces where the registers allow)
constexpr int GRAD_TT = 32;        // tokens per step

template <int RB>
struct GradWalk {
    static constexpr int CT = GRAD_CT<RB>;
    static constexpr int RPITCH = CT * 2 + 16;             // LDS row pitch of the R tile in bytes
    static constexpr int LP = 2 * RB * 16 * 2 + 16;        // LDS row pitch of the L tile (value | residual) in bytes
    static constexpr int R_BYTES = GRAD_TT * RPITCH, L_BYTES = GRAD_TT * LP, BYTES = R_BYTES + L_BYTES;
};
template <int RB, bool CMAJOR>
__device__ __forceinline__ void lora_grad_walk(const GradParams& p, const GradItem& it, const SegDesc& sd, int block, unsigned char* sR, unsigned char* sL) {
    constexpr int CT = GradWalk<RB>::CT, NI = CT / 64;      // columns per workgroup, 16-column blocks per wavefront
    constexpr int RPITCH = GradWalk<RB>::RPITCH, LP = GradWalk<RB>::LP;
    constexpr int LPRW = CT / 8, NRC = GRAD_TT * LPRW / 256;   // 16-byte chunks per R row, R chunks per thread
    const int s = it.seg;
    const int t_lo = it.t_lo, t_hi = it.t_hi;
    const bf16* const rbase = p.R_seg ? p.R_seg[s] - (size_t)p.off[s] * p.ncols : p.R;
    const int c0 = block * CT;
    const int nb = sd.rpad >> 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    floatx4 acc[NI][RB];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < RB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    // R tile: 32 rows x CT/8 chunks of 8 columns, NRC per thread.  L tile: 32 x (rpad/4) chunks,
    // at most NLC per thread.  Two register sets: the chunks of tokens t0 + 64 are requested as soon as those
    // of t0 are in LDS (their set is free then), so a request has two steps to arrive (a step is far shorter than the memory
    // latency, and a launch over a few segments has too few workgroups per CU to hide it otherwise).
    // Every load is unconditional: out-of-range chunks read a valid address and count as zero when they go
    // to LDS, two steps later.  (With the zeroing next to the load the compiler puts the load under the
    // condition, and a load that may or may not have been issued makes it wait for all of them, the
    // newest request included.)
    constexpr int NLC = (GRAD_TT * 4 * RB + 255) / 256;
    const int lw = sd.rpad >> 2;                       // 16-byte chunks per L row: 2 * rpad bf16
    const int l_chunks = GRAD_TT * lw;
    struct Stage { u32x4 rr[NRC]; u32x4 lv[NLC]; };
    const bool col_ok = (c0 + (tid % LPRW) * 8) < p.ncols;
    auto fetch = [&](Stage& sg, int t0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NRC; ++i) {
            const int c = tid + i * 256, tr = c / LPRW, cc = c % LPRW;
            sg.rr[i] = ld_glb16(rbase + (size_t)min(t0 + tr, t_hi - 1) * p.ncols + c0 + (col_ok ? cc * 8 : 0));
        }
#pragma unroll
        for (int i = 0; i < NLC; ++i) {
            const int c = tid + i * 256, tr = c / lw, pc = c % lw;
            sg.lv[i] = ld_glb16(p.L + (size_t)min(t0 + tr, t_hi - 1) * p.l_pitch + pc * 8);
        }
    };
    // the chunks of tokens t0.., landed (see step), go to LDS
    auto put = [&](const Stage& sg, int t0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NRC; ++i) {
            const int c = tid + i * 256, tr = c / LPRW, cc = c % LPRW;
            const bool ok = (t0 + tr) < t_hi && col_ok;
            *reinterpret_cast<u32x4*>(sR + tr * RPITCH + cc * 16) = ok ? sg.rr[i] : u32x4{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (int i = 0; i < NLC; ++i) {
            const int c = tid + i * 256, tr = c / lw, pc = c % lw;
            if (c < l_chunks) *reinterpret_cast<u32x4*>(sL + tr * LP + pc * 16) = (t0 + tr) < t_hi ? sg.lv[i] : u32x4{0u, 0u, 0u, 0u};
        }
    };
    auto multiply = [&]() __attribute__((always_inline)) {
        bf16x8 rf[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) rf[i] = lds_read_tr_16x32(sR, RPITCH, wave * (NI * 16) + i * 16, lane);
#pragma unroll
        for (int j = 0; j < RB; ++j) {
            if (j < nb) {
#pragma unroll
                for (int half = 0; half < 2; ++half) {      // bf16 value, then its rounding residual
                    const bf16x8 lf = lds_read_tr_16x32(sL, LP, half * sd.rpad + j * 16, lane);
#pragma unroll
                    for (int i = 0; i < NI; ++i) {
                        if constexpr (CMAJOR) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lf, rf[i], acc[i][j], 0, 0, 0);
                        else acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(rf[i], lf, acc[i][j], 0, 0, 0);
                    }
                }
            }
        }
    };
    if (t_lo < t_hi) {
        Stage sg0, sg1;
        fetch(sg0, t_lo);
        fetch(sg1, t_lo + GRAD_TT);
        // Two register sets, two tiles in flight: a set is free again as soon as its tile is in LDS, so the
        // tile two steps ahead is requested into it; cur was requested two fetches ago, and the wait for it
        // leaves the newest fetch in flight.
        auto step = [&](Stage& cur, int t0) __attribute__((always_inline)) {
            __syncthreads();     // previous step's LDS reads are done
            put(cur, t0);
            __syncthreads();
            fetch(cur, t0 + 2 * GRAD_TT);
            multiply();
        };
        for (int t0 = t_lo; t0 < t_hi; t0 += 2 * GRAD_TT) {
            step(sg0, t0);
            if (t0 + GRAD_TT < t_hi) step(sg1, t0 + GRAD_TT);
        }
    }
    float* out = it.direct ? (CMAJOR ? sd.dB : sd.dA) : p.partial + it.partial_off;
    const bool accumulate = it.direct && p.accumulate;
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < RB; ++j) {
            if (j < nb) {
                if constexpr (CMAJOR) {
                    // lane: column c = .. + (lane & 15); registers: pp = j*16 + 4*(lane >> 4) + q
                    const int c = c0 + wave * (NI * 16) + i * 16 + (lane & 15);
                    if (c < p.ncols) {
                        const int pp0 = j * 16 + ((lane >> 4) << 2);
                        float* dst = out + (size_t)c * sd.rank + pp0;
                        float old[4] = {0.f, 0.f, 0.f, 0.f};        // all four read before the first store
                        if (accumulate) {
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                if (pp0 + q < sd.rank) old[q] = dst[q];
                        }
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (pp0 + q < sd.rank) dst[q] = old[q] + acc[i][j][q];
                    }
                } else {
                    // lane: pp = j*16 + (lane & 15); registers: column c = .. + 4*(lane >> 4) + q
                    const int pp = j * 16 + (lane & 15);
                    const int c = c0 + wave * (NI * 16) + i * 16 + ((lane >> 4) << 2);
                    if (pp < sd.rank && c < p.ncols) {
                        float4* dst = reinterpret_cast<float4*>(out + (size_t)pp * p.ncols + c);
                        float4 v = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
                        if (accumulate) { const float4 o = *dst; v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w; }
                        *dst = v;
                    }
                }
            }
        }
}

template <int RB, bool CMAJOR>
SYMB_KERNEL void __launch_bounds__(256)
symb_lora_grad_kernel(const GradParams p) {
    __shared__ __attribute__((aligned(16))) unsigned char sR[GradWalk<RB>::R_BYTES], sL[GradWalk<RB>::L_BYTES];
    const GradItem it = p.items[blockIdx.y];
    const SegDesc sd = p.seg[it.seg];
    lora_grad_walk<RB, CMAJOR>(p, it, sd, blockIdx.x, sR, sL);
}

// -------------------------------------------------------------------------------------------
// The same gradients for ranks up to 64, with the tokens of a work item dealt out over the wavefronts: each takes every fourth
// slice of 32 tokens, brings its rows of R and L in by LDS DMA into two buffers of its own (no workgroup barrier in the loop) and
// accumulates all 128 columns; the wavefronts' sums meet in LDS in a fixed order at the end.  Bound by HBM (R once).  A launch of few
// workgroups lasts as long as its longest walk, which is a quarter as many steps as in symb_lora_grad_kernel: dB of 16 segments of 1024 tokens,
// 256 columns, rank 8, 25.3 -> 12.2 us; 13 runs of 5120 tokens of ranks 8 to 64, 4096 columns, dB 43.5 -> 34.3, dA 35.5 -> 26.9.  But a workgroup
// takes 80 to 128 KiB of LDS, where the other kernel's takes 17 to 19, and adds four sets of sums up, so launches of many workgroups, and short
// segments, are that kernel's (16-row segments, 64 of them, dA + dB on 4096 columns: rank 8 17 us against 30, rank 32 34 / 77): grad_wave()
// in the host code has the line.  Above rank 64 the L rows, re-read by every column block, outweigh R and their LDS halves the tile (20 clients of
// 1024 tokens at rank 128 on 6144 -> 256: the gradient call 387 us against 300): those segments always keep that walk.  So does dB of layers of
// GRAD_WIDE columns and more, where one pass over dY forms dB and dH in that kernel's order, and the two ways to a gradient give the
// same bits.
// R slice: 32 token rows of 128 columns, L slice: 32 rows of 2 rpad, 32-byte pieces of row t stored at piece ^ skinny_bt_swz (rows of
// 64 elements and more).  Tokens past the item's last one repeat it and are masked in the fragments of the last slice.
// -------------------------------------------------------------------------------------------
constexpr int GRAD_WIDE = 63 * 256 + 1;       // more than 63 blocks of 256 columns
constexpr int GRAD_WAVE_CT = 128, GRAD_WAVE_RANK = 64;
template <int RB>
struct GradWave {
    static constexpr int CT = GRAD_WAVE_CT, RREQ = CT / 16, LREQ = 2 * RB, REQ = RREQ + LREQ, NBUF = 2;
    static constexpr int SLICE = REQ * 1024, WAVE = NBUF * SLICE, BYTES = 4 * WAVE, NI = CT / 16;
    static_assert(4 * NI * RB * 1024 <= BYTES, "the wavefronts' sums fit the slice buffers");
};
template <int RB, bool CMAJOR>
__device__ __forceinline__ void lora_grad_wave(const GradParams& p, const GradItem& it, const SegDesc& sd, int block, unsigned char* smem) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    using GW = GradWave<RB>;
    constexpr int CT = GW::CT, NI = GW::NI;
    const int s = it.seg;
    const int t_lo = it.t_lo, t_hi = it.t_hi;
    const bf16* const rbase = p.R_seg ? p.R_seg[s] - (size_t)p.off[s] * p.ncols : p.R;
    const int c0 = block * CT, nb = sd.rpad >> 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l15 = lane & 15, kq = lane >> 4;
    unsigned char* const wbuf = smem + wave * GW::WAVE;
    // this lane's 16 bytes of every DMA request of a slice: token of the slice and column
    constexpr int RPR = 512 / CT;                        // R rows per request
    int rcol[GW::RREQ], ltok[GW::LREQ], lcol[GW::LREQ];
#pragma unroll
    for (int i = 0; i < GW::RREQ; ++i) {
        const int t = i * RPR + lane / (CT / 8), slot = lane % (CT / 8);
        rcol[i] = min(c0 + ((slot ^ (skinny_bt_swz(CT, t) << 1)) * 8), p.ncols - 8);
    }
    const int lw = sd.rpad >> 2;                         // 16-byte chunks per L row
#pragma unroll
    for (int i = 0; i < GW::LREQ; ++i) {
        const int x = min(i * 64 + lane, 32 * lw - 1);
        ltok[i] = x / lw;
        lcol[i] = ((x - ltok[i] * lw) ^ (skinny_bt_swz(2 * sd.rpad, ltok[i]) << 1)) * 8;
    }
    unsigned roff[NI], loff[RB][2];
    const int k0 = kq * 8 + (l15 >> 2);                  // first of the two transposing reads; the second is 4 tokens further
#pragma unroll
    for (int i = 0; i < NI; ++i) roff[i] = (unsigned)(size_t)wbuf + (unsigned)(k0 * CT * 2 + ((i ^ skinny_bt_swz(CT, k0)) * 32) + (l15 & 3) * 8);
#pragma unroll
    for (int j = 0; j < RB; ++j)
#pragma unroll
        for (int half = 0; half < 2; ++half)
            loff[j][half] = (unsigned)(size_t)wbuf + (unsigned)(GW::RREQ * 1024 + k0 * 4 * sd.rpad + (((half * nb + min(j, nb - 1)) ^ skinny_bt_swz(2 * sd.rpad, k0)) * 32) + (l15 & 3) * 8);
    floatx4 acc[NI][RB];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < RB; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto dma = [&](int buf, int t0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < GW::RREQ; ++i)
            __builtin_amdgcn_global_load_lds((glb_void_t*)(rbase + (size_t)min(t0 + i * RPR + lane / (CT / 8), t_hi - 1) * p.ncols + rcol[i]),
                                             (lds_void_t*)(wbuf + buf * GW::SLICE + i * 1024), 16, 0, 0);
#pragma unroll
        for (int i = 0; i < GW::LREQ; ++i)
            __builtin_amdgcn_global_load_lds((glb_void_t*)(p.L + (size_t)min(t0 + ltok[i], t_hi - 1) * p.l_pitch + lcol[i]),
                                             (lds_void_t*)(wbuf + buf * GW::SLICE + (GW::RREQ + i) * 1024), 16, 0, 0);
    };
    // fragment reads with a wait of their own (see the skinny kernel); returns with the buffer free again
    auto mul = [&](int buf, int t0) __attribute__((always_inline)) {
        u32x2 rt[NI][2], lt[RB][2][2];
        const unsigned at = (unsigned)(buf * GW::SLICE), lrow = 16 * sd.rpad;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(rt[i][0]) : "v"(roff[i] + at));
            asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(rt[i][1]) : "v"(roff[i] + at), "n"(CT * 8));
        }
#pragma unroll
        for (int j = 0; j < RB; ++j)
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(lt[j][half][0]) : "v"(loff[j][half] + at));
                asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(lt[j][half][1]) : "v"(loff[j][half] + at + lrow));
            }
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
#pragma unroll
        for (int i = 0; i < NI; ++i) { asm volatile("" : "+v"(rt[i][0])); asm volatile("" : "+v"(rt[i][1])); }
#pragma unroll
        for (int j = 0; j < RB; ++j)
#pragma unroll
            for (int half = 0; half < 2; ++half) { asm volatile("" : "+v"(lt[j][half][0])); asm volatile("" : "+v"(lt[j][half][1])); }
        u32x4 rf[NI], lf[RB][2];
#pragma unroll
        for (int i = 0; i < NI; ++i) rf[i] = __builtin_shufflevector(rt[i][0], rt[i][1], 0, 1, 2, 3);
#pragma unroll
        for (int j = 0; j < RB; ++j)
#pragma unroll
            for (int half = 0; half < 2; ++half) lf[j][half] = __builtin_shufflevector(lt[j][half][0], lt[j][half][1], 0, 1, 2, 3);
        if (t0 + 32 > t_hi) {                            // a lane holds tokens t0 + 8 kq + 0..7: those past the end count as zero, in both operands
            const int left = t_hi - (t0 + kq * 8);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const unsigned keep = 2 * q + 1 < left ? 0xffffffffu : 2 * q < left ? 0xffffu : 0u;
#pragma unroll
                for (int i = 0; i < NI; ++i) rf[i][q] &= keep;
#pragma unroll
                for (int j = 0; j < RB; ++j) { lf[j][0][q] &= keep; lf[j][1][q] &= keep; }
            }
        }
#pragma unroll
        for (int j = 0; j < RB; ++j)
            if (j < nb) {
#pragma unroll
                for (int half = 0; half < 2; ++half)     // bf16 value, then its rounding residual
#pragma unroll
                    for (int i = 0; i < NI; ++i) {
                        const bf16x8 l = __builtin_bit_cast(bf16x8, lf[j][half]), r = __builtin_bit_cast(bf16x8, rf[i]);
                        acc[i][j] = CMAJOR ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(l, r, acc[i][j], 0, 0, 0)
                                           : __builtin_amdgcn_mfma_f32_16x16x32_bf16(r, l, acc[i][j], 0, 0, 0);
                    }
            }
    };
    const int nsl = (t_hi - t_lo + 31) >> 5, ns = nsl > wave ? (nsl - wave + 3) >> 2 : 0;
    int t = t_lo + wave * 32;
    if (ns > 0) dma(0, t);
    if (ns > 1) dma(1, t + 128);
    for (int q = 0; q < ns; ++q, t += 128) {
        if (q + 1 < ns) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(GW::REQ) : "memory");       // the next slice may still be in flight
        else asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        mul(q & 1, t);
        if (q + 2 < ns) dma(q & 1, t + 256);
    }
    floatx4* const red = reinterpret_cast<floatx4*>(smem);
    __syncthreads();                                     // every wavefront is done with its slice buffers
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < RB; ++j) red[((wave * NI + i) * RB + j) * 64 + lane] = acc[i][j];
    __syncthreads();
    float* const out = it.direct ? (CMAJOR ? sd.dB : sd.dA) : p.partial + it.partial_off;
    const bool accumulate = it.direct && p.accumulate;
#pragma unroll
    for (int b = 0; b < NI * RB; ++b) {
        const int i = b / RB, j = b % RB;
        if ((b & 3) != wave || j >= nb) continue;
        floatx4 v = red[b * 64 + lane];
#pragma unroll
        for (int w = 1; w < 4; ++w) v += red[(w * NI * RB + b) * 64 + lane];
        if constexpr (CMAJOR) {
            // lane: column c = .. + l15; registers: pp = 16 j + 4 kq + q
            const int c = c0 + i * 16 + l15, pp0 = j * 16 + kq * 4;
            if (c < p.ncols) {
                float* const dst = out + (size_t)c * sd.rank + pp0;
                float old[4] = {0.f, 0.f, 0.f, 0.f};     // all four read before the first store
                if (accumulate) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (pp0 + q < sd.rank) old[q] = dst[q];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (pp0 + q < sd.rank) dst[q] = old[q] + v[q];
            }
        } else {
            // lane: pp = 16 j + l15; registers: column c = .. + 4 kq + q
            const int pp = j * 16 + l15, c = c0 + i * 16 + kq * 4;
            if (pp < sd.rank && c < p.ncols) {
                floatx4* const dst = reinterpret_cast<floatx4*>(out + (size_t)pp * p.ncols + c);
                *dst = accumulate ? v + *dst : v;
            }
        }
    }
}

// RB: rank blocks of the widest segment of the launch.  The segments' own ones decide what each workgroup runs (above rank 64 the other
// kernel's walk): one launch lets the short walks of low ranks fill the CUs beside the long ones.
template <int RB, bool CMAJOR>
SYMB_KERNEL void __launch_bounds__(256)
symb_lora_grad_wave_kernel(const GradParams p) {
    constexpr int WB = RB < 4 ? RB : 4;
    __shared__ __attribute__((aligned(16))) unsigned char smem[GradWave<WB>::BYTES];
    static_assert(GRAD_CT<8> == GRAD_WAVE_CT && GradWalk<8>::BYTES <= GradWave<4>::BYTES, "both walks share a grid and the LDS");
    const GradItem it = p.items[blockIdx.y];
    const SegDesc sd = p.seg[it.seg];
    if (sd.rpad <= 16) lora_grad_wave<1, CMAJOR>(p, it, sd, blockIdx.x, smem);
    else if constexpr (RB >= 2) {
        if (sd.rpad <= 32) lora_grad_wave<2, CMAJOR>(p, it, sd, blockIdx.x, smem);
        else if constexpr (RB >= 4) {
            if (sd.rpad <= GRAD_WAVE_RANK) lora_grad_wave<4, CMAJOR>(p, it, sd, blockIdx.x, smem);
            else if constexpr (RB >= 8) lora_grad_walk<8, CMAJOR>(p, it, sd, blockIdx.x, smem, smem + GradWalk<8>::R_BYTES);
        }
    }
}

// dH of a gradient call beside its dB, ranks up to 64: nchunks workgroups of the backward shrink, then those of dB.  Neither needs the
// other's result, and a small call's time is its launches: training step of 4 x 64 tokens on 768 columns 46.9 -> 43.0 us.  wave: see grad_wave()
// in the host code (without it ranks above 32, whose walk has blocks of 128 columns too).
template <int RB>
SYMB_KERNEL void __launch_bounds__(256)
symb_lora_grad_pair_kernel(const SkinnyParams sp, int nchunks, const GradParams gp, int col_blocks, int wave) {
    constexpr int BYTES = SkinnyBuild<RB, SKINNY_DEEP>::BYTES > GradWave<RB>::BYTES ? SkinnyBuild<RB, SKINNY_DEEP>::BYTES : GradWave<RB>::BYTES;
    __shared__ __attribute__((aligned(16))) unsigned char smem[BYTES];
    if ((int)blockIdx.x < nchunks) {
        skinny_chunk<RB, SKINNY_DEEP, true>(sp, blockIdx.x, smem);
        return;
    }
    const int g = blockIdx.x - nchunks, block = g % col_blocks;
    const GradItem it = gp.items[g / col_blocks];
    const SegDesc sd = gp.seg[it.seg];
    if constexpr (RB == 4) {
        static_assert(GRAD_CT<4> == GRAD_WAVE_CT && GradWalk<4>::BYTES <= BYTES, "both walks share a grid and the LDS");
        if (!wave) {
            lora_grad_walk<4, true>(gp, it, sd, block, smem, smem + GradWalk<4>::R_BYTES);
            return;
        }
    }
    if (sd.rpad <= 16) lora_grad_wave<1, true>(gp, it, sd, block, smem);
    else if constexpr (RB >= 2) {
        if (sd.rpad <= 32) lora_grad_wave<2, true>(gp, it, sd, block, smem);
        else if constexpr (RB >= 4) lora_grad_wave<4, true>(gp, it, sd, block, smem);
    }
}

// -------------------------------------------------------------------------------------------
// dA, dB and dH of short segments (at most 64 tokens, ranks up to 16) in one launch.  Such a call is its launches: dA wants dH, so that beside dB in one launch (above) dH
// still was a launch before dA's.  Here every workgroup of dA forms dH of its whole segment itself, (tokens + 16) d_out products' operands from L2, while its columns of X are on
// their way; the first of a segment leaves it in the workspace.  A segment's tokens are at most two steps of the matrix cores: the eight wavefronts take 16 of the workgroup's 128 columns
// each, with no sums between them.  Training step of 16 tokens, 4096 x 4096, 9.8 us in two launches, 7.1 here, the step 34.7 -> 31.0; of 4 x 64 tokens on
// 768 columns 26.5 -> 25.7 (bound by the host's three calls).
// -------------------------------------------------------------------------------------------
constexpr int GRAD_SHORT_TOKENS = 64, GRAD_SHORT_CT = 128;
struct GradShort {
    using ST1 = SkinnyStage<1, 3, true, 1, 8>;           // up to 16 tokens
    using ST2 = SkinnyStage<1, 2, true, 2, 8>;           // 32 at a time
    static constexpr int STAGE = ST1::BYTES > ST2::BYTES ? ST1::BYTES : ST2::BYTES;
    static constexpr int X_BYTES = GRAD_SHORT_TOKENS * GRAD_SHORT_CT * 2, L_BYTES = GRAD_SHORT_TOKENS * 64, BYTES = STAGE + X_BYTES + L_BYTES;
    static_assert(8 * 32 * 20 * 4 <= STAGE, "the wavefronts' sums of dH");
};
template <bool CMAJOR>
__device__ __forceinline__ void lora_grad_short(const GradParams& p, const SkinnyParams& sp, const GradItem& it, const SegDesc& sd, int block, unsigned char* smem) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    constexpr int CT = GRAD_SHORT_CT;
    const int s = it.seg, t_lo = it.t_lo, n = it.t_hi - it.t_lo;
    const bf16* const rbase = p.R_seg ? p.R_seg[s] - (size_t)p.off[s] * p.ncols : p.R;
    const int c0 = block * CT, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l15 = lane & 15, kq = lane >> 4;
    unsigned char* const sX = smem + GradShort::STAGE;   // [token][128 columns], 32-byte pieces of row t at piece ^ skinny_bt_swz
    unsigned char* const sL = sX + GradShort::X_BYTES;   // [token][16 values | 16 residuals]
    for (int i = wave; i * 4 < n; i += 8) {              // four rows of X (dY) per request; past the last token it again
        const int t = i * 4 + (lane >> 4), slot = lane & 15;
        const bf16* const src = rbase + (size_t)(t_lo + min(t, n - 1)) * p.ncols + min(c0 + ((slot ^ (skinny_bt_swz(CT, t) << 1)) * 8), p.ncols - 8);
        __builtin_amdgcn_global_load_lds((glb_void_t*)src, (lds_void_t*)(sX + i * 1024), 16, 0, 0);
    }
    if constexpr (CMAJOR) {
        for (int i = wave; i * 16 < n; i += 8)
            __builtin_amdgcn_global_load_lds((glb_void_t*)(p.L + (size_t)(t_lo + min(i * 16 + (lane >> 2), n - 1)) * p.l_pitch + (lane & 3) * 8), (lds_void_t*)(sL + i * 1024), 16, 0, 0);
    } else {
        auto part = [&](auto STC, int at, int rows) __attribute__((always_inline)) {
            using ST = typename decltype(STC)::type;
            skinny_rows<1, ST, true>(sp, RowChunk{s, t_lo + at, rows, 0}, sd, smem, [&](int t, int pp, uint2 hi, uint2 lo) __attribute__((always_inline)) {
                *reinterpret_cast<uint2*>(sL + (at + t) * 64 + pp * 2) = hi;
                *reinterpret_cast<uint2*>(sL + (at + t) * 64 + 32 + pp * 2) = lo;
                if (block) return;
                bf16* const row = sp.out + (size_t)(t_lo + at + t) * sp.out_pitch + pp;
                *reinterpret_cast<uint2*>(row) = hi;
                *reinterpret_cast<uint2*>(row + 16) = lo;
            });
        };
        if (n <= 16) part(std::enable_if<true, GradShort::ST1>{}, 0, n);
        else
            for (int at = 0; at < n; at += 32) {
                if (at) __syncthreads();                 // the sums of the first 32 tokens are read
                part(std::enable_if<true, GradShort::ST2>{}, at, min(n - at, 32));
            }
    }
    asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
    __syncthreads();
    // fragment reads with a wait of their own (see the skinny kernel)
    const int k0 = kq * 8 + (l15 >> 2);                  // first of the two transposing reads; the second is 4 tokens further
    const unsigned roff = (unsigned)(size_t)sX + (unsigned)(k0 * CT * 2 + ((wave ^ skinny_bt_swz(CT, k0)) * 32) + (l15 & 3) * 8);
    const unsigned loff = (unsigned)(size_t)sL + (unsigned)(k0 * 64 + (l15 & 3) * 8);
    floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};           // a sum per 32 tokens, added up: the bits of the kernel that deals them out over its wavefronts
    for (int t0 = 0; t0 < n; t0 += 32) {
        floatx4 part = floatx4{0.f, 0.f, 0.f, 0.f};
        u32x2 rt[2], lt[2][2];
        const unsigned ra = roff + t0 * CT * 2, la = loff + t0 * 64;
        asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(rt[0]) : "v"(ra));
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:1024" : "=v"(rt[1]) : "v"(ra));
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(lt[half][0]) : "v"(la + half * 32));
            asm volatile("ds_read_b64_tr_b16 %0, %1 offset:256" : "=v"(lt[half][1]) : "v"(la + half * 32));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
        asm volatile("" : "+v"(rt[0])); asm volatile("" : "+v"(rt[1]));
#pragma unroll
        for (int half = 0; half < 2; ++half) { asm volatile("" : "+v"(lt[half][0])); asm volatile("" : "+v"(lt[half][1])); }
        u32x4 rf = __builtin_shufflevector(rt[0], rt[1], 0, 1, 2, 3);
        u32x4 lf[2] = {__builtin_shufflevector(lt[0][0], lt[0][1], 0, 1, 2, 3), __builtin_shufflevector(lt[1][0], lt[1][1], 0, 1, 2, 3)};
        const int left = n - (t0 + kq * 8);              // a lane holds tokens t0 + 8 kq + 0..7: those past the end count as zero, in both operands
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned keep = 2 * q + 1 < left ? 0xffffffffu : 2 * q < left ? 0xffffu : 0u;
            rf[q] &= keep;
            lf[0][q] &= keep;
            lf[1][q] &= keep;
        }
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const bf16x8 l = __builtin_bit_cast(bf16x8, lf[half]), r = __builtin_bit_cast(bf16x8, rf);
            part = CMAJOR ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(l, r, part, 0, 0, 0) : __builtin_amdgcn_mfma_f32_16x16x32_bf16(r, l, part, 0, 0, 0);
        }
        acc += part;
    }
    if constexpr (CMAJOR) {                              // lane: column l15 of the wavefront's; registers: ranks 4 kq ..
        const int c = c0 + wave * 16 + l15;
        float* const dst = sd.dB + (size_t)c * sd.rank + kq * 4;
        if (c >= p.ncols) return;
        float old[4] = {0.f, 0.f, 0.f, 0.f};             // all four read before the first store
        if (p.accumulate) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (kq * 4 + q < sd.rank) old[q] = dst[q];
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (kq * 4 + q < sd.rank) dst[q] = old[q] + acc[q];
    } else {                                             // lane: rank l15; registers: columns 4 kq ..
        const int c = c0 + wave * 16 + kq * 4;
        if (l15 >= sd.rank || c >= p.ncols) return;
        floatx4* const dst = reinterpret_cast<floatx4*>(sd.dA + (size_t)l15 * p.ncols + c);
        *dst = p.accumulate ? acc + *dst : acc;
    }
}
// grid = (column blocks of dA) x segments, then (column blocks of dB) x segments; sp: the shrink of the backward, without chunks.
SYMB_KERNEL void __launch_bounds__(512)
symb_lora_grad_short_kernel(const SkinnyParams sp, const GradParams ga, int a_blocks, int a_groups, const GradParams gb, int b_blocks) {
    __shared__ __attribute__((aligned(16))) unsigned char smem[GradShort::BYTES];
    if ((int)blockIdx.x < a_groups) {
        const GradItem it = ga.items[blockIdx.x / a_blocks];
        lora_grad_short<false>(ga, sp, it, ga.seg[it.seg], blockIdx.x % a_blocks, smem);
    } else {
        const int g = blockIdx.x - a_groups;
        const GradItem it = gb.items[g / b_blocks];
        lora_grad_short<true>(gb, sp, it, gb.seg[it.seg], g % b_blocks, smem);
    }
}

// -------------------------------------------------------------------------------------------
// dB_i and dH_i in ONE pass over dY (ranks up to 16).  Both products contract dY:
//   dB_i[c][pp] = sum_t dY[t][c] * Hs[t][pp]            (over the segment's tokens)
//   dH[t][pp]   = s_i * sum_c dY[t][c] * B_i[c][pp]     (over the output columns)
// and dY is by far the largest tensor either reads (T x d_out), so reading it once instead of
// twice saves its bytes.  A workgroup owns G column blocks of 256 columns of one work item
// (a segment, or a run of a long one) and walks its tokens 32 at a time; per step it visits its
// column blocks in turn: the dY tile goes through LDS as in symb_lora_grad_kernel and feeds
// (a) the dB accumulators of that block (transposing LDS reads, token-contracted) and (b) a
// 32 x 16 partial of dH over the block's columns (plain LDS reads, B_i^T fragments held
// in registers).  After the last block of a step the four wavefronts' dH partials
// meet in LDS and the sum goes to dh_partial[group][t][16]; symb_dh_finish_kernel adds the
// groups in order, scales by s_i and writes dH as value + residual.  Fixed summation order
// everywhere: deterministic, no atomics.  dB comes out bit-identical to symb_lora_grad_kernel's.
// -------------------------------------------------------------------------------------------
struct DhDbParams {
    const bf16* R;            // dY [T][ncols]
    const bf16* L;            // Hs [T][l_pitch]: per row 16 values then 16 residuals
    int ncols, l_pitch;
    const int32_t* off;
    const SegDesc* seg;
    const GradItem* items;
    int accumulate;
    const bf16* const* R_seg;
    float* partial;           // dB runs of split segments
    float* dh_partial;        // [gridDim.x][T][16] fp32
    int T;
};

template <int I0, int I1, class F>
__device__ __forceinline__ void grad_static_for(F&& f) {
    if constexpr (I0 < I1) {
        f(std::integral_constant<int, I0>{});
        grad_static_for<I0 + 1, I1>(f);
    }
}

template <int G>
SYMB_KERNEL void __launch_bounds__(256)
symb_lora_dhdb_kernel(const DhDbParams p) {
    constexpr int CT = 256, NI = CT / 64;
    constexpr int RPITCH = CT * 2 + 16, LPRW = CT / 8, NRC = GRAD_TT * LPRW / 256;
    constexpr int LP = 2 * 16 * 2 + 16;
    __shared__ __attribute__((aligned(16))) unsigned char sR[GRAD_TT * RPITCH];
    __shared__ __attribute__((aligned(16))) unsigned char sL[GRAD_TT * LP];
    __shared__ __attribute__((aligned(16))) float red[4][GRAD_TT][16 + 4];
    const GradItem it = p.items[blockIdx.y];
    const int s = it.seg;
    const SegDesc sd = p.seg[s];
    const int t_lo = it.t_lo, t_hi = it.t_hi;
    const bf16* const rbase = p.R_seg ? p.R_seg[s] - (size_t)p.off[s] * p.ncols : p.R;
    const int nblk = (p.ncols + CT - 1) / CT;
    const int cb0 = blockIdx.x * G, ncb = min(G, nblk - cb0);     // this workgroup's column blocks (uniform)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    floatx4 acc[G][NI];                                  // dB of every block of the group
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int i = 0; i < NI; ++i) acc[g][i] = floatx4{0.f, 0.f, 0.f, 0.f};
    // B_i^T fragments of this wavefront's 64 columns of every block: lane holds rank row lane & 15,
    // columns 8 (lane >> 4) .. + 7 of each of the two 32-column steps
    u32x4 btf[G][2];
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int c = (cb0 + g) * CT + wave * 64 + ks * 32 + (lane >> 4) * 8;
            const bool ok = g < ncb && c < p.ncols;
            // (element loads from B_i [ncols][rank]: once per workgroup)
            const int pr = lane & 15;
            const unsigned short* const e = reinterpret_cast<const unsigned short*>(sd.B) + (size_t)(ok ? c : 0) * sd.rank + min(pr, sd.rank - 1);
#pragma unroll
            for (int q = 0; q < 4; ++q) btf[g][ks][q] = e[(size_t)(2 * q) * sd.rank] | ((unsigned)e[(size_t)(2 * q + 1) * sd.rank] << 16);
            if (!ok || pr >= sd.rank) btf[g][ks] = u32x4{0u, 0u, 0u, 0u};
        }

    struct Stage { u32x4 rr[NRC]; u32x4 lv; };
    const int l_chunks = GRAD_TT * 4;                    // 16-byte chunks of the L tile: 32 rows x 64 bytes (16 values + 16 residuals)
    const int l_tr = (tid & 127) >> 2, l_pc = tid & 3;    // this thread's chunk of it
    // unconditional loads, zeroed on their way to LDS (see symb_lora_grad_kernel)
    auto fetch = [&](Stage& sg, int t0, int g) __attribute__((always_inline)) {
        const int c0 = (cb0 + min(g, ncb - 1)) * CT;
        const bool col_ok = (c0 + (tid % LPRW) * 8) < p.ncols;
#pragma unroll
        for (int i = 0; i < NRC; ++i) {
            const int c = tid + i * 256, tr = c / LPRW, cc = c % LPRW;
            sg.rr[i] = ld_glb16(rbase + (size_t)min(t0 + tr, t_hi - 1) * p.ncols + c0 + (col_ok ? cc * 8 : 0));
        }
        sg.lv = ld_glb16(p.L + (size_t)min(t0 + l_tr, t_hi - 1) * p.l_pitch + l_pc * 8);
    };
    auto put = [&](const Stage& sg, int t0, int g) __attribute__((always_inline)) {
        const int c0 = (cb0 + g) * CT;
        const bool col_ok = (c0 + (tid % LPRW) * 8) < p.ncols;
#pragma unroll
        for (int i = 0; i < NRC; ++i) {
            const int c = tid + i * 256, tr = c / LPRW, cc = c % LPRW;
            const bool ok = (t0 + tr) < t_hi && col_ok;
            *reinterpret_cast<u32x4*>(sR + tr * RPITCH + cc * 16) = ok ? sg.rr[i] : u32x4{0u, 0u, 0u, 0u};
        }
        if (g == 0 && tid < l_chunks)                    // the Hs rows of a step are the same for all its blocks
            *reinterpret_cast<u32x4*>(sL + l_tr * LP + l_pc * 16) = (t0 + l_tr) < t_hi ? sg.lv : u32x4{0u, 0u, 0u, 0u};
    };
    floatx4 dh[2];                                       // dH partial of the step: token blocks 0 / 1, this wavefront's columns
    auto multiply = [&](auto GC) __attribute__((always_inline)) {
        constexpr int g = decltype(GC)::value;
        bf16x8 rf[NI];
#pragma unroll
        for (int i = 0; i < NI; ++i) rf[i] = lds_read_tr_16x32(sR, RPITCH, wave * (NI * 16) + i * 16, lane);
#pragma unroll
        for (int half = 0; half < 2; ++half) {           // Hs value, then its rounding residual
            const bf16x8 lf = lds_read_tr_16x32(sL, LP, half * 16, lane);
#pragma unroll
            for (int i = 0; i < NI; ++i) acc[g][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lf, rf[i], acc[g][i], 0, 0, 0);
        }
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const u32x4 yv = *reinterpret_cast<const u32x4*>(sR + (tb * 16 + (lane & 15)) * RPITCH + (wave * 64 + ks * 32 + (lane >> 4) * 8) * 2);
                dh[tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, btf[g][ks]), __builtin_bit_cast(bf16x8, yv), dh[tb], 0, 0, 0);
            }
    };
    // One tile = (token step, column block), blocks fastest.  Two register sets, the tile two ahead is
    // requested as soon as the current one is in LDS.
    auto advance = [&](int& t0, int& g) __attribute__((always_inline)) {
        if (++g == ncb) { g = 0; t0 += GRAD_TT; }
    };
    if (t_lo < t_hi) {
        Stage sg0, sg1;
        int ft = t_lo, fg = 0;                           // the next tile to request
        fetch(sg0, ft, fg); advance(ft, fg);
        fetch(sg1, ft, fg); advance(ft, fg);
        int t0 = t_lo, g = 0;                            // the tile being computed
        auto step = [&](Stage& cur) __attribute__((always_inline)) {
            if (g == 0) dh[0] = dh[1] = floatx4{0.f, 0.f, 0.f, 0.f};
            __syncthreads();                             // the previous tile's LDS reads are done
            put(cur, t0, g);
            __syncthreads();
            fetch(cur, ft, fg); advance(ft, fg);         // the set is free again: the tile two steps ahead goes into it
            // the block index selects registers: dispatch on it (uniform)
            grad_static_for<0, G>([&](auto GC) __attribute__((always_inline)) {
                if (g == decltype(GC)::value) multiply(GC);
            });
            if (g == ncb - 1) {
                // the step's dH partial over this workgroup's columns: wavefronts meet in LDS, fixed order
#pragma unroll
                for (int tb = 0; tb < 2; ++tb)
                    *reinterpret_cast<float4*>(&red[wave][tb * 16 + (lane & 15)][(lane >> 4) * 4]) = make_float4(dh[tb][0], dh[tb][1], dh[tb][2], dh[tb][3]);
                __syncthreads();
                if (tid < GRAD_TT * 4) {
                    const int tr = tid >> 2, q = (tid & 3) * 4;
                    if (t0 + tr < t_hi) {
                        float4 v = *reinterpret_cast<const float4*>(&red[0][tr][q]);
#pragma unroll
                        for (int w = 1; w < 4; ++w) {
                            const float4 a = *reinterpret_cast<const float4*>(&red[w][tr][q]);
                            v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w;
                        }
                        *reinterpret_cast<float4*>(p.dh_partial + ((size_t)blockIdx.x * p.T + t0 + tr) * 16 + q) = v;
                    }
                }
            }
            advance(t0, g);
        };
        while (t0 < t_hi) {
            step(sg0);
            if (t0 < t_hi) step(sg1);
        }
    }
    // ---- dB of every block, as symb_lora_grad_kernel<1, true> writes it
    float* out = it.direct ? sd.dB : p.partial + it.partial_off;
    const bool accumulate = it.direct && p.accumulate;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        if (g < ncb) {
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int c = (cb0 + g) * CT + wave * (NI * 16) + i * 16 + (lane & 15);
                if (c < p.ncols) {
                    const int pp0 = (lane >> 4) << 2;
                    float* dst = out + (size_t)c * sd.rank + pp0;
                    float old[4] = {0.f, 0.f, 0.f, 0.f};
                    if (accumulate) {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (pp0 + q < sd.rank) old[q] = dst[q];
                    }
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (pp0 + q < sd.rank) dst[q] = old[q] + acc[g][i][q];
                }
            }
        }
    }
}

// dH of the rows of one chunk from the groups' partial sums: dH[t][pp] = s_i * (group 0 + group 1 + ...),
// written as a bf16 value plus its bf16 rounding residual (the layout the skinny kernel writes).
struct DhFinishParams {
    const float* dh_partial;  // [groups][T][16]
    int groups, T;
    bf16* out;                // [T][out_pitch]
    int out_pitch;
    const RowChunk* chunks;
    const SegDesc* seg;
};
SYMB_KERNEL void __launch_bounds__(128)
symb_dh_finish_kernel(const DhFinishParams p) {
    const RowChunk ch = p.chunks[blockIdx.x];
    const SegDesc sd = p.seg[ch.seg];
    const int tr = threadIdx.x >> 2, q = (threadIdx.x & 3) * 4;
    if (tr >= ch.nrows) return;
    const size_t row = (size_t)(ch.row0 + tr);
    float4 v = *reinterpret_cast<const float4*>(p.dh_partial + row * 16 + q);
    for (int g = 1; g < p.groups; ++g) {
        const float4 a = *reinterpret_cast<const float4*>(p.dh_partial + ((size_t)g * p.T + row) * 16 + q);
        v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w;
    }
    v.x *= sd.scale; v.y *= sd.scale; v.z *= sd.scale; v.w *= sd.scale;
    const unsigned h01 = pack2_bf16(v.x, v.y), h23 = pack2_bf16(v.z, v.w);
    uint2 hi2, lo2;
    hi2.x = h01;
    hi2.y = h23;
    lo2.x = pack2_bf16(v.x - bf16_bits_to_f32((unsigned short)(h01 & 0xffffu)), v.y - bf16_bits_to_f32((unsigned short)(h01 >> 16)));
    lo2.y = pack2_bf16(v.z - bf16_bits_to_f32((unsigned short)(h23 & 0xffffu)), v.w - bf16_bits_to_f32((unsigned short)(h23 >> 16)));
    bf16* o = p.out + row * p.out_pitch;
    *reinterpret_cast<uint2*>(o + q) = hi2;
    *reinterpret_cast<uint2*>(o + sd.rpad + q) = lo2;
}

// Sums the runs of the split segments (see GradItem) into their dA / dB: element by element,
//   out = (accumulate ? out : 0) + (run 0 + run 1 + ...), the runs in this order.
// grid.y indexes the split segments; every thread owns four consecutive floats at a time.
struct GradReduceItem {
    int32_t seg, nruns;
    int64_t partial_off;      // run 0, in floats; run q follows at + q * rank * ncols
};
struct GradReduceParams {
    const SegDesc* seg;
    const GradReduceItem* items;
    const float* partial;
    int ncols, cmajor, accumulate;
};
SYMB_KERNEL void __launch_bounds__(256) symb_grad_reduce_kernel(const GradReduceParams p) {
    const GradReduceItem it = p.items[blockIdx.y];
    const SegDesc sd = p.seg[it.seg];
    const size_t n = (size_t)sd.rank * p.ncols;          // a multiple of 4: ncols is a multiple of 8
    float* const out = p.cmajor ? sd.dB : sd.dA;
    const float* const run0 = p.partial + it.partial_off;
    for (size_t e = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4; e < n; e += (size_t)gridDim.x * 1024) {
        float4 v = *reinterpret_cast<const float4*>(run0 + e);
        for (int q = 1; q < it.nruns; ++q) {
            const float4 a = *reinterpret_cast<const float4*>(run0 + (size_t)q * n + e);
            v.x += a.x; v.y += a.y; v.z += a.z; v.w += a.w;
        }
        if (p.accumulate) { const float4 o = *reinterpret_cast<const float4*>(out + e); v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w; }
        *reinterpret_cast<float4*>(out + e) = v;
    }
}

// -------------------------------------------------------------------------------------------
// IA3 vector gradient:  dl_i[j] = sum_{t in segment i} dY[t][j] * Y0[t][j]
// grid.x covers d_out in blocks of COLS columns, grid.y indexes the IA3 segments that want it.
// A thread owns 8 columns (16-byte loads) and every LN-th token, four tokens per step in flight;
// partial sums meet in LDS in a fixed order.  Bound by HBM (4 bytes per element).  Two shapes:
//   long   1024 threads, 128 tokens side by side on 64 columns (one 128-byte line per row): a launch lasts as long as its longest
//          segment's walk.  11 segments of 8200 tokens together, 11008 wide: 84 us (4.3 TB/s), 96 in the short shape; one segment of 4096 tokens on
//          4096 columns 22 / 39.
//   short  256 threads, 16 tokens side by side on 128 columns: an eighth of the threads per segment.  64 segments of 16 tokens, 11008 wide:
//          13 us, 71 in the long shape; 16 of 256 tokens, 4096 wide, 1.12 times the long shape's speed.
// (Long shape on 128 columns 87 us, on 256 105; starting the longest segments first changes nothing.)
// -------------------------------------------------------------------------------------------
struct Ia3GradParams {
    const bf16* dY;
    const bf16* Y0;
    int d_out;
    const int32_t* off;
    const SegDesc* seg;
    const int32_t* seg_list;
    int accumulate;
    const bf16* const* dY_seg;   // device [S] or null: per-segment buffers of the first / second operand
    const bf16* const* Y0_seg;
};
constexpr int ia3_grad_cols(bool lng) { return lng ? 64 : 128; }
constexpr int ia3_grad_threads(bool lng) { return lng ? 1024 : 256; }
template <bool LONG>
SYMB_KERNEL void __launch_bounds__(ia3_grad_threads(LONG)) symb_ia3_grad_kernel(const Ia3GradParams p) {
    constexpr int COLS = ia3_grad_cols(LONG), THREADS = ia3_grad_threads(LONG), CHUNKS = COLS / 8, LN = THREADS / CHUNKS;
    constexpr int WL = 64 / CHUNKS, NW = THREADS / 64;   // token lanes per wavefront; wavefronts
    __shared__ float red[NW][COLS];
    const int s = p.seg_list[blockIdx.y];
    const int t_lo = p.off[s], t_hi = p.off[s + 1];
    const bf16* const gbase = p.dY_seg ? p.dY_seg[s] - (size_t)t_lo * p.d_out : p.dY;
    const bf16* const ybase = p.Y0_seg ? p.Y0_seg[s] - (size_t)t_lo * p.d_out : p.Y0;
    const int cc = threadIdx.x % CHUNKS, tl = threadIdx.x / CHUNKS;
    const int c = blockIdx.x * COLS + cc * 8;
    float a[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    auto fma8 = [&](const uint4& g, const uint4& y) __attribute__((always_inline)) {
        const unsigned int gw[4] = {g.x, g.y, g.z, g.w}, yw[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            a[2 * q] += bf16_bits_to_f32((unsigned short)(gw[q] & 0xffffu)) * bf16_bits_to_f32((unsigned short)(yw[q] & 0xffffu));
            a[2 * q + 1] += bf16_bits_to_f32((unsigned short)(gw[q] >> 16)) * bf16_bits_to_f32((unsigned short)(yw[q] >> 16));
        }
    };
    if (c < p.d_out) {
        int t = t_lo + tl;
        for (; t + 3 * LN < t_hi; t += 4 * LN) {
            uint4 g[4], y[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                g[u] = *reinterpret_cast<const uint4*>(gbase + (size_t)(t + LN * u) * p.d_out + c);
                y[u] = *reinterpret_cast<const uint4*>(ybase + (size_t)(t + LN * u) * p.d_out + c);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) fma8(g[u], y[u]);
        }
        for (; t < t_hi; t += LN) {
            const uint4 g = *reinterpret_cast<const uint4*>(gbase + (size_t)t * p.d_out + c);
            const uint4 y = *reinterpret_cast<const uint4*>(ybase + (size_t)t * p.d_out + c);
            fma8(g, y);
        }
    }
    // the token lanes of a wavefront first (lanes CHUNKS apart hold the same columns), then the wavefronts
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int m = CHUNKS; m < 64; m *= 2) a[q] += __shfl_xor(a[q], m);
    static_assert(WL * CHUNKS == 64, "whole rows of chunks per wavefront");
    if ((tl % WL) == 0) {
#pragma unroll
        for (int q = 0; q < 8; ++q) red[tl / WL][cc * 8 + q] = a[q];
    }
    __syncthreads();
    const int j = blockIdx.x * COLS + threadIdx.x;
    if (threadIdx.x < COLS && j < p.d_out) {
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) v += red[w][threadIdx.x];
        float* const out = p.seg[s].dA + j;
        *out = p.accumulate ? (*out + v) : v;
    }
}

constexpr int ROWPASS_ROWS = 8;        // rows per thread (a divisor of the row chunk's SKINNY_ROWS)
constexpr int ROWPASS_COLS = 128;      // threads per workgroup, one 16-byte column each

// -------------------------------------------------------------------------------------------
// Row scale for the IA3 backward:  out[t][j] = bf16( dY[t][j] * l_seg(t)[j] ) for IA3 rows,
// a plain copy for the others (and, with X and kind = IA3_IN, the input scale of the forward).  Bound by
// HBM: 4 bytes per element.  Measured on 8200 IA3 rows of 11008: 84.1 us with a workgroup per 32-row chunk
// walking its rows four at a time (257 workgroups), 55.2 us (6.6 TB/s) with 8 rows x 1024 columns each.
// -------------------------------------------------------------------------------------------
struct ScaleParams {
    const bf16* dY;           // [T][d_out]: rows to scale (dY for the IA3 backward, X for the IA3_IN forward)
    bf16* out;
    int d_out;                // row width
    const RowChunk* chunks;
    const SegDesc* seg;
    int kind;                 // segments of this kind are scaled by their vector, the others copied
    const bf16* const* in_seg;// device [S] or null: input rows of segment i start at in_seg[i]
    const int32_t* off;       // device [S+1] (read only with in_seg)
};
// grid = (blocks of ROWPASS_COLS 16-byte columns, row chunks, SKINNY_ROWS / ROWPASS_ROWS); see the noise prepass below
SYMB_KERNEL void __launch_bounds__(ROWPASS_COLS) symb_ia3_scale_rows_kernel(const ScaleParams p) {
    const RowChunk ch = p.chunks[blockIdx.y];
    const SegDesc sd = p.seg[ch.seg];
    const bool ia3 = sd.kind == p.kind;
    const bf16* const in = p.in_seg ? p.in_seg[ch.seg] - (size_t)p.off[ch.seg] * p.d_out : p.dY;
    const int r0 = blockIdx.z * ROWPASS_ROWS, nr = min(ch.nrows - r0, ROWPASS_ROWS);
    const int c = blockIdx.x * ROWPASS_COLS + threadIdx.x;
    if (nr <= 0 || c >= (p.d_out >> 3)) return;
    const size_t col = (size_t)c * 8;
    const int row0 = ch.row0 + r0;
    uint4 g[ROWPASS_ROWS];                               // rows past the last one repeat it and are not stored
#pragma unroll
    for (int u = 0; u < ROWPASS_ROWS; ++u) g[u] = *reinterpret_cast<const uint4*>(in + (size_t)(row0 + min(u, nr - 1)) * p.d_out + col);
    if (ia3) {
        const uint4 l = *reinterpret_cast<const uint4*>(sd.A + col);
        const unsigned int lw[4] = {l.x, l.y, l.z, l.w};
#pragma unroll
        for (int u = 0; u < ROWPASS_ROWS; ++u) {
            unsigned int gw[4] = {g[u].x, g[u].y, g[u].z, g[u].w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float lo = bf16_bits_to_f32((unsigned short)(gw[q] & 0xffffu)) * bf16_bits_to_f32((unsigned short)(lw[q] & 0xffffu));
                const float hi = bf16_bits_to_f32((unsigned short)(gw[q] >> 16)) * bf16_bits_to_f32((unsigned short)(lw[q] >> 16));
                gw[q] = pack2_bf16(lo, hi);
            }
            g[u] = make_uint4(gw[0], gw[1], gw[2], gw[3]);
        }
    }
#pragma unroll
    for (int u = 0; u < ROWPASS_ROWS; ++u)
        if (u < nr) *reinterpret_cast<uint4*>(p.out + (size_t)(row0 + u) * p.d_out + col) = g[u];
}

// -------------------------------------------------------------------------------------------
// Noise prepass of the privacy flow:  out[t][k] = bf16( X[t][k] + n_seg(t)[r][k] ), r = 0 for a
// broadcast row, else the token's index inside its segment; rows of segments without noise are
// copied.  fp32 sum, one rounding.  Bound by HBM (6 bytes per element).  A workgroup takes ROWPASS_ROWS
// rows x ROWPASS_COLS 16-byte columns of one row chunk, all its loads in flight at once: a chunk per workgroup,
// its rows one after the other, left three quarters of the chip idle on small batches (2000 rows of 4608
// with a noise row each: 63 workgroups, 60.9 us, 0.9 TB/s; now 1260, about 13 us, and the call with its
// forward 178.5 -> 131.0 us).
// -------------------------------------------------------------------------------------------
struct NoiseAddParams {
    const bf16* X;
    bf16* out;
    int width;
    const RowChunk* chunks;
    const int32_t* off;
    const NoiseDesc* noise;
};
// grid = (blocks of ROWPASS_COLS 16-byte columns, row chunks, SKINNY_ROWS / ROWPASS_ROWS)
SYMB_KERNEL void __launch_bounds__(ROWPASS_COLS) symb_noise_add_kernel(const NoiseAddParams p) {
    const RowChunk ch = p.chunks[blockIdx.y];
    const NoiseDesc nd = p.noise[ch.seg];
    const int r0 = blockIdx.z * ROWPASS_ROWS, nr = min(ch.nrows - r0, ROWPASS_ROWS), seg0 = p.off[ch.seg];
    const int c = blockIdx.x * ROWPASS_COLS + threadIdx.x;
    if (nr <= 0 || c >= (p.width >> 3)) return;
    const size_t col = (size_t)c * 8;
    const int row0 = ch.row0 + r0;
    uint4 x[ROWPASS_ROWS], n[ROWPASS_ROWS];              // rows past the last one repeat it and are not stored
#pragma unroll
    for (int u = 0; u < ROWPASS_ROWS; ++u) x[u] = *reinterpret_cast<const uint4*>(p.X + (size_t)(row0 + min(u, nr - 1)) * p.width + col);
    if (nd.ptr) {
#pragma unroll
        for (int u = 0; u < ROWPASS_ROWS; ++u)
            n[u] = *reinterpret_cast<const uint4*>(nd.ptr + (size_t)(nd.rows == 1 ? 0 : row0 + min(u, nr - 1) - seg0) * p.width + col);
#pragma unroll
        for (int u = 0; u < ROWPASS_ROWS; ++u) {
            unsigned int xw[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
            const unsigned int nw[4] = {n[u].x, n[u].y, n[u].z, n[u].w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float lo = bf16_bits_to_f32((unsigned short)(xw[q] & 0xffffu)) + bf16_bits_to_f32((unsigned short)(nw[q] & 0xffffu));
                const float hi = bf16_bits_to_f32((unsigned short)(xw[q] >> 16)) + bf16_bits_to_f32((unsigned short)(nw[q] >> 16));
                xw[q] = pack2_bf16(lo, hi);
            }
            x[u] = make_uint4(xw[0], xw[1], xw[2], xw[3]);
        }
    }
#pragma unroll
    for (int u = 0; u < ROWPASS_ROWS; ++u)
        if (u < nr) *reinterpret_cast<uint4*>(p.out + (size_t)(row0 + u) * p.width + col) = x[u];
}

// -------------------------------------------------------------------------------------------
// Row scatter of a per-segment call whose output went through a flat copy in the workspace:
// row t of segment i moves from in[t] to out_seg[i][t - off[i]].  One workgroup per row chunk.
// -------------------------------------------------------------------------------------------
struct ScatterParams {
    const bf16* in;           // [T][width]
    int width;
    const RowChunk* chunks;
    bf16* const* out_seg;     // device [S]
    const int32_t* off;       // device [S+1]
};
SYMB_KERNEL void __launch_bounds__(256) symb_scatter_rows_kernel(const ScatterParams p) {
    const RowChunk ch = p.chunks[blockIdx.x];
    const int nchunk = p.width >> 3;
    bf16* const out = p.out_seg[ch.seg] - (size_t)p.off[ch.seg] * p.width;
    for (int e = threadIdx.x; e < ch.nrows * nchunk; e += 256) {
        const size_t at = (size_t)(ch.row0 + e / nchunk) * p.width + (size_t)(e % nchunk) * 8;
        *reinterpret_cast<uint4*>(out + at) = *reinterpret_cast<const uint4*>(p.in + at);
    }
}

SYMB_KERNEL void __launch_bounds__(256) symb_fill_zero_kernel(float* dst, size_t n) {
    for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) dst[i] = 0.f;
}

}  // namespace symb
