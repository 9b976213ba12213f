// Input gradient of a layer of few outputs (64 to 256) over many rows: dX = dY W + dH A_i.  The tiled kernel walks two to four stages per tile, so that its time is
// the tiles' prologues and stores, one behind the other; here the inner dimension is short enough that a wavefront keeps its 64 columns of W in registers (128 of them at
// 256 outputs) and streams rows past them.
//
// 16384 rows of 6144 <- 256, 201 MB of dX: 85 us in 256x256 tiles, 80 here with a wait for every chunk's stores, 73 with those left open (three sets of operands in turn); 6000 rows 39.2, 29.4, 26.1.  That is 2.8 TB/s
// of stores: a kernel that only stores reaches 6.9, a copy writes 2.7, so the stores alone are not what bounds it; what does has not been measured.  A workgroup is 4 wavefronts, 256 columns; its 32-row chunks (with adapters never across a segment)
// come in by LDS DMA through a ring of three, one barrier per chunk, and every wavefront multiplies all 32 rows with its own columns.  Two workgroups per CU, so that one's stores run beside the
// other's products.  The columns of a wavefront are dealt out so that a lane ends up with 16 consecutive ones of a row, 32 bytes: output goes to memory from the registers, whole
// 128-byte lines per row between four lanes, with no staging.
#pragma once
#include "adapter_kernels.hpp"

namespace symb {

constexpr int SHORTK_COLS = 256;

struct ShortKParams {
    const bf16* G;            // dY [M][K], K = 32 KS
    const bf16* W;            // [K][N]
    bf16* C;                  // dX [M][N]
    const bf16* h_rows;       // [M][32]: dH, 16 values and 16 residuals; null: no LoRA term
    int N, num_chunks, groups, per_group;
    const RowChunk* chunks;   // device: at most 32 rows each, with h_rows of one segment; a workgroup takes per_group of them
    const SegDesc* seg;       // LoRA segments: ranks up to 16
};

// Column of a wavefront's 64 that index i of its column block c stands for (see above).
__device__ __forceinline__ int shortk_col(int c, int i) { return (i >> 2) * 16 + c * 4 + (i & 3); }

template <int KS>
SYMB_KERNEL void __launch_bounds__(256, 2)
symb_gemm_shortk_kernel(const ShortKParams p) {
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    constexpr int K = 32 * KS, CPR = 4 * KS, ROW = K * 2, STAGE = 32 * ROW, NBUF = 3, REQ = KS / 2;      // 16-byte chunks per row; bytes; requests of a wavefront per chunk of rows
    constexpr int WK = KS < 4 ? KS : 4;                  // 32-k steps of the weight that pass through LDS at a time, a wavefront's 4 KiB each
    constexpr int SWZ = CPR % 16 == 0 ? 15 : 7;
    static_assert(KS % 2 == 0 && KS <= 8, "whole requests; the weight fits the registers");
    constexpr int H_AT = STAGE, BUF = STAGE + 32 * 64;   // a buffer: rows of dY, rows of dH
    constexpr int BYTES = NBUF * BUF > 4 * WK * 4096 ? NBUF * BUF : 4 * WK * 4096;
    __shared__ __attribute__((aligned(16))) unsigned char smem[BYTES];
    const int strips = (p.N + SHORTK_COLS - 1) / SHORTK_COLS, total = strips * p.groups, per_xcd = (total + 7) >> 3;
    const int lin = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (lin >= total || (int)(blockIdx.x >> 3) >= per_xcd) return;
    const int first = lin / strips * p.per_group, last = min(first + p.per_group, p.num_chunks);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l15 = lane & 15, kq = lane >> 4;
    const int N = p.N, n0 = lin % strips * SHORTK_COLS + wave * 64;
    if (first >= last) return;
    const unsigned lds0 = (unsigned)(size_t)smem;

    // ---- this wavefront's columns of W, through its own part of the LDS: rows of 64 columns, 32-byte pieces of row k at piece ^ skinny_bt_swz
    u32x4 wf[KS][4];
    {
        unsigned char* const mine = smem + wave * (WK * 4096);
        const int k0 = kq * 8 + (l15 >> 2);              // first of the two transposing reads; the second is 4 k further
        const unsigned at = (unsigned)(size_t)mine + (unsigned)(k0 * 128 + (((l15 & 3) ^ skinny_bt_swz(64, k0)) * 32));
#pragma unroll
        for (int g = 0; g < KS; g += WK) {
#pragma unroll
            for (int i = 0; i < WK * 4; ++i) {           // 8 k-rows of 128 bytes per request; columns past the last ones repeat those
                if (g * 4 + i >= KS * 4) continue;
                const int k = i * 8 + (lane >> 3), slot = lane & 7, col = (((slot >> 1) ^ skinny_bt_swz(64, k)) << 4) | ((slot & 1) << 3);
                __builtin_amdgcn_global_load_lds((glb_void_t*)(p.W + (size_t)(g * 32 + k) * N + min(n0 + col, N - 8)), (lds_void_t*)(mine + i * 1024), 16, 0, 0);
            }
            asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
            u32x2 t[WK][4][2];
#pragma unroll
            for (int s = 0; s < WK; ++s)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(t[s][c][0]) : "v"(at), "n"(s * 4096 + c * 8));
                    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(t[s][c][1]) : "v"(at), "n"(s * 4096 + c * 8 + 512));
                }
            asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
#pragma unroll
            for (int s = 0; s < WK; ++s)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    asm volatile("" : "+v"(t[s][c][0])); asm volatile("" : "+v"(t[s][c][1]));
                    if (g + s < KS) wf[g + s][c] = __builtin_shufflevector(t[s][c][0], t[s][c][1], 0, 1, 2, 3);
                }
        }
    }
    __syncthreads();                                     // the ring takes the place

    // ---- the rows: chunk x of a request's 64 is row x / CPR, position x % CPR, which holds 16-byte chunk position ^ row % (SWZ + 1) of it
    const bf16* src0[REQ];
    int srow[REQ];
#pragma unroll
    for (int i = 0; i < REQ; ++i) {
        const int x = (wave * REQ + i) * 64 + lane, r = x / CPR, pos = x % CPR;
        srow[i] = r;
        src0[i] = p.G + ((pos & ~SWZ) | ((pos ^ r) & SWZ)) * 8;
    }
    // dH, eight rows of 64 bytes per wavefront, lanes 0 to 31: position pos of row r holds chunk pos ^ (r / 2) % 4
    const int hrow = wave * 8 + ((lane & 31) >> 2);
    const bf16* const hsrc = p.h_rows + ((lane & 3) ^ ((hrow >> 1) & 3)) * 8;
    const bool h = p.h_rows != nullptr;
    // (scalar loads: a vector load's wait would be one for all stores before it)
    auto chunk = [&](int i) __attribute__((always_inline)) {
        const __attribute__((address_space(4))) int* const c = (const __attribute__((address_space(4))) int*)reinterpret_cast<const int*>(p.chunks + min(i, last - 1));
        return RowChunk{c[0], c[1], c[2], 0};
    };
    auto dma = [&](int buf, const RowChunk& ch) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < REQ; ++i)
            __builtin_amdgcn_global_load_lds((glb_void_t*)(src0[i] + (size_t)(ch.row0 + min(srow[i], ch.nrows - 1)) * K), (lds_void_t*)(smem + buf * BUF + (wave * REQ + i) * 1024), 16, 0, 0);
        if (h && lane < 32)
            __builtin_amdgcn_global_load_lds((glb_void_t*)(hsrc + (size_t)(ch.row0 + min(hrow, ch.nrows - 1)) * 32), (lds_void_t*)(smem + buf * BUF + H_AT + wave * 512), 16, 0, 0);
    };
    u32x4 lf[4] = {};
    int seg = -1;
    bool lora = false;
    RowChunk cur = chunk(first), next = chunk(first + 1), after = chunk(first + 2);
    dma(0, cur);
    if (first + 1 < last) dma(1, next);
    // Stores that the last two chunks issued for certain: four each, where the chunk reaches into its second 16 rows and this wavefront's columns are all there.
    const bool inside = n0 + 64 <= N;
    bool four1 = false, four2 = false;
    int buf = 0;
    for (int it = first; it < last; ++it) {
        const RowChunk later = chunk(it + 3);
        if (cur.seg != seg) {                            // (uniform) A_i: columns as in wf, ranks 8 (kq % 2) .. + 7, for both halves of the step
            seg = cur.seg;
            const SegDesc sd = p.seg[seg];
            lora = h && sd.kind == KIND_LORA;
            if (lora) {
                const __attribute__((address_space(1))) unsigned short* const a =
                    (const __attribute__((address_space(1))) unsigned short*)reinterpret_cast<const unsigned short*>(sd.A);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int n = min(n0 + shortk_col(c, l15), N - 1), q0 = (kq & 1) * 8;
                    unsigned e[8];
#pragma unroll
                    for (int q = 0; q < 8; ++q) e[q] = a[(size_t)min(q0 + q, sd.rank - 1) * N + n];
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        lf[c][q] = (q0 + 2 * q < sd.rank ? e[2 * q] : 0u) | (q0 + 2 * q + 1 < sd.rank ? e[2 * q + 1] << 16 : 0u);
                }
            }
        }
        // This wavefront's part of the chunk has landed; behind the barrier everybody's has, and the buffer of the chunk before is free.  Behind its requests came the stores of the
        // chunk two before, the next chunk's requests and the stores of the chunk before: those may stay open.  (Requests and stores are counted together and come back in order, so
        // that a wait for fewer, or one that the compiler adds for a vector load of its own, is one for the stores just made.)
        const bool more = it + 1 < last;
        auto landed = [&](auto REQS) __attribute__((always_inline)) {
            constexpr int R = decltype(REQS)::value;
            if (four1 && four2) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(R + 8) : "memory");
            else if (four1) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(R + 4) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0)" : : "n"(R) : "memory");
        };
        if (!more) landed(std::integral_constant<int, 0>{});
        else if (h) landed(std::integral_constant<int, REQ + 1>{});
        else landed(std::integral_constant<int, REQ>{});
        __builtin_amdgcn_s_barrier();
        const int nb = buf + 2 >= NBUF ? buf + 2 - NBUF : buf + 2;
        if (it + 2 < last) dma(nb, after);
        floatx4 acc[2][4];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[b][c] = floatx4{0.f, 0.f, 0.f, 0.f};
        const unsigned base = lds0 + (unsigned)(buf * BUF + l15 * ROW);
#pragma unroll
        for (int g = 0; g < KS; g += 2) {
            u32x4 x[2][2];
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    const int ck = (g + s) * 4 + kq;
                    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(x[s][b]) : "v"(base + (unsigned)(((ck & ~SWZ) | ((ck ^ l15) & SWZ)) * 16)), "n"(b * 16 * ROW));
                }
            asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int b = 0; b < 2; ++b) asm volatile("" : "+v"(x[s][b]));
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        acc[b][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wf[g + s][c]), __builtin_bit_cast(bf16x8, x[s][b]), acc[b][c], 0, 0, 0);
        }
        if (lora) {
            u32x4 hv[2];
            const unsigned hat = lds0 + (unsigned)(buf * BUF + H_AT + l15 * 64 + ((kq ^ ((l15 >> 1) & 3)) * 16));
#pragma unroll
            for (int b = 0; b < 2; ++b) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(hv[b]) : "v"(hat), "n"(b * 1024));
            asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
#pragma unroll
            for (int b = 0; b < 2; ++b) asm volatile("" : "+v"(hv[b]));
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    acc[b][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, lf[c]), __builtin_bit_cast(bf16x8, hv[b]), acc[b][c], 0, 0, 0);
        }
        // C[row b * 16 + l15][n0 + 16 kq ..]: block c holds columns 4 c .. + 3 of the lane's 16
        const int n = n0 + kq * 16;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            if (b * 16 + l15 >= cur.nrows) continue;
            bf16* const out = p.C + (size_t)(cur.row0 + b * 16 + l15) * N + n;
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                const floatx4 &u = acc[b][2 * half], &v = acc[b][2 * half + 1];
                if (n + half * 8 < N) *reinterpret_cast<uint4*>(out + half * 8) = make_uint4(pack2_bf16(u[0], u[1]), pack2_bf16(u[2], u[3]), pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3]));
            }
        }
        four2 = four1;
        four1 = inside && cur.nrows > 16;
        cur = next;
        next = after;
        after = later;
        buf = buf + 1 == NBUF ? 0 : buf + 1;
    }
}

}  // namespace symb
