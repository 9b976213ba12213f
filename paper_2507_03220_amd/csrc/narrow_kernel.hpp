// Forward of a narrow layer (129 to 256 outputs) over many rows, LoRA shrink included: every workgroup takes 64 rows of one segment and all columns, so that X,
// by far the largest tensor, is read once for the product and for H = X A_i^T together.  As two launches, shrink and tiled product, each read it.
//
// Bound by HBM: 2 K bytes per row.  16384 rows of 6144 -> 256 in 16 rank-8 segments: shrink 61 us and product 59 before, now 94 to 102
// (90 without other work on the chip; 82 with X in cache, and 82 without the matrix instructions: what is left is the arrival of the weight's 32 KiB per stage).  A workgroup
// is 4 wavefronts of 64 columns each; K goes by in stages of 64, by LDS DMA, one barrier per stage: the weight (32 KiB, from L2) and the 16 rows of A_i (2 KiB) through a ring of
// three, X (8 KiB, from HBM) through one of seven.  Requests return in order to the wavefront that made them, so one wavefront requests X alone, six stages ahead, and the
// others the rest, two ahead: with all of it two ahead 4 MB of X were on their way on the whole chip, 2.5 TB/s (112 us).  64 rows make one workgroup per CU of
// 16384 rows, and a stage's 42 KiB are less than what a CU takes in (64 bytes per clock) while HBM delivers its share of X.  Every XCD starts at another eighth of
// K and walks around the end (in step they all ask for the same few columns of X at a time: 93 us; every workgroup at a stage of its own, so that an XCD's L2 has to hold the whole
// weight, 93).  The next stage's fragments read under this one's matrix instructions: 111 us, dropped.  A chunk of rows never crosses a segment, so
// that one adapter belongs to it; H stays in the accumulators of one wavefront per 16 rows, leaves as value + residual for a gradient call, and meets
// B_i as one more 32-wide step, as in the tiled kernels.
#pragma once
#include "adapter_kernels.hpp"

namespace symb {

constexpr int NARROW_ROWS = 64, NARROW_COLS = 256;

struct NarrowParams {
    const bf16* X;            // [M][K], K a multiple of 64
    const bf16* W;            // [N][K], N <= 256
    const bf16* bias;         // [N] or null
    bf16* C;                  // [M][N]
    bf16* h_rows;             // [M][h_pitch]: value + residual of LoRA segments' rows
    int N, K, h_pitch;
    const RowChunk* chunks;   // device: at most NARROW_ROWS rows of one segment each
    const SegDesc* seg;       // LoRA segments: ranks up to 16
};

struct Narrow {
    static constexpr int X_STAGE = NARROW_ROWS * 128, W_BYTES = NARROW_COLS * 128, W_STAGE = W_BYTES + 16 * 128, XBUF = 7, WBUF = 3;
    static constexpr int W_AT = XBUF * X_STAGE, BYTES = W_AT + WBUF * W_STAGE;
    static constexpr int XREQ = X_STAGE / 1024, WREQ = 12;           // requests of 1 KiB per stage: of wavefront 0; of each other one (32 of the weight, two of A_i, those two again)
    static constexpr int C_PITCH = NARROW_COLS * 2 + 16;
    static_assert(BYTES <= 160 << 10 && NARROW_ROWS * (64 + C_PITCH) <= BYTES, "a CU's LDS; H and the staged output fit the rings");
};

SYMB_KERNEL void __launch_bounds__(256)
symb_gemm_narrow_kernel(const NarrowParams p) {
    using ST = Narrow;
    __shared__ __attribute__((aligned(16))) unsigned char smem[ST::BYTES];
    const RowChunk ch = p.chunks[blockIdx.x];
    const SegDesc sd = p.seg[ch.seg];
    const bool lora = sd.kind == KIND_LORA;              // uniform
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l15 = lane & 15, kq = lane >> 4;
    const int K = p.K, N = p.N, n0 = wave * 64;
    // this lane's 16 bytes of each request, 8 rows of 128 bytes: chunk c of row r lies at c ^ (r / 2) % 8; rows and columns past the last one repeat it
    const bf16* src[ST::WREQ];
    unsigned dst[ST::WREQ];                              // inside a stage
#pragma unroll
    for (int i = 0; i < ST::WREQ; ++i) {
        const bf16* row;
        int r;
        if (wave == 0) {
            r = min(i, ST::XREQ - 1) * 8 + (lane >> 3);
            row = p.X + (size_t)(ch.row0 + min(r, ch.nrows - 1)) * K;
            dst[i] = (unsigned)(min(i, ST::XREQ - 1) * 1024);
        } else {
            const int q = (wave - 1) * ST::WREQ + i;     // 0 .. 31: the weight; then A_i (without an adapter: the weight's first row, not used)
            r = (q < 32 ? q : q & 1) * 8 + (lane >> 3);
            row = q < 32 ? p.W + (size_t)min(r, N - 1) * K : lora ? sd.A + (size_t)min(r, sd.rank - 1) * K : p.W;
            dst[i] = (unsigned)(q < 32 ? q * 1024 : ST::W_BYTES + (q & 1) * 1024);
        }
        src[i] = row + ((lane & 7) ^ ((r >> 1) & 7)) * 8;
    }
    const unsigned lds0 = (unsigned)(size_t)smem;
    const int ns = K >> 6;
    int at_k = (int)((blockIdx.x & 7) * (unsigned)ns / 8);       // the stage to request next
    auto dma_x = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < ST::XREQ; ++i) __builtin_amdgcn_global_load_lds((glb_void_t*)(src[i] + at_k * 64), (lds_void_t*)(smem + buf * ST::X_STAGE + dst[i]), 16, 0, 0);
        at_k = at_k + 1 == ns ? 0 : at_k + 1;
    };
    auto dma_w = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < ST::WREQ; ++i)
            __builtin_amdgcn_global_load_lds((glb_void_t*)(src[i] + at_k * 64), (lds_void_t*)(smem + ST::W_AT + buf * ST::W_STAGE + dst[i]), 16, 0, 0);
        at_k = at_k + 1 == ns ? 0 : at_k + 1;
    };
    // fragment of block 0 of 32-k step h; block b of the weight is 2 KiB further.  Row block b of a wavefront is number (b + wave) % 4 of the chunk, so that block 0
    // is the one whose H it forms
    unsigned xoff[2], woff[2], aoff[2], xblk[4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        xoff[h] = lds0 + (unsigned)(l15 * 128 + (((h * 4 + kq) ^ ((l15 >> 1) & 7)) * 16));
        woff[h] = xoff[h] + (unsigned)(ST::W_AT + n0 * 128);
        aoff[h] = xoff[h] + ST::W_AT + ST::W_BYTES;
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) xblk[b] = (unsigned)(((b + wave) & 3) * 2048);
    floatx4 acc[4][4], acch = floatx4{0.f, 0.f, 0.f, 0.f};           // [row block][column block]
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[b][c] = floatx4{0.f, 0.f, 0.f, 0.f};
    // Fragment reads with waits of their own (see the skinny kernel), nine per 32-k step, each step's behind the one before in the other set, so that they arrive under its matrix instructions.
    struct Frags { u32x4 x[4], w[4], a; } f0, f1;        // of the two 32-k steps
    auto read = [&](Frags& f, int h, int xbuf, int wbuf) __attribute__((always_inline)) {
        const unsigned xat = xoff[h] + (unsigned)(xbuf * ST::X_STAGE), wat = (unsigned)(wbuf * ST::W_STAGE);
#pragma unroll
        for (int b = 0; b < 4; ++b) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(f.w[b]) : "v"(woff[h] + wat), "n"(b * 2048));
#pragma unroll
        for (int b = 0; b < 4; ++b) asm volatile("ds_read_b128 %0, %1" : "=v"(f.x[b]) : "v"(xat + xblk[b]));
        asm volatile("ds_read_b128 %0, %1" : "=v"(f.a) : "v"(aoff[h] + wat));
    };
    auto mul = [&](const Frags& f) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                acc[b][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f.w[c]), __builtin_bit_cast(bf16x8, f.x[b]), acc[b][c], 0, 0, 0);
        acch = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f.a), __builtin_bit_cast(bf16x8, f.x[0]), acch, 0, 0, 0);
    };
    auto landed = [&](Frags& f) __attribute__((always_inline)) {     // (each result is tied to the wait that covers it)
#pragma unroll
        for (int b = 0; b < 4; ++b) { asm volatile("" : "+v"(f.w[b])); asm volatile("" : "+v"(f.x[b])); }
        asm volatile("" : "+v"(f.a));
    };
    if (wave == 0)
        for (int d = 0; d < min(ns, ST::XBUF - 1); ++d) dma_x(d);
    else
        for (int d = 0; d < min(ns, ST::WBUF - 1); ++d) dma_w(d);
    int x = 0, xn = ST::XBUF - 1, w = 0, wn = ST::WBUF - 1;          // buffers of this stage, of the one to request
    for (int s = 0; s < ns; ++s) {
        // this wavefront's part of stage s has landed; behind the barrier everybody's has, and the buffers of stage s - 1 are free
        if (wave == 0) {
            if (s + ST::XBUF - 1 <= ns) asm volatile("s_waitcnt vmcnt(%0)" : : "n"((ST::XBUF - 2) * ST::XREQ) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        } else {
            if (s + 1 < ns) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(ST::WREQ) : "memory");
            else asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
        }
        __builtin_amdgcn_s_barrier();
        read(f0, 0, x, w);
        read(f1, 1, x, w);
        if (wave == 0) {
            if (s + ST::XBUF - 1 < ns) dma_x(xn);
        } else if (s + ST::WBUF - 1 < ns) dma_w(wn);
        asm volatile("s_waitcnt lgkmcnt(9)" : : : "memory");
        landed(f0);
        mul(f0);
        asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");
        landed(f1);
        mul(f1);
        x = x + 1 == ST::XBUF ? 0 : x + 1;
        xn = xn + 1 == ST::XBUF ? 0 : xn + 1;
        w = w + 1 == ST::WBUF ? 0 : w + 1;
        wn = wn + 1 == ST::WBUF ? 0 : wn + 1;
    }
    __syncthreads();                                     // every wavefront is done with the rings
    unsigned char* const sH = smem;                      // [row][16 values | 16 residuals]
    unsigned char* const sC = smem + NARROW_ROWS * 64;
    if (lora) {
        // B_i: columns n0 + 16 c + l15, ranks 8 (kq % 2) .. + 7 (both halves of the step meet the same ones)
        u32x4 bw[4];
        const int q0 = (kq & 1) * 8;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int n = min(n0 + c * 16 + l15, N - 1);
            if ((sd.rank & 7) == 0) bw[c] = ld_glb16(sd.B + (size_t)n * sd.rank + min(q0, sd.rank - 8));
            else {
                const unsigned short* const e = reinterpret_cast<const unsigned short*>(sd.B) + (size_t)n * sd.rank;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const unsigned a = e[min(q0 + 2 * q, sd.rank - 1)], b = e[min(q0 + 2 * q + 1, sd.rank - 1)];
                    bw[c][q] = (q0 + 2 * q < sd.rank ? a : 0u) | (q0 + 2 * q + 1 < sd.rank ? b << 16 : 0u);
                }
            }
            if (q0 >= sd.rank) bw[c] = u32x4{0u, 0u, 0u, 0u};
        }
        // H[16 wave + l15][4 kq + q]; ranks past the last one repeated its row of A_i: zero
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = kq * 4 + q < sd.rank ? sd.scale * acch[q] : 0.f;
        const unsigned h01 = pack2_bf16(v[0], v[1]), h23 = pack2_bf16(v[2], v[3]);
        const uint2 hi = make_uint2(h01, h23);
        const uint2 lo = make_uint2(pack2_bf16(v[0] - bf16_bits_to_f32((unsigned short)(h01 & 0xffffu)), v[1] - bf16_bits_to_f32((unsigned short)(h01 >> 16))),
                                    pack2_bf16(v[2] - bf16_bits_to_f32((unsigned short)(h23 & 0xffffu)), v[3] - bf16_bits_to_f32((unsigned short)(h23 >> 16))));
        const int t = wave * 16 + l15;
        *reinterpret_cast<uint2*>(sH + t * 64 + kq * 8) = hi;
        *reinterpret_cast<uint2*>(sH + t * 64 + 32 + kq * 8) = lo;
        if (t < ch.nrows) {
            bf16* const row = p.h_rows + (size_t)(ch.row0 + t) * p.h_pitch + kq * 4;
            *reinterpret_cast<uint2*>(row) = hi;
            *reinterpret_cast<uint2*>(row + 16) = lo;
        }
        __syncthreads();
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const bf16x8 hf = *reinterpret_cast<const bf16x8*>(sH + (((b + wave) & 3) * 16 + l15) * 64 + kq * 16);
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[b][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, bw[c]), hf, acc[b][c], 0, 0, 0);
        }
    }
    // bias, IA3 scale of the chunk's segment, one rounding; C[16 ((b + wave) % 4) + l15][n0 + 16 c + 4 kq ..] through LDS, whole rows to memory
    const bool ia3 = sd.kind == KIND_IA3;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int n = min(n0 + c * 16 + kq * 4, N - 4);
        const uint2 bv = p.bias ? *reinterpret_cast<const uint2*>(p.bias + n) : make_uint2(0u, 0u);
        const uint2 lv = ia3 ? *reinterpret_cast<const uint2*>(sd.A + n) : make_uint2(0x3f803f80u, 0x3f803f80u);
        auto lo16 = [](unsigned x) { return bf16_bits_to_f32((unsigned short)(x & 0xffffu)); };
        auto hi16 = [](unsigned x) { return bf16_bits_to_f32((unsigned short)(x >> 16)); };
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            floatx4 v = acc[b][c];
            if (p.bias) v += floatx4{lo16(bv.x), hi16(bv.x), lo16(bv.y), hi16(bv.y)};
            if (ia3) v *= floatx4{lo16(lv.x), hi16(lv.x), lo16(lv.y), hi16(lv.y)};
            *reinterpret_cast<uint2*>(sC + (((b + wave) & 3) * 16 + l15) * ST::C_PITCH + (n0 + c * 16 + kq * 4) * 2) = make_uint2(pack2_bf16(v[0], v[1]), pack2_bf16(v[2], v[3]));
        }
    }
    __syncthreads();
    const int col = (tid & 31) * 8;
#pragma unroll
    for (int i = 0; i < NARROW_ROWS / 8; ++i) {
        const int t = i * 8 + (tid >> 5);
        if (t < ch.nrows && col < N) *reinterpret_cast<uint4*>(p.C + (size_t)(ch.row0 + t) * N + col) = *reinterpret_cast<const uint4*>(sC + t * ST::C_PITCH + col * 2);
    }
}

}  // namespace symb
