// GENERATED by gen_gemm16_asm.py -- do not edit by hand.
// Assembly of the 4-wavefront base GEMM on v_mfma_f32_16x16x32_bf16 for gfx950, for a 256x256 tile
// (macros SYMB_GEMM16_*), a 128x128 tile (SYMB_GEMM16S_*) and a 256x128 tile (SYMB_GEMM16T_*).  The accumulators are not operands:
// every template names the accumulation registers literally.  The main loop zeroes the
// accumulators itself (after issuing its first loads); *_ZERO is for a K extent without a single
// full stage.
#pragma once
// ---- 256x256 tile: a wavefront owns 8x8 blocks, block (i, j) in a[4(8i+j) : 4(8i+j)+3].
// Main loop operands: %0-%3 A fragment lane offsets inside an A unit (32-k step 0 first / second
// read, step 1 first / second read); %4-%11 B fragment lane offsets inside a B unit (K-contiguous W:
// as for A in %4-%7; N-contiguous W: one per 16-column block); %12-%19 / %20-%27 global byte offsets
// of this lane's 8 A / 8 B loads per stage; %28,%29 global base of the A / B stage (64-bit SGPR);
// %30 byte stride of B between stages; %31 number of 64-k stages (>= 1); %32 LDS byte address of the
// dynamic segment + this wavefront's first load inside a unit (wave * 8192).  LDS: units of
// 32 KiB, A at unit 0/1/2, B at unit 3/4.  Fixed registers: s80-s91, v116-v255 (fragment sets at
// v128 and v192), a0-a255.
#define SYMB_GEMM16_LOOP_NT \
    "s_mov_b64 s[80:81], %28\n\t" \
    "s_mov_b64 s[82:83], %29\n\t" \
    "s_sub_u32 s84, %31, 2\n\t" \
    "s_mov_b32 s85, 0\n\t" \
    "s_mov_b32 s86, 32768\n\t" \
    "s_mov_b32 s87, 65536\n\t" \
    "s_mov_b32 s88, 98304\n\t" \
    "s_mov_b32 s89, 131072\n\t" \
    "s_add_u32 s90, s85, %32\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %12, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %13, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %14, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %15, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %16, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 5120\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %17, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 6144\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %18, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 7168\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %19, s[80:81]\n\t" \
    "s_cmp_gt_u32 %31, 1\n\t" \
    "s_cselect_b32 s91, 128, 0\n\t" \
    "s_add_u32 s80, s80, s91\n\t" \
    "s_addc_u32 s81, s81, 0\n\t" \
    "s_add_u32 s90, s88, %32\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %20, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %21, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %22, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %23, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %24, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 5120\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %25, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 6144\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %26, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 7168\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %27, s[82:83]\n\t" \
    "s_cmp_gt_u32 %31, 1\n\t" \
    "s_cselect_b32 s91, %30, 0\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, 0\n\t" \
    "s_add_u32 s90, s86, %32\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %12, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %13, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %14, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %15, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %16, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 5120\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %17, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 6144\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %18, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 7168\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %19, s[80:81]\n\t" \
    "s_add_u32 s80, s80, 128\n\t" \
    "s_addc_u32 s81, s81, 0\n\t" \
    "s_add_u32 s90, s89, %32\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %20, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %21, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %22, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %23, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %24, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 5120\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %25, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 6144\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %26, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 7168\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %27, s[82:83]\n\t" \
    "s_mov_b32 s91, %30\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, 0\n\t" \
    "v_accvgpr_write_b32 a0, 0\n\t" \
    "v_accvgpr_write_b32 a1, 0\n\t" \
    "v_accvgpr_write_b32 a2, 0\n\t" \
    "v_accvgpr_write_b32 a3, 0\n\t" \
    "v_accvgpr_write_b32 a4, 0\n\t" \
    "v_accvgpr_write_b32 a5, 0\n\t" \
    "v_accvgpr_write_b32 a6, 0\n\t" \
    "v_accvgpr_write_b32 a7, 0\n\t" \
    "v_accvgpr_write_b32 a8, 0\n\t" \
    "v_accvgpr_write_b32 a9, 0\n\t" \
    "v_accvgpr_write_b32 a10, 0\n\t" \
    "v_accvgpr_write_b32 a11, 0\n\t" \
    "v_accvgpr_write_b32 a12, 0\n\t" \
    "v_accvgpr_write_b32 a13, 0\n\t" \
    "v_accvgpr_write_b32 a14, 0\n\t" \
    "v_accvgpr_write_b32 a15, 0\n\t" \
    "v_accvgpr_write_b32 a16, 0\n\t" \
    "v_accvgpr_write_b32 a17, 0\n\t" \
    "v_accvgpr_write_b32 a18, 0\n\t" \
    "v_accvgpr_write_b32 a19, 0\n\t" \
    "v_accvgpr_write_b32 a20, 0\n\t" \
    "v_accvgpr_write_b32 a21, 0\n\t" \
    "v_accvgpr_write_b32 a22, 0\n\t" \
    "v_accvgpr_write_b32 a23, 0\n\t" \
    "v_accvgpr_write_b32 a24, 0\n\t" \
    "v_accvgpr_write_b32 a25, 0\n\t" \
    "v_accvgpr_write_b32 a26, 0\n\t" \
    "v_accvgpr_write_b32 a27, 0\n\t" \
    "v_accvgpr_write_b32 a28, 0\n\t" \
    "v_accvgpr_write_b32 a29, 0\n\t" \
    "v_accvgpr_write_b32 a30, 0\n\t" \
    "v_accvgpr_write_b32 a31, 0\n\t" \
    "v_accvgpr_write_b32 a32, 0\n\t" \
    "v_accvgpr_write_b32 a33, 0\n\t" \
    "v_accvgpr_write_b32 a34, 0\n\t" \
    "v_accvgpr_write_b32 a35, 0\n\t" \
    "v_accvgpr_write_b32 a36, 0\n\t" \
    "v_accvgpr_write_b32 a37, 0\n\t" \
    "v_accvgpr_write_b32 a38, 0\n\t" \
    "v_accvgpr_write_b32 a39, 0\n\t" \
    "v_accvgpr_write_b32 a40, 0\n\t" \
    "v_accvgpr_write_b32 a41, 0\n\t" \
    "v_accvgpr_write_b32 a42, 0\n\t" \
    "v_accvgpr_write_b32 a43, 0\n\t" \
    "v_accvgpr_write_b32 a44, 0\n\t" \
    "v_accvgpr_write_b32 a45, 0\n\t" \
    "v_accvgpr_write_b32 a46, 0\n\t" \
    "v_accvgpr_write_b32 a47, 0\n\t" \
    "v_accvgpr_write_b32 a48, 0\n\t" \
    "v_accvgpr_write_b32 a49, 0\n\t" \
    "v_accvgpr_write_b32 a50, 0\n\t" \
    "v_accvgpr_write_b32 a51, 0\n\t" \
    "v_accvgpr_write_b32 a52, 0\n\t" \
    "v_accvgpr_write_b32 a53, 0\n\t" \
    "v_accvgpr_write_b32 a54, 0\n\t" \
    "v_accvgpr_write_b32 a55, 0\n\t" \
    "v_accvgpr_write_b32 a56, 0\n\t" \
    "v_accvgpr_write_b32 a57, 0\n\t" \
    "v_accvgpr_write_b32 a58, 0\n\t" \
    "v_accvgpr_write_b32 a59, 0\n\t" \
    "v_accvgpr_write_b32 a60, 0\n\t" \
    "v_accvgpr_write_b32 a61, 0\n\t" \
    "v_accvgpr_write_b32 a62, 0\n\t" \
    "v_accvgpr_write_b32 a63, 0\n\t" \
    "v_accvgpr_write_b32 a64, 0\n\t" \
    "v_accvgpr_write_b32 a65, 0\n\t" \
    "v_accvgpr_write_b32 a66, 0\n\t" \
    "v_accvgpr_write_b32 a67, 0\n\t" \
    "v_accvgpr_write_b32 a68, 0\n\t" \
    "v_accvgpr_write_b32 a69, 0\n\t" \
    "v_accvgpr_write_b32 a70, 0\n\t" \
    "v_accvgpr_write_b32 a71, 0\n\t" \
    "v_accvgpr_write_b32 a72, 0\n\t" \
    "v_accvgpr_write_b32 a73, 0\n\t" \
    "v_accvgpr_write_b32 a74, 0\n\t" \
    "v_accvgpr_write_b32 a75, 0\n\t" \
    "v_accvgpr_write_b32 a76, 0\n\t" \
    "v_accvgpr_write_b32 a77, 0\n\t" \
    "v_accvgpr_write_b32 a78, 0\n\t" \
    "v_accvgpr_write_b32 a79, 0\n\t" \
    "v_accvgpr_write_b32 a80, 0\n\t" \
    "v_accvgpr_write_b32 a81, 0\n\t" \
    "v_accvgpr_write_b32 a82, 0\n\t" \
    "v_accvgpr_write_b32 a83, 0\n\t" \
    "v_accvgpr_write_b32 a84, 0\n\t" \
    "v_accvgpr_write_b32 a85, 0\n\t" \
    "v_accvgpr_write_b32 a86, 0\n\t" \
    "v_accvgpr_write_b32 a87, 0\n\t" \
    "v_accvgpr_write_b32 a88, 0\n\t" \
    "v_accvgpr_write_b32 a89, 0\n\t" \
    "v_accvgpr_write_b32 a90, 0\n\t" \
    "v_accvgpr_write_b32 a91, 0\n\t" \
    "v_accvgpr_write_b32 a92, 0\n\t" \
    "v_accvgpr_write_b32 a93, 0\n\t" \
    "v_accvgpr_write_b32 a94, 0\n\t" \
    "v_accvgpr_write_b32 a95, 0\n\t" \
    "v_accvgpr_write_b32 a96, 0\n\t" \
    "v_accvgpr_write_b32 a97, 0\n\t" \
    "v_accvgpr_write_b32 a98, 0\n\t" \
    "v_accvgpr_write_b32 a99, 0\n\t" \
    "v_accvgpr_write_b32 a100, 0\n\t" \
    "v_accvgpr_write_b32 a101, 0\n\t" \
    "v_accvgpr_write_b32 a102, 0\n\t" \
    "v_accvgpr_write_b32 a103, 0\n\t" \
    "v_accvgpr_write_b32 a104, 0\n\t" \
    "v_accvgpr_write_b32 a105, 0\n\t" \
    "v_accvgpr_write_b32 a106, 0\n\t" \
    "v_accvgpr_write_b32 a107, 0\n\t" \
    "v_accvgpr_write_b32 a108, 0\n\t" \
    "v_accvgpr_write_b32 a109, 0\n\t" \
    "v_accvgpr_write_b32 a110, 0\n\t" \
    "v_accvgpr_write_b32 a111, 0\n\t" \
    "v_accvgpr_write_b32 a112, 0\n\t" \
    "v_accvgpr_write_b32 a113, 0\n\t" \
    "v_accvgpr_write_b32 a114, 0\n\t" \
    "v_accvgpr_write_b32 a115, 0\n\t" \
    "v_accvgpr_write_b32 a116, 0\n\t" \
    "v_accvgpr_write_b32 a117, 0\n\t" \
    "v_accvgpr_write_b32 a118, 0\n\t" \
    "v_accvgpr_write_b32 a119, 0\n\t" \
    "v_accvgpr_write_b32 a120, 0\n\t" \
    "v_accvgpr_write_b32 a121, 0\n\t" \
    "v_accvgpr_write_b32 a122, 0\n\t" \
    "v_accvgpr_write_b32 a123, 0\n\t" \
    "v_accvgpr_write_b32 a124, 0\n\t" \
    "v_accvgpr_write_b32 a125, 0\n\t" \
    "v_accvgpr_write_b32 a126, 0\n\t" \
    "v_accvgpr_write_b32 a127, 0\n\t" \
    "v_accvgpr_write_b32 a128, 0\n\t" \
    "v_accvgpr_write_b32 a129, 0\n\t" \
    "v_accvgpr_write_b32 a130, 0\n\t" \
    "v_accvgpr_write_b32 a131, 0\n\t" \
    "v_accvgpr_write_b32 a132, 0\n\t" \
    "v_accvgpr_write_b32 a133, 0\n\t" \
    "v_accvgpr_write_b32 a134, 0\n\t" \
    "v_accvgpr_write_b32 a135, 0\n\t" \
    "v_accvgpr_write_b32 a136, 0\n\t" \
    "v_accvgpr_write_b32 a137, 0\n\t" \
    "v_accvgpr_write_b32 a138, 0\n\t" \
    "v_accvgpr_write_b32 a139, 0\n\t" \
    "v_accvgpr_write_b32 a140, 0\n\t" \
    "v_accvgpr_write_b32 a141, 0\n\t" \
    "v_accvgpr_write_b32 a142, 0\n\t" \
    "v_accvgpr_write_b32 a143, 0\n\t" \
    "v_accvgpr_write_b32 a144, 0\n\t" \
    "v_accvgpr_write_b32 a145, 0\n\t" \
    "v_accvgpr_write_b32 a146, 0\n\t" \
    "v_accvgpr_write_b32 a147, 0\n\t" \
    "v_accvgpr_write_b32 a148, 0\n\t" \
    "v_accvgpr_write_b32 a149, 0\n\t" \
    "v_accvgpr_write_b32 a150, 0\n\t" \
    "v_accvgpr_write_b32 a151, 0\n\t" \
    "v_accvgpr_write_b32 a152, 0\n\t" \
    "v_accvgpr_write_b32 a153, 0\n\t" \
    "v_accvgpr_write_b32 a154, 0\n\t" \
    "v_accvgpr_write_b32 a155, 0\n\t" \
    "v_accvgpr_write_b32 a156, 0\n\t" \
    "v_accvgpr_write_b32 a157, 0\n\t" \
    "v_accvgpr_write_b32 a158, 0\n\t" \
    "v_accvgpr_write_b32 a159, 0\n\t" \
    "v_accvgpr_write_b32 a160, 0\n\t" \
    "v_accvgpr_write_b32 a161, 0\n\t" \
    "v_accvgpr_write_b32 a162, 0\n\t" \
    "v_accvgpr_write_b32 a163, 0\n\t" \
    "v_accvgpr_write_b32 a164, 0\n\t" \
    "v_accvgpr_write_b32 a165, 0\n\t" \
    "v_accvgpr_write_b32 a166, 0\n\t" \
    "v_accvgpr_write_b32 a167, 0\n\t" \
    "v_accvgpr_write_b32 a168, 0\n\t" \
    "v_accvgpr_write_b32 a169, 0\n\t" \
    "v_accvgpr_write_b32 a170, 0\n\t" \
    "v_accvgpr_write_b32 a171, 0\n\t" \
    "v_accvgpr_write_b32 a172, 0\n\t" \
    "v_accvgpr_write_b32 a173, 0\n\t" \
    "v_accvgpr_write_b32 a174, 0\n\t" \
    "v_accvgpr_write_b32 a175, 0\n\t" \
    "v_accvgpr_write_b32 a176, 0\n\t" \
    "v_accvgpr_write_b32 a177, 0\n\t" \
    "v_accvgpr_write_b32 a178, 0\n\t" \
    "v_accvgpr_write_b32 a179, 0\n\t" \
    "v_accvgpr_write_b32 a180, 0\n\t" \
    "v_accvgpr_write_b32 a181, 0\n\t" \
    "v_accvgpr_write_b32 a182, 0\n\t" \
    "v_accvgpr_write_b32 a183, 0\n\t" \
    "v_accvgpr_write_b32 a184, 0\n\t" \
    "v_accvgpr_write_b32 a185, 0\n\t" \
    "v_accvgpr_write_b32 a186, 0\n\t" \
    "v_accvgpr_write_b32 a187, 0\n\t" \
    "v_accvgpr_write_b32 a188, 0\n\t" \
    "v_accvgpr_write_b32 a189, 0\n\t" \
    "v_accvgpr_write_b32 a190, 0\n\t" \
    "v_accvgpr_write_b32 a191, 0\n\t" \
    "v_accvgpr_write_b32 a192, 0\n\t" \
    "v_accvgpr_write_b32 a193, 0\n\t" \
    "v_accvgpr_write_b32 a194, 0\n\t" \
    "v_accvgpr_write_b32 a195, 0\n\t" \
    "v_accvgpr_write_b32 a196, 0\n\t" \
    "v_accvgpr_write_b32 a197, 0\n\t" \
    "v_accvgpr_write_b32 a198, 0\n\t" \
    "v_accvgpr_write_b32 a199, 0\n\t" \
    "v_accvgpr_write_b32 a200, 0\n\t" \
    "v_accvgpr_write_b32 a201, 0\n\t" \
    "v_accvgpr_write_b32 a202, 0\n\t" \
    "v_accvgpr_write_b32 a203, 0\n\t" \
    "v_accvgpr_write_b32 a204, 0\n\t" \
    "v_accvgpr_write_b32 a205, 0\n\t" \
    "v_accvgpr_write_b32 a206, 0\n\t" \
    "v_accvgpr_write_b32 a207, 0\n\t" \
    "v_accvgpr_write_b32 a208, 0\n\t" \
    "v_accvgpr_write_b32 a209, 0\n\t" \
    "v_accvgpr_write_b32 a210, 0\n\t" \
    "v_accvgpr_write_b32 a211, 0\n\t" \
    "v_accvgpr_write_b32 a212, 0\n\t" \
    "v_accvgpr_write_b32 a213, 0\n\t" \
    "v_accvgpr_write_b32 a214, 0\n\t" \
    "v_accvgpr_write_b32 a215, 0\n\t" \
    "v_accvgpr_write_b32 a216, 0\n\t" \
    "v_accvgpr_write_b32 a217, 0\n\t" \
    "v_accvgpr_write_b32 a218, 0\n\t" \
    "v_accvgpr_write_b32 a219, 0\n\t" \
    "v_accvgpr_write_b32 a220, 0\n\t" \
    "v_accvgpr_write_b32 a221, 0\n\t" \
    "v_accvgpr_write_b32 a222, 0\n\t" \
    "v_accvgpr_write_b32 a223, 0\n\t" \
    "v_accvgpr_write_b32 a224, 0\n\t" \
    "v_accvgpr_write_b32 a225, 0\n\t" \
    "v_accvgpr_write_b32 a226, 0\n\t" \
    "v_accvgpr_write_b32 a227, 0\n\t" \
    "v_accvgpr_write_b32 a228, 0\n\t" \
    "v_accvgpr_write_b32 a229, 0\n\t" \
    "v_accvgpr_write_b32 a230, 0\n\t" \
    "v_accvgpr_write_b32 a231, 0\n\t" \
    "v_accvgpr_write_b32 a232, 0\n\t" \
    "v_accvgpr_write_b32 a233, 0\n\t" \
    "v_accvgpr_write_b32 a234, 0\n\t" \
    "v_accvgpr_write_b32 a235, 0\n\t" \
    "v_accvgpr_write_b32 a236, 0\n\t" \
    "v_accvgpr_write_b32 a237, 0\n\t" \
    "v_accvgpr_write_b32 a238, 0\n\t" \
    "v_accvgpr_write_b32 a239, 0\n\t" \
    "v_accvgpr_write_b32 a240, 0\n\t" \
    "v_accvgpr_write_b32 a241, 0\n\t" \
    "v_accvgpr_write_b32 a242, 0\n\t" \
    "v_accvgpr_write_b32 a243, 0\n\t" \
    "v_accvgpr_write_b32 a244, 0\n\t" \
    "v_accvgpr_write_b32 a245, 0\n\t" \
    "v_accvgpr_write_b32 a246, 0\n\t" \
    "v_accvgpr_write_b32 a247, 0\n\t" \
    "v_accvgpr_write_b32 a248, 0\n\t" \
    "v_accvgpr_write_b32 a249, 0\n\t" \
    "v_accvgpr_write_b32 a250, 0\n\t" \
    "v_accvgpr_write_b32 a251, 0\n\t" \
    "v_accvgpr_write_b32 a252, 0\n\t" \
    "v_accvgpr_write_b32 a253, 0\n\t" \
    "v_accvgpr_write_b32 a254, 0\n\t" \
    "v_accvgpr_write_b32 a255, 0\n\t" \
    "s_nop 3\n\t" \
    "s_waitcnt vmcnt(16)\n\t" \
    "s_barrier\n\t" \
    "v_add_u32 v116, s85, %0\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "ds_read_b64 v[144:145], v116 offset:8192\n\t" \
    "ds_read_b64 v[148:149], v116 offset:10240\n\t" \
    "ds_read_b64 v[152:153], v116 offset:12288\n\t" \
    "ds_read_b64 v[156:157], v116 offset:14336\n\t" \
    "v_add_u32 v117, s85, %1\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "ds_read_b64 v[146:147], v117 offset:8192\n\t" \
    "ds_read_b64 v[150:151], v117 offset:10240\n\t" \
    "ds_read_b64 v[154:155], v117 offset:12288\n\t" \
    "ds_read_b64 v[158:159], v117 offset:14336\n\t" \
    "v_add_u32 v118, s88, %4\n\t" \
    "ds_read_b64 v[160:161], v118 offset:0\n\t" \
    "ds_read_b64 v[164:165], v118 offset:2048\n\t" \
    "ds_read_b64 v[168:169], v118 offset:4096\n\t" \
    "ds_read_b64 v[172:173], v118 offset:6144\n\t" \
    "ds_read_b64 v[176:177], v118 offset:8192\n\t" \
    "ds_read_b64 v[180:181], v118 offset:10240\n\t" \
    "ds_read_b64 v[184:185], v118 offset:12288\n\t" \
    "ds_read_b64 v[188:189], v118 offset:14336\n\t" \
    "v_add_u32 v119, s88, %5\n\t" \
    "ds_read_b64 v[162:163], v119 offset:0\n\t" \
    "ds_read_b64 v[166:167], v119 offset:2048\n\t" \
    "ds_read_b64 v[170:171], v119 offset:4096\n\t" \
    "ds_read_b64 v[174:175], v119 offset:6144\n\t" \
    "ds_read_b64 v[178:179], v119 offset:8192\n\t" \
    "ds_read_b64 v[182:183], v119 offset:10240\n\t" \
    "ds_read_b64 v[186:187], v119 offset:12288\n\t" \
    "ds_read_b64 v[190:191], v119 offset:14336\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_cmp_lt_u32 %31, 3\n\t" \
    "s_cbranch_scc1 2f\n\t" \
    "1:\n\t" \
    "s_add_u32 s90, s87, %32\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "ds_read_b64 v[192:193], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "ds_read_b64 v[196:197], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "global_load_lds_dwordx4 %12, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[176:179], v[128:131], a[16:19]\n\t" \
    "ds_read_b64 v[200:201], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[180:183], v[128:131], a[20:23]\n\t" \
    "ds_read_b64 v[204:205], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[184:187], v[128:131], a[24:27]\n\t" \
    "ds_read_b64 v[208:209], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[188:191], v[128:131], a[28:31]\n\t" \
    "ds_read_b64 v[212:213], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[132:135], a[32:35]\n\t" \
    "ds_read_b64 v[216:217], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[132:135], a[36:39]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[132:135], a[40:43]\n\t" \
    "global_load_lds_dwordx4 %13, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[132:135], a[44:47]\n\t" \
    "ds_read_b64 v[220:221], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[176:179], v[132:135], a[48:51]\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[194:195], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[180:183], v[132:135], a[52:55]\n\t" \
    "ds_read_b64 v[198:199], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[184:187], v[132:135], a[56:59]\n\t" \
    "ds_read_b64 v[202:203], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[188:191], v[132:135], a[60:63]\n\t" \
    "ds_read_b64 v[206:207], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[136:139], a[64:67]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[136:139], a[68:71]\n\t" \
    "global_load_lds_dwordx4 %14, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[136:139], a[72:75]\n\t" \
    "ds_read_b64 v[210:211], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[136:139], a[76:79]\n\t" \
    "ds_read_b64 v[214:215], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[176:179], v[136:139], a[80:83]\n\t" \
    "ds_read_b64 v[218:219], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[180:183], v[136:139], a[84:87]\n\t" \
    "ds_read_b64 v[222:223], v117 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[184:187], v[136:139], a[88:91]\n\t" \
    "v_add_u32 v118, s88, %6\n\t" \
    "ds_read_b64 v[224:225], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[188:191], v[136:139], a[92:95]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[140:143], a[96:99]\n\t" \
    "global_load_lds_dwordx4 %15, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[140:143], a[100:103]\n\t" \
    "ds_read_b64 v[228:229], v118 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[140:143], a[104:107]\n\t" \
    "ds_read_b64 v[232:233], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[140:143], a[108:111]\n\t" \
    "ds_read_b64 v[236:237], v118 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[176:179], v[140:143], a[112:115]\n\t" \
    "ds_read_b64 v[240:241], v118 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[180:183], v[140:143], a[116:119]\n\t" \
    "ds_read_b64 v[244:245], v118 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[184:187], v[140:143], a[120:123]\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[188:191], v[140:143], a[124:127]\n\t" \
    "global_load_lds_dwordx4 %16, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[128:131], v[160:163], v[144:147], a[128:131]\n\t" \
    "ds_read_b64 v[248:249], v118 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[132:135], v[164:167], v[144:147], a[132:135]\n\t" \
    "ds_read_b64 v[252:253], v118 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[136:139], v[168:171], v[144:147], a[136:139]\n\t" \
    "v_add_u32 v119, s88, %7\n\t" \
    "ds_read_b64 v[226:227], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[140:143], v[172:175], v[144:147], a[140:143]\n\t" \
    "ds_read_b64 v[230:231], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[144:147], v[176:179], v[144:147], a[144:147]\n\t" \
    "ds_read_b64 v[234:235], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[148:151], v[180:183], v[144:147], a[148:151]\n\t" \
    "s_add_u32 m0, s90, 5120\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[152:155], v[184:187], v[144:147], a[152:155]\n\t" \
    "global_load_lds_dwordx4 %17, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[156:159], v[188:191], v[144:147], a[156:159]\n\t" \
    "ds_read_b64 v[238:239], v119 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[160:163], v[160:163], v[148:151], a[160:163]\n\t" \
    "ds_read_b64 v[242:243], v119 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[164:167], v[164:167], v[148:151], a[164:167]\n\t" \
    "ds_read_b64 v[246:247], v119 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[168:171], v[168:171], v[148:151], a[168:171]\n\t" \
    "ds_read_b64 v[250:251], v119 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[172:175], v[172:175], v[148:151], a[172:175]\n\t" \
    "ds_read_b64 v[254:255], v119 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[176:179], v[176:179], v[148:151], a[176:179]\n\t" \
    "s_add_u32 m0, s90, 6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[180:183], v[180:183], v[148:151], a[180:183]\n\t" \
    "global_load_lds_dwordx4 %18, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[184:187], v[184:187], v[148:151], a[184:187]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[188:191], v[188:191], v[148:151], a[188:191]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[192:195], v[160:163], v[152:155], a[192:195]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[196:199], v[164:167], v[152:155], a[196:199]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[200:203], v[168:171], v[152:155], a[200:203]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[204:207], v[172:175], v[152:155], a[204:207]\n\t" \
    "s_add_u32 m0, s90, 7168\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[208:211], v[176:179], v[152:155], a[208:211]\n\t" \
    "global_load_lds_dwordx4 %19, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[212:215], v[180:183], v[152:155], a[212:215]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[216:219], v[184:187], v[152:155], a[216:219]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[220:223], v[188:191], v[152:155], a[220:223]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[224:227], v[160:163], v[156:159], a[224:227]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[228:231], v[164:167], v[156:159], a[228:231]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[232:235], v[168:171], v[156:159], a[232:235]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[236:239], v[172:175], v[156:159], a[236:239]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[240:243], v[176:179], v[156:159], a[240:243]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[244:247], v[180:183], v[156:159], a[244:247]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[248:251], v[184:187], v[156:159], a[248:251]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[252:255], v[188:191], v[156:159], a[252:255]\n\t" \
    "s_add_u32 s80, s80, 128\n\t" \
    "s_addc_u32 s81, s81, 0\n\t" \
    "s_waitcnt vmcnt(8) lgkmcnt(0)\n\t" \
    "s_barrier\n\t" \
    "s_add_u32 s90, s88, %32\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[224:227], v[192:195], a[0:3]\n\t" \
    "v_add_u32 v116, s86, %0\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[228:231], v[192:195], a[4:7]\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[232:235], v[192:195], a[8:11]\n\t" \
    "global_load_lds_dwordx4 %20, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[236:239], v[192:195], a[12:15]\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[240:243], v[192:195], a[16:19]\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[244:247], v[192:195], a[20:23]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[248:251], v[192:195], a[24:27]\n\t" \
    "global_load_lds_dwordx4 %21, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[252:255], v[192:195], a[28:31]\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[224:227], v[196:199], a[32:35]\n\t" \
    "ds_read_b64 v[144:145], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[228:231], v[196:199], a[36:39]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[232:235], v[196:199], a[40:43]\n\t" \
    "global_load_lds_dwordx4 %22, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[236:239], v[196:199], a[44:47]\n\t" \
    "ds_read_b64 v[148:149], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[240:243], v[196:199], a[48:51]\n\t" \
    "ds_read_b64 v[152:153], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[244:247], v[196:199], a[52:55]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[248:251], v[196:199], a[56:59]\n\t" \
    "global_load_lds_dwordx4 %23, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[252:255], v[196:199], a[60:63]\n\t" \
    "ds_read_b64 v[156:157], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[224:227], v[200:203], a[64:67]\n\t" \
    "v_add_u32 v117, s86, %1\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[228:231], v[200:203], a[68:71]\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[232:235], v[200:203], a[72:75]\n\t" \
    "global_load_lds_dwordx4 %24, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[236:239], v[200:203], a[76:79]\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[240:243], v[200:203], a[80:83]\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[244:247], v[200:203], a[84:87]\n\t" \
    "s_add_u32 m0, s90, 5120\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[248:251], v[200:203], a[88:91]\n\t" \
    "global_load_lds_dwordx4 %25, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[252:255], v[200:203], a[92:95]\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[224:227], v[204:207], a[96:99]\n\t" \
    "ds_read_b64 v[146:147], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[228:231], v[204:207], a[100:103]\n\t" \
    "s_add_u32 m0, s90, 6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[232:235], v[204:207], a[104:107]\n\t" \
    "global_load_lds_dwordx4 %26, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[236:239], v[204:207], a[108:111]\n\t" \
    "ds_read_b64 v[150:151], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[240:243], v[204:207], a[112:115]\n\t" \
    "ds_read_b64 v[154:155], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[244:247], v[204:207], a[116:119]\n\t" \
    "s_add_u32 m0, s90, 7168\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[248:251], v[204:207], a[120:123]\n\t" \
    "global_load_lds_dwordx4 %27, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[252:255], v[204:207], a[124:127]\n\t" \
    "ds_read_b64 v[158:159], v117 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[128:131], v[224:227], v[208:211], a[128:131]\n\t" \
    "v_add_u32 v118, s89, %4\n\t" \
    "ds_read_b64 v[160:161], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[132:135], v[228:231], v[208:211], a[132:135]\n\t" \
    "ds_read_b64 v[164:165], v118 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[136:139], v[232:235], v[208:211], a[136:139]\n\t" \
    "ds_read_b64 v[168:169], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[140:143], v[236:239], v[208:211], a[140:143]\n\t" \
    "ds_read_b64 v[172:173], v118 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[144:147], v[240:243], v[208:211], a[144:147]\n\t" \
    "ds_read_b64 v[176:177], v118 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[148:151], v[244:247], v[208:211], a[148:151]\n\t" \
    "ds_read_b64 v[180:181], v118 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[152:155], v[248:251], v[208:211], a[152:155]\n\t" \
    "ds_read_b64 v[184:185], v118 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[156:159], v[252:255], v[208:211], a[156:159]\n\t" \
    "ds_read_b64 v[188:189], v118 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[160:163], v[224:227], v[212:215], a[160:163]\n\t" \
    "v_add_u32 v119, s89, %5\n\t" \
    "ds_read_b64 v[162:163], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[164:167], v[228:231], v[212:215], a[164:167]\n\t" \
    "ds_read_b64 v[166:167], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[168:171], v[232:235], v[212:215], a[168:171]\n\t" \
    "ds_read_b64 v[170:171], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[172:175], v[236:239], v[212:215], a[172:175]\n\t" \
    "ds_read_b64 v[174:175], v119 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[176:179], v[240:243], v[212:215], a[176:179]\n\t" \
    "ds_read_b64 v[178:179], v119 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[180:183], v[244:247], v[212:215], a[180:183]\n\t" \
    "ds_read_b64 v[182:183], v119 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[184:187], v[248:251], v[212:215], a[184:187]\n\t" \
    "ds_read_b64 v[186:187], v119 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[188:191], v[252:255], v[212:215], a[188:191]\n\t" \
    "ds_read_b64 v[190:191], v119 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[192:195], v[224:227], v[216:219], a[192:195]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[196:199], v[228:231], v[216:219], a[196:199]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[200:203], v[232:235], v[216:219], a[200:203]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[204:207], v[236:239], v[216:219], a[204:207]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[208:211], v[240:243], v[216:219], a[208:211]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[212:215], v[244:247], v[216:219], a[212:215]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[216:219], v[248:251], v[216:219], a[216:219]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[220:223], v[252:255], v[216:219], a[220:223]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[224:227], v[224:227], v[220:223], a[224:227]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[228:231], v[228:231], v[220:223], a[228:231]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[232:235], v[232:235], v[220:223], a[232:235]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[236:239], v[236:239], v[220:223], a[236:239]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[240:243], v[240:243], v[220:223], a[240:243]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[244:247], v[244:247], v[220:223], a[244:247]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[248:251], v[248:251], v[220:223], a[248:251]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[252:255], v[252:255], v[220:223], a[252:255]\n\t" \
    "s_mov_b32 s91, %30\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, 0\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_mov_b32 s90, s85\n\t" \
    "s_mov_b32 s85, s86\n\t" \
    "s_mov_b32 s86, s87\n\t" \
    "s_mov_b32 s87, s90\n\t" \
    "s_mov_b32 s90, s88\n\t" \
    "s_mov_b32 s88, s89\n\t" \
    "s_mov_b32 s89, s90\n\t" \
    "s_sub_u32 s84, s84, 1\n\t" \
    "s_cmp_lg_u32 s84, 0\n\t" \
    "s_cbranch_scc1 1b\n\t" \
    "2:\n\t" \
    "s_cmp_lt_u32 %31, 2\n\t" \
    "s_cbranch_scc1 3f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "ds_read_b64 v[192:193], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "ds_read_b64 v[196:197], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "ds_read_b64 v[200:201], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "ds_read_b64 v[204:205], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[176:179], v[128:131], a[16:19]\n\t" \
    "ds_read_b64 v[208:209], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[180:183], v[128:131], a[20:23]\n\t" \
    "ds_read_b64 v[212:213], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[184:187], v[128:131], a[24:27]\n\t" \
    "ds_read_b64 v[216:217], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[188:191], v[128:131], a[28:31]\n\t" \
    "ds_read_b64 v[220:221], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[132:135], a[32:35]\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[194:195], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[132:135], a[36:39]\n\t" \
    "ds_read_b64 v[198:199], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[132:135], a[40:43]\n\t" \
    "ds_read_b64 v[202:203], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[132:135], a[44:47]\n\t" \
    "ds_read_b64 v[206:207], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[176:179], v[132:135], a[48:51]\n\t" \
    "ds_read_b64 v[210:211], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[180:183], v[132:135], a[52:55]\n\t" \
    "ds_read_b64 v[214:215], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[184:187], v[132:135], a[56:59]\n\t" \
    "ds_read_b64 v[218:219], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[188:191], v[132:135], a[60:63]\n\t" \
    "ds_read_b64 v[222:223], v117 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[136:139], a[64:67]\n\t" \
    "v_add_u32 v118, s88, %6\n\t" \
    "ds_read_b64 v[224:225], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[136:139], a[68:71]\n\t" \
    "ds_read_b64 v[228:229], v118 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[136:139], a[72:75]\n\t" \
    "ds_read_b64 v[232:233], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[136:139], a[76:79]\n\t" \
    "ds_read_b64 v[236:237], v118 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[176:179], v[136:139], a[80:83]\n\t" \
    "ds_read_b64 v[240:241], v118 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[180:183], v[136:139], a[84:87]\n\t" \
    "ds_read_b64 v[244:245], v118 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[184:187], v[136:139], a[88:91]\n\t" \
    "ds_read_b64 v[248:249], v118 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[188:191], v[136:139], a[92:95]\n\t" \
    "ds_read_b64 v[252:253], v118 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[140:143], a[96:99]\n\t" \
    "v_add_u32 v119, s88, %7\n\t" \
    "ds_read_b64 v[226:227], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[140:143], a[100:103]\n\t" \
    "ds_read_b64 v[230:231], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[140:143], a[104:107]\n\t" \
    "ds_read_b64 v[234:235], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[140:143], a[108:111]\n\t" \
    "ds_read_b64 v[238:239], v119 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[176:179], v[140:143], a[112:115]\n\t" \
    "ds_read_b64 v[242:243], v119 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[180:183], v[140:143], a[116:119]\n\t" \
    "ds_read_b64 v[246:247], v119 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[184:187], v[140:143], a[120:123]\n\t" \
    "ds_read_b64 v[250:251], v119 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[188:191], v[140:143], a[124:127]\n\t" \
    "ds_read_b64 v[254:255], v119 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[128:131], v[160:163], v[144:147], a[128:131]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[132:135], v[164:167], v[144:147], a[132:135]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[136:139], v[168:171], v[144:147], a[136:139]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[140:143], v[172:175], v[144:147], a[140:143]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[144:147], v[176:179], v[144:147], a[144:147]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[148:151], v[180:183], v[144:147], a[148:151]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[152:155], v[184:187], v[144:147], a[152:155]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[156:159], v[188:191], v[144:147], a[156:159]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[160:163], v[160:163], v[148:151], a[160:163]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[164:167], v[164:167], v[148:151], a[164:167]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[168:171], v[168:171], v[148:151], a[168:171]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[172:175], v[172:175], v[148:151], a[172:175]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[176:179], v[176:179], v[148:151], a[176:179]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[180:183], v[180:183], v[148:151], a[180:183]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[184:187], v[184:187], v[148:151], a[184:187]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[188:191], v[188:191], v[148:151], a[188:191]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[192:195], v[160:163], v[152:155], a[192:195]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[196:199], v[164:167], v[152:155], a[196:199]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[200:203], v[168:171], v[152:155], a[200:203]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[204:207], v[172:175], v[152:155], a[204:207]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[208:211], v[176:179], v[152:155], a[208:211]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[212:215], v[180:183], v[152:155], a[212:215]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[216:219], v[184:187], v[152:155], a[216:219]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[220:223], v[188:191], v[152:155], a[220:223]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[224:227], v[160:163], v[156:159], a[224:227]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[228:231], v[164:167], v[156:159], a[228:231]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[232:235], v[168:171], v[156:159], a[232:235]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[236:239], v[172:175], v[156:159], a[236:239]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[240:243], v[176:179], v[156:159], a[240:243]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[244:247], v[180:183], v[156:159], a[244:247]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[248:251], v[184:187], v[156:159], a[248:251]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[252:255], v[188:191], v[156:159], a[252:255]\n\t" \
    "s_waitcnt vmcnt(0) lgkmcnt(0)\n\t" \
    "s_barrier\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[224:227], v[192:195], a[0:3]\n\t" \
    "v_add_u32 v116, s86, %0\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[228:231], v[192:195], a[4:7]\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[232:235], v[192:195], a[8:11]\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[236:239], v[192:195], a[12:15]\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[240:243], v[192:195], a[16:19]\n\t" \
    "ds_read_b64 v[144:145], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[244:247], v[192:195], a[20:23]\n\t" \
    "ds_read_b64 v[148:149], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[248:251], v[192:195], a[24:27]\n\t" \
    "ds_read_b64 v[152:153], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[252:255], v[192:195], a[28:31]\n\t" \
    "ds_read_b64 v[156:157], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[224:227], v[196:199], a[32:35]\n\t" \
    "v_add_u32 v117, s86, %1\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[228:231], v[196:199], a[36:39]\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[232:235], v[196:199], a[40:43]\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[236:239], v[196:199], a[44:47]\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[240:243], v[196:199], a[48:51]\n\t" \
    "ds_read_b64 v[146:147], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[244:247], v[196:199], a[52:55]\n\t" \
    "ds_read_b64 v[150:151], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[248:251], v[196:199], a[56:59]\n\t" \
    "ds_read_b64 v[154:155], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[252:255], v[196:199], a[60:63]\n\t" \
    "ds_read_b64 v[158:159], v117 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[224:227], v[200:203], a[64:67]\n\t" \
    "v_add_u32 v118, s89, %4\n\t" \
    "ds_read_b64 v[160:161], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[228:231], v[200:203], a[68:71]\n\t" \
    "ds_read_b64 v[164:165], v118 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[232:235], v[200:203], a[72:75]\n\t" \
    "ds_read_b64 v[168:169], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[236:239], v[200:203], a[76:79]\n\t" \
    "ds_read_b64 v[172:173], v118 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[240:243], v[200:203], a[80:83]\n\t" \
    "ds_read_b64 v[176:177], v118 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[244:247], v[200:203], a[84:87]\n\t" \
    "ds_read_b64 v[180:181], v118 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[248:251], v[200:203], a[88:91]\n\t" \
    "ds_read_b64 v[184:185], v118 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[252:255], v[200:203], a[92:95]\n\t" \
    "ds_read_b64 v[188:189], v118 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[224:227], v[204:207], a[96:99]\n\t" \
    "v_add_u32 v119, s89, %5\n\t" \
    "ds_read_b64 v[162:163], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[228:231], v[204:207], a[100:103]\n\t" \
    "ds_read_b64 v[166:167], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[232:235], v[204:207], a[104:107]\n\t" \
    "ds_read_b64 v[170:171], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[236:239], v[204:207], a[108:111]\n\t" \
    "ds_read_b64 v[174:175], v119 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[240:243], v[204:207], a[112:115]\n\t" \
    "ds_read_b64 v[178:179], v119 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[244:247], v[204:207], a[116:119]\n\t" \
    "ds_read_b64 v[182:183], v119 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[248:251], v[204:207], a[120:123]\n\t" \
    "ds_read_b64 v[186:187], v119 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[252:255], v[204:207], a[124:127]\n\t" \
    "ds_read_b64 v[190:191], v119 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[128:131], v[224:227], v[208:211], a[128:131]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[132:135], v[228:231], v[208:211], a[132:135]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[136:139], v[232:235], v[208:211], a[136:139]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[140:143], v[236:239], v[208:211], a[140:143]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[144:147], v[240:243], v[208:211], a[144:147]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[148:151], v[244:247], v[208:211], a[148:151]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[152:155], v[248:251], v[208:211], a[152:155]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[156:159], v[252:255], v[208:211], a[156:159]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[160:163], v[224:227], v[212:215], a[160:163]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[164:167], v[228:231], v[212:215], a[164:167]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[168:171], v[232:235], v[212:215], a[168:171]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[172:175], v[236:239], v[212:215], a[172:175]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[176:179], v[240:243], v[212:215], a[176:179]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[180:183], v[244:247], v[212:215], a[180:183]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[184:187], v[248:251], v[212:215], a[184:187]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[188:191], v[252:255], v[212:215], a[188:191]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[192:195], v[224:227], v[216:219], a[192:195]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[196:199], v[228:231], v[216:219], a[196:199]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[200:203], v[232:235], v[216:219], a[200:203]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[204:207], v[236:239], v[216:219], a[204:207]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[208:211], v[240:243], v[216:219], a[208:211]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[212:215], v[244:247], v[216:219], a[212:215]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[216:219], v[248:251], v[216:219], a[216:219]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[220:223], v[252:255], v[216:219], a[220:223]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[224:227], v[224:227], v[220:223], a[224:227]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[228:231], v[228:231], v[220:223], a[228:231]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[232:235], v[232:235], v[220:223], a[232:235]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[236:239], v[236:239], v[220:223], a[236:239]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[240:243], v[240:243], v[220:223], a[240:243]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[244:247], v[244:247], v[220:223], a[244:247]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[248:251], v[248:251], v[220:223], a[248:251]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[252:255], v[252:255], v[220:223], a[252:255]\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_mov_b32 s90, s85\n\t" \
    "s_mov_b32 s85, s86\n\t" \
    "s_mov_b32 s86, s87\n\t" \
    "s_mov_b32 s87, s90\n\t" \
    "s_mov_b32 s90, s88\n\t" \
    "s_mov_b32 s88, s89\n\t" \
    "s_mov_b32 s89, s90\n\t" \
    "3:\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "ds_read_b64 v[192:193], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "ds_read_b64 v[196:197], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "ds_read_b64 v[200:201], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "ds_read_b64 v[204:205], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[176:179], v[128:131], a[16:19]\n\t" \
    "ds_read_b64 v[208:209], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[180:183], v[128:131], a[20:23]\n\t" \
    "ds_read_b64 v[212:213], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[184:187], v[128:131], a[24:27]\n\t" \
    "ds_read_b64 v[216:217], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[188:191], v[128:131], a[28:31]\n\t" \
    "ds_read_b64 v[220:221], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[132:135], a[32:35]\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[194:195], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[132:135], a[36:39]\n\t" \
    "ds_read_b64 v[198:199], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[132:135], a[40:43]\n\t" \
    "ds_read_b64 v[202:203], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[132:135], a[44:47]\n\t" \
    "ds_read_b64 v[206:207], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[176:179], v[132:135], a[48:51]\n\t" \
    "ds_read_b64 v[210:211], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[180:183], v[132:135], a[52:55]\n\t" \
    "ds_read_b64 v[214:215], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[184:187], v[132:135], a[56:59]\n\t" \
    "ds_read_b64 v[218:219], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[188:191], v[132:135], a[60:63]\n\t" \
    "ds_read_b64 v[222:223], v117 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[136:139], a[64:67]\n\t" \
    "v_add_u32 v118, s88, %6\n\t" \
    "ds_read_b64 v[224:225], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[136:139], a[68:71]\n\t" \
    "ds_read_b64 v[228:229], v118 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[136:139], a[72:75]\n\t" \
    "ds_read_b64 v[232:233], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[136:139], a[76:79]\n\t" \
    "ds_read_b64 v[236:237], v118 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[176:179], v[136:139], a[80:83]\n\t" \
    "ds_read_b64 v[240:241], v118 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[180:183], v[136:139], a[84:87]\n\t" \
    "ds_read_b64 v[244:245], v118 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[184:187], v[136:139], a[88:91]\n\t" \
    "ds_read_b64 v[248:249], v118 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[188:191], v[136:139], a[92:95]\n\t" \
    "ds_read_b64 v[252:253], v118 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[140:143], a[96:99]\n\t" \
    "v_add_u32 v119, s88, %7\n\t" \
    "ds_read_b64 v[226:227], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[140:143], a[100:103]\n\t" \
    "ds_read_b64 v[230:231], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[140:143], a[104:107]\n\t" \
    "ds_read_b64 v[234:235], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[140:143], a[108:111]\n\t" \
    "ds_read_b64 v[238:239], v119 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[176:179], v[140:143], a[112:115]\n\t" \
    "ds_read_b64 v[242:243], v119 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[180:183], v[140:143], a[116:119]\n\t" \
    "ds_read_b64 v[246:247], v119 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[184:187], v[140:143], a[120:123]\n\t" \
    "ds_read_b64 v[250:251], v119 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[188:191], v[140:143], a[124:127]\n\t" \
    "ds_read_b64 v[254:255], v119 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[128:131], v[160:163], v[144:147], a[128:131]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[132:135], v[164:167], v[144:147], a[132:135]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[136:139], v[168:171], v[144:147], a[136:139]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[140:143], v[172:175], v[144:147], a[140:143]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[144:147], v[176:179], v[144:147], a[144:147]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[148:151], v[180:183], v[144:147], a[148:151]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[152:155], v[184:187], v[144:147], a[152:155]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[156:159], v[188:191], v[144:147], a[156:159]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[160:163], v[160:163], v[148:151], a[160:163]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[164:167], v[164:167], v[148:151], a[164:167]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[168:171], v[168:171], v[148:151], a[168:171]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[172:175], v[172:175], v[148:151], a[172:175]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[176:179], v[176:179], v[148:151], a[176:179]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[180:183], v[180:183], v[148:151], a[180:183]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[184:187], v[184:187], v[148:151], a[184:187]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[188:191], v[188:191], v[148:151], a[188:191]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[192:195], v[160:163], v[152:155], a[192:195]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[196:199], v[164:167], v[152:155], a[196:199]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[200:203], v[168:171], v[152:155], a[200:203]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[204:207], v[172:175], v[152:155], a[204:207]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[208:211], v[176:179], v[152:155], a[208:211]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[212:215], v[180:183], v[152:155], a[212:215]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[216:219], v[184:187], v[152:155], a[216:219]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[220:223], v[188:191], v[152:155], a[220:223]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[224:227], v[160:163], v[156:159], a[224:227]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[228:231], v[164:167], v[156:159], a[228:231]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[232:235], v[168:171], v[156:159], a[232:235]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[236:239], v[172:175], v[156:159], a[236:239]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[240:243], v[176:179], v[156:159], a[240:243]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[244:247], v[180:183], v[156:159], a[244:247]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[248:251], v[184:187], v[156:159], a[248:251]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[252:255], v[188:191], v[156:159], a[252:255]\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[224:227], v[192:195], a[0:3]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[228:231], v[192:195], a[4:7]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[232:235], v[192:195], a[8:11]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[236:239], v[192:195], a[12:15]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[240:243], v[192:195], a[16:19]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[244:247], v[192:195], a[20:23]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[248:251], v[192:195], a[24:27]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[252:255], v[192:195], a[28:31]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[224:227], v[196:199], a[32:35]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[228:231], v[196:199], a[36:39]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[232:235], v[196:199], a[40:43]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[236:239], v[196:199], a[44:47]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[240:243], v[196:199], a[48:51]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[244:247], v[196:199], a[52:55]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[248:251], v[196:199], a[56:59]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[252:255], v[196:199], a[60:63]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[224:227], v[200:203], a[64:67]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[228:231], v[200:203], a[68:71]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[232:235], v[200:203], a[72:75]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[236:239], v[200:203], a[76:79]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[240:243], v[200:203], a[80:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[244:247], v[200:203], a[84:87]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[248:251], v[200:203], a[88:91]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[252:255], v[200:203], a[92:95]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[224:227], v[204:207], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[228:231], v[204:207], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[232:235], v[204:207], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[236:239], v[204:207], a[108:111]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[240:243], v[204:207], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[244:247], v[204:207], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[248:251], v[204:207], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[252:255], v[204:207], a[124:127]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[128:131], v[224:227], v[208:211], a[128:131]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[132:135], v[228:231], v[208:211], a[132:135]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[136:139], v[232:235], v[208:211], a[136:139]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[140:143], v[236:239], v[208:211], a[140:143]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[144:147], v[240:243], v[208:211], a[144:147]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[148:151], v[244:247], v[208:211], a[148:151]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[152:155], v[248:251], v[208:211], a[152:155]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[156:159], v[252:255], v[208:211], a[156:159]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[160:163], v[224:227], v[212:215], a[160:163]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[164:167], v[228:231], v[212:215], a[164:167]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[168:171], v[232:235], v[212:215], a[168:171]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[172:175], v[236:239], v[212:215], a[172:175]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[176:179], v[240:243], v[212:215], a[176:179]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[180:183], v[244:247], v[212:215], a[180:183]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[184:187], v[248:251], v[212:215], a[184:187]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[188:191], v[252:255], v[212:215], a[188:191]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[192:195], v[224:227], v[216:219], a[192:195]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[196:199], v[228:231], v[216:219], a[196:199]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[200:203], v[232:235], v[216:219], a[200:203]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[204:207], v[236:239], v[216:219], a[204:207]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[208:211], v[240:243], v[216:219], a[208:211]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[212:215], v[244:247], v[216:219], a[212:215]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[216:219], v[248:251], v[216:219], a[216:219]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[220:223], v[252:255], v[216:219], a[220:223]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[224:227], v[224:227], v[220:223], a[224:227]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[228:231], v[228:231], v[220:223], a[228:231]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[232:235], v[232:235], v[220:223], a[232:235]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[236:239], v[236:239], v[220:223], a[236:239]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[240:243], v[240:243], v[220:223], a[240:243]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[244:247], v[244:247], v[220:223], a[244:247]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[248:251], v[248:251], v[220:223], a[248:251]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[252:255], v[252:255], v[220:223], a[252:255]\n\t" \
    "s_waitcnt vmcnt(0)\n\t" \
    "s_nop 15\n\t" \
    "s_nop 7\n\t" \
    ""

#define SYMB_GEMM16_LOOP_NN \
    "s_mov_b64 s[80:81], %28\n\t" \
    "s_mov_b64 s[82:83], %29\n\t" \
    "s_sub_u32 s84, %31, 2\n\t" \
    "s_mov_b32 s85, 0\n\t" \
    "s_mov_b32 s86, 32768\n\t" \
    "s_mov_b32 s87, 65536\n\t" \
    "s_mov_b32 s88, 98304\n\t" \
    "s_mov_b32 s89, 131072\n\t" \
    "s_add_u32 s90, s85, %32\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %12, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %13, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %14, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %15, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %16, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 5120\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %17, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 6144\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %18, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 7168\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %19, s[80:81]\n\t" \
    "s_cmp_gt_u32 %31, 1\n\t" \
    "s_cselect_b32 s91, 128, 0\n\t" \
    "s_add_u32 s80, s80, s91\n\t" \
    "s_addc_u32 s81, s81, 0\n\t" \
    "s_add_u32 s90, s88, %32\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %20, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %21, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %22, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %23, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %24, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 5120\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %25, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 6144\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %26, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 7168\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %27, s[82:83]\n\t" \
    "s_cmp_gt_u32 %31, 1\n\t" \
    "s_cselect_b32 s91, %30, 0\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, 0\n\t" \
    "s_add_u32 s90, s86, %32\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %12, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %13, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %14, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %15, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %16, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 5120\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %17, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 6144\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %18, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 7168\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %19, s[80:81]\n\t" \
    "s_add_u32 s80, s80, 128\n\t" \
    "s_addc_u32 s81, s81, 0\n\t" \
    "s_add_u32 s90, s89, %32\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %20, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %21, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %22, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %23, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %24, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 5120\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %25, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 6144\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %26, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 7168\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %27, s[82:83]\n\t" \
    "s_mov_b32 s91, %30\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, 0\n\t" \
    "v_accvgpr_write_b32 a0, 0\n\t" \
    "v_accvgpr_write_b32 a1, 0\n\t" \
    "v_accvgpr_write_b32 a2, 0\n\t" \
    "v_accvgpr_write_b32 a3, 0\n\t" \
    "v_accvgpr_write_b32 a4, 0\n\t" \
    "v_accvgpr_write_b32 a5, 0\n\t" \
    "v_accvgpr_write_b32 a6, 0\n\t" \
    "v_accvgpr_write_b32 a7, 0\n\t" \
    "v_accvgpr_write_b32 a8, 0\n\t" \
    "v_accvgpr_write_b32 a9, 0\n\t" \
    "v_accvgpr_write_b32 a10, 0\n\t" \
    "v_accvgpr_write_b32 a11, 0\n\t" \
    "v_accvgpr_write_b32 a12, 0\n\t" \
    "v_accvgpr_write_b32 a13, 0\n\t" \
    "v_accvgpr_write_b32 a14, 0\n\t" \
    "v_accvgpr_write_b32 a15, 0\n\t" \
    "v_accvgpr_write_b32 a16, 0\n\t" \
    "v_accvgpr_write_b32 a17, 0\n\t" \
    "v_accvgpr_write_b32 a18, 0\n\t" \
    "v_accvgpr_write_b32 a19, 0\n\t" \
    "v_accvgpr_write_b32 a20, 0\n\t" \
    "v_accvgpr_write_b32 a21, 0\n\t" \
    "v_accvgpr_write_b32 a22, 0\n\t" \
    "v_accvgpr_write_b32 a23, 0\n\t" \
    "v_accvgpr_write_b32 a24, 0\n\t" \
    "v_accvgpr_write_b32 a25, 0\n\t" \
    "v_accvgpr_write_b32 a26, 0\n\t" \
    "v_accvgpr_write_b32 a27, 0\n\t" \
    "v_accvgpr_write_b32 a28, 0\n\t" \
    "v_accvgpr_write_b32 a29, 0\n\t" \
    "v_accvgpr_write_b32 a30, 0\n\t" \
    "v_accvgpr_write_b32 a31, 0\n\t" \
    "v_accvgpr_write_b32 a32, 0\n\t" \
    "v_accvgpr_write_b32 a33, 0\n\t" \
    "v_accvgpr_write_b32 a34, 0\n\t" \
    "v_accvgpr_write_b32 a35, 0\n\t" \
    "v_accvgpr_write_b32 a36, 0\n\t" \
    "v_accvgpr_write_b32 a37, 0\n\t" \
    "v_accvgpr_write_b32 a38, 0\n\t" \
    "v_accvgpr_write_b32 a39, 0\n\t" \
    "v_accvgpr_write_b32 a40, 0\n\t" \
    "v_accvgpr_write_b32 a41, 0\n\t" \
    "v_accvgpr_write_b32 a42, 0\n\t" \
    "v_accvgpr_write_b32 a43, 0\n\t" \
    "v_accvgpr_write_b32 a44, 0\n\t" \
    "v_accvgpr_write_b32 a45, 0\n\t" \
    "v_accvgpr_write_b32 a46, 0\n\t" \
    "v_accvgpr_write_b32 a47, 0\n\t" \
    "v_accvgpr_write_b32 a48, 0\n\t" \
    "v_accvgpr_write_b32 a49, 0\n\t" \
    "v_accvgpr_write_b32 a50, 0\n\t" \
    "v_accvgpr_write_b32 a51, 0\n\t" \
    "v_accvgpr_write_b32 a52, 0\n\t" \
    "v_accvgpr_write_b32 a53, 0\n\t" \
    "v_accvgpr_write_b32 a54, 0\n\t" \
    "v_accvgpr_write_b32 a55, 0\n\t" \
    "v_accvgpr_write_b32 a56, 0\n\t" \
    "v_accvgpr_write_b32 a57, 0\n\t" \
    "v_accvgpr_write_b32 a58, 0\n\t" \
    "v_accvgpr_write_b32 a59, 0\n\t" \
    "v_accvgpr_write_b32 a60, 0\n\t" \
    "v_accvgpr_write_b32 a61, 0\n\t" \
    "v_accvgpr_write_b32 a62, 0\n\t" \
    "v_accvgpr_write_b32 a63, 0\n\t" \
    "v_accvgpr_write_b32 a64, 0\n\t" \
    "v_accvgpr_write_b32 a65, 0\n\t" \
    "v_accvgpr_write_b32 a66, 0\n\t" \
    "v_accvgpr_write_b32 a67, 0\n\t" \
    "v_accvgpr_write_b32 a68, 0\n\t" \
    "v_accvgpr_write_b32 a69, 0\n\t" \
    "v_accvgpr_write_b32 a70, 0\n\t" \
    "v_accvgpr_write_b32 a71, 0\n\t" \
    "v_accvgpr_write_b32 a72, 0\n\t" \
    "v_accvgpr_write_b32 a73, 0\n\t" \
    "v_accvgpr_write_b32 a74, 0\n\t" \
    "v_accvgpr_write_b32 a75, 0\n\t" \
    "v_accvgpr_write_b32 a76, 0\n\t" \
    "v_accvgpr_write_b32 a77, 0\n\t" \
    "v_accvgpr_write_b32 a78, 0\n\t" \
    "v_accvgpr_write_b32 a79, 0\n\t" \
    "v_accvgpr_write_b32 a80, 0\n\t" \
    "v_accvgpr_write_b32 a81, 0\n\t" \
    "v_accvgpr_write_b32 a82, 0\n\t" \
    "v_accvgpr_write_b32 a83, 0\n\t" \
    "v_accvgpr_write_b32 a84, 0\n\t" \
    "v_accvgpr_write_b32 a85, 0\n\t" \
    "v_accvgpr_write_b32 a86, 0\n\t" \
    "v_accvgpr_write_b32 a87, 0\n\t" \
    "v_accvgpr_write_b32 a88, 0\n\t" \
    "v_accvgpr_write_b32 a89, 0\n\t" \
    "v_accvgpr_write_b32 a90, 0\n\t" \
    "v_accvgpr_write_b32 a91, 0\n\t" \
    "v_accvgpr_write_b32 a92, 0\n\t" \
    "v_accvgpr_write_b32 a93, 0\n\t" \
    "v_accvgpr_write_b32 a94, 0\n\t" \
    "v_accvgpr_write_b32 a95, 0\n\t" \
    "v_accvgpr_write_b32 a96, 0\n\t" \
    "v_accvgpr_write_b32 a97, 0\n\t" \
    "v_accvgpr_write_b32 a98, 0\n\t" \
    "v_accvgpr_write_b32 a99, 0\n\t" \
    "v_accvgpr_write_b32 a100, 0\n\t" \
    "v_accvgpr_write_b32 a101, 0\n\t" \
    "v_accvgpr_write_b32 a102, 0\n\t" \
    "v_accvgpr_write_b32 a103, 0\n\t" \
    "v_accvgpr_write_b32 a104, 0\n\t" \
    "v_accvgpr_write_b32 a105, 0\n\t" \
    "v_accvgpr_write_b32 a106, 0\n\t" \
    "v_accvgpr_write_b32 a107, 0\n\t" \
    "v_accvgpr_write_b32 a108, 0\n\t" \
    "v_accvgpr_write_b32 a109, 0\n\t" \
    "v_accvgpr_write_b32 a110, 0\n\t" \
    "v_accvgpr_write_b32 a111, 0\n\t" \
    "v_accvgpr_write_b32 a112, 0\n\t" \
    "v_accvgpr_write_b32 a113, 0\n\t" \
    "v_accvgpr_write_b32 a114, 0\n\t" \
    "v_accvgpr_write_b32 a115, 0\n\t" \
    "v_accvgpr_write_b32 a116, 0\n\t" \
    "v_accvgpr_write_b32 a117, 0\n\t" \
    "v_accvgpr_write_b32 a118, 0\n\t" \
    "v_accvgpr_write_b32 a119, 0\n\t" \
    "v_accvgpr_write_b32 a120, 0\n\t" \
    "v_accvgpr_write_b32 a121, 0\n\t" \
    "v_accvgpr_write_b32 a122, 0\n\t" \
    "v_accvgpr_write_b32 a123, 0\n\t" \
    "v_accvgpr_write_b32 a124, 0\n\t" \
    "v_accvgpr_write_b32 a125, 0\n\t" \
    "v_accvgpr_write_b32 a126, 0\n\t" \
    "v_accvgpr_write_b32 a127, 0\n\t" \
    "v_accvgpr_write_b32 a128, 0\n\t" \
    "v_accvgpr_write_b32 a129, 0\n\t" \
    "v_accvgpr_write_b32 a130, 0\n\t" \
    "v_accvgpr_write_b32 a131, 0\n\t" \
    "v_accvgpr_write_b32 a132, 0\n\t" \
    "v_accvgpr_write_b32 a133, 0\n\t" \
    "v_accvgpr_write_b32 a134, 0\n\t" \
    "v_accvgpr_write_b32 a135, 0\n\t" \
    "v_accvgpr_write_b32 a136, 0\n\t" \
    "v_accvgpr_write_b32 a137, 0\n\t" \
    "v_accvgpr_write_b32 a138, 0\n\t" \
    "v_accvgpr_write_b32 a139, 0\n\t" \
    "v_accvgpr_write_b32 a140, 0\n\t" \
    "v_accvgpr_write_b32 a141, 0\n\t" \
    "v_accvgpr_write_b32 a142, 0\n\t" \
    "v_accvgpr_write_b32 a143, 0\n\t" \
    "v_accvgpr_write_b32 a144, 0\n\t" \
    "v_accvgpr_write_b32 a145, 0\n\t" \
    "v_accvgpr_write_b32 a146, 0\n\t" \
    "v_accvgpr_write_b32 a147, 0\n\t" \
    "v_accvgpr_write_b32 a148, 0\n\t" \
    "v_accvgpr_write_b32 a149, 0\n\t" \
    "v_accvgpr_write_b32 a150, 0\n\t" \
    "v_accvgpr_write_b32 a151, 0\n\t" \
    "v_accvgpr_write_b32 a152, 0\n\t" \
    "v_accvgpr_write_b32 a153, 0\n\t" \
    "v_accvgpr_write_b32 a154, 0\n\t" \
    "v_accvgpr_write_b32 a155, 0\n\t" \
    "v_accvgpr_write_b32 a156, 0\n\t" \
    "v_accvgpr_write_b32 a157, 0\n\t" \
    "v_accvgpr_write_b32 a158, 0\n\t" \
    "v_accvgpr_write_b32 a159, 0\n\t" \
    "v_accvgpr_write_b32 a160, 0\n\t" \
    "v_accvgpr_write_b32 a161, 0\n\t" \
    "v_accvgpr_write_b32 a162, 0\n\t" \
    "v_accvgpr_write_b32 a163, 0\n\t" \
    "v_accvgpr_write_b32 a164, 0\n\t" \
    "v_accvgpr_write_b32 a165, 0\n\t" \
    "v_accvgpr_write_b32 a166, 0\n\t" \
    "v_accvgpr_write_b32 a167, 0\n\t" \
    "v_accvgpr_write_b32 a168, 0\n\t" \
    "v_accvgpr_write_b32 a169, 0\n\t" \
    "v_accvgpr_write_b32 a170, 0\n\t" \
    "v_accvgpr_write_b32 a171, 0\n\t" \
    "v_accvgpr_write_b32 a172, 0\n\t" \
    "v_accvgpr_write_b32 a173, 0\n\t" \
    "v_accvgpr_write_b32 a174, 0\n\t" \
    "v_accvgpr_write_b32 a175, 0\n\t" \
    "v_accvgpr_write_b32 a176, 0\n\t" \
    "v_accvgpr_write_b32 a177, 0\n\t" \
    "v_accvgpr_write_b32 a178, 0\n\t" \
    "v_accvgpr_write_b32 a179, 0\n\t" \
    "v_accvgpr_write_b32 a180, 0\n\t" \
    "v_accvgpr_write_b32 a181, 0\n\t" \
    "v_accvgpr_write_b32 a182, 0\n\t" \
    "v_accvgpr_write_b32 a183, 0\n\t" \
    "v_accvgpr_write_b32 a184, 0\n\t" \
    "v_accvgpr_write_b32 a185, 0\n\t" \
    "v_accvgpr_write_b32 a186, 0\n\t" \
    "v_accvgpr_write_b32 a187, 0\n\t" \
    "v_accvgpr_write_b32 a188, 0\n\t" \
    "v_accvgpr_write_b32 a189, 0\n\t" \
    "v_accvgpr_write_b32 a190, 0\n\t" \
    "v_accvgpr_write_b32 a191, 0\n\t" \
    "v_accvgpr_write_b32 a192, 0\n\t" \
    "v_accvgpr_write_b32 a193, 0\n\t" \
    "v_accvgpr_write_b32 a194, 0\n\t" \
    "v_accvgpr_write_b32 a195, 0\n\t" \
    "v_accvgpr_write_b32 a196, 0\n\t" \
    "v_accvgpr_write_b32 a197, 0\n\t" \
    "v_accvgpr_write_b32 a198, 0\n\t" \
    "v_accvgpr_write_b32 a199, 0\n\t" \
    "v_accvgpr_write_b32 a200, 0\n\t" \
    "v_accvgpr_write_b32 a201, 0\n\t" \
    "v_accvgpr_write_b32 a202, 0\n\t" \
    "v_accvgpr_write_b32 a203, 0\n\t" \
    "v_accvgpr_write_b32 a204, 0\n\t" \
    "v_accvgpr_write_b32 a205, 0\n\t" \
    "v_accvgpr_write_b32 a206, 0\n\t" \
    "v_accvgpr_write_b32 a207, 0\n\t" \
    "v_accvgpr_write_b32 a208, 0\n\t" \
    "v_accvgpr_write_b32 a209, 0\n\t" \
    "v_accvgpr_write_b32 a210, 0\n\t" \
    "v_accvgpr_write_b32 a211, 0\n\t" \
    "v_accvgpr_write_b32 a212, 0\n\t" \
    "v_accvgpr_write_b32 a213, 0\n\t" \
    "v_accvgpr_write_b32 a214, 0\n\t" \
    "v_accvgpr_write_b32 a215, 0\n\t" \
    "v_accvgpr_write_b32 a216, 0\n\t" \
    "v_accvgpr_write_b32 a217, 0\n\t" \
    "v_accvgpr_write_b32 a218, 0\n\t" \
    "v_accvgpr_write_b32 a219, 0\n\t" \
    "v_accvgpr_write_b32 a220, 0\n\t" \
    "v_accvgpr_write_b32 a221, 0\n\t" \
    "v_accvgpr_write_b32 a222, 0\n\t" \
    "v_accvgpr_write_b32 a223, 0\n\t" \
    "v_accvgpr_write_b32 a224, 0\n\t" \
    "v_accvgpr_write_b32 a225, 0\n\t" \
    "v_accvgpr_write_b32 a226, 0\n\t" \
    "v_accvgpr_write_b32 a227, 0\n\t" \
    "v_accvgpr_write_b32 a228, 0\n\t" \
    "v_accvgpr_write_b32 a229, 0\n\t" \
    "v_accvgpr_write_b32 a230, 0\n\t" \
    "v_accvgpr_write_b32 a231, 0\n\t" \
    "v_accvgpr_write_b32 a232, 0\n\t" \
    "v_accvgpr_write_b32 a233, 0\n\t" \
    "v_accvgpr_write_b32 a234, 0\n\t" \
    "v_accvgpr_write_b32 a235, 0\n\t" \
    "v_accvgpr_write_b32 a236, 0\n\t" \
    "v_accvgpr_write_b32 a237, 0\n\t" \
    "v_accvgpr_write_b32 a238, 0\n\t" \
    "v_accvgpr_write_b32 a239, 0\n\t" \
    "v_accvgpr_write_b32 a240, 0\n\t" \
    "v_accvgpr_write_b32 a241, 0\n\t" \
    "v_accvgpr_write_b32 a242, 0\n\t" \
    "v_accvgpr_write_b32 a243, 0\n\t" \
    "v_accvgpr_write_b32 a244, 0\n\t" \
    "v_accvgpr_write_b32 a245, 0\n\t" \
    "v_accvgpr_write_b32 a246, 0\n\t" \
    "v_accvgpr_write_b32 a247, 0\n\t" \
    "v_accvgpr_write_b32 a248, 0\n\t" \
    "v_accvgpr_write_b32 a249, 0\n\t" \
    "v_accvgpr_write_b32 a250, 0\n\t" \
    "v_accvgpr_write_b32 a251, 0\n\t" \
    "v_accvgpr_write_b32 a252, 0\n\t" \
    "v_accvgpr_write_b32 a253, 0\n\t" \
    "v_accvgpr_write_b32 a254, 0\n\t" \
    "v_accvgpr_write_b32 a255, 0\n\t" \
    "s_nop 3\n\t" \
    "s_waitcnt vmcnt(16)\n\t" \
    "s_barrier\n\t" \
    "v_add_u32 v116, s85, %0\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "ds_read_b64 v[144:145], v116 offset:8192\n\t" \
    "ds_read_b64 v[148:149], v116 offset:10240\n\t" \
    "ds_read_b64 v[152:153], v116 offset:12288\n\t" \
    "ds_read_b64 v[156:157], v116 offset:14336\n\t" \
    "v_add_u32 v117, s85, %1\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "ds_read_b64 v[146:147], v117 offset:8192\n\t" \
    "ds_read_b64 v[150:151], v117 offset:10240\n\t" \
    "ds_read_b64 v[154:155], v117 offset:12288\n\t" \
    "ds_read_b64 v[158:159], v117 offset:14336\n\t" \
    "v_add_u32 v118, s88, %4\n\t" \
    "ds_read_b64_tr_b16 v[160:161], v118 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[162:163], v118 offset:8192\n\t" \
    "v_add_u32 v119, s88, %5\n\t" \
    "ds_read_b64_tr_b16 v[164:165], v119 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[166:167], v119 offset:8192\n\t" \
    "v_add_u32 v120, s88, %6\n\t" \
    "ds_read_b64_tr_b16 v[168:169], v120 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[170:171], v120 offset:8192\n\t" \
    "v_add_u32 v121, s88, %7\n\t" \
    "ds_read_b64_tr_b16 v[172:173], v121 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[174:175], v121 offset:8192\n\t" \
    "v_add_u32 v122, s88, %8\n\t" \
    "ds_read_b64_tr_b16 v[176:177], v122 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[178:179], v122 offset:8192\n\t" \
    "v_add_u32 v123, s88, %9\n\t" \
    "ds_read_b64_tr_b16 v[180:181], v123 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[182:183], v123 offset:8192\n\t" \
    "v_add_u32 v124, s88, %10\n\t" \
    "ds_read_b64_tr_b16 v[184:185], v124 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[186:187], v124 offset:8192\n\t" \
    "v_add_u32 v125, s88, %11\n\t" \
    "ds_read_b64_tr_b16 v[188:189], v125 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[190:191], v125 offset:8192\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_cmp_lt_u32 %31, 3\n\t" \
    "s_cbranch_scc1 2f\n\t" \
    "1:\n\t" \
    "s_add_u32 s90, s87, %32\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "ds_read_b64 v[192:193], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "ds_read_b64 v[196:197], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "global_load_lds_dwordx4 %12, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[176:179], v[128:131], a[16:19]\n\t" \
    "ds_read_b64 v[200:201], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[180:183], v[128:131], a[20:23]\n\t" \
    "ds_read_b64 v[204:205], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[184:187], v[128:131], a[24:27]\n\t" \
    "ds_read_b64 v[208:209], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[188:191], v[128:131], a[28:31]\n\t" \
    "ds_read_b64 v[212:213], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[132:135], a[32:35]\n\t" \
    "ds_read_b64 v[216:217], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[132:135], a[36:39]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[132:135], a[40:43]\n\t" \
    "global_load_lds_dwordx4 %13, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[132:135], a[44:47]\n\t" \
    "ds_read_b64 v[220:221], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[176:179], v[132:135], a[48:51]\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[194:195], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[180:183], v[132:135], a[52:55]\n\t" \
    "ds_read_b64 v[198:199], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[184:187], v[132:135], a[56:59]\n\t" \
    "ds_read_b64 v[202:203], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[188:191], v[132:135], a[60:63]\n\t" \
    "ds_read_b64 v[206:207], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[136:139], a[64:67]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[136:139], a[68:71]\n\t" \
    "global_load_lds_dwordx4 %14, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[136:139], a[72:75]\n\t" \
    "ds_read_b64 v[210:211], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[136:139], a[76:79]\n\t" \
    "ds_read_b64 v[214:215], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[176:179], v[136:139], a[80:83]\n\t" \
    "ds_read_b64 v[218:219], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[180:183], v[136:139], a[84:87]\n\t" \
    "ds_read_b64 v[222:223], v117 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[184:187], v[136:139], a[88:91]\n\t" \
    "v_add_u32 v118, s88, %4\n\t" \
    "ds_read_b64_tr_b16 v[224:225], v118 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[188:191], v[136:139], a[92:95]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[140:143], a[96:99]\n\t" \
    "global_load_lds_dwordx4 %15, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[140:143], a[100:103]\n\t" \
    "ds_read_b64_tr_b16 v[226:227], v118 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[140:143], a[104:107]\n\t" \
    "v_add_u32 v119, s88, %5\n\t" \
    "ds_read_b64_tr_b16 v[228:229], v119 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[140:143], a[108:111]\n\t" \
    "ds_read_b64_tr_b16 v[230:231], v119 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[176:179], v[140:143], a[112:115]\n\t" \
    "v_add_u32 v120, s88, %6\n\t" \
    "ds_read_b64_tr_b16 v[232:233], v120 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[180:183], v[140:143], a[116:119]\n\t" \
    "ds_read_b64_tr_b16 v[234:235], v120 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[184:187], v[140:143], a[120:123]\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[188:191], v[140:143], a[124:127]\n\t" \
    "global_load_lds_dwordx4 %16, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[128:131], v[160:163], v[144:147], a[128:131]\n\t" \
    "v_add_u32 v121, s88, %7\n\t" \
    "ds_read_b64_tr_b16 v[236:237], v121 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[132:135], v[164:167], v[144:147], a[132:135]\n\t" \
    "ds_read_b64_tr_b16 v[238:239], v121 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[136:139], v[168:171], v[144:147], a[136:139]\n\t" \
    "v_add_u32 v122, s88, %8\n\t" \
    "ds_read_b64_tr_b16 v[240:241], v122 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[140:143], v[172:175], v[144:147], a[140:143]\n\t" \
    "ds_read_b64_tr_b16 v[242:243], v122 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[144:147], v[176:179], v[144:147], a[144:147]\n\t" \
    "v_add_u32 v123, s88, %9\n\t" \
    "ds_read_b64_tr_b16 v[244:245], v123 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[148:151], v[180:183], v[144:147], a[148:151]\n\t" \
    "s_add_u32 m0, s90, 5120\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[152:155], v[184:187], v[144:147], a[152:155]\n\t" \
    "global_load_lds_dwordx4 %17, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[156:159], v[188:191], v[144:147], a[156:159]\n\t" \
    "ds_read_b64_tr_b16 v[246:247], v123 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[160:163], v[160:163], v[148:151], a[160:163]\n\t" \
    "v_add_u32 v124, s88, %10\n\t" \
    "ds_read_b64_tr_b16 v[248:249], v124 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[164:167], v[164:167], v[148:151], a[164:167]\n\t" \
    "ds_read_b64_tr_b16 v[250:251], v124 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[168:171], v[168:171], v[148:151], a[168:171]\n\t" \
    "v_add_u32 v125, s88, %11\n\t" \
    "ds_read_b64_tr_b16 v[252:253], v125 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[172:175], v[172:175], v[148:151], a[172:175]\n\t" \
    "ds_read_b64_tr_b16 v[254:255], v125 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[176:179], v[176:179], v[148:151], a[176:179]\n\t" \
    "s_add_u32 m0, s90, 6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[180:183], v[180:183], v[148:151], a[180:183]\n\t" \
    "global_load_lds_dwordx4 %18, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[184:187], v[184:187], v[148:151], a[184:187]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[188:191], v[188:191], v[148:151], a[188:191]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[192:195], v[160:163], v[152:155], a[192:195]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[196:199], v[164:167], v[152:155], a[196:199]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[200:203], v[168:171], v[152:155], a[200:203]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[204:207], v[172:175], v[152:155], a[204:207]\n\t" \
    "s_add_u32 m0, s90, 7168\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[208:211], v[176:179], v[152:155], a[208:211]\n\t" \
    "global_load_lds_dwordx4 %19, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[212:215], v[180:183], v[152:155], a[212:215]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[216:219], v[184:187], v[152:155], a[216:219]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[220:223], v[188:191], v[152:155], a[220:223]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[224:227], v[160:163], v[156:159], a[224:227]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[228:231], v[164:167], v[156:159], a[228:231]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[232:235], v[168:171], v[156:159], a[232:235]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[236:239], v[172:175], v[156:159], a[236:239]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[240:243], v[176:179], v[156:159], a[240:243]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[244:247], v[180:183], v[156:159], a[244:247]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[248:251], v[184:187], v[156:159], a[248:251]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[252:255], v[188:191], v[156:159], a[252:255]\n\t" \
    "s_add_u32 s80, s80, 128\n\t" \
    "s_addc_u32 s81, s81, 0\n\t" \
    "s_waitcnt vmcnt(8) lgkmcnt(0)\n\t" \
    "s_barrier\n\t" \
    "s_add_u32 s90, s88, %32\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[224:227], v[192:195], a[0:3]\n\t" \
    "v_add_u32 v116, s86, %0\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[228:231], v[192:195], a[4:7]\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[232:235], v[192:195], a[8:11]\n\t" \
    "global_load_lds_dwordx4 %20, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[236:239], v[192:195], a[12:15]\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[240:243], v[192:195], a[16:19]\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[244:247], v[192:195], a[20:23]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[248:251], v[192:195], a[24:27]\n\t" \
    "global_load_lds_dwordx4 %21, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[252:255], v[192:195], a[28:31]\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[224:227], v[196:199], a[32:35]\n\t" \
    "ds_read_b64 v[144:145], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[228:231], v[196:199], a[36:39]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[232:235], v[196:199], a[40:43]\n\t" \
    "global_load_lds_dwordx4 %22, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[236:239], v[196:199], a[44:47]\n\t" \
    "ds_read_b64 v[148:149], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[240:243], v[196:199], a[48:51]\n\t" \
    "ds_read_b64 v[152:153], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[244:247], v[196:199], a[52:55]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[248:251], v[196:199], a[56:59]\n\t" \
    "global_load_lds_dwordx4 %23, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[252:255], v[196:199], a[60:63]\n\t" \
    "ds_read_b64 v[156:157], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[224:227], v[200:203], a[64:67]\n\t" \
    "v_add_u32 v117, s86, %1\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[228:231], v[200:203], a[68:71]\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[232:235], v[200:203], a[72:75]\n\t" \
    "global_load_lds_dwordx4 %24, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[236:239], v[200:203], a[76:79]\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[240:243], v[200:203], a[80:83]\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[244:247], v[200:203], a[84:87]\n\t" \
    "s_add_u32 m0, s90, 5120\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[248:251], v[200:203], a[88:91]\n\t" \
    "global_load_lds_dwordx4 %25, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[252:255], v[200:203], a[92:95]\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[224:227], v[204:207], a[96:99]\n\t" \
    "ds_read_b64 v[146:147], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[228:231], v[204:207], a[100:103]\n\t" \
    "s_add_u32 m0, s90, 6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[232:235], v[204:207], a[104:107]\n\t" \
    "global_load_lds_dwordx4 %26, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[236:239], v[204:207], a[108:111]\n\t" \
    "ds_read_b64 v[150:151], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[240:243], v[204:207], a[112:115]\n\t" \
    "ds_read_b64 v[154:155], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[244:247], v[204:207], a[116:119]\n\t" \
    "s_add_u32 m0, s90, 7168\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[248:251], v[204:207], a[120:123]\n\t" \
    "global_load_lds_dwordx4 %27, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[252:255], v[204:207], a[124:127]\n\t" \
    "ds_read_b64 v[158:159], v117 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[128:131], v[224:227], v[208:211], a[128:131]\n\t" \
    "v_add_u32 v118, s89, %4\n\t" \
    "ds_read_b64_tr_b16 v[160:161], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[132:135], v[228:231], v[208:211], a[132:135]\n\t" \
    "ds_read_b64_tr_b16 v[162:163], v118 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[136:139], v[232:235], v[208:211], a[136:139]\n\t" \
    "v_add_u32 v119, s89, %5\n\t" \
    "ds_read_b64_tr_b16 v[164:165], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[140:143], v[236:239], v[208:211], a[140:143]\n\t" \
    "ds_read_b64_tr_b16 v[166:167], v119 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[144:147], v[240:243], v[208:211], a[144:147]\n\t" \
    "v_add_u32 v120, s89, %6\n\t" \
    "ds_read_b64_tr_b16 v[168:169], v120 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[148:151], v[244:247], v[208:211], a[148:151]\n\t" \
    "ds_read_b64_tr_b16 v[170:171], v120 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[152:155], v[248:251], v[208:211], a[152:155]\n\t" \
    "v_add_u32 v121, s89, %7\n\t" \
    "ds_read_b64_tr_b16 v[172:173], v121 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[156:159], v[252:255], v[208:211], a[156:159]\n\t" \
    "ds_read_b64_tr_b16 v[174:175], v121 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[160:163], v[224:227], v[212:215], a[160:163]\n\t" \
    "v_add_u32 v122, s89, %8\n\t" \
    "ds_read_b64_tr_b16 v[176:177], v122 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[164:167], v[228:231], v[212:215], a[164:167]\n\t" \
    "ds_read_b64_tr_b16 v[178:179], v122 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[168:171], v[232:235], v[212:215], a[168:171]\n\t" \
    "v_add_u32 v123, s89, %9\n\t" \
    "ds_read_b64_tr_b16 v[180:181], v123 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[172:175], v[236:239], v[212:215], a[172:175]\n\t" \
    "ds_read_b64_tr_b16 v[182:183], v123 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[176:179], v[240:243], v[212:215], a[176:179]\n\t" \
    "v_add_u32 v124, s89, %10\n\t" \
    "ds_read_b64_tr_b16 v[184:185], v124 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[180:183], v[244:247], v[212:215], a[180:183]\n\t" \
    "ds_read_b64_tr_b16 v[186:187], v124 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[184:187], v[248:251], v[212:215], a[184:187]\n\t" \
    "v_add_u32 v125, s89, %11\n\t" \
    "ds_read_b64_tr_b16 v[188:189], v125 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[188:191], v[252:255], v[212:215], a[188:191]\n\t" \
    "ds_read_b64_tr_b16 v[190:191], v125 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[192:195], v[224:227], v[216:219], a[192:195]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[196:199], v[228:231], v[216:219], a[196:199]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[200:203], v[232:235], v[216:219], a[200:203]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[204:207], v[236:239], v[216:219], a[204:207]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[208:211], v[240:243], v[216:219], a[208:211]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[212:215], v[244:247], v[216:219], a[212:215]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[216:219], v[248:251], v[216:219], a[216:219]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[220:223], v[252:255], v[216:219], a[220:223]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[224:227], v[224:227], v[220:223], a[224:227]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[228:231], v[228:231], v[220:223], a[228:231]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[232:235], v[232:235], v[220:223], a[232:235]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[236:239], v[236:239], v[220:223], a[236:239]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[240:243], v[240:243], v[220:223], a[240:243]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[244:247], v[244:247], v[220:223], a[244:247]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[248:251], v[248:251], v[220:223], a[248:251]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[252:255], v[252:255], v[220:223], a[252:255]\n\t" \
    "s_mov_b32 s91, %30\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, 0\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_mov_b32 s90, s85\n\t" \
    "s_mov_b32 s85, s86\n\t" \
    "s_mov_b32 s86, s87\n\t" \
    "s_mov_b32 s87, s90\n\t" \
    "s_mov_b32 s90, s88\n\t" \
    "s_mov_b32 s88, s89\n\t" \
    "s_mov_b32 s89, s90\n\t" \
    "s_sub_u32 s84, s84, 1\n\t" \
    "s_cmp_lg_u32 s84, 0\n\t" \
    "s_cbranch_scc1 1b\n\t" \
    "2:\n\t" \
    "s_cmp_lt_u32 %31, 2\n\t" \
    "s_cbranch_scc1 3f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "ds_read_b64 v[192:193], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "ds_read_b64 v[196:197], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "ds_read_b64 v[200:201], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "ds_read_b64 v[204:205], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[176:179], v[128:131], a[16:19]\n\t" \
    "ds_read_b64 v[208:209], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[180:183], v[128:131], a[20:23]\n\t" \
    "ds_read_b64 v[212:213], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[184:187], v[128:131], a[24:27]\n\t" \
    "ds_read_b64 v[216:217], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[188:191], v[128:131], a[28:31]\n\t" \
    "ds_read_b64 v[220:221], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[132:135], a[32:35]\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[194:195], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[132:135], a[36:39]\n\t" \
    "ds_read_b64 v[198:199], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[132:135], a[40:43]\n\t" \
    "ds_read_b64 v[202:203], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[132:135], a[44:47]\n\t" \
    "ds_read_b64 v[206:207], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[176:179], v[132:135], a[48:51]\n\t" \
    "ds_read_b64 v[210:211], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[180:183], v[132:135], a[52:55]\n\t" \
    "ds_read_b64 v[214:215], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[184:187], v[132:135], a[56:59]\n\t" \
    "ds_read_b64 v[218:219], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[188:191], v[132:135], a[60:63]\n\t" \
    "ds_read_b64 v[222:223], v117 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[136:139], a[64:67]\n\t" \
    "v_add_u32 v118, s88, %4\n\t" \
    "ds_read_b64_tr_b16 v[224:225], v118 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[136:139], a[68:71]\n\t" \
    "ds_read_b64_tr_b16 v[226:227], v118 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[136:139], a[72:75]\n\t" \
    "v_add_u32 v119, s88, %5\n\t" \
    "ds_read_b64_tr_b16 v[228:229], v119 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[136:139], a[76:79]\n\t" \
    "ds_read_b64_tr_b16 v[230:231], v119 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[176:179], v[136:139], a[80:83]\n\t" \
    "v_add_u32 v120, s88, %6\n\t" \
    "ds_read_b64_tr_b16 v[232:233], v120 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[180:183], v[136:139], a[84:87]\n\t" \
    "ds_read_b64_tr_b16 v[234:235], v120 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[184:187], v[136:139], a[88:91]\n\t" \
    "v_add_u32 v121, s88, %7\n\t" \
    "ds_read_b64_tr_b16 v[236:237], v121 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[188:191], v[136:139], a[92:95]\n\t" \
    "ds_read_b64_tr_b16 v[238:239], v121 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[140:143], a[96:99]\n\t" \
    "v_add_u32 v122, s88, %8\n\t" \
    "ds_read_b64_tr_b16 v[240:241], v122 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[140:143], a[100:103]\n\t" \
    "ds_read_b64_tr_b16 v[242:243], v122 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[140:143], a[104:107]\n\t" \
    "v_add_u32 v123, s88, %9\n\t" \
    "ds_read_b64_tr_b16 v[244:245], v123 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[140:143], a[108:111]\n\t" \
    "ds_read_b64_tr_b16 v[246:247], v123 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[176:179], v[140:143], a[112:115]\n\t" \
    "v_add_u32 v124, s88, %10\n\t" \
    "ds_read_b64_tr_b16 v[248:249], v124 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[180:183], v[140:143], a[116:119]\n\t" \
    "ds_read_b64_tr_b16 v[250:251], v124 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[184:187], v[140:143], a[120:123]\n\t" \
    "v_add_u32 v125, s88, %11\n\t" \
    "ds_read_b64_tr_b16 v[252:253], v125 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[188:191], v[140:143], a[124:127]\n\t" \
    "ds_read_b64_tr_b16 v[254:255], v125 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[128:131], v[160:163], v[144:147], a[128:131]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[132:135], v[164:167], v[144:147], a[132:135]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[136:139], v[168:171], v[144:147], a[136:139]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[140:143], v[172:175], v[144:147], a[140:143]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[144:147], v[176:179], v[144:147], a[144:147]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[148:151], v[180:183], v[144:147], a[148:151]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[152:155], v[184:187], v[144:147], a[152:155]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[156:159], v[188:191], v[144:147], a[156:159]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[160:163], v[160:163], v[148:151], a[160:163]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[164:167], v[164:167], v[148:151], a[164:167]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[168:171], v[168:171], v[148:151], a[168:171]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[172:175], v[172:175], v[148:151], a[172:175]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[176:179], v[176:179], v[148:151], a[176:179]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[180:183], v[180:183], v[148:151], a[180:183]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[184:187], v[184:187], v[148:151], a[184:187]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[188:191], v[188:191], v[148:151], a[188:191]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[192:195], v[160:163], v[152:155], a[192:195]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[196:199], v[164:167], v[152:155], a[196:199]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[200:203], v[168:171], v[152:155], a[200:203]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[204:207], v[172:175], v[152:155], a[204:207]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[208:211], v[176:179], v[152:155], a[208:211]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[212:215], v[180:183], v[152:155], a[212:215]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[216:219], v[184:187], v[152:155], a[216:219]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[220:223], v[188:191], v[152:155], a[220:223]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[224:227], v[160:163], v[156:159], a[224:227]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[228:231], v[164:167], v[156:159], a[228:231]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[232:235], v[168:171], v[156:159], a[232:235]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[236:239], v[172:175], v[156:159], a[236:239]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[240:243], v[176:179], v[156:159], a[240:243]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[244:247], v[180:183], v[156:159], a[244:247]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[248:251], v[184:187], v[156:159], a[248:251]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[252:255], v[188:191], v[156:159], a[252:255]\n\t" \
    "s_waitcnt vmcnt(0) lgkmcnt(0)\n\t" \
    "s_barrier\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[224:227], v[192:195], a[0:3]\n\t" \
    "v_add_u32 v116, s86, %0\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[228:231], v[192:195], a[4:7]\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[232:235], v[192:195], a[8:11]\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[236:239], v[192:195], a[12:15]\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[240:243], v[192:195], a[16:19]\n\t" \
    "ds_read_b64 v[144:145], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[244:247], v[192:195], a[20:23]\n\t" \
    "ds_read_b64 v[148:149], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[248:251], v[192:195], a[24:27]\n\t" \
    "ds_read_b64 v[152:153], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[252:255], v[192:195], a[28:31]\n\t" \
    "ds_read_b64 v[156:157], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[224:227], v[196:199], a[32:35]\n\t" \
    "v_add_u32 v117, s86, %1\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[228:231], v[196:199], a[36:39]\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[232:235], v[196:199], a[40:43]\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[236:239], v[196:199], a[44:47]\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[240:243], v[196:199], a[48:51]\n\t" \
    "ds_read_b64 v[146:147], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[244:247], v[196:199], a[52:55]\n\t" \
    "ds_read_b64 v[150:151], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[248:251], v[196:199], a[56:59]\n\t" \
    "ds_read_b64 v[154:155], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[252:255], v[196:199], a[60:63]\n\t" \
    "ds_read_b64 v[158:159], v117 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[224:227], v[200:203], a[64:67]\n\t" \
    "v_add_u32 v118, s89, %4\n\t" \
    "ds_read_b64_tr_b16 v[160:161], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[228:231], v[200:203], a[68:71]\n\t" \
    "ds_read_b64_tr_b16 v[162:163], v118 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[232:235], v[200:203], a[72:75]\n\t" \
    "v_add_u32 v119, s89, %5\n\t" \
    "ds_read_b64_tr_b16 v[164:165], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[236:239], v[200:203], a[76:79]\n\t" \
    "ds_read_b64_tr_b16 v[166:167], v119 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[240:243], v[200:203], a[80:83]\n\t" \
    "v_add_u32 v120, s89, %6\n\t" \
    "ds_read_b64_tr_b16 v[168:169], v120 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[244:247], v[200:203], a[84:87]\n\t" \
    "ds_read_b64_tr_b16 v[170:171], v120 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[248:251], v[200:203], a[88:91]\n\t" \
    "v_add_u32 v121, s89, %7\n\t" \
    "ds_read_b64_tr_b16 v[172:173], v121 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[252:255], v[200:203], a[92:95]\n\t" \
    "ds_read_b64_tr_b16 v[174:175], v121 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[224:227], v[204:207], a[96:99]\n\t" \
    "v_add_u32 v122, s89, %8\n\t" \
    "ds_read_b64_tr_b16 v[176:177], v122 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[228:231], v[204:207], a[100:103]\n\t" \
    "ds_read_b64_tr_b16 v[178:179], v122 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[232:235], v[204:207], a[104:107]\n\t" \
    "v_add_u32 v123, s89, %9\n\t" \
    "ds_read_b64_tr_b16 v[180:181], v123 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[236:239], v[204:207], a[108:111]\n\t" \
    "ds_read_b64_tr_b16 v[182:183], v123 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[240:243], v[204:207], a[112:115]\n\t" \
    "v_add_u32 v124, s89, %10\n\t" \
    "ds_read_b64_tr_b16 v[184:185], v124 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[244:247], v[204:207], a[116:119]\n\t" \
    "ds_read_b64_tr_b16 v[186:187], v124 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[248:251], v[204:207], a[120:123]\n\t" \
    "v_add_u32 v125, s89, %11\n\t" \
    "ds_read_b64_tr_b16 v[188:189], v125 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[252:255], v[204:207], a[124:127]\n\t" \
    "ds_read_b64_tr_b16 v[190:191], v125 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[128:131], v[224:227], v[208:211], a[128:131]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[132:135], v[228:231], v[208:211], a[132:135]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[136:139], v[232:235], v[208:211], a[136:139]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[140:143], v[236:239], v[208:211], a[140:143]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[144:147], v[240:243], v[208:211], a[144:147]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[148:151], v[244:247], v[208:211], a[148:151]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[152:155], v[248:251], v[208:211], a[152:155]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[156:159], v[252:255], v[208:211], a[156:159]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[160:163], v[224:227], v[212:215], a[160:163]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[164:167], v[228:231], v[212:215], a[164:167]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[168:171], v[232:235], v[212:215], a[168:171]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[172:175], v[236:239], v[212:215], a[172:175]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[176:179], v[240:243], v[212:215], a[176:179]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[180:183], v[244:247], v[212:215], a[180:183]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[184:187], v[248:251], v[212:215], a[184:187]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[188:191], v[252:255], v[212:215], a[188:191]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[192:195], v[224:227], v[216:219], a[192:195]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[196:199], v[228:231], v[216:219], a[196:199]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[200:203], v[232:235], v[216:219], a[200:203]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[204:207], v[236:239], v[216:219], a[204:207]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[208:211], v[240:243], v[216:219], a[208:211]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[212:215], v[244:247], v[216:219], a[212:215]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[216:219], v[248:251], v[216:219], a[216:219]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[220:223], v[252:255], v[216:219], a[220:223]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[224:227], v[224:227], v[220:223], a[224:227]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[228:231], v[228:231], v[220:223], a[228:231]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[232:235], v[232:235], v[220:223], a[232:235]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[236:239], v[236:239], v[220:223], a[236:239]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[240:243], v[240:243], v[220:223], a[240:243]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[244:247], v[244:247], v[220:223], a[244:247]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[248:251], v[248:251], v[220:223], a[248:251]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[252:255], v[252:255], v[220:223], a[252:255]\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_mov_b32 s90, s85\n\t" \
    "s_mov_b32 s85, s86\n\t" \
    "s_mov_b32 s86, s87\n\t" \
    "s_mov_b32 s87, s90\n\t" \
    "s_mov_b32 s90, s88\n\t" \
    "s_mov_b32 s88, s89\n\t" \
    "s_mov_b32 s89, s90\n\t" \
    "3:\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "ds_read_b64 v[192:193], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "ds_read_b64 v[196:197], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "ds_read_b64 v[200:201], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "ds_read_b64 v[204:205], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[176:179], v[128:131], a[16:19]\n\t" \
    "ds_read_b64 v[208:209], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[180:183], v[128:131], a[20:23]\n\t" \
    "ds_read_b64 v[212:213], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[184:187], v[128:131], a[24:27]\n\t" \
    "ds_read_b64 v[216:217], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[188:191], v[128:131], a[28:31]\n\t" \
    "ds_read_b64 v[220:221], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[132:135], a[32:35]\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[194:195], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[132:135], a[36:39]\n\t" \
    "ds_read_b64 v[198:199], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[132:135], a[40:43]\n\t" \
    "ds_read_b64 v[202:203], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[132:135], a[44:47]\n\t" \
    "ds_read_b64 v[206:207], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[176:179], v[132:135], a[48:51]\n\t" \
    "ds_read_b64 v[210:211], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[180:183], v[132:135], a[52:55]\n\t" \
    "ds_read_b64 v[214:215], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[184:187], v[132:135], a[56:59]\n\t" \
    "ds_read_b64 v[218:219], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[188:191], v[132:135], a[60:63]\n\t" \
    "ds_read_b64 v[222:223], v117 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[136:139], a[64:67]\n\t" \
    "v_add_u32 v118, s88, %4\n\t" \
    "ds_read_b64_tr_b16 v[224:225], v118 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[136:139], a[68:71]\n\t" \
    "ds_read_b64_tr_b16 v[226:227], v118 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[136:139], a[72:75]\n\t" \
    "v_add_u32 v119, s88, %5\n\t" \
    "ds_read_b64_tr_b16 v[228:229], v119 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[136:139], a[76:79]\n\t" \
    "ds_read_b64_tr_b16 v[230:231], v119 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[176:179], v[136:139], a[80:83]\n\t" \
    "v_add_u32 v120, s88, %6\n\t" \
    "ds_read_b64_tr_b16 v[232:233], v120 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[180:183], v[136:139], a[84:87]\n\t" \
    "ds_read_b64_tr_b16 v[234:235], v120 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[184:187], v[136:139], a[88:91]\n\t" \
    "v_add_u32 v121, s88, %7\n\t" \
    "ds_read_b64_tr_b16 v[236:237], v121 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[188:191], v[136:139], a[92:95]\n\t" \
    "ds_read_b64_tr_b16 v[238:239], v121 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[140:143], a[96:99]\n\t" \
    "v_add_u32 v122, s88, %8\n\t" \
    "ds_read_b64_tr_b16 v[240:241], v122 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[140:143], a[100:103]\n\t" \
    "ds_read_b64_tr_b16 v[242:243], v122 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[140:143], a[104:107]\n\t" \
    "v_add_u32 v123, s88, %9\n\t" \
    "ds_read_b64_tr_b16 v[244:245], v123 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[140:143], a[108:111]\n\t" \
    "ds_read_b64_tr_b16 v[246:247], v123 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[176:179], v[140:143], a[112:115]\n\t" \
    "v_add_u32 v124, s88, %10\n\t" \
    "ds_read_b64_tr_b16 v[248:249], v124 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[180:183], v[140:143], a[116:119]\n\t" \
    "ds_read_b64_tr_b16 v[250:251], v124 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[184:187], v[140:143], a[120:123]\n\t" \
    "v_add_u32 v125, s88, %11\n\t" \
    "ds_read_b64_tr_b16 v[252:253], v125 offset:16384\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[188:191], v[140:143], a[124:127]\n\t" \
    "ds_read_b64_tr_b16 v[254:255], v125 offset:24576\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[128:131], v[160:163], v[144:147], a[128:131]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[132:135], v[164:167], v[144:147], a[132:135]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[136:139], v[168:171], v[144:147], a[136:139]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[140:143], v[172:175], v[144:147], a[140:143]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[144:147], v[176:179], v[144:147], a[144:147]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[148:151], v[180:183], v[144:147], a[148:151]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[152:155], v[184:187], v[144:147], a[152:155]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[156:159], v[188:191], v[144:147], a[156:159]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[160:163], v[160:163], v[148:151], a[160:163]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[164:167], v[164:167], v[148:151], a[164:167]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[168:171], v[168:171], v[148:151], a[168:171]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[172:175], v[172:175], v[148:151], a[172:175]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[176:179], v[176:179], v[148:151], a[176:179]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[180:183], v[180:183], v[148:151], a[180:183]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[184:187], v[184:187], v[148:151], a[184:187]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[188:191], v[188:191], v[148:151], a[188:191]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[192:195], v[160:163], v[152:155], a[192:195]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[196:199], v[164:167], v[152:155], a[196:199]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[200:203], v[168:171], v[152:155], a[200:203]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[204:207], v[172:175], v[152:155], a[204:207]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[208:211], v[176:179], v[152:155], a[208:211]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[212:215], v[180:183], v[152:155], a[212:215]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[216:219], v[184:187], v[152:155], a[216:219]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[220:223], v[188:191], v[152:155], a[220:223]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[224:227], v[160:163], v[156:159], a[224:227]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[228:231], v[164:167], v[156:159], a[228:231]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[232:235], v[168:171], v[156:159], a[232:235]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[236:239], v[172:175], v[156:159], a[236:239]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[240:243], v[176:179], v[156:159], a[240:243]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[244:247], v[180:183], v[156:159], a[244:247]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[248:251], v[184:187], v[156:159], a[248:251]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[252:255], v[188:191], v[156:159], a[252:255]\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[224:227], v[192:195], a[0:3]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[228:231], v[192:195], a[4:7]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[232:235], v[192:195], a[8:11]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[236:239], v[192:195], a[12:15]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[240:243], v[192:195], a[16:19]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[244:247], v[192:195], a[20:23]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[248:251], v[192:195], a[24:27]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[252:255], v[192:195], a[28:31]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[224:227], v[196:199], a[32:35]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[228:231], v[196:199], a[36:39]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[232:235], v[196:199], a[40:43]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[236:239], v[196:199], a[44:47]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[240:243], v[196:199], a[48:51]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[244:247], v[196:199], a[52:55]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[248:251], v[196:199], a[56:59]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[252:255], v[196:199], a[60:63]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[224:227], v[200:203], a[64:67]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[228:231], v[200:203], a[68:71]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[232:235], v[200:203], a[72:75]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[236:239], v[200:203], a[76:79]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[240:243], v[200:203], a[80:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[244:247], v[200:203], a[84:87]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[248:251], v[200:203], a[88:91]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[252:255], v[200:203], a[92:95]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[224:227], v[204:207], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[228:231], v[204:207], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[232:235], v[204:207], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[236:239], v[204:207], a[108:111]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[240:243], v[204:207], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[244:247], v[204:207], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[248:251], v[204:207], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[252:255], v[204:207], a[124:127]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[128:131], v[224:227], v[208:211], a[128:131]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[132:135], v[228:231], v[208:211], a[132:135]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[136:139], v[232:235], v[208:211], a[136:139]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[140:143], v[236:239], v[208:211], a[140:143]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[144:147], v[240:243], v[208:211], a[144:147]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[148:151], v[244:247], v[208:211], a[148:151]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[152:155], v[248:251], v[208:211], a[152:155]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[156:159], v[252:255], v[208:211], a[156:159]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[160:163], v[224:227], v[212:215], a[160:163]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[164:167], v[228:231], v[212:215], a[164:167]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[168:171], v[232:235], v[212:215], a[168:171]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[172:175], v[236:239], v[212:215], a[172:175]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[176:179], v[240:243], v[212:215], a[176:179]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[180:183], v[244:247], v[212:215], a[180:183]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[184:187], v[248:251], v[212:215], a[184:187]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[188:191], v[252:255], v[212:215], a[188:191]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[192:195], v[224:227], v[216:219], a[192:195]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[196:199], v[228:231], v[216:219], a[196:199]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[200:203], v[232:235], v[216:219], a[200:203]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[204:207], v[236:239], v[216:219], a[204:207]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[208:211], v[240:243], v[216:219], a[208:211]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[212:215], v[244:247], v[216:219], a[212:215]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[216:219], v[248:251], v[216:219], a[216:219]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[220:223], v[252:255], v[216:219], a[220:223]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[224:227], v[224:227], v[220:223], a[224:227]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[228:231], v[228:231], v[220:223], a[228:231]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[232:235], v[232:235], v[220:223], a[232:235]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[236:239], v[236:239], v[220:223], a[236:239]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[240:243], v[240:243], v[220:223], a[240:243]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[244:247], v[244:247], v[220:223], a[244:247]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[248:251], v[248:251], v[220:223], a[248:251]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[252:255], v[252:255], v[220:223], a[252:255]\n\t" \
    "s_waitcnt vmcnt(0)\n\t" \
    "s_nop 15\n\t" \
    "s_nop 7\n\t" \
    ""

#define SYMB_GEMM16_KSTEP32_NT \
    "s_cmp_eq_u32 %4, 0\n\t" \
    "s_cbranch_scc1 19f\n\t" \
    "ds_read_b64 v[160:161], %2 offset:0\n\t" \
    "ds_read_b64 v[164:165], %2 offset:2048\n\t" \
    "ds_read_b64 v[168:169], %2 offset:4096\n\t" \
    "ds_read_b64 v[172:173], %2 offset:6144\n\t" \
    "ds_read_b64 v[176:177], %2 offset:8192\n\t" \
    "ds_read_b64 v[180:181], %2 offset:10240\n\t" \
    "ds_read_b64 v[184:185], %2 offset:12288\n\t" \
    "ds_read_b64 v[188:189], %2 offset:14336\n\t" \
    "ds_read_b64 v[162:163], %3 offset:0\n\t" \
    "ds_read_b64 v[166:167], %3 offset:2048\n\t" \
    "ds_read_b64 v[170:171], %3 offset:4096\n\t" \
    "ds_read_b64 v[174:175], %3 offset:6144\n\t" \
    "ds_read_b64 v[178:179], %3 offset:8192\n\t" \
    "ds_read_b64 v[182:183], %3 offset:10240\n\t" \
    "ds_read_b64 v[186:187], %3 offset:12288\n\t" \
    "ds_read_b64 v[190:191], %3 offset:14336\n\t" \
    "s_bitcmp1_b32 %4, 0\n\t" \
    "s_cbranch_scc0 20f\n\t" \
    "ds_read_b64 v[128:129], %0 offset:0\n\t" \
    "ds_read_b64 v[130:131], %1 offset:0\n\t" \
    "20:\n\t" \
    "s_bitcmp1_b32 %4, 1\n\t" \
    "s_cbranch_scc0 21f\n\t" \
    "ds_read_b64 v[132:133], %0 offset:2048\n\t" \
    "ds_read_b64 v[134:135], %1 offset:2048\n\t" \
    "21:\n\t" \
    "s_bitcmp1_b32 %4, 2\n\t" \
    "s_cbranch_scc0 22f\n\t" \
    "ds_read_b64 v[136:137], %0 offset:4096\n\t" \
    "ds_read_b64 v[138:139], %1 offset:4096\n\t" \
    "22:\n\t" \
    "s_bitcmp1_b32 %4, 3\n\t" \
    "s_cbranch_scc0 23f\n\t" \
    "ds_read_b64 v[140:141], %0 offset:6144\n\t" \
    "ds_read_b64 v[142:143], %1 offset:6144\n\t" \
    "23:\n\t" \
    "s_bitcmp1_b32 %4, 4\n\t" \
    "s_cbranch_scc0 24f\n\t" \
    "ds_read_b64 v[144:145], %0 offset:8192\n\t" \
    "ds_read_b64 v[146:147], %1 offset:8192\n\t" \
    "24:\n\t" \
    "s_bitcmp1_b32 %4, 5\n\t" \
    "s_cbranch_scc0 25f\n\t" \
    "ds_read_b64 v[148:149], %0 offset:10240\n\t" \
    "ds_read_b64 v[150:151], %1 offset:10240\n\t" \
    "25:\n\t" \
    "s_bitcmp1_b32 %4, 6\n\t" \
    "s_cbranch_scc0 26f\n\t" \
    "ds_read_b64 v[152:153], %0 offset:12288\n\t" \
    "ds_read_b64 v[154:155], %1 offset:12288\n\t" \
    "26:\n\t" \
    "s_bitcmp1_b32 %4, 7\n\t" \
    "s_cbranch_scc0 27f\n\t" \
    "ds_read_b64 v[156:157], %0 offset:14336\n\t" \
    "ds_read_b64 v[158:159], %1 offset:14336\n\t" \
    "27:\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_bitcmp1_b32 %4, 0\n\t" \
    "s_cbranch_scc0 30f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[176:179], v[128:131], a[16:19]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[180:183], v[128:131], a[20:23]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[184:187], v[128:131], a[24:27]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[188:191], v[128:131], a[28:31]\n\t" \
    "30:\n\t" \
    "s_bitcmp1_b32 %4, 1\n\t" \
    "s_cbranch_scc0 31f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[132:135], a[32:35]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[132:135], a[36:39]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[132:135], a[40:43]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[132:135], a[44:47]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[176:179], v[132:135], a[48:51]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[180:183], v[132:135], a[52:55]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[184:187], v[132:135], a[56:59]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[188:191], v[132:135], a[60:63]\n\t" \
    "31:\n\t" \
    "s_bitcmp1_b32 %4, 2\n\t" \
    "s_cbranch_scc0 32f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[136:139], a[64:67]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[136:139], a[68:71]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[136:139], a[72:75]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[136:139], a[76:79]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[176:179], v[136:139], a[80:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[180:183], v[136:139], a[84:87]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[184:187], v[136:139], a[88:91]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[188:191], v[136:139], a[92:95]\n\t" \
    "32:\n\t" \
    "s_bitcmp1_b32 %4, 3\n\t" \
    "s_cbranch_scc0 33f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[140:143], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[140:143], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[140:143], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[140:143], a[108:111]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[176:179], v[140:143], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[180:183], v[140:143], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[184:187], v[140:143], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[188:191], v[140:143], a[124:127]\n\t" \
    "33:\n\t" \
    "s_bitcmp1_b32 %4, 4\n\t" \
    "s_cbranch_scc0 34f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[128:131], v[160:163], v[144:147], a[128:131]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[132:135], v[164:167], v[144:147], a[132:135]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[136:139], v[168:171], v[144:147], a[136:139]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[140:143], v[172:175], v[144:147], a[140:143]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[144:147], v[176:179], v[144:147], a[144:147]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[148:151], v[180:183], v[144:147], a[148:151]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[152:155], v[184:187], v[144:147], a[152:155]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[156:159], v[188:191], v[144:147], a[156:159]\n\t" \
    "34:\n\t" \
    "s_bitcmp1_b32 %4, 5\n\t" \
    "s_cbranch_scc0 35f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[160:163], v[160:163], v[148:151], a[160:163]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[164:167], v[164:167], v[148:151], a[164:167]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[168:171], v[168:171], v[148:151], a[168:171]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[172:175], v[172:175], v[148:151], a[172:175]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[176:179], v[176:179], v[148:151], a[176:179]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[180:183], v[180:183], v[148:151], a[180:183]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[184:187], v[184:187], v[148:151], a[184:187]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[188:191], v[188:191], v[148:151], a[188:191]\n\t" \
    "35:\n\t" \
    "s_bitcmp1_b32 %4, 6\n\t" \
    "s_cbranch_scc0 36f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[192:195], v[160:163], v[152:155], a[192:195]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[196:199], v[164:167], v[152:155], a[196:199]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[200:203], v[168:171], v[152:155], a[200:203]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[204:207], v[172:175], v[152:155], a[204:207]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[208:211], v[176:179], v[152:155], a[208:211]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[212:215], v[180:183], v[152:155], a[212:215]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[216:219], v[184:187], v[152:155], a[216:219]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[220:223], v[188:191], v[152:155], a[220:223]\n\t" \
    "36:\n\t" \
    "s_bitcmp1_b32 %4, 7\n\t" \
    "s_cbranch_scc0 37f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[224:227], v[160:163], v[156:159], a[224:227]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[228:231], v[164:167], v[156:159], a[228:231]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[232:235], v[168:171], v[156:159], a[232:235]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[236:239], v[172:175], v[156:159], a[236:239]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[240:243], v[176:179], v[156:159], a[240:243]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[244:247], v[180:183], v[156:159], a[244:247]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[248:251], v[184:187], v[156:159], a[248:251]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[252:255], v[188:191], v[156:159], a[252:255]\n\t" \
    "37:\n\t" \
    "s_nop 15\n\t" \
    "s_nop 7\n\t" \
    "19:\n\t" \
    ""

#define SYMB_GEMM16_KSTEP32_NN \
    "s_cmp_eq_u32 %10, 0\n\t" \
    "s_cbranch_scc1 19f\n\t" \
    "ds_read_b64_tr_b16 v[160:161], %2 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[162:163], %2 offset:8192\n\t" \
    "ds_read_b64_tr_b16 v[164:165], %3 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[166:167], %3 offset:8192\n\t" \
    "ds_read_b64_tr_b16 v[168:169], %4 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[170:171], %4 offset:8192\n\t" \
    "ds_read_b64_tr_b16 v[172:173], %5 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[174:175], %5 offset:8192\n\t" \
    "ds_read_b64_tr_b16 v[176:177], %6 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[178:179], %6 offset:8192\n\t" \
    "ds_read_b64_tr_b16 v[180:181], %7 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[182:183], %7 offset:8192\n\t" \
    "ds_read_b64_tr_b16 v[184:185], %8 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[186:187], %8 offset:8192\n\t" \
    "ds_read_b64_tr_b16 v[188:189], %9 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[190:191], %9 offset:8192\n\t" \
    "s_bitcmp1_b32 %10, 0\n\t" \
    "s_cbranch_scc0 20f\n\t" \
    "ds_read_b64 v[128:129], %0 offset:0\n\t" \
    "ds_read_b64 v[130:131], %1 offset:0\n\t" \
    "20:\n\t" \
    "s_bitcmp1_b32 %10, 1\n\t" \
    "s_cbranch_scc0 21f\n\t" \
    "ds_read_b64 v[132:133], %0 offset:2048\n\t" \
    "ds_read_b64 v[134:135], %1 offset:2048\n\t" \
    "21:\n\t" \
    "s_bitcmp1_b32 %10, 2\n\t" \
    "s_cbranch_scc0 22f\n\t" \
    "ds_read_b64 v[136:137], %0 offset:4096\n\t" \
    "ds_read_b64 v[138:139], %1 offset:4096\n\t" \
    "22:\n\t" \
    "s_bitcmp1_b32 %10, 3\n\t" \
    "s_cbranch_scc0 23f\n\t" \
    "ds_read_b64 v[140:141], %0 offset:6144\n\t" \
    "ds_read_b64 v[142:143], %1 offset:6144\n\t" \
    "23:\n\t" \
    "s_bitcmp1_b32 %10, 4\n\t" \
    "s_cbranch_scc0 24f\n\t" \
    "ds_read_b64 v[144:145], %0 offset:8192\n\t" \
    "ds_read_b64 v[146:147], %1 offset:8192\n\t" \
    "24:\n\t" \
    "s_bitcmp1_b32 %10, 5\n\t" \
    "s_cbranch_scc0 25f\n\t" \
    "ds_read_b64 v[148:149], %0 offset:10240\n\t" \
    "ds_read_b64 v[150:151], %1 offset:10240\n\t" \
    "25:\n\t" \
    "s_bitcmp1_b32 %10, 6\n\t" \
    "s_cbranch_scc0 26f\n\t" \
    "ds_read_b64 v[152:153], %0 offset:12288\n\t" \
    "ds_read_b64 v[154:155], %1 offset:12288\n\t" \
    "26:\n\t" \
    "s_bitcmp1_b32 %10, 7\n\t" \
    "s_cbranch_scc0 27f\n\t" \
    "ds_read_b64 v[156:157], %0 offset:14336\n\t" \
    "ds_read_b64 v[158:159], %1 offset:14336\n\t" \
    "27:\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_bitcmp1_b32 %10, 0\n\t" \
    "s_cbranch_scc0 30f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[176:179], v[128:131], a[16:19]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[180:183], v[128:131], a[20:23]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[184:187], v[128:131], a[24:27]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[188:191], v[128:131], a[28:31]\n\t" \
    "30:\n\t" \
    "s_bitcmp1_b32 %10, 1\n\t" \
    "s_cbranch_scc0 31f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[132:135], a[32:35]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[132:135], a[36:39]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[132:135], a[40:43]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[132:135], a[44:47]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[176:179], v[132:135], a[48:51]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[180:183], v[132:135], a[52:55]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[184:187], v[132:135], a[56:59]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[188:191], v[132:135], a[60:63]\n\t" \
    "31:\n\t" \
    "s_bitcmp1_b32 %10, 2\n\t" \
    "s_cbranch_scc0 32f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[136:139], a[64:67]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[136:139], a[68:71]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[136:139], a[72:75]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[136:139], a[76:79]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[176:179], v[136:139], a[80:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[180:183], v[136:139], a[84:87]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[184:187], v[136:139], a[88:91]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[188:191], v[136:139], a[92:95]\n\t" \
    "32:\n\t" \
    "s_bitcmp1_b32 %10, 3\n\t" \
    "s_cbranch_scc0 33f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[140:143], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[140:143], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[140:143], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[140:143], a[108:111]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[176:179], v[140:143], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[180:183], v[140:143], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[184:187], v[140:143], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[188:191], v[140:143], a[124:127]\n\t" \
    "33:\n\t" \
    "s_bitcmp1_b32 %10, 4\n\t" \
    "s_cbranch_scc0 34f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[128:131], v[160:163], v[144:147], a[128:131]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[132:135], v[164:167], v[144:147], a[132:135]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[136:139], v[168:171], v[144:147], a[136:139]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[140:143], v[172:175], v[144:147], a[140:143]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[144:147], v[176:179], v[144:147], a[144:147]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[148:151], v[180:183], v[144:147], a[148:151]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[152:155], v[184:187], v[144:147], a[152:155]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[156:159], v[188:191], v[144:147], a[156:159]\n\t" \
    "34:\n\t" \
    "s_bitcmp1_b32 %10, 5\n\t" \
    "s_cbranch_scc0 35f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[160:163], v[160:163], v[148:151], a[160:163]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[164:167], v[164:167], v[148:151], a[164:167]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[168:171], v[168:171], v[148:151], a[168:171]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[172:175], v[172:175], v[148:151], a[172:175]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[176:179], v[176:179], v[148:151], a[176:179]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[180:183], v[180:183], v[148:151], a[180:183]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[184:187], v[184:187], v[148:151], a[184:187]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[188:191], v[188:191], v[148:151], a[188:191]\n\t" \
    "35:\n\t" \
    "s_bitcmp1_b32 %10, 6\n\t" \
    "s_cbranch_scc0 36f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[192:195], v[160:163], v[152:155], a[192:195]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[196:199], v[164:167], v[152:155], a[196:199]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[200:203], v[168:171], v[152:155], a[200:203]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[204:207], v[172:175], v[152:155], a[204:207]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[208:211], v[176:179], v[152:155], a[208:211]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[212:215], v[180:183], v[152:155], a[212:215]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[216:219], v[184:187], v[152:155], a[216:219]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[220:223], v[188:191], v[152:155], a[220:223]\n\t" \
    "36:\n\t" \
    "s_bitcmp1_b32 %10, 7\n\t" \
    "s_cbranch_scc0 37f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[224:227], v[160:163], v[156:159], a[224:227]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[228:231], v[164:167], v[156:159], a[228:231]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[232:235], v[168:171], v[156:159], a[232:235]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[236:239], v[172:175], v[156:159], a[236:239]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[240:243], v[176:179], v[156:159], a[240:243]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[244:247], v[180:183], v[156:159], a[244:247]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[248:251], v[184:187], v[156:159], a[248:251]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[252:255], v[188:191], v[156:159], a[252:255]\n\t" \
    "37:\n\t" \
    "s_nop 15\n\t" \
    "s_nop 7\n\t" \
    "19:\n\t" \
    ""

#define SYMB_GEMM16_ZERO \
    "v_accvgpr_write_b32 a0, 0\n\t" \
    "v_accvgpr_write_b32 a1, 0\n\t" \
    "v_accvgpr_write_b32 a2, 0\n\t" \
    "v_accvgpr_write_b32 a3, 0\n\t" \
    "v_accvgpr_write_b32 a4, 0\n\t" \
    "v_accvgpr_write_b32 a5, 0\n\t" \
    "v_accvgpr_write_b32 a6, 0\n\t" \
    "v_accvgpr_write_b32 a7, 0\n\t" \
    "v_accvgpr_write_b32 a8, 0\n\t" \
    "v_accvgpr_write_b32 a9, 0\n\t" \
    "v_accvgpr_write_b32 a10, 0\n\t" \
    "v_accvgpr_write_b32 a11, 0\n\t" \
    "v_accvgpr_write_b32 a12, 0\n\t" \
    "v_accvgpr_write_b32 a13, 0\n\t" \
    "v_accvgpr_write_b32 a14, 0\n\t" \
    "v_accvgpr_write_b32 a15, 0\n\t" \
    "v_accvgpr_write_b32 a16, 0\n\t" \
    "v_accvgpr_write_b32 a17, 0\n\t" \
    "v_accvgpr_write_b32 a18, 0\n\t" \
    "v_accvgpr_write_b32 a19, 0\n\t" \
    "v_accvgpr_write_b32 a20, 0\n\t" \
    "v_accvgpr_write_b32 a21, 0\n\t" \
    "v_accvgpr_write_b32 a22, 0\n\t" \
    "v_accvgpr_write_b32 a23, 0\n\t" \
    "v_accvgpr_write_b32 a24, 0\n\t" \
    "v_accvgpr_write_b32 a25, 0\n\t" \
    "v_accvgpr_write_b32 a26, 0\n\t" \
    "v_accvgpr_write_b32 a27, 0\n\t" \
    "v_accvgpr_write_b32 a28, 0\n\t" \
    "v_accvgpr_write_b32 a29, 0\n\t" \
    "v_accvgpr_write_b32 a30, 0\n\t" \
    "v_accvgpr_write_b32 a31, 0\n\t" \
    "v_accvgpr_write_b32 a32, 0\n\t" \
    "v_accvgpr_write_b32 a33, 0\n\t" \
    "v_accvgpr_write_b32 a34, 0\n\t" \
    "v_accvgpr_write_b32 a35, 0\n\t" \
    "v_accvgpr_write_b32 a36, 0\n\t" \
    "v_accvgpr_write_b32 a37, 0\n\t" \
    "v_accvgpr_write_b32 a38, 0\n\t" \
    "v_accvgpr_write_b32 a39, 0\n\t" \
    "v_accvgpr_write_b32 a40, 0\n\t" \
    "v_accvgpr_write_b32 a41, 0\n\t" \
    "v_accvgpr_write_b32 a42, 0\n\t" \
    "v_accvgpr_write_b32 a43, 0\n\t" \
    "v_accvgpr_write_b32 a44, 0\n\t" \
    "v_accvgpr_write_b32 a45, 0\n\t" \
    "v_accvgpr_write_b32 a46, 0\n\t" \
    "v_accvgpr_write_b32 a47, 0\n\t" \
    "v_accvgpr_write_b32 a48, 0\n\t" \
    "v_accvgpr_write_b32 a49, 0\n\t" \
    "v_accvgpr_write_b32 a50, 0\n\t" \
    "v_accvgpr_write_b32 a51, 0\n\t" \
    "v_accvgpr_write_b32 a52, 0\n\t" \
    "v_accvgpr_write_b32 a53, 0\n\t" \
    "v_accvgpr_write_b32 a54, 0\n\t" \
    "v_accvgpr_write_b32 a55, 0\n\t" \
    "v_accvgpr_write_b32 a56, 0\n\t" \
    "v_accvgpr_write_b32 a57, 0\n\t" \
    "v_accvgpr_write_b32 a58, 0\n\t" \
    "v_accvgpr_write_b32 a59, 0\n\t" \
    "v_accvgpr_write_b32 a60, 0\n\t" \
    "v_accvgpr_write_b32 a61, 0\n\t" \
    "v_accvgpr_write_b32 a62, 0\n\t" \
    "v_accvgpr_write_b32 a63, 0\n\t" \
    "v_accvgpr_write_b32 a64, 0\n\t" \
    "v_accvgpr_write_b32 a65, 0\n\t" \
    "v_accvgpr_write_b32 a66, 0\n\t" \
    "v_accvgpr_write_b32 a67, 0\n\t" \
    "v_accvgpr_write_b32 a68, 0\n\t" \
    "v_accvgpr_write_b32 a69, 0\n\t" \
    "v_accvgpr_write_b32 a70, 0\n\t" \
    "v_accvgpr_write_b32 a71, 0\n\t" \
    "v_accvgpr_write_b32 a72, 0\n\t" \
    "v_accvgpr_write_b32 a73, 0\n\t" \
    "v_accvgpr_write_b32 a74, 0\n\t" \
    "v_accvgpr_write_b32 a75, 0\n\t" \
    "v_accvgpr_write_b32 a76, 0\n\t" \
    "v_accvgpr_write_b32 a77, 0\n\t" \
    "v_accvgpr_write_b32 a78, 0\n\t" \
    "v_accvgpr_write_b32 a79, 0\n\t" \
    "v_accvgpr_write_b32 a80, 0\n\t" \
    "v_accvgpr_write_b32 a81, 0\n\t" \
    "v_accvgpr_write_b32 a82, 0\n\t" \
    "v_accvgpr_write_b32 a83, 0\n\t" \
    "v_accvgpr_write_b32 a84, 0\n\t" \
    "v_accvgpr_write_b32 a85, 0\n\t" \
    "v_accvgpr_write_b32 a86, 0\n\t" \
    "v_accvgpr_write_b32 a87, 0\n\t" \
    "v_accvgpr_write_b32 a88, 0\n\t" \
    "v_accvgpr_write_b32 a89, 0\n\t" \
    "v_accvgpr_write_b32 a90, 0\n\t" \
    "v_accvgpr_write_b32 a91, 0\n\t" \
    "v_accvgpr_write_b32 a92, 0\n\t" \
    "v_accvgpr_write_b32 a93, 0\n\t" \
    "v_accvgpr_write_b32 a94, 0\n\t" \
    "v_accvgpr_write_b32 a95, 0\n\t" \
    "v_accvgpr_write_b32 a96, 0\n\t" \
    "v_accvgpr_write_b32 a97, 0\n\t" \
    "v_accvgpr_write_b32 a98, 0\n\t" \
    "v_accvgpr_write_b32 a99, 0\n\t" \
    "v_accvgpr_write_b32 a100, 0\n\t" \
    "v_accvgpr_write_b32 a101, 0\n\t" \
    "v_accvgpr_write_b32 a102, 0\n\t" \
    "v_accvgpr_write_b32 a103, 0\n\t" \
    "v_accvgpr_write_b32 a104, 0\n\t" \
    "v_accvgpr_write_b32 a105, 0\n\t" \
    "v_accvgpr_write_b32 a106, 0\n\t" \
    "v_accvgpr_write_b32 a107, 0\n\t" \
    "v_accvgpr_write_b32 a108, 0\n\t" \
    "v_accvgpr_write_b32 a109, 0\n\t" \
    "v_accvgpr_write_b32 a110, 0\n\t" \
    "v_accvgpr_write_b32 a111, 0\n\t" \
    "v_accvgpr_write_b32 a112, 0\n\t" \
    "v_accvgpr_write_b32 a113, 0\n\t" \
    "v_accvgpr_write_b32 a114, 0\n\t" \
    "v_accvgpr_write_b32 a115, 0\n\t" \
    "v_accvgpr_write_b32 a116, 0\n\t" \
    "v_accvgpr_write_b32 a117, 0\n\t" \
    "v_accvgpr_write_b32 a118, 0\n\t" \
    "v_accvgpr_write_b32 a119, 0\n\t" \
    "v_accvgpr_write_b32 a120, 0\n\t" \
    "v_accvgpr_write_b32 a121, 0\n\t" \
    "v_accvgpr_write_b32 a122, 0\n\t" \
    "v_accvgpr_write_b32 a123, 0\n\t" \
    "v_accvgpr_write_b32 a124, 0\n\t" \
    "v_accvgpr_write_b32 a125, 0\n\t" \
    "v_accvgpr_write_b32 a126, 0\n\t" \
    "v_accvgpr_write_b32 a127, 0\n\t" \
    "v_accvgpr_write_b32 a128, 0\n\t" \
    "v_accvgpr_write_b32 a129, 0\n\t" \
    "v_accvgpr_write_b32 a130, 0\n\t" \
    "v_accvgpr_write_b32 a131, 0\n\t" \
    "v_accvgpr_write_b32 a132, 0\n\t" \
    "v_accvgpr_write_b32 a133, 0\n\t" \
    "v_accvgpr_write_b32 a134, 0\n\t" \
    "v_accvgpr_write_b32 a135, 0\n\t" \
    "v_accvgpr_write_b32 a136, 0\n\t" \
    "v_accvgpr_write_b32 a137, 0\n\t" \
    "v_accvgpr_write_b32 a138, 0\n\t" \
    "v_accvgpr_write_b32 a139, 0\n\t" \
    "v_accvgpr_write_b32 a140, 0\n\t" \
    "v_accvgpr_write_b32 a141, 0\n\t" \
    "v_accvgpr_write_b32 a142, 0\n\t" \
    "v_accvgpr_write_b32 a143, 0\n\t" \
    "v_accvgpr_write_b32 a144, 0\n\t" \
    "v_accvgpr_write_b32 a145, 0\n\t" \
    "v_accvgpr_write_b32 a146, 0\n\t" \
    "v_accvgpr_write_b32 a147, 0\n\t" \
    "v_accvgpr_write_b32 a148, 0\n\t" \
    "v_accvgpr_write_b32 a149, 0\n\t" \
    "v_accvgpr_write_b32 a150, 0\n\t" \
    "v_accvgpr_write_b32 a151, 0\n\t" \
    "v_accvgpr_write_b32 a152, 0\n\t" \
    "v_accvgpr_write_b32 a153, 0\n\t" \
    "v_accvgpr_write_b32 a154, 0\n\t" \
    "v_accvgpr_write_b32 a155, 0\n\t" \
    "v_accvgpr_write_b32 a156, 0\n\t" \
    "v_accvgpr_write_b32 a157, 0\n\t" \
    "v_accvgpr_write_b32 a158, 0\n\t" \
    "v_accvgpr_write_b32 a159, 0\n\t" \
    "v_accvgpr_write_b32 a160, 0\n\t" \
    "v_accvgpr_write_b32 a161, 0\n\t" \
    "v_accvgpr_write_b32 a162, 0\n\t" \
    "v_accvgpr_write_b32 a163, 0\n\t" \
    "v_accvgpr_write_b32 a164, 0\n\t" \
    "v_accvgpr_write_b32 a165, 0\n\t" \
    "v_accvgpr_write_b32 a166, 0\n\t" \
    "v_accvgpr_write_b32 a167, 0\n\t" \
    "v_accvgpr_write_b32 a168, 0\n\t" \
    "v_accvgpr_write_b32 a169, 0\n\t" \
    "v_accvgpr_write_b32 a170, 0\n\t" \
    "v_accvgpr_write_b32 a171, 0\n\t" \
    "v_accvgpr_write_b32 a172, 0\n\t" \
    "v_accvgpr_write_b32 a173, 0\n\t" \
    "v_accvgpr_write_b32 a174, 0\n\t" \
    "v_accvgpr_write_b32 a175, 0\n\t" \
    "v_accvgpr_write_b32 a176, 0\n\t" \
    "v_accvgpr_write_b32 a177, 0\n\t" \
    "v_accvgpr_write_b32 a178, 0\n\t" \
    "v_accvgpr_write_b32 a179, 0\n\t" \
    "v_accvgpr_write_b32 a180, 0\n\t" \
    "v_accvgpr_write_b32 a181, 0\n\t" \
    "v_accvgpr_write_b32 a182, 0\n\t" \
    "v_accvgpr_write_b32 a183, 0\n\t" \
    "v_accvgpr_write_b32 a184, 0\n\t" \
    "v_accvgpr_write_b32 a185, 0\n\t" \
    "v_accvgpr_write_b32 a186, 0\n\t" \
    "v_accvgpr_write_b32 a187, 0\n\t" \
    "v_accvgpr_write_b32 a188, 0\n\t" \
    "v_accvgpr_write_b32 a189, 0\n\t" \
    "v_accvgpr_write_b32 a190, 0\n\t" \
    "v_accvgpr_write_b32 a191, 0\n\t" \
    "v_accvgpr_write_b32 a192, 0\n\t" \
    "v_accvgpr_write_b32 a193, 0\n\t" \
    "v_accvgpr_write_b32 a194, 0\n\t" \
    "v_accvgpr_write_b32 a195, 0\n\t" \
    "v_accvgpr_write_b32 a196, 0\n\t" \
    "v_accvgpr_write_b32 a197, 0\n\t" \
    "v_accvgpr_write_b32 a198, 0\n\t" \
    "v_accvgpr_write_b32 a199, 0\n\t" \
    "v_accvgpr_write_b32 a200, 0\n\t" \
    "v_accvgpr_write_b32 a201, 0\n\t" \
    "v_accvgpr_write_b32 a202, 0\n\t" \
    "v_accvgpr_write_b32 a203, 0\n\t" \
    "v_accvgpr_write_b32 a204, 0\n\t" \
    "v_accvgpr_write_b32 a205, 0\n\t" \
    "v_accvgpr_write_b32 a206, 0\n\t" \
    "v_accvgpr_write_b32 a207, 0\n\t" \
    "v_accvgpr_write_b32 a208, 0\n\t" \
    "v_accvgpr_write_b32 a209, 0\n\t" \
    "v_accvgpr_write_b32 a210, 0\n\t" \
    "v_accvgpr_write_b32 a211, 0\n\t" \
    "v_accvgpr_write_b32 a212, 0\n\t" \
    "v_accvgpr_write_b32 a213, 0\n\t" \
    "v_accvgpr_write_b32 a214, 0\n\t" \
    "v_accvgpr_write_b32 a215, 0\n\t" \
    "v_accvgpr_write_b32 a216, 0\n\t" \
    "v_accvgpr_write_b32 a217, 0\n\t" \
    "v_accvgpr_write_b32 a218, 0\n\t" \
    "v_accvgpr_write_b32 a219, 0\n\t" \
    "v_accvgpr_write_b32 a220, 0\n\t" \
    "v_accvgpr_write_b32 a221, 0\n\t" \
    "v_accvgpr_write_b32 a222, 0\n\t" \
    "v_accvgpr_write_b32 a223, 0\n\t" \
    "v_accvgpr_write_b32 a224, 0\n\t" \
    "v_accvgpr_write_b32 a225, 0\n\t" \
    "v_accvgpr_write_b32 a226, 0\n\t" \
    "v_accvgpr_write_b32 a227, 0\n\t" \
    "v_accvgpr_write_b32 a228, 0\n\t" \
    "v_accvgpr_write_b32 a229, 0\n\t" \
    "v_accvgpr_write_b32 a230, 0\n\t" \
    "v_accvgpr_write_b32 a231, 0\n\t" \
    "v_accvgpr_write_b32 a232, 0\n\t" \
    "v_accvgpr_write_b32 a233, 0\n\t" \
    "v_accvgpr_write_b32 a234, 0\n\t" \
    "v_accvgpr_write_b32 a235, 0\n\t" \
    "v_accvgpr_write_b32 a236, 0\n\t" \
    "v_accvgpr_write_b32 a237, 0\n\t" \
    "v_accvgpr_write_b32 a238, 0\n\t" \
    "v_accvgpr_write_b32 a239, 0\n\t" \
    "v_accvgpr_write_b32 a240, 0\n\t" \
    "v_accvgpr_write_b32 a241, 0\n\t" \
    "v_accvgpr_write_b32 a242, 0\n\t" \
    "v_accvgpr_write_b32 a243, 0\n\t" \
    "v_accvgpr_write_b32 a244, 0\n\t" \
    "v_accvgpr_write_b32 a245, 0\n\t" \
    "v_accvgpr_write_b32 a246, 0\n\t" \
    "v_accvgpr_write_b32 a247, 0\n\t" \
    "v_accvgpr_write_b32 a248, 0\n\t" \
    "v_accvgpr_write_b32 a249, 0\n\t" \
    "v_accvgpr_write_b32 a250, 0\n\t" \
    "v_accvgpr_write_b32 a251, 0\n\t" \
    "v_accvgpr_write_b32 a252, 0\n\t" \
    "v_accvgpr_write_b32 a253, 0\n\t" \
    "v_accvgpr_write_b32 a254, 0\n\t" \
    "v_accvgpr_write_b32 a255, 0\n\t" \
    "s_nop 3\n\t" \
    ""

#define SYMB_GEMM16_STAGE_OUT \
    "v_accvgpr_read_b32 v128, a0\n\t" \
    "v_accvgpr_read_b32 v129, a1\n\t" \
    "v_accvgpr_read_b32 v130, a2\n\t" \
    "v_accvgpr_read_b32 v131, a3\n\t" \
    "v_cvt_pk_bf16_f32 v132, v128, v129\n\t" \
    "v_cvt_pk_bf16_f32 v133, v130, v131\n\t" \
    "ds_write_b64 %0, v[132:133] offset:0\n\t" \
    "v_accvgpr_read_b32 v134, a4\n\t" \
    "v_accvgpr_read_b32 v135, a5\n\t" \
    "v_accvgpr_read_b32 v136, a6\n\t" \
    "v_accvgpr_read_b32 v137, a7\n\t" \
    "v_cvt_pk_bf16_f32 v138, v134, v135\n\t" \
    "v_cvt_pk_bf16_f32 v139, v136, v137\n\t" \
    "ds_write_b64 %0, v[138:139] offset:32\n\t" \
    "v_accvgpr_read_b32 v140, a8\n\t" \
    "v_accvgpr_read_b32 v141, a9\n\t" \
    "v_accvgpr_read_b32 v142, a10\n\t" \
    "v_accvgpr_read_b32 v143, a11\n\t" \
    "v_cvt_pk_bf16_f32 v144, v140, v141\n\t" \
    "v_cvt_pk_bf16_f32 v145, v142, v143\n\t" \
    "ds_write_b64 %0, v[144:145] offset:64\n\t" \
    "v_accvgpr_read_b32 v146, a12\n\t" \
    "v_accvgpr_read_b32 v147, a13\n\t" \
    "v_accvgpr_read_b32 v148, a14\n\t" \
    "v_accvgpr_read_b32 v149, a15\n\t" \
    "v_cvt_pk_bf16_f32 v150, v146, v147\n\t" \
    "v_cvt_pk_bf16_f32 v151, v148, v149\n\t" \
    "ds_write_b64 %0, v[150:151] offset:96\n\t" \
    "v_accvgpr_read_b32 v152, a16\n\t" \
    "v_accvgpr_read_b32 v153, a17\n\t" \
    "v_accvgpr_read_b32 v154, a18\n\t" \
    "v_accvgpr_read_b32 v155, a19\n\t" \
    "v_cvt_pk_bf16_f32 v156, v152, v153\n\t" \
    "v_cvt_pk_bf16_f32 v157, v154, v155\n\t" \
    "ds_write_b64 %0, v[156:157] offset:128\n\t" \
    "v_accvgpr_read_b32 v158, a20\n\t" \
    "v_accvgpr_read_b32 v159, a21\n\t" \
    "v_accvgpr_read_b32 v160, a22\n\t" \
    "v_accvgpr_read_b32 v161, a23\n\t" \
    "v_cvt_pk_bf16_f32 v162, v158, v159\n\t" \
    "v_cvt_pk_bf16_f32 v163, v160, v161\n\t" \
    "ds_write_b64 %0, v[162:163] offset:160\n\t" \
    "v_accvgpr_read_b32 v164, a24\n\t" \
    "v_accvgpr_read_b32 v165, a25\n\t" \
    "v_accvgpr_read_b32 v166, a26\n\t" \
    "v_accvgpr_read_b32 v167, a27\n\t" \
    "v_cvt_pk_bf16_f32 v168, v164, v165\n\t" \
    "v_cvt_pk_bf16_f32 v169, v166, v167\n\t" \
    "ds_write_b64 %0, v[168:169] offset:192\n\t" \
    "v_accvgpr_read_b32 v170, a28\n\t" \
    "v_accvgpr_read_b32 v171, a29\n\t" \
    "v_accvgpr_read_b32 v172, a30\n\t" \
    "v_accvgpr_read_b32 v173, a31\n\t" \
    "v_cvt_pk_bf16_f32 v174, v170, v171\n\t" \
    "v_cvt_pk_bf16_f32 v175, v172, v173\n\t" \
    "ds_write_b64 %0, v[174:175] offset:224\n\t" \
    "v_accvgpr_read_b32 v128, a32\n\t" \
    "v_accvgpr_read_b32 v129, a33\n\t" \
    "v_accvgpr_read_b32 v130, a34\n\t" \
    "v_accvgpr_read_b32 v131, a35\n\t" \
    "v_cvt_pk_bf16_f32 v132, v128, v129\n\t" \
    "v_cvt_pk_bf16_f32 v133, v130, v131\n\t" \
    "ds_write_b64 %0, v[132:133] offset:8448\n\t" \
    "v_accvgpr_read_b32 v134, a36\n\t" \
    "v_accvgpr_read_b32 v135, a37\n\t" \
    "v_accvgpr_read_b32 v136, a38\n\t" \
    "v_accvgpr_read_b32 v137, a39\n\t" \
    "v_cvt_pk_bf16_f32 v138, v134, v135\n\t" \
    "v_cvt_pk_bf16_f32 v139, v136, v137\n\t" \
    "ds_write_b64 %0, v[138:139] offset:8480\n\t" \
    "v_accvgpr_read_b32 v140, a40\n\t" \
    "v_accvgpr_read_b32 v141, a41\n\t" \
    "v_accvgpr_read_b32 v142, a42\n\t" \
    "v_accvgpr_read_b32 v143, a43\n\t" \
    "v_cvt_pk_bf16_f32 v144, v140, v141\n\t" \
    "v_cvt_pk_bf16_f32 v145, v142, v143\n\t" \
    "ds_write_b64 %0, v[144:145] offset:8512\n\t" \
    "v_accvgpr_read_b32 v146, a44\n\t" \
    "v_accvgpr_read_b32 v147, a45\n\t" \
    "v_accvgpr_read_b32 v148, a46\n\t" \
    "v_accvgpr_read_b32 v149, a47\n\t" \
    "v_cvt_pk_bf16_f32 v150, v146, v147\n\t" \
    "v_cvt_pk_bf16_f32 v151, v148, v149\n\t" \
    "ds_write_b64 %0, v[150:151] offset:8544\n\t" \
    "v_accvgpr_read_b32 v152, a48\n\t" \
    "v_accvgpr_read_b32 v153, a49\n\t" \
    "v_accvgpr_read_b32 v154, a50\n\t" \
    "v_accvgpr_read_b32 v155, a51\n\t" \
    "v_cvt_pk_bf16_f32 v156, v152, v153\n\t" \
    "v_cvt_pk_bf16_f32 v157, v154, v155\n\t" \
    "ds_write_b64 %0, v[156:157] offset:8576\n\t" \
    "v_accvgpr_read_b32 v158, a52\n\t" \
    "v_accvgpr_read_b32 v159, a53\n\t" \
    "v_accvgpr_read_b32 v160, a54\n\t" \
    "v_accvgpr_read_b32 v161, a55\n\t" \
    "v_cvt_pk_bf16_f32 v162, v158, v159\n\t" \
    "v_cvt_pk_bf16_f32 v163, v160, v161\n\t" \
    "ds_write_b64 %0, v[162:163] offset:8608\n\t" \
    "v_accvgpr_read_b32 v164, a56\n\t" \
    "v_accvgpr_read_b32 v165, a57\n\t" \
    "v_accvgpr_read_b32 v166, a58\n\t" \
    "v_accvgpr_read_b32 v167, a59\n\t" \
    "v_cvt_pk_bf16_f32 v168, v164, v165\n\t" \
    "v_cvt_pk_bf16_f32 v169, v166, v167\n\t" \
    "ds_write_b64 %0, v[168:169] offset:8640\n\t" \
    "v_accvgpr_read_b32 v170, a60\n\t" \
    "v_accvgpr_read_b32 v171, a61\n\t" \
    "v_accvgpr_read_b32 v172, a62\n\t" \
    "v_accvgpr_read_b32 v173, a63\n\t" \
    "v_cvt_pk_bf16_f32 v174, v170, v171\n\t" \
    "v_cvt_pk_bf16_f32 v175, v172, v173\n\t" \
    "ds_write_b64 %0, v[174:175] offset:8672\n\t" \
    "v_accvgpr_read_b32 v128, a64\n\t" \
    "v_accvgpr_read_b32 v129, a65\n\t" \
    "v_accvgpr_read_b32 v130, a66\n\t" \
    "v_accvgpr_read_b32 v131, a67\n\t" \
    "v_cvt_pk_bf16_f32 v132, v128, v129\n\t" \
    "v_cvt_pk_bf16_f32 v133, v130, v131\n\t" \
    "ds_write_b64 %0, v[132:133] offset:16896\n\t" \
    "v_accvgpr_read_b32 v134, a68\n\t" \
    "v_accvgpr_read_b32 v135, a69\n\t" \
    "v_accvgpr_read_b32 v136, a70\n\t" \
    "v_accvgpr_read_b32 v137, a71\n\t" \
    "v_cvt_pk_bf16_f32 v138, v134, v135\n\t" \
    "v_cvt_pk_bf16_f32 v139, v136, v137\n\t" \
    "ds_write_b64 %0, v[138:139] offset:16928\n\t" \
    "v_accvgpr_read_b32 v140, a72\n\t" \
    "v_accvgpr_read_b32 v141, a73\n\t" \
    "v_accvgpr_read_b32 v142, a74\n\t" \
    "v_accvgpr_read_b32 v143, a75\n\t" \
    "v_cvt_pk_bf16_f32 v144, v140, v141\n\t" \
    "v_cvt_pk_bf16_f32 v145, v142, v143\n\t" \
    "ds_write_b64 %0, v[144:145] offset:16960\n\t" \
    "v_accvgpr_read_b32 v146, a76\n\t" \
    "v_accvgpr_read_b32 v147, a77\n\t" \
    "v_accvgpr_read_b32 v148, a78\n\t" \
    "v_accvgpr_read_b32 v149, a79\n\t" \
    "v_cvt_pk_bf16_f32 v150, v146, v147\n\t" \
    "v_cvt_pk_bf16_f32 v151, v148, v149\n\t" \
    "ds_write_b64 %0, v[150:151] offset:16992\n\t" \
    "v_accvgpr_read_b32 v152, a80\n\t" \
    "v_accvgpr_read_b32 v153, a81\n\t" \
    "v_accvgpr_read_b32 v154, a82\n\t" \
    "v_accvgpr_read_b32 v155, a83\n\t" \
    "v_cvt_pk_bf16_f32 v156, v152, v153\n\t" \
    "v_cvt_pk_bf16_f32 v157, v154, v155\n\t" \
    "ds_write_b64 %0, v[156:157] offset:17024\n\t" \
    "v_accvgpr_read_b32 v158, a84\n\t" \
    "v_accvgpr_read_b32 v159, a85\n\t" \
    "v_accvgpr_read_b32 v160, a86\n\t" \
    "v_accvgpr_read_b32 v161, a87\n\t" \
    "v_cvt_pk_bf16_f32 v162, v158, v159\n\t" \
    "v_cvt_pk_bf16_f32 v163, v160, v161\n\t" \
    "ds_write_b64 %0, v[162:163] offset:17056\n\t" \
    "v_accvgpr_read_b32 v164, a88\n\t" \
    "v_accvgpr_read_b32 v165, a89\n\t" \
    "v_accvgpr_read_b32 v166, a90\n\t" \
    "v_accvgpr_read_b32 v167, a91\n\t" \
    "v_cvt_pk_bf16_f32 v168, v164, v165\n\t" \
    "v_cvt_pk_bf16_f32 v169, v166, v167\n\t" \
    "ds_write_b64 %0, v[168:169] offset:17088\n\t" \
    "v_accvgpr_read_b32 v170, a92\n\t" \
    "v_accvgpr_read_b32 v171, a93\n\t" \
    "v_accvgpr_read_b32 v172, a94\n\t" \
    "v_accvgpr_read_b32 v173, a95\n\t" \
    "v_cvt_pk_bf16_f32 v174, v170, v171\n\t" \
    "v_cvt_pk_bf16_f32 v175, v172, v173\n\t" \
    "ds_write_b64 %0, v[174:175] offset:17120\n\t" \
    "v_accvgpr_read_b32 v128, a96\n\t" \
    "v_accvgpr_read_b32 v129, a97\n\t" \
    "v_accvgpr_read_b32 v130, a98\n\t" \
    "v_accvgpr_read_b32 v131, a99\n\t" \
    "v_cvt_pk_bf16_f32 v132, v128, v129\n\t" \
    "v_cvt_pk_bf16_f32 v133, v130, v131\n\t" \
    "ds_write_b64 %0, v[132:133] offset:25344\n\t" \
    "v_accvgpr_read_b32 v134, a100\n\t" \
    "v_accvgpr_read_b32 v135, a101\n\t" \
    "v_accvgpr_read_b32 v136, a102\n\t" \
    "v_accvgpr_read_b32 v137, a103\n\t" \
    "v_cvt_pk_bf16_f32 v138, v134, v135\n\t" \
    "v_cvt_pk_bf16_f32 v139, v136, v137\n\t" \
    "ds_write_b64 %0, v[138:139] offset:25376\n\t" \
    "v_accvgpr_read_b32 v140, a104\n\t" \
    "v_accvgpr_read_b32 v141, a105\n\t" \
    "v_accvgpr_read_b32 v142, a106\n\t" \
    "v_accvgpr_read_b32 v143, a107\n\t" \
    "v_cvt_pk_bf16_f32 v144, v140, v141\n\t" \
    "v_cvt_pk_bf16_f32 v145, v142, v143\n\t" \
    "ds_write_b64 %0, v[144:145] offset:25408\n\t" \
    "v_accvgpr_read_b32 v146, a108\n\t" \
    "v_accvgpr_read_b32 v147, a109\n\t" \
    "v_accvgpr_read_b32 v148, a110\n\t" \
    "v_accvgpr_read_b32 v149, a111\n\t" \
    "v_cvt_pk_bf16_f32 v150, v146, v147\n\t" \
    "v_cvt_pk_bf16_f32 v151, v148, v149\n\t" \
    "ds_write_b64 %0, v[150:151] offset:25440\n\t" \
    "v_accvgpr_read_b32 v152, a112\n\t" \
    "v_accvgpr_read_b32 v153, a113\n\t" \
    "v_accvgpr_read_b32 v154, a114\n\t" \
    "v_accvgpr_read_b32 v155, a115\n\t" \
    "v_cvt_pk_bf16_f32 v156, v152, v153\n\t" \
    "v_cvt_pk_bf16_f32 v157, v154, v155\n\t" \
    "ds_write_b64 %0, v[156:157] offset:25472\n\t" \
    "v_accvgpr_read_b32 v158, a116\n\t" \
    "v_accvgpr_read_b32 v159, a117\n\t" \
    "v_accvgpr_read_b32 v160, a118\n\t" \
    "v_accvgpr_read_b32 v161, a119\n\t" \
    "v_cvt_pk_bf16_f32 v162, v158, v159\n\t" \
    "v_cvt_pk_bf16_f32 v163, v160, v161\n\t" \
    "ds_write_b64 %0, v[162:163] offset:25504\n\t" \
    "v_accvgpr_read_b32 v164, a120\n\t" \
    "v_accvgpr_read_b32 v165, a121\n\t" \
    "v_accvgpr_read_b32 v166, a122\n\t" \
    "v_accvgpr_read_b32 v167, a123\n\t" \
    "v_cvt_pk_bf16_f32 v168, v164, v165\n\t" \
    "v_cvt_pk_bf16_f32 v169, v166, v167\n\t" \
    "ds_write_b64 %0, v[168:169] offset:25536\n\t" \
    "v_accvgpr_read_b32 v170, a124\n\t" \
    "v_accvgpr_read_b32 v171, a125\n\t" \
    "v_accvgpr_read_b32 v172, a126\n\t" \
    "v_accvgpr_read_b32 v173, a127\n\t" \
    "v_cvt_pk_bf16_f32 v174, v170, v171\n\t" \
    "v_cvt_pk_bf16_f32 v175, v172, v173\n\t" \
    "ds_write_b64 %0, v[174:175] offset:25568\n\t" \
    "v_accvgpr_read_b32 v128, a128\n\t" \
    "v_accvgpr_read_b32 v129, a129\n\t" \
    "v_accvgpr_read_b32 v130, a130\n\t" \
    "v_accvgpr_read_b32 v131, a131\n\t" \
    "v_cvt_pk_bf16_f32 v132, v128, v129\n\t" \
    "v_cvt_pk_bf16_f32 v133, v130, v131\n\t" \
    "ds_write_b64 %0, v[132:133] offset:33792\n\t" \
    "v_accvgpr_read_b32 v134, a132\n\t" \
    "v_accvgpr_read_b32 v135, a133\n\t" \
    "v_accvgpr_read_b32 v136, a134\n\t" \
    "v_accvgpr_read_b32 v137, a135\n\t" \
    "v_cvt_pk_bf16_f32 v138, v134, v135\n\t" \
    "v_cvt_pk_bf16_f32 v139, v136, v137\n\t" \
    "ds_write_b64 %0, v[138:139] offset:33824\n\t" \
    "v_accvgpr_read_b32 v140, a136\n\t" \
    "v_accvgpr_read_b32 v141, a137\n\t" \
    "v_accvgpr_read_b32 v142, a138\n\t" \
    "v_accvgpr_read_b32 v143, a139\n\t" \
    "v_cvt_pk_bf16_f32 v144, v140, v141\n\t" \
    "v_cvt_pk_bf16_f32 v145, v142, v143\n\t" \
    "ds_write_b64 %0, v[144:145] offset:33856\n\t" \
    "v_accvgpr_read_b32 v146, a140\n\t" \
    "v_accvgpr_read_b32 v147, a141\n\t" \
    "v_accvgpr_read_b32 v148, a142\n\t" \
    "v_accvgpr_read_b32 v149, a143\n\t" \
    "v_cvt_pk_bf16_f32 v150, v146, v147\n\t" \
    "v_cvt_pk_bf16_f32 v151, v148, v149\n\t" \
    "ds_write_b64 %0, v[150:151] offset:33888\n\t" \
    "v_accvgpr_read_b32 v152, a144\n\t" \
    "v_accvgpr_read_b32 v153, a145\n\t" \
    "v_accvgpr_read_b32 v154, a146\n\t" \
    "v_accvgpr_read_b32 v155, a147\n\t" \
    "v_cvt_pk_bf16_f32 v156, v152, v153\n\t" \
    "v_cvt_pk_bf16_f32 v157, v154, v155\n\t" \
    "ds_write_b64 %0, v[156:157] offset:33920\n\t" \
    "v_accvgpr_read_b32 v158, a148\n\t" \
    "v_accvgpr_read_b32 v159, a149\n\t" \
    "v_accvgpr_read_b32 v160, a150\n\t" \
    "v_accvgpr_read_b32 v161, a151\n\t" \
    "v_cvt_pk_bf16_f32 v162, v158, v159\n\t" \
    "v_cvt_pk_bf16_f32 v163, v160, v161\n\t" \
    "ds_write_b64 %0, v[162:163] offset:33952\n\t" \
    "v_accvgpr_read_b32 v164, a152\n\t" \
    "v_accvgpr_read_b32 v165, a153\n\t" \
    "v_accvgpr_read_b32 v166, a154\n\t" \
    "v_accvgpr_read_b32 v167, a155\n\t" \
    "v_cvt_pk_bf16_f32 v168, v164, v165\n\t" \
    "v_cvt_pk_bf16_f32 v169, v166, v167\n\t" \
    "ds_write_b64 %0, v[168:169] offset:33984\n\t" \
    "v_accvgpr_read_b32 v170, a156\n\t" \
    "v_accvgpr_read_b32 v171, a157\n\t" \
    "v_accvgpr_read_b32 v172, a158\n\t" \
    "v_accvgpr_read_b32 v173, a159\n\t" \
    "v_cvt_pk_bf16_f32 v174, v170, v171\n\t" \
    "v_cvt_pk_bf16_f32 v175, v172, v173\n\t" \
    "ds_write_b64 %0, v[174:175] offset:34016\n\t" \
    "v_accvgpr_read_b32 v128, a160\n\t" \
    "v_accvgpr_read_b32 v129, a161\n\t" \
    "v_accvgpr_read_b32 v130, a162\n\t" \
    "v_accvgpr_read_b32 v131, a163\n\t" \
    "v_cvt_pk_bf16_f32 v132, v128, v129\n\t" \
    "v_cvt_pk_bf16_f32 v133, v130, v131\n\t" \
    "ds_write_b64 %0, v[132:133] offset:42240\n\t" \
    "v_accvgpr_read_b32 v134, a164\n\t" \
    "v_accvgpr_read_b32 v135, a165\n\t" \
    "v_accvgpr_read_b32 v136, a166\n\t" \
    "v_accvgpr_read_b32 v137, a167\n\t" \
    "v_cvt_pk_bf16_f32 v138, v134, v135\n\t" \
    "v_cvt_pk_bf16_f32 v139, v136, v137\n\t" \
    "ds_write_b64 %0, v[138:139] offset:42272\n\t" \
    "v_accvgpr_read_b32 v140, a168\n\t" \
    "v_accvgpr_read_b32 v141, a169\n\t" \
    "v_accvgpr_read_b32 v142, a170\n\t" \
    "v_accvgpr_read_b32 v143, a171\n\t" \
    "v_cvt_pk_bf16_f32 v144, v140, v141\n\t" \
    "v_cvt_pk_bf16_f32 v145, v142, v143\n\t" \
    "ds_write_b64 %0, v[144:145] offset:42304\n\t" \
    "v_accvgpr_read_b32 v146, a172\n\t" \
    "v_accvgpr_read_b32 v147, a173\n\t" \
    "v_accvgpr_read_b32 v148, a174\n\t" \
    "v_accvgpr_read_b32 v149, a175\n\t" \
    "v_cvt_pk_bf16_f32 v150, v146, v147\n\t" \
    "v_cvt_pk_bf16_f32 v151, v148, v149\n\t" \
    "ds_write_b64 %0, v[150:151] offset:42336\n\t" \
    "v_accvgpr_read_b32 v152, a176\n\t" \
    "v_accvgpr_read_b32 v153, a177\n\t" \
    "v_accvgpr_read_b32 v154, a178\n\t" \
    "v_accvgpr_read_b32 v155, a179\n\t" \
    "v_cvt_pk_bf16_f32 v156, v152, v153\n\t" \
    "v_cvt_pk_bf16_f32 v157, v154, v155\n\t" \
    "ds_write_b64 %0, v[156:157] offset:42368\n\t" \
    "v_accvgpr_read_b32 v158, a180\n\t" \
    "v_accvgpr_read_b32 v159, a181\n\t" \
    "v_accvgpr_read_b32 v160, a182\n\t" \
    "v_accvgpr_read_b32 v161, a183\n\t" \
    "v_cvt_pk_bf16_f32 v162, v158, v159\n\t" \
    "v_cvt_pk_bf16_f32 v163, v160, v161\n\t" \
    "ds_write_b64 %0, v[162:163] offset:42400\n\t" \
    "v_accvgpr_read_b32 v164, a184\n\t" \
    "v_accvgpr_read_b32 v165, a185\n\t" \
    "v_accvgpr_read_b32 v166, a186\n\t" \
    "v_accvgpr_read_b32 v167, a187\n\t" \
    "v_cvt_pk_bf16_f32 v168, v164, v165\n\t" \
    "v_cvt_pk_bf16_f32 v169, v166, v167\n\t" \
    "ds_write_b64 %0, v[168:169] offset:42432\n\t" \
    "v_accvgpr_read_b32 v170, a188\n\t" \
    "v_accvgpr_read_b32 v171, a189\n\t" \
    "v_accvgpr_read_b32 v172, a190\n\t" \
    "v_accvgpr_read_b32 v173, a191\n\t" \
    "v_cvt_pk_bf16_f32 v174, v170, v171\n\t" \
    "v_cvt_pk_bf16_f32 v175, v172, v173\n\t" \
    "ds_write_b64 %0, v[174:175] offset:42464\n\t" \
    "v_accvgpr_read_b32 v128, a192\n\t" \
    "v_accvgpr_read_b32 v129, a193\n\t" \
    "v_accvgpr_read_b32 v130, a194\n\t" \
    "v_accvgpr_read_b32 v131, a195\n\t" \
    "v_cvt_pk_bf16_f32 v132, v128, v129\n\t" \
    "v_cvt_pk_bf16_f32 v133, v130, v131\n\t" \
    "ds_write_b64 %0, v[132:133] offset:50688\n\t" \
    "v_accvgpr_read_b32 v134, a196\n\t" \
    "v_accvgpr_read_b32 v135, a197\n\t" \
    "v_accvgpr_read_b32 v136, a198\n\t" \
    "v_accvgpr_read_b32 v137, a199\n\t" \
    "v_cvt_pk_bf16_f32 v138, v134, v135\n\t" \
    "v_cvt_pk_bf16_f32 v139, v136, v137\n\t" \
    "ds_write_b64 %0, v[138:139] offset:50720\n\t" \
    "v_accvgpr_read_b32 v140, a200\n\t" \
    "v_accvgpr_read_b32 v141, a201\n\t" \
    "v_accvgpr_read_b32 v142, a202\n\t" \
    "v_accvgpr_read_b32 v143, a203\n\t" \
    "v_cvt_pk_bf16_f32 v144, v140, v141\n\t" \
    "v_cvt_pk_bf16_f32 v145, v142, v143\n\t" \
    "ds_write_b64 %0, v[144:145] offset:50752\n\t" \
    "v_accvgpr_read_b32 v146, a204\n\t" \
    "v_accvgpr_read_b32 v147, a205\n\t" \
    "v_accvgpr_read_b32 v148, a206\n\t" \
    "v_accvgpr_read_b32 v149, a207\n\t" \
    "v_cvt_pk_bf16_f32 v150, v146, v147\n\t" \
    "v_cvt_pk_bf16_f32 v151, v148, v149\n\t" \
    "ds_write_b64 %0, v[150:151] offset:50784\n\t" \
    "v_accvgpr_read_b32 v152, a208\n\t" \
    "v_accvgpr_read_b32 v153, a209\n\t" \
    "v_accvgpr_read_b32 v154, a210\n\t" \
    "v_accvgpr_read_b32 v155, a211\n\t" \
    "v_cvt_pk_bf16_f32 v156, v152, v153\n\t" \
    "v_cvt_pk_bf16_f32 v157, v154, v155\n\t" \
    "ds_write_b64 %0, v[156:157] offset:50816\n\t" \
    "v_accvgpr_read_b32 v158, a212\n\t" \
    "v_accvgpr_read_b32 v159, a213\n\t" \
    "v_accvgpr_read_b32 v160, a214\n\t" \
    "v_accvgpr_read_b32 v161, a215\n\t" \
    "v_cvt_pk_bf16_f32 v162, v158, v159\n\t" \
    "v_cvt_pk_bf16_f32 v163, v160, v161\n\t" \
    "ds_write_b64 %0, v[162:163] offset:50848\n\t" \
    "v_accvgpr_read_b32 v164, a216\n\t" \
    "v_accvgpr_read_b32 v165, a217\n\t" \
    "v_accvgpr_read_b32 v166, a218\n\t" \
    "v_accvgpr_read_b32 v167, a219\n\t" \
    "v_cvt_pk_bf16_f32 v168, v164, v165\n\t" \
    "v_cvt_pk_bf16_f32 v169, v166, v167\n\t" \
    "ds_write_b64 %0, v[168:169] offset:50880\n\t" \
    "v_accvgpr_read_b32 v170, a220\n\t" \
    "v_accvgpr_read_b32 v171, a221\n\t" \
    "v_accvgpr_read_b32 v172, a222\n\t" \
    "v_accvgpr_read_b32 v173, a223\n\t" \
    "v_cvt_pk_bf16_f32 v174, v170, v171\n\t" \
    "v_cvt_pk_bf16_f32 v175, v172, v173\n\t" \
    "ds_write_b64 %0, v[174:175] offset:50912\n\t" \
    "v_accvgpr_read_b32 v128, a224\n\t" \
    "v_accvgpr_read_b32 v129, a225\n\t" \
    "v_accvgpr_read_b32 v130, a226\n\t" \
    "v_accvgpr_read_b32 v131, a227\n\t" \
    "v_cvt_pk_bf16_f32 v132, v128, v129\n\t" \
    "v_cvt_pk_bf16_f32 v133, v130, v131\n\t" \
    "ds_write_b64 %0, v[132:133] offset:59136\n\t" \
    "v_accvgpr_read_b32 v134, a228\n\t" \
    "v_accvgpr_read_b32 v135, a229\n\t" \
    "v_accvgpr_read_b32 v136, a230\n\t" \
    "v_accvgpr_read_b32 v137, a231\n\t" \
    "v_cvt_pk_bf16_f32 v138, v134, v135\n\t" \
    "v_cvt_pk_bf16_f32 v139, v136, v137\n\t" \
    "ds_write_b64 %0, v[138:139] offset:59168\n\t" \
    "v_accvgpr_read_b32 v140, a232\n\t" \
    "v_accvgpr_read_b32 v141, a233\n\t" \
    "v_accvgpr_read_b32 v142, a234\n\t" \
    "v_accvgpr_read_b32 v143, a235\n\t" \
    "v_cvt_pk_bf16_f32 v144, v140, v141\n\t" \
    "v_cvt_pk_bf16_f32 v145, v142, v143\n\t" \
    "ds_write_b64 %0, v[144:145] offset:59200\n\t" \
    "v_accvgpr_read_b32 v146, a236\n\t" \
    "v_accvgpr_read_b32 v147, a237\n\t" \
    "v_accvgpr_read_b32 v148, a238\n\t" \
    "v_accvgpr_read_b32 v149, a239\n\t" \
    "v_cvt_pk_bf16_f32 v150, v146, v147\n\t" \
    "v_cvt_pk_bf16_f32 v151, v148, v149\n\t" \
    "ds_write_b64 %0, v[150:151] offset:59232\n\t" \
    "v_accvgpr_read_b32 v152, a240\n\t" \
    "v_accvgpr_read_b32 v153, a241\n\t" \
    "v_accvgpr_read_b32 v154, a242\n\t" \
    "v_accvgpr_read_b32 v155, a243\n\t" \
    "v_cvt_pk_bf16_f32 v156, v152, v153\n\t" \
    "v_cvt_pk_bf16_f32 v157, v154, v155\n\t" \
    "ds_write_b64 %0, v[156:157] offset:59264\n\t" \
    "v_accvgpr_read_b32 v158, a244\n\t" \
    "v_accvgpr_read_b32 v159, a245\n\t" \
    "v_accvgpr_read_b32 v160, a246\n\t" \
    "v_accvgpr_read_b32 v161, a247\n\t" \
    "v_cvt_pk_bf16_f32 v162, v158, v159\n\t" \
    "v_cvt_pk_bf16_f32 v163, v160, v161\n\t" \
    "ds_write_b64 %0, v[162:163] offset:59296\n\t" \
    "v_accvgpr_read_b32 v164, a248\n\t" \
    "v_accvgpr_read_b32 v165, a249\n\t" \
    "v_accvgpr_read_b32 v166, a250\n\t" \
    "v_accvgpr_read_b32 v167, a251\n\t" \
    "v_cvt_pk_bf16_f32 v168, v164, v165\n\t" \
    "v_cvt_pk_bf16_f32 v169, v166, v167\n\t" \
    "ds_write_b64 %0, v[168:169] offset:59328\n\t" \
    "v_accvgpr_read_b32 v170, a252\n\t" \
    "v_accvgpr_read_b32 v171, a253\n\t" \
    "v_accvgpr_read_b32 v172, a254\n\t" \
    "v_accvgpr_read_b32 v173, a255\n\t" \
    "v_cvt_pk_bf16_f32 v174, v170, v171\n\t" \
    "v_cvt_pk_bf16_f32 v175, v172, v173\n\t" \
    "ds_write_b64 %0, v[174:175] offset:59360\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    ""

#define SYMB_GEMM16_STORE_PARTIAL \
    "v_mov_b32 v116, %0\n\t" \
    "global_store_dwordx4 v116, a[0:3], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[4:7], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[8:11], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[12:15], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[16:19], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[20:23], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[24:27], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[28:31], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[32:35], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[36:39], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[40:43], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[44:47], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[48:51], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[52:55], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[56:59], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[60:63], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[64:67], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[68:71], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[72:75], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[76:79], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[80:83], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[84:87], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[88:91], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[92:95], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[96:99], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[100:103], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[104:107], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[108:111], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[112:115], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[116:119], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[120:123], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[124:127], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[128:131], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[132:135], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[136:139], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[140:143], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[144:147], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[148:151], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[152:155], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[156:159], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[160:163], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[164:167], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[168:171], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[172:175], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[176:179], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[180:183], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[184:187], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[188:191], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[192:195], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[196:199], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[200:203], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[204:207], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[208:211], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[212:215], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[216:219], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[220:223], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[224:227], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[228:231], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[232:235], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[236:239], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[240:243], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[244:247], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[248:251], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[252:255], %1 offset:3072\n\t" \
    "s_waitcnt vmcnt(0)\n\t" \
    ""

#define SYMB_GEMM16_VCLOBBERS "v116", "v117", "v118", "v119", "v120", "v121", "v122", "v123", "v124", "v125", "v126", "v127", "v128", "v129", "v130", "v131", "v132", "v133", "v134", "v135", "v136", "v137", "v138", "v139", "v140", "v141", "v142", "v143", "v144", "v145", "v146", "v147", "v148", "v149", "v150", "v151", "v152", "v153", "v154", "v155", "v156", "v157", "v158", "v159", "v160", "v161", "v162", "v163", "v164", "v165", "v166", "v167", "v168", "v169", "v170", "v171", "v172", "v173", "v174", "v175", "v176", "v177", "v178", "v179", "v180", "v181", "v182", "v183", "v184", "v185", "v186", "v187", "v188", "v189", "v190", "v191", "v192", "v193", "v194", "v195", "v196", "v197", "v198", "v199", "v200", "v201", "v202", "v203", "v204", "v205", "v206", "v207", "v208", "v209", "v210", "v211", "v212", "v213", "v214", "v215", "v216", "v217", "v218", "v219", "v220", "v221", "v222", "v223", "v224", "v225", "v226", "v227", "v228", "v229", "v230", "v231", "v232", "v233", "v234", "v235", "v236", "v237", "v238", "v239", "v240", "v241", "v242", "v243", "v244", "v245", "v246", "v247", "v248", "v249", "v250", "v251", "v252", "v253", "v254", "v255"
#define SYMB_GEMM16_ACLOBBERS "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15", "a16", "a17", "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31", "a32", "a33", "a34", "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46", "a47", "a48", "a49", "a50", "a51", "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61", "a62", "a63", "a64", "a65", "a66", "a67", "a68", "a69", "a70", "a71", "a72", "a73", "a74", "a75", "a76", "a77", "a78", "a79", "a80", "a81", "a82", "a83", "a84", "a85", "a86", "a87", "a88", "a89", "a90", "a91", "a92", "a93", "a94", "a95", "a96", "a97", "a98", "a99", "a100", "a101", "a102", "a103", "a104", "a105", "a106", "a107", "a108", "a109", "a110", "a111", "a112", "a113", "a114", "a115", "a116", "a117", "a118", "a119", "a120", "a121", "a122", "a123", "a124", "a125", "a126", "a127", "a128", "a129", "a130", "a131", "a132", "a133", "a134", "a135", "a136", "a137", "a138", "a139", "a140", "a141", "a142", "a143", "a144", "a145", "a146", "a147", "a148", "a149", "a150", "a151", "a152", "a153", "a154", "a155", "a156", "a157", "a158", "a159", "a160", "a161", "a162", "a163", "a164", "a165", "a166", "a167", "a168", "a169", "a170", "a171", "a172", "a173", "a174", "a175", "a176", "a177", "a178", "a179", "a180", "a181", "a182", "a183", "a184", "a185", "a186", "a187", "a188", "a189", "a190", "a191", "a192", "a193", "a194", "a195", "a196", "a197", "a198", "a199", "a200", "a201", "a202", "a203", "a204", "a205", "a206", "a207", "a208", "a209", "a210", "a211", "a212", "a213", "a214", "a215", "a216", "a217", "a218", "a219", "a220", "a221", "a222", "a223", "a224", "a225", "a226", "a227", "a228", "a229", "a230", "a231", "a232", "a233", "a234", "a235", "a236", "a237", "a238", "a239", "a240", "a241", "a242", "a243", "a244", "a245", "a246", "a247", "a248", "a249", "a250", "a251", "a252", "a253", "a254", "a255"

// ---- 128x128 tile: a wavefront owns 4x4 blocks, block (i, j) in a[4(4i+j) : 4(4i+j)+3].
// Main loop operands: %0-%3 A fragment lane offsets inside an A unit (32-k step 0 first / second
// read, step 1 first / second read); %4-%7 B fragment lane offsets inside a B unit (K-contiguous W:
// as for A in %4-%7; N-contiguous W: one per 16-column block); %8-%11 / %12-%15 global byte offsets
// of this lane's 4 A / 4 B loads per stage; %16,%17 global base of the A / B stage (64-bit SGPR);
// %18 byte stride of B between stages; %19 number of 64-k stages (>= 1); %20 LDS byte address of the
// dynamic segment + this wavefront's first load inside a unit (wave * 4096).  LDS: units of
// 16 KiB, A at unit 0/1/2, B at unit 3/4.  Fixed registers: s80-s91, v116-v191 (fragment sets at
// v128 and v160), a0-a63.
#define SYMB_GEMM16S_LOOP_NT \
    "s_mov_b64 s[80:81], %16\n\t" \
    "s_mov_b64 s[82:83], %17\n\t" \
    "s_sub_u32 s84, %19, 2\n\t" \
    "s_mov_b32 s85, 0\n\t" \
    "s_mov_b32 s86, 16384\n\t" \
    "s_mov_b32 s87, 32768\n\t" \
    "s_mov_b32 s88, 49152\n\t" \
    "s_mov_b32 s89, 65536\n\t" \
    "s_add_u32 s90, s85, %20\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %8, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %9, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %10, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %11, s[80:81]\n\t" \
    "s_cmp_gt_u32 %19, 1\n\t" \
    "s_cselect_b32 s91, 128, 0\n\t" \
    "s_add_u32 s80, s80, s91\n\t" \
    "s_addc_u32 s81, s81, 0\n\t" \
    "s_add_u32 s90, s88, %20\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %12, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %13, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %14, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %15, s[82:83]\n\t" \
    "s_cmp_gt_u32 %19, 1\n\t" \
    "s_cselect_b32 s91, %18, 0\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, 0\n\t" \
    "s_add_u32 s90, s86, %20\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %8, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %9, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %10, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %11, s[80:81]\n\t" \
    "s_add_u32 s80, s80, 128\n\t" \
    "s_addc_u32 s81, s81, 0\n\t" \
    "s_add_u32 s90, s89, %20\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %12, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %13, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %14, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %15, s[82:83]\n\t" \
    "s_mov_b32 s91, %18\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, 0\n\t" \
    "v_accvgpr_write_b32 a0, 0\n\t" \
    "v_accvgpr_write_b32 a1, 0\n\t" \
    "v_accvgpr_write_b32 a2, 0\n\t" \
    "v_accvgpr_write_b32 a3, 0\n\t" \
    "v_accvgpr_write_b32 a4, 0\n\t" \
    "v_accvgpr_write_b32 a5, 0\n\t" \
    "v_accvgpr_write_b32 a6, 0\n\t" \
    "v_accvgpr_write_b32 a7, 0\n\t" \
    "v_accvgpr_write_b32 a8, 0\n\t" \
    "v_accvgpr_write_b32 a9, 0\n\t" \
    "v_accvgpr_write_b32 a10, 0\n\t" \
    "v_accvgpr_write_b32 a11, 0\n\t" \
    "v_accvgpr_write_b32 a12, 0\n\t" \
    "v_accvgpr_write_b32 a13, 0\n\t" \
    "v_accvgpr_write_b32 a14, 0\n\t" \
    "v_accvgpr_write_b32 a15, 0\n\t" \
    "v_accvgpr_write_b32 a16, 0\n\t" \
    "v_accvgpr_write_b32 a17, 0\n\t" \
    "v_accvgpr_write_b32 a18, 0\n\t" \
    "v_accvgpr_write_b32 a19, 0\n\t" \
    "v_accvgpr_write_b32 a20, 0\n\t" \
    "v_accvgpr_write_b32 a21, 0\n\t" \
    "v_accvgpr_write_b32 a22, 0\n\t" \
    "v_accvgpr_write_b32 a23, 0\n\t" \
    "v_accvgpr_write_b32 a24, 0\n\t" \
    "v_accvgpr_write_b32 a25, 0\n\t" \
    "v_accvgpr_write_b32 a26, 0\n\t" \
    "v_accvgpr_write_b32 a27, 0\n\t" \
    "v_accvgpr_write_b32 a28, 0\n\t" \
    "v_accvgpr_write_b32 a29, 0\n\t" \
    "v_accvgpr_write_b32 a30, 0\n\t" \
    "v_accvgpr_write_b32 a31, 0\n\t" \
    "v_accvgpr_write_b32 a32, 0\n\t" \
    "v_accvgpr_write_b32 a33, 0\n\t" \
    "v_accvgpr_write_b32 a34, 0\n\t" \
    "v_accvgpr_write_b32 a35, 0\n\t" \
    "v_accvgpr_write_b32 a36, 0\n\t" \
    "v_accvgpr_write_b32 a37, 0\n\t" \
    "v_accvgpr_write_b32 a38, 0\n\t" \
    "v_accvgpr_write_b32 a39, 0\n\t" \
    "v_accvgpr_write_b32 a40, 0\n\t" \
    "v_accvgpr_write_b32 a41, 0\n\t" \
    "v_accvgpr_write_b32 a42, 0\n\t" \
    "v_accvgpr_write_b32 a43, 0\n\t" \
    "v_accvgpr_write_b32 a44, 0\n\t" \
    "v_accvgpr_write_b32 a45, 0\n\t" \
    "v_accvgpr_write_b32 a46, 0\n\t" \
    "v_accvgpr_write_b32 a47, 0\n\t" \
    "v_accvgpr_write_b32 a48, 0\n\t" \
    "v_accvgpr_write_b32 a49, 0\n\t" \
    "v_accvgpr_write_b32 a50, 0\n\t" \
    "v_accvgpr_write_b32 a51, 0\n\t" \
    "v_accvgpr_write_b32 a52, 0\n\t" \
    "v_accvgpr_write_b32 a53, 0\n\t" \
    "v_accvgpr_write_b32 a54, 0\n\t" \
    "v_accvgpr_write_b32 a55, 0\n\t" \
    "v_accvgpr_write_b32 a56, 0\n\t" \
    "v_accvgpr_write_b32 a57, 0\n\t" \
    "v_accvgpr_write_b32 a58, 0\n\t" \
    "v_accvgpr_write_b32 a59, 0\n\t" \
    "v_accvgpr_write_b32 a60, 0\n\t" \
    "v_accvgpr_write_b32 a61, 0\n\t" \
    "v_accvgpr_write_b32 a62, 0\n\t" \
    "v_accvgpr_write_b32 a63, 0\n\t" \
    "s_nop 3\n\t" \
    "s_waitcnt vmcnt(8)\n\t" \
    "s_barrier\n\t" \
    "v_add_u32 v116, s85, %0\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "v_add_u32 v117, s85, %1\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "v_add_u32 v118, s88, %4\n\t" \
    "ds_read_b64 v[144:145], v118 offset:0\n\t" \
    "ds_read_b64 v[148:149], v118 offset:2048\n\t" \
    "ds_read_b64 v[152:153], v118 offset:4096\n\t" \
    "ds_read_b64 v[156:157], v118 offset:6144\n\t" \
    "v_add_u32 v119, s88, %5\n\t" \
    "ds_read_b64 v[146:147], v119 offset:0\n\t" \
    "ds_read_b64 v[150:151], v119 offset:2048\n\t" \
    "ds_read_b64 v[154:155], v119 offset:4096\n\t" \
    "ds_read_b64 v[158:159], v119 offset:6144\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_cmp_lt_u32 %19, 3\n\t" \
    "s_cbranch_scc1 2f\n\t" \
    "1:\n\t" \
    "s_add_u32 s90, s87, %20\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[144:147], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "ds_read_b64 v[160:161], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[148:151], v[128:131], a[4:7]\n\t" \
    "ds_read_b64 v[164:165], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[152:155], v[128:131], a[8:11]\n\t" \
    "ds_read_b64 v[168:169], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[156:159], v[128:131], a[12:15]\n\t" \
    "ds_read_b64 v[172:173], v116 offset:6144\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %8, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[144:147], v[132:135], a[16:19]\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[162:163], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[148:151], v[132:135], a[20:23]\n\t" \
    "ds_read_b64 v[166:167], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[152:155], v[132:135], a[24:27]\n\t" \
    "ds_read_b64 v[170:171], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[156:159], v[132:135], a[28:31]\n\t" \
    "ds_read_b64 v[174:175], v117 offset:6144\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %9, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[144:147], v[136:139], a[32:35]\n\t" \
    "v_add_u32 v118, s88, %6\n\t" \
    "ds_read_b64 v[176:177], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[148:151], v[136:139], a[36:39]\n\t" \
    "ds_read_b64 v[180:181], v118 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[152:155], v[136:139], a[40:43]\n\t" \
    "ds_read_b64 v[184:185], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[156:159], v[136:139], a[44:47]\n\t" \
    "ds_read_b64 v[188:189], v118 offset:6144\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %10, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[144:147], v[140:143], a[48:51]\n\t" \
    "v_add_u32 v119, s88, %7\n\t" \
    "ds_read_b64 v[178:179], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[148:151], v[140:143], a[52:55]\n\t" \
    "ds_read_b64 v[182:183], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[152:155], v[140:143], a[56:59]\n\t" \
    "ds_read_b64 v[186:187], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[156:159], v[140:143], a[60:63]\n\t" \
    "ds_read_b64 v[190:191], v119 offset:6144\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %11, s[80:81]\n\t" \
    "s_add_u32 s80, s80, 128\n\t" \
    "s_addc_u32 s81, s81, 0\n\t" \
    "s_waitcnt vmcnt(4) lgkmcnt(0)\n\t" \
    "s_barrier\n\t" \
    "s_add_u32 s90, s88, %20\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[176:179], v[160:163], a[0:3]\n\t" \
    "v_add_u32 v116, s86, %0\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[180:183], v[160:163], a[4:7]\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[184:187], v[160:163], a[8:11]\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[188:191], v[160:163], a[12:15]\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %12, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[176:179], v[164:167], a[16:19]\n\t" \
    "v_add_u32 v117, s86, %1\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[180:183], v[164:167], a[20:23]\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[184:187], v[164:167], a[24:27]\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[188:191], v[164:167], a[28:31]\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %13, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[176:179], v[168:171], a[32:35]\n\t" \
    "v_add_u32 v118, s89, %4\n\t" \
    "ds_read_b64 v[144:145], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[180:183], v[168:171], a[36:39]\n\t" \
    "ds_read_b64 v[148:149], v118 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[184:187], v[168:171], a[40:43]\n\t" \
    "ds_read_b64 v[152:153], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[188:191], v[168:171], a[44:47]\n\t" \
    "ds_read_b64 v[156:157], v118 offset:6144\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %14, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[176:179], v[172:175], a[48:51]\n\t" \
    "v_add_u32 v119, s89, %5\n\t" \
    "ds_read_b64 v[146:147], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[180:183], v[172:175], a[52:55]\n\t" \
    "ds_read_b64 v[150:151], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[184:187], v[172:175], a[56:59]\n\t" \
    "ds_read_b64 v[154:155], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[188:191], v[172:175], a[60:63]\n\t" \
    "ds_read_b64 v[158:159], v119 offset:6144\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %15, s[82:83]\n\t" \
    "s_mov_b32 s91, %18\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, 0\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_mov_b32 s90, s85\n\t" \
    "s_mov_b32 s85, s86\n\t" \
    "s_mov_b32 s86, s87\n\t" \
    "s_mov_b32 s87, s90\n\t" \
    "s_mov_b32 s90, s88\n\t" \
    "s_mov_b32 s88, s89\n\t" \
    "s_mov_b32 s89, s90\n\t" \
    "s_sub_u32 s84, s84, 1\n\t" \
    "s_cmp_lg_u32 s84, 0\n\t" \
    "s_cbranch_scc1 1b\n\t" \
    "2:\n\t" \
    "s_cmp_lt_u32 %19, 2\n\t" \
    "s_cbranch_scc1 3f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[144:147], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "ds_read_b64 v[160:161], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[148:151], v[128:131], a[4:7]\n\t" \
    "ds_read_b64 v[164:165], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[152:155], v[128:131], a[8:11]\n\t" \
    "ds_read_b64 v[168:169], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[156:159], v[128:131], a[12:15]\n\t" \
    "ds_read_b64 v[172:173], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[144:147], v[132:135], a[16:19]\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[162:163], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[148:151], v[132:135], a[20:23]\n\t" \
    "ds_read_b64 v[166:167], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[152:155], v[132:135], a[24:27]\n\t" \
    "ds_read_b64 v[170:171], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[156:159], v[132:135], a[28:31]\n\t" \
    "ds_read_b64 v[174:175], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[144:147], v[136:139], a[32:35]\n\t" \
    "v_add_u32 v118, s88, %6\n\t" \
    "ds_read_b64 v[176:177], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[148:151], v[136:139], a[36:39]\n\t" \
    "ds_read_b64 v[180:181], v118 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[152:155], v[136:139], a[40:43]\n\t" \
    "ds_read_b64 v[184:185], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[156:159], v[136:139], a[44:47]\n\t" \
    "ds_read_b64 v[188:189], v118 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[144:147], v[140:143], a[48:51]\n\t" \
    "v_add_u32 v119, s88, %7\n\t" \
    "ds_read_b64 v[178:179], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[148:151], v[140:143], a[52:55]\n\t" \
    "ds_read_b64 v[182:183], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[152:155], v[140:143], a[56:59]\n\t" \
    "ds_read_b64 v[186:187], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[156:159], v[140:143], a[60:63]\n\t" \
    "ds_read_b64 v[190:191], v119 offset:6144\n\t" \
    "s_waitcnt vmcnt(0) lgkmcnt(0)\n\t" \
    "s_barrier\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[176:179], v[160:163], a[0:3]\n\t" \
    "v_add_u32 v116, s86, %0\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[180:183], v[160:163], a[4:7]\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[184:187], v[160:163], a[8:11]\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[188:191], v[160:163], a[12:15]\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[176:179], v[164:167], a[16:19]\n\t" \
    "v_add_u32 v117, s86, %1\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[180:183], v[164:167], a[20:23]\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[184:187], v[164:167], a[24:27]\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[188:191], v[164:167], a[28:31]\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[176:179], v[168:171], a[32:35]\n\t" \
    "v_add_u32 v118, s89, %4\n\t" \
    "ds_read_b64 v[144:145], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[180:183], v[168:171], a[36:39]\n\t" \
    "ds_read_b64 v[148:149], v118 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[184:187], v[168:171], a[40:43]\n\t" \
    "ds_read_b64 v[152:153], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[188:191], v[168:171], a[44:47]\n\t" \
    "ds_read_b64 v[156:157], v118 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[176:179], v[172:175], a[48:51]\n\t" \
    "v_add_u32 v119, s89, %5\n\t" \
    "ds_read_b64 v[146:147], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[180:183], v[172:175], a[52:55]\n\t" \
    "ds_read_b64 v[150:151], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[184:187], v[172:175], a[56:59]\n\t" \
    "ds_read_b64 v[154:155], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[188:191], v[172:175], a[60:63]\n\t" \
    "ds_read_b64 v[158:159], v119 offset:6144\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_mov_b32 s90, s85\n\t" \
    "s_mov_b32 s85, s86\n\t" \
    "s_mov_b32 s86, s87\n\t" \
    "s_mov_b32 s87, s90\n\t" \
    "s_mov_b32 s90, s88\n\t" \
    "s_mov_b32 s88, s89\n\t" \
    "s_mov_b32 s89, s90\n\t" \
    "3:\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[144:147], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "ds_read_b64 v[160:161], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[148:151], v[128:131], a[4:7]\n\t" \
    "ds_read_b64 v[164:165], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[152:155], v[128:131], a[8:11]\n\t" \
    "ds_read_b64 v[168:169], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[156:159], v[128:131], a[12:15]\n\t" \
    "ds_read_b64 v[172:173], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[144:147], v[132:135], a[16:19]\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[162:163], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[148:151], v[132:135], a[20:23]\n\t" \
    "ds_read_b64 v[166:167], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[152:155], v[132:135], a[24:27]\n\t" \
    "ds_read_b64 v[170:171], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[156:159], v[132:135], a[28:31]\n\t" \
    "ds_read_b64 v[174:175], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[144:147], v[136:139], a[32:35]\n\t" \
    "v_add_u32 v118, s88, %6\n\t" \
    "ds_read_b64 v[176:177], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[148:151], v[136:139], a[36:39]\n\t" \
    "ds_read_b64 v[180:181], v118 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[152:155], v[136:139], a[40:43]\n\t" \
    "ds_read_b64 v[184:185], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[156:159], v[136:139], a[44:47]\n\t" \
    "ds_read_b64 v[188:189], v118 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[144:147], v[140:143], a[48:51]\n\t" \
    "v_add_u32 v119, s88, %7\n\t" \
    "ds_read_b64 v[178:179], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[148:151], v[140:143], a[52:55]\n\t" \
    "ds_read_b64 v[182:183], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[152:155], v[140:143], a[56:59]\n\t" \
    "ds_read_b64 v[186:187], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[156:159], v[140:143], a[60:63]\n\t" \
    "ds_read_b64 v[190:191], v119 offset:6144\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[176:179], v[160:163], a[0:3]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[180:183], v[160:163], a[4:7]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[184:187], v[160:163], a[8:11]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[188:191], v[160:163], a[12:15]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[176:179], v[164:167], a[16:19]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[180:183], v[164:167], a[20:23]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[184:187], v[164:167], a[24:27]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[188:191], v[164:167], a[28:31]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[176:179], v[168:171], a[32:35]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[180:183], v[168:171], a[36:39]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[184:187], v[168:171], a[40:43]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[188:191], v[168:171], a[44:47]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[176:179], v[172:175], a[48:51]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[180:183], v[172:175], a[52:55]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[184:187], v[172:175], a[56:59]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[188:191], v[172:175], a[60:63]\n\t" \
    "s_waitcnt vmcnt(0)\n\t" \
    "s_nop 15\n\t" \
    "s_nop 7\n\t" \
    ""

#define SYMB_GEMM16S_LOOP_NN \
    "s_mov_b64 s[80:81], %16\n\t" \
    "s_mov_b64 s[82:83], %17\n\t" \
    "s_sub_u32 s84, %19, 2\n\t" \
    "s_mov_b32 s85, 0\n\t" \
    "s_mov_b32 s86, 16384\n\t" \
    "s_mov_b32 s87, 32768\n\t" \
    "s_mov_b32 s88, 49152\n\t" \
    "s_mov_b32 s89, 65536\n\t" \
    "s_add_u32 s90, s85, %20\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %8, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %9, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %10, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %11, s[80:81]\n\t" \
    "s_cmp_gt_u32 %19, 1\n\t" \
    "s_cselect_b32 s91, 128, 0\n\t" \
    "s_add_u32 s80, s80, s91\n\t" \
    "s_addc_u32 s81, s81, 0\n\t" \
    "s_add_u32 s90, s88, %20\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %12, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %13, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %14, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %15, s[82:83]\n\t" \
    "s_cmp_gt_u32 %19, 1\n\t" \
    "s_cselect_b32 s91, %18, 0\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, 0\n\t" \
    "s_add_u32 s90, s86, %20\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %8, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %9, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %10, s[80:81]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %11, s[80:81]\n\t" \
    "s_add_u32 s80, s80, 128\n\t" \
    "s_addc_u32 s81, s81, 0\n\t" \
    "s_add_u32 s90, s89, %20\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %12, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %13, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %14, s[82:83]\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %15, s[82:83]\n\t" \
    "s_mov_b32 s91, %18\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, 0\n\t" \
    "v_accvgpr_write_b32 a0, 0\n\t" \
    "v_accvgpr_write_b32 a1, 0\n\t" \
    "v_accvgpr_write_b32 a2, 0\n\t" \
    "v_accvgpr_write_b32 a3, 0\n\t" \
    "v_accvgpr_write_b32 a4, 0\n\t" \
    "v_accvgpr_write_b32 a5, 0\n\t" \
    "v_accvgpr_write_b32 a6, 0\n\t" \
    "v_accvgpr_write_b32 a7, 0\n\t" \
    "v_accvgpr_write_b32 a8, 0\n\t" \
    "v_accvgpr_write_b32 a9, 0\n\t" \
    "v_accvgpr_write_b32 a10, 0\n\t" \
    "v_accvgpr_write_b32 a11, 0\n\t" \
    "v_accvgpr_write_b32 a12, 0\n\t" \
    "v_accvgpr_write_b32 a13, 0\n\t" \
    "v_accvgpr_write_b32 a14, 0\n\t" \
    "v_accvgpr_write_b32 a15, 0\n\t" \
    "v_accvgpr_write_b32 a16, 0\n\t" \
    "v_accvgpr_write_b32 a17, 0\n\t" \
    "v_accvgpr_write_b32 a18, 0\n\t" \
    "v_accvgpr_write_b32 a19, 0\n\t" \
    "v_accvgpr_write_b32 a20, 0\n\t" \
    "v_accvgpr_write_b32 a21, 0\n\t" \
    "v_accvgpr_write_b32 a22, 0\n\t" \
    "v_accvgpr_write_b32 a23, 0\n\t" \
    "v_accvgpr_write_b32 a24, 0\n\t" \
    "v_accvgpr_write_b32 a25, 0\n\t" \
    "v_accvgpr_write_b32 a26, 0\n\t" \
    "v_accvgpr_write_b32 a27, 0\n\t" \
    "v_accvgpr_write_b32 a28, 0\n\t" \
    "v_accvgpr_write_b32 a29, 0\n\t" \
    "v_accvgpr_write_b32 a30, 0\n\t" \
    "v_accvgpr_write_b32 a31, 0\n\t" \
    "v_accvgpr_write_b32 a32, 0\n\t" \
    "v_accvgpr_write_b32 a33, 0\n\t" \
    "v_accvgpr_write_b32 a34, 0\n\t" \
    "v_accvgpr_write_b32 a35, 0\n\t" \
    "v_accvgpr_write_b32 a36, 0\n\t" \
    "v_accvgpr_write_b32 a37, 0\n\t" \
    "v_accvgpr_write_b32 a38, 0\n\t" \
    "v_accvgpr_write_b32 a39, 0\n\t" \
    "v_accvgpr_write_b32 a40, 0\n\t" \
    "v_accvgpr_write_b32 a41, 0\n\t" \
    "v_accvgpr_write_b32 a42, 0\n\t" \
    "v_accvgpr_write_b32 a43, 0\n\t" \
    "v_accvgpr_write_b32 a44, 0\n\t" \
    "v_accvgpr_write_b32 a45, 0\n\t" \
    "v_accvgpr_write_b32 a46, 0\n\t" \
    "v_accvgpr_write_b32 a47, 0\n\t" \
    "v_accvgpr_write_b32 a48, 0\n\t" \
    "v_accvgpr_write_b32 a49, 0\n\t" \
    "v_accvgpr_write_b32 a50, 0\n\t" \
    "v_accvgpr_write_b32 a51, 0\n\t" \
    "v_accvgpr_write_b32 a52, 0\n\t" \
    "v_accvgpr_write_b32 a53, 0\n\t" \
    "v_accvgpr_write_b32 a54, 0\n\t" \
    "v_accvgpr_write_b32 a55, 0\n\t" \
    "v_accvgpr_write_b32 a56, 0\n\t" \
    "v_accvgpr_write_b32 a57, 0\n\t" \
    "v_accvgpr_write_b32 a58, 0\n\t" \
    "v_accvgpr_write_b32 a59, 0\n\t" \
    "v_accvgpr_write_b32 a60, 0\n\t" \
    "v_accvgpr_write_b32 a61, 0\n\t" \
    "v_accvgpr_write_b32 a62, 0\n\t" \
    "v_accvgpr_write_b32 a63, 0\n\t" \
    "s_nop 3\n\t" \
    "s_waitcnt vmcnt(8)\n\t" \
    "s_barrier\n\t" \
    "v_add_u32 v116, s85, %0\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "v_add_u32 v117, s85, %1\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "v_add_u32 v118, s88, %4\n\t" \
    "ds_read_b64_tr_b16 v[144:145], v118 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[146:147], v118 offset:4096\n\t" \
    "v_add_u32 v119, s88, %5\n\t" \
    "ds_read_b64_tr_b16 v[148:149], v119 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[150:151], v119 offset:4096\n\t" \
    "v_add_u32 v120, s88, %6\n\t" \
    "ds_read_b64_tr_b16 v[152:153], v120 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[154:155], v120 offset:4096\n\t" \
    "v_add_u32 v121, s88, %7\n\t" \
    "ds_read_b64_tr_b16 v[156:157], v121 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[158:159], v121 offset:4096\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_cmp_lt_u32 %19, 3\n\t" \
    "s_cbranch_scc1 2f\n\t" \
    "1:\n\t" \
    "s_add_u32 s90, s87, %20\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[144:147], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "ds_read_b64 v[160:161], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[148:151], v[128:131], a[4:7]\n\t" \
    "ds_read_b64 v[164:165], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[152:155], v[128:131], a[8:11]\n\t" \
    "ds_read_b64 v[168:169], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[156:159], v[128:131], a[12:15]\n\t" \
    "ds_read_b64 v[172:173], v116 offset:6144\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %8, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[144:147], v[132:135], a[16:19]\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[162:163], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[148:151], v[132:135], a[20:23]\n\t" \
    "ds_read_b64 v[166:167], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[152:155], v[132:135], a[24:27]\n\t" \
    "ds_read_b64 v[170:171], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[156:159], v[132:135], a[28:31]\n\t" \
    "ds_read_b64 v[174:175], v117 offset:6144\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %9, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[144:147], v[136:139], a[32:35]\n\t" \
    "v_add_u32 v118, s88, %4\n\t" \
    "ds_read_b64_tr_b16 v[176:177], v118 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[148:151], v[136:139], a[36:39]\n\t" \
    "ds_read_b64_tr_b16 v[178:179], v118 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[152:155], v[136:139], a[40:43]\n\t" \
    "v_add_u32 v119, s88, %5\n\t" \
    "ds_read_b64_tr_b16 v[180:181], v119 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[156:159], v[136:139], a[44:47]\n\t" \
    "ds_read_b64_tr_b16 v[182:183], v119 offset:12288\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %10, s[80:81]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[144:147], v[140:143], a[48:51]\n\t" \
    "v_add_u32 v120, s88, %6\n\t" \
    "ds_read_b64_tr_b16 v[184:185], v120 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[148:151], v[140:143], a[52:55]\n\t" \
    "ds_read_b64_tr_b16 v[186:187], v120 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[152:155], v[140:143], a[56:59]\n\t" \
    "v_add_u32 v121, s88, %7\n\t" \
    "ds_read_b64_tr_b16 v[188:189], v121 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[156:159], v[140:143], a[60:63]\n\t" \
    "ds_read_b64_tr_b16 v[190:191], v121 offset:12288\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %11, s[80:81]\n\t" \
    "s_add_u32 s80, s80, 128\n\t" \
    "s_addc_u32 s81, s81, 0\n\t" \
    "s_waitcnt vmcnt(4) lgkmcnt(0)\n\t" \
    "s_barrier\n\t" \
    "s_add_u32 s90, s88, %20\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[176:179], v[160:163], a[0:3]\n\t" \
    "v_add_u32 v116, s86, %0\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[180:183], v[160:163], a[4:7]\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[184:187], v[160:163], a[8:11]\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[188:191], v[160:163], a[12:15]\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %12, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[176:179], v[164:167], a[16:19]\n\t" \
    "v_add_u32 v117, s86, %1\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[180:183], v[164:167], a[20:23]\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[184:187], v[164:167], a[24:27]\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[188:191], v[164:167], a[28:31]\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "s_add_u32 m0, s90, 1024\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %13, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[176:179], v[168:171], a[32:35]\n\t" \
    "v_add_u32 v118, s89, %4\n\t" \
    "ds_read_b64_tr_b16 v[144:145], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[180:183], v[168:171], a[36:39]\n\t" \
    "ds_read_b64_tr_b16 v[146:147], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[184:187], v[168:171], a[40:43]\n\t" \
    "v_add_u32 v119, s89, %5\n\t" \
    "ds_read_b64_tr_b16 v[148:149], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[188:191], v[168:171], a[44:47]\n\t" \
    "ds_read_b64_tr_b16 v[150:151], v119 offset:4096\n\t" \
    "s_add_u32 m0, s90, 2048\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %14, s[82:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[176:179], v[172:175], a[48:51]\n\t" \
    "v_add_u32 v120, s89, %6\n\t" \
    "ds_read_b64_tr_b16 v[152:153], v120 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[180:183], v[172:175], a[52:55]\n\t" \
    "ds_read_b64_tr_b16 v[154:155], v120 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[184:187], v[172:175], a[56:59]\n\t" \
    "v_add_u32 v121, s89, %7\n\t" \
    "ds_read_b64_tr_b16 v[156:157], v121 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[188:191], v[172:175], a[60:63]\n\t" \
    "ds_read_b64_tr_b16 v[158:159], v121 offset:4096\n\t" \
    "s_add_u32 m0, s90, 3072\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %15, s[82:83]\n\t" \
    "s_mov_b32 s91, %18\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, 0\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_mov_b32 s90, s85\n\t" \
    "s_mov_b32 s85, s86\n\t" \
    "s_mov_b32 s86, s87\n\t" \
    "s_mov_b32 s87, s90\n\t" \
    "s_mov_b32 s90, s88\n\t" \
    "s_mov_b32 s88, s89\n\t" \
    "s_mov_b32 s89, s90\n\t" \
    "s_sub_u32 s84, s84, 1\n\t" \
    "s_cmp_lg_u32 s84, 0\n\t" \
    "s_cbranch_scc1 1b\n\t" \
    "2:\n\t" \
    "s_cmp_lt_u32 %19, 2\n\t" \
    "s_cbranch_scc1 3f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[144:147], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "ds_read_b64 v[160:161], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[148:151], v[128:131], a[4:7]\n\t" \
    "ds_read_b64 v[164:165], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[152:155], v[128:131], a[8:11]\n\t" \
    "ds_read_b64 v[168:169], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[156:159], v[128:131], a[12:15]\n\t" \
    "ds_read_b64 v[172:173], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[144:147], v[132:135], a[16:19]\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[162:163], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[148:151], v[132:135], a[20:23]\n\t" \
    "ds_read_b64 v[166:167], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[152:155], v[132:135], a[24:27]\n\t" \
    "ds_read_b64 v[170:171], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[156:159], v[132:135], a[28:31]\n\t" \
    "ds_read_b64 v[174:175], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[144:147], v[136:139], a[32:35]\n\t" \
    "v_add_u32 v118, s88, %4\n\t" \
    "ds_read_b64_tr_b16 v[176:177], v118 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[148:151], v[136:139], a[36:39]\n\t" \
    "ds_read_b64_tr_b16 v[178:179], v118 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[152:155], v[136:139], a[40:43]\n\t" \
    "v_add_u32 v119, s88, %5\n\t" \
    "ds_read_b64_tr_b16 v[180:181], v119 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[156:159], v[136:139], a[44:47]\n\t" \
    "ds_read_b64_tr_b16 v[182:183], v119 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[144:147], v[140:143], a[48:51]\n\t" \
    "v_add_u32 v120, s88, %6\n\t" \
    "ds_read_b64_tr_b16 v[184:185], v120 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[148:151], v[140:143], a[52:55]\n\t" \
    "ds_read_b64_tr_b16 v[186:187], v120 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[152:155], v[140:143], a[56:59]\n\t" \
    "v_add_u32 v121, s88, %7\n\t" \
    "ds_read_b64_tr_b16 v[188:189], v121 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[156:159], v[140:143], a[60:63]\n\t" \
    "ds_read_b64_tr_b16 v[190:191], v121 offset:12288\n\t" \
    "s_waitcnt vmcnt(0) lgkmcnt(0)\n\t" \
    "s_barrier\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[176:179], v[160:163], a[0:3]\n\t" \
    "v_add_u32 v116, s86, %0\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[180:183], v[160:163], a[4:7]\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[184:187], v[160:163], a[8:11]\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[188:191], v[160:163], a[12:15]\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[176:179], v[164:167], a[16:19]\n\t" \
    "v_add_u32 v117, s86, %1\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[180:183], v[164:167], a[20:23]\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[184:187], v[164:167], a[24:27]\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[188:191], v[164:167], a[28:31]\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[176:179], v[168:171], a[32:35]\n\t" \
    "v_add_u32 v118, s89, %4\n\t" \
    "ds_read_b64_tr_b16 v[144:145], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[180:183], v[168:171], a[36:39]\n\t" \
    "ds_read_b64_tr_b16 v[146:147], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[184:187], v[168:171], a[40:43]\n\t" \
    "v_add_u32 v119, s89, %5\n\t" \
    "ds_read_b64_tr_b16 v[148:149], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[188:191], v[168:171], a[44:47]\n\t" \
    "ds_read_b64_tr_b16 v[150:151], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[176:179], v[172:175], a[48:51]\n\t" \
    "v_add_u32 v120, s89, %6\n\t" \
    "ds_read_b64_tr_b16 v[152:153], v120 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[180:183], v[172:175], a[52:55]\n\t" \
    "ds_read_b64_tr_b16 v[154:155], v120 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[184:187], v[172:175], a[56:59]\n\t" \
    "v_add_u32 v121, s89, %7\n\t" \
    "ds_read_b64_tr_b16 v[156:157], v121 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[188:191], v[172:175], a[60:63]\n\t" \
    "ds_read_b64_tr_b16 v[158:159], v121 offset:4096\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_mov_b32 s90, s85\n\t" \
    "s_mov_b32 s85, s86\n\t" \
    "s_mov_b32 s86, s87\n\t" \
    "s_mov_b32 s87, s90\n\t" \
    "s_mov_b32 s90, s88\n\t" \
    "s_mov_b32 s88, s89\n\t" \
    "s_mov_b32 s89, s90\n\t" \
    "3:\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[144:147], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "ds_read_b64 v[160:161], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[148:151], v[128:131], a[4:7]\n\t" \
    "ds_read_b64 v[164:165], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[152:155], v[128:131], a[8:11]\n\t" \
    "ds_read_b64 v[168:169], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[156:159], v[128:131], a[12:15]\n\t" \
    "ds_read_b64 v[172:173], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[144:147], v[132:135], a[16:19]\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[162:163], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[148:151], v[132:135], a[20:23]\n\t" \
    "ds_read_b64 v[166:167], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[152:155], v[132:135], a[24:27]\n\t" \
    "ds_read_b64 v[170:171], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[156:159], v[132:135], a[28:31]\n\t" \
    "ds_read_b64 v[174:175], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[144:147], v[136:139], a[32:35]\n\t" \
    "v_add_u32 v118, s88, %4\n\t" \
    "ds_read_b64_tr_b16 v[176:177], v118 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[148:151], v[136:139], a[36:39]\n\t" \
    "ds_read_b64_tr_b16 v[178:179], v118 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[152:155], v[136:139], a[40:43]\n\t" \
    "v_add_u32 v119, s88, %5\n\t" \
    "ds_read_b64_tr_b16 v[180:181], v119 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[156:159], v[136:139], a[44:47]\n\t" \
    "ds_read_b64_tr_b16 v[182:183], v119 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[144:147], v[140:143], a[48:51]\n\t" \
    "v_add_u32 v120, s88, %6\n\t" \
    "ds_read_b64_tr_b16 v[184:185], v120 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[148:151], v[140:143], a[52:55]\n\t" \
    "ds_read_b64_tr_b16 v[186:187], v120 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[152:155], v[140:143], a[56:59]\n\t" \
    "v_add_u32 v121, s88, %7\n\t" \
    "ds_read_b64_tr_b16 v[188:189], v121 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[156:159], v[140:143], a[60:63]\n\t" \
    "ds_read_b64_tr_b16 v[190:191], v121 offset:12288\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[176:179], v[160:163], a[0:3]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[180:183], v[160:163], a[4:7]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[184:187], v[160:163], a[8:11]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[188:191], v[160:163], a[12:15]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[176:179], v[164:167], a[16:19]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[180:183], v[164:167], a[20:23]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[184:187], v[164:167], a[24:27]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[188:191], v[164:167], a[28:31]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[176:179], v[168:171], a[32:35]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[180:183], v[168:171], a[36:39]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[184:187], v[168:171], a[40:43]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[188:191], v[168:171], a[44:47]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[176:179], v[172:175], a[48:51]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[180:183], v[172:175], a[52:55]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[184:187], v[172:175], a[56:59]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[188:191], v[172:175], a[60:63]\n\t" \
    "s_waitcnt vmcnt(0)\n\t" \
    "s_nop 15\n\t" \
    "s_nop 7\n\t" \
    ""

#define SYMB_GEMM16S_KSTEP32_NT \
    "s_cmp_eq_u32 %4, 0\n\t" \
    "s_cbranch_scc1 19f\n\t" \
    "ds_read_b64 v[144:145], %2 offset:0\n\t" \
    "ds_read_b64 v[148:149], %2 offset:2048\n\t" \
    "ds_read_b64 v[152:153], %2 offset:4096\n\t" \
    "ds_read_b64 v[156:157], %2 offset:6144\n\t" \
    "ds_read_b64 v[146:147], %3 offset:0\n\t" \
    "ds_read_b64 v[150:151], %3 offset:2048\n\t" \
    "ds_read_b64 v[154:155], %3 offset:4096\n\t" \
    "ds_read_b64 v[158:159], %3 offset:6144\n\t" \
    "s_bitcmp1_b32 %4, 0\n\t" \
    "s_cbranch_scc0 20f\n\t" \
    "ds_read_b64 v[128:129], %0 offset:0\n\t" \
    "ds_read_b64 v[130:131], %1 offset:0\n\t" \
    "20:\n\t" \
    "s_bitcmp1_b32 %4, 1\n\t" \
    "s_cbranch_scc0 21f\n\t" \
    "ds_read_b64 v[132:133], %0 offset:2048\n\t" \
    "ds_read_b64 v[134:135], %1 offset:2048\n\t" \
    "21:\n\t" \
    "s_bitcmp1_b32 %4, 2\n\t" \
    "s_cbranch_scc0 22f\n\t" \
    "ds_read_b64 v[136:137], %0 offset:4096\n\t" \
    "ds_read_b64 v[138:139], %1 offset:4096\n\t" \
    "22:\n\t" \
    "s_bitcmp1_b32 %4, 3\n\t" \
    "s_cbranch_scc0 23f\n\t" \
    "ds_read_b64 v[140:141], %0 offset:6144\n\t" \
    "ds_read_b64 v[142:143], %1 offset:6144\n\t" \
    "23:\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_bitcmp1_b32 %4, 0\n\t" \
    "s_cbranch_scc0 30f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[144:147], v[128:131], a[0:3]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[148:151], v[128:131], a[4:7]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[152:155], v[128:131], a[8:11]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[156:159], v[128:131], a[12:15]\n\t" \
    "30:\n\t" \
    "s_bitcmp1_b32 %4, 1\n\t" \
    "s_cbranch_scc0 31f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[144:147], v[132:135], a[16:19]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[148:151], v[132:135], a[20:23]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[152:155], v[132:135], a[24:27]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[156:159], v[132:135], a[28:31]\n\t" \
    "31:\n\t" \
    "s_bitcmp1_b32 %4, 2\n\t" \
    "s_cbranch_scc0 32f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[144:147], v[136:139], a[32:35]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[148:151], v[136:139], a[36:39]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[152:155], v[136:139], a[40:43]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[156:159], v[136:139], a[44:47]\n\t" \
    "32:\n\t" \
    "s_bitcmp1_b32 %4, 3\n\t" \
    "s_cbranch_scc0 33f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[144:147], v[140:143], a[48:51]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[148:151], v[140:143], a[52:55]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[152:155], v[140:143], a[56:59]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[156:159], v[140:143], a[60:63]\n\t" \
    "33:\n\t" \
    "s_nop 15\n\t" \
    "s_nop 7\n\t" \
    "19:\n\t" \
    ""

#define SYMB_GEMM16S_KSTEP32_NN \
    "s_cmp_eq_u32 %6, 0\n\t" \
    "s_cbranch_scc1 19f\n\t" \
    "ds_read_b64_tr_b16 v[144:145], %2 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[146:147], %2 offset:4096\n\t" \
    "ds_read_b64_tr_b16 v[148:149], %3 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[150:151], %3 offset:4096\n\t" \
    "ds_read_b64_tr_b16 v[152:153], %4 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[154:155], %4 offset:4096\n\t" \
    "ds_read_b64_tr_b16 v[156:157], %5 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[158:159], %5 offset:4096\n\t" \
    "s_bitcmp1_b32 %6, 0\n\t" \
    "s_cbranch_scc0 20f\n\t" \
    "ds_read_b64 v[128:129], %0 offset:0\n\t" \
    "ds_read_b64 v[130:131], %1 offset:0\n\t" \
    "20:\n\t" \
    "s_bitcmp1_b32 %6, 1\n\t" \
    "s_cbranch_scc0 21f\n\t" \
    "ds_read_b64 v[132:133], %0 offset:2048\n\t" \
    "ds_read_b64 v[134:135], %1 offset:2048\n\t" \
    "21:\n\t" \
    "s_bitcmp1_b32 %6, 2\n\t" \
    "s_cbranch_scc0 22f\n\t" \
    "ds_read_b64 v[136:137], %0 offset:4096\n\t" \
    "ds_read_b64 v[138:139], %1 offset:4096\n\t" \
    "22:\n\t" \
    "s_bitcmp1_b32 %6, 3\n\t" \
    "s_cbranch_scc0 23f\n\t" \
    "ds_read_b64 v[140:141], %0 offset:6144\n\t" \
    "ds_read_b64 v[142:143], %1 offset:6144\n\t" \
    "23:\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_bitcmp1_b32 %6, 0\n\t" \
    "s_cbranch_scc0 30f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[144:147], v[128:131], a[0:3]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[148:151], v[128:131], a[4:7]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[152:155], v[128:131], a[8:11]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[156:159], v[128:131], a[12:15]\n\t" \
    "30:\n\t" \
    "s_bitcmp1_b32 %6, 1\n\t" \
    "s_cbranch_scc0 31f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[144:147], v[132:135], a[16:19]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[148:151], v[132:135], a[20:23]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[152:155], v[132:135], a[24:27]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[156:159], v[132:135], a[28:31]\n\t" \
    "31:\n\t" \
    "s_bitcmp1_b32 %6, 2\n\t" \
    "s_cbranch_scc0 32f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[144:147], v[136:139], a[32:35]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[148:151], v[136:139], a[36:39]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[152:155], v[136:139], a[40:43]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[156:159], v[136:139], a[44:47]\n\t" \
    "32:\n\t" \
    "s_bitcmp1_b32 %6, 3\n\t" \
    "s_cbranch_scc0 33f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[144:147], v[140:143], a[48:51]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[148:151], v[140:143], a[52:55]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[152:155], v[140:143], a[56:59]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[156:159], v[140:143], a[60:63]\n\t" \
    "33:\n\t" \
    "s_nop 15\n\t" \
    "s_nop 7\n\t" \
    "19:\n\t" \
    ""

#define SYMB_GEMM16S_ZERO \
    "v_accvgpr_write_b32 a0, 0\n\t" \
    "v_accvgpr_write_b32 a1, 0\n\t" \
    "v_accvgpr_write_b32 a2, 0\n\t" \
    "v_accvgpr_write_b32 a3, 0\n\t" \
    "v_accvgpr_write_b32 a4, 0\n\t" \
    "v_accvgpr_write_b32 a5, 0\n\t" \
    "v_accvgpr_write_b32 a6, 0\n\t" \
    "v_accvgpr_write_b32 a7, 0\n\t" \
    "v_accvgpr_write_b32 a8, 0\n\t" \
    "v_accvgpr_write_b32 a9, 0\n\t" \
    "v_accvgpr_write_b32 a10, 0\n\t" \
    "v_accvgpr_write_b32 a11, 0\n\t" \
    "v_accvgpr_write_b32 a12, 0\n\t" \
    "v_accvgpr_write_b32 a13, 0\n\t" \
    "v_accvgpr_write_b32 a14, 0\n\t" \
    "v_accvgpr_write_b32 a15, 0\n\t" \
    "v_accvgpr_write_b32 a16, 0\n\t" \
    "v_accvgpr_write_b32 a17, 0\n\t" \
    "v_accvgpr_write_b32 a18, 0\n\t" \
    "v_accvgpr_write_b32 a19, 0\n\t" \
    "v_accvgpr_write_b32 a20, 0\n\t" \
    "v_accvgpr_write_b32 a21, 0\n\t" \
    "v_accvgpr_write_b32 a22, 0\n\t" \
    "v_accvgpr_write_b32 a23, 0\n\t" \
    "v_accvgpr_write_b32 a24, 0\n\t" \
    "v_accvgpr_write_b32 a25, 0\n\t" \
    "v_accvgpr_write_b32 a26, 0\n\t" \
    "v_accvgpr_write_b32 a27, 0\n\t" \
    "v_accvgpr_write_b32 a28, 0\n\t" \
    "v_accvgpr_write_b32 a29, 0\n\t" \
    "v_accvgpr_write_b32 a30, 0\n\t" \
    "v_accvgpr_write_b32 a31, 0\n\t" \
    "v_accvgpr_write_b32 a32, 0\n\t" \
    "v_accvgpr_write_b32 a33, 0\n\t" \
    "v_accvgpr_write_b32 a34, 0\n\t" \
    "v_accvgpr_write_b32 a35, 0\n\t" \
    "v_accvgpr_write_b32 a36, 0\n\t" \
    "v_accvgpr_write_b32 a37, 0\n\t" \
    "v_accvgpr_write_b32 a38, 0\n\t" \
    "v_accvgpr_write_b32 a39, 0\n\t" \
    "v_accvgpr_write_b32 a40, 0\n\t" \
    "v_accvgpr_write_b32 a41, 0\n\t" \
    "v_accvgpr_write_b32 a42, 0\n\t" \
    "v_accvgpr_write_b32 a43, 0\n\t" \
    "v_accvgpr_write_b32 a44, 0\n\t" \
    "v_accvgpr_write_b32 a45, 0\n\t" \
    "v_accvgpr_write_b32 a46, 0\n\t" \
    "v_accvgpr_write_b32 a47, 0\n\t" \
    "v_accvgpr_write_b32 a48, 0\n\t" \
    "v_accvgpr_write_b32 a49, 0\n\t" \
    "v_accvgpr_write_b32 a50, 0\n\t" \
    "v_accvgpr_write_b32 a51, 0\n\t" \
    "v_accvgpr_write_b32 a52, 0\n\t" \
    "v_accvgpr_write_b32 a53, 0\n\t" \
    "v_accvgpr_write_b32 a54, 0\n\t" \
    "v_accvgpr_write_b32 a55, 0\n\t" \
    "v_accvgpr_write_b32 a56, 0\n\t" \
    "v_accvgpr_write_b32 a57, 0\n\t" \
    "v_accvgpr_write_b32 a58, 0\n\t" \
    "v_accvgpr_write_b32 a59, 0\n\t" \
    "v_accvgpr_write_b32 a60, 0\n\t" \
    "v_accvgpr_write_b32 a61, 0\n\t" \
    "v_accvgpr_write_b32 a62, 0\n\t" \
    "v_accvgpr_write_b32 a63, 0\n\t" \
    "s_nop 3\n\t" \
    ""

#define SYMB_GEMM16S_STAGE_OUT \
    "v_accvgpr_read_b32 v128, a0\n\t" \
    "v_accvgpr_read_b32 v129, a1\n\t" \
    "v_accvgpr_read_b32 v130, a2\n\t" \
    "v_accvgpr_read_b32 v131, a3\n\t" \
    "v_cvt_pk_bf16_f32 v132, v128, v129\n\t" \
    "v_cvt_pk_bf16_f32 v133, v130, v131\n\t" \
    "ds_write_b64 %0, v[132:133] offset:0\n\t" \
    "v_accvgpr_read_b32 v134, a4\n\t" \
    "v_accvgpr_read_b32 v135, a5\n\t" \
    "v_accvgpr_read_b32 v136, a6\n\t" \
    "v_accvgpr_read_b32 v137, a7\n\t" \
    "v_cvt_pk_bf16_f32 v138, v134, v135\n\t" \
    "v_cvt_pk_bf16_f32 v139, v136, v137\n\t" \
    "ds_write_b64 %0, v[138:139] offset:32\n\t" \
    "v_accvgpr_read_b32 v140, a8\n\t" \
    "v_accvgpr_read_b32 v141, a9\n\t" \
    "v_accvgpr_read_b32 v142, a10\n\t" \
    "v_accvgpr_read_b32 v143, a11\n\t" \
    "v_cvt_pk_bf16_f32 v144, v140, v141\n\t" \
    "v_cvt_pk_bf16_f32 v145, v142, v143\n\t" \
    "ds_write_b64 %0, v[144:145] offset:64\n\t" \
    "v_accvgpr_read_b32 v146, a12\n\t" \
    "v_accvgpr_read_b32 v147, a13\n\t" \
    "v_accvgpr_read_b32 v148, a14\n\t" \
    "v_accvgpr_read_b32 v149, a15\n\t" \
    "v_cvt_pk_bf16_f32 v150, v146, v147\n\t" \
    "v_cvt_pk_bf16_f32 v151, v148, v149\n\t" \
    "ds_write_b64 %0, v[150:151] offset:96\n\t" \
    "v_accvgpr_read_b32 v152, a16\n\t" \
    "v_accvgpr_read_b32 v153, a17\n\t" \
    "v_accvgpr_read_b32 v154, a18\n\t" \
    "v_accvgpr_read_b32 v155, a19\n\t" \
    "v_cvt_pk_bf16_f32 v156, v152, v153\n\t" \
    "v_cvt_pk_bf16_f32 v157, v154, v155\n\t" \
    "ds_write_b64 %0, v[156:157] offset:4352\n\t" \
    "v_accvgpr_read_b32 v158, a20\n\t" \
    "v_accvgpr_read_b32 v159, a21\n\t" \
    "v_accvgpr_read_b32 v160, a22\n\t" \
    "v_accvgpr_read_b32 v161, a23\n\t" \
    "v_cvt_pk_bf16_f32 v162, v158, v159\n\t" \
    "v_cvt_pk_bf16_f32 v163, v160, v161\n\t" \
    "ds_write_b64 %0, v[162:163] offset:4384\n\t" \
    "v_accvgpr_read_b32 v164, a24\n\t" \
    "v_accvgpr_read_b32 v165, a25\n\t" \
    "v_accvgpr_read_b32 v166, a26\n\t" \
    "v_accvgpr_read_b32 v167, a27\n\t" \
    "v_cvt_pk_bf16_f32 v168, v164, v165\n\t" \
    "v_cvt_pk_bf16_f32 v169, v166, v167\n\t" \
    "ds_write_b64 %0, v[168:169] offset:4416\n\t" \
    "v_accvgpr_read_b32 v170, a28\n\t" \
    "v_accvgpr_read_b32 v171, a29\n\t" \
    "v_accvgpr_read_b32 v172, a30\n\t" \
    "v_accvgpr_read_b32 v173, a31\n\t" \
    "v_cvt_pk_bf16_f32 v174, v170, v171\n\t" \
    "v_cvt_pk_bf16_f32 v175, v172, v173\n\t" \
    "ds_write_b64 %0, v[174:175] offset:4448\n\t" \
    "v_accvgpr_read_b32 v128, a32\n\t" \
    "v_accvgpr_read_b32 v129, a33\n\t" \
    "v_accvgpr_read_b32 v130, a34\n\t" \
    "v_accvgpr_read_b32 v131, a35\n\t" \
    "v_cvt_pk_bf16_f32 v132, v128, v129\n\t" \
    "v_cvt_pk_bf16_f32 v133, v130, v131\n\t" \
    "ds_write_b64 %0, v[132:133] offset:8704\n\t" \
    "v_accvgpr_read_b32 v134, a36\n\t" \
    "v_accvgpr_read_b32 v135, a37\n\t" \
    "v_accvgpr_read_b32 v136, a38\n\t" \
    "v_accvgpr_read_b32 v137, a39\n\t" \
    "v_cvt_pk_bf16_f32 v138, v134, v135\n\t" \
    "v_cvt_pk_bf16_f32 v139, v136, v137\n\t" \
    "ds_write_b64 %0, v[138:139] offset:8736\n\t" \
    "v_accvgpr_read_b32 v140, a40\n\t" \
    "v_accvgpr_read_b32 v141, a41\n\t" \
    "v_accvgpr_read_b32 v142, a42\n\t" \
    "v_accvgpr_read_b32 v143, a43\n\t" \
    "v_cvt_pk_bf16_f32 v144, v140, v141\n\t" \
    "v_cvt_pk_bf16_f32 v145, v142, v143\n\t" \
    "ds_write_b64 %0, v[144:145] offset:8768\n\t" \
    "v_accvgpr_read_b32 v146, a44\n\t" \
    "v_accvgpr_read_b32 v147, a45\n\t" \
    "v_accvgpr_read_b32 v148, a46\n\t" \
    "v_accvgpr_read_b32 v149, a47\n\t" \
    "v_cvt_pk_bf16_f32 v150, v146, v147\n\t" \
    "v_cvt_pk_bf16_f32 v151, v148, v149\n\t" \
    "ds_write_b64 %0, v[150:151] offset:8800\n\t" \
    "v_accvgpr_read_b32 v152, a48\n\t" \
    "v_accvgpr_read_b32 v153, a49\n\t" \
    "v_accvgpr_read_b32 v154, a50\n\t" \
    "v_accvgpr_read_b32 v155, a51\n\t" \
    "v_cvt_pk_bf16_f32 v156, v152, v153\n\t" \
    "v_cvt_pk_bf16_f32 v157, v154, v155\n\t" \
    "ds_write_b64 %0, v[156:157] offset:13056\n\t" \
    "v_accvgpr_read_b32 v158, a52\n\t" \
    "v_accvgpr_read_b32 v159, a53\n\t" \
    "v_accvgpr_read_b32 v160, a54\n\t" \
    "v_accvgpr_read_b32 v161, a55\n\t" \
    "v_cvt_pk_bf16_f32 v162, v158, v159\n\t" \
    "v_cvt_pk_bf16_f32 v163, v160, v161\n\t" \
    "ds_write_b64 %0, v[162:163] offset:13088\n\t" \
    "v_accvgpr_read_b32 v164, a56\n\t" \
    "v_accvgpr_read_b32 v165, a57\n\t" \
    "v_accvgpr_read_b32 v166, a58\n\t" \
    "v_accvgpr_read_b32 v167, a59\n\t" \
    "v_cvt_pk_bf16_f32 v168, v164, v165\n\t" \
    "v_cvt_pk_bf16_f32 v169, v166, v167\n\t" \
    "ds_write_b64 %0, v[168:169] offset:13120\n\t" \
    "v_accvgpr_read_b32 v170, a60\n\t" \
    "v_accvgpr_read_b32 v171, a61\n\t" \
    "v_accvgpr_read_b32 v172, a62\n\t" \
    "v_accvgpr_read_b32 v173, a63\n\t" \
    "v_cvt_pk_bf16_f32 v174, v170, v171\n\t" \
    "v_cvt_pk_bf16_f32 v175, v172, v173\n\t" \
    "ds_write_b64 %0, v[174:175] offset:13152\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    ""

#define SYMB_GEMM16S_STORE_PARTIAL \
    "v_mov_b32 v116, %0\n\t" \
    "global_store_dwordx4 v116, a[0:3], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[4:7], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[8:11], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[12:15], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[16:19], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[20:23], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[24:27], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[28:31], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[32:35], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[36:39], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[40:43], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[44:47], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[48:51], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[52:55], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[56:59], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[60:63], %1 offset:3072\n\t" \
    "s_waitcnt vmcnt(0)\n\t" \
    ""

#define SYMB_GEMM16S_VCLOBBERS "v116", "v117", "v118", "v119", "v120", "v121", "v122", "v123", "v124", "v125", "v126", "v127", "v128", "v129", "v130", "v131", "v132", "v133", "v134", "v135", "v136", "v137", "v138", "v139", "v140", "v141", "v142", "v143", "v144", "v145", "v146", "v147", "v148", "v149", "v150", "v151", "v152", "v153", "v154", "v155", "v156", "v157", "v158", "v159", "v160", "v161", "v162", "v163", "v164", "v165", "v166", "v167", "v168", "v169", "v170", "v171", "v172", "v173", "v174", "v175", "v176", "v177", "v178", "v179", "v180", "v181", "v182", "v183", "v184", "v185", "v186", "v187", "v188", "v189", "v190", "v191"
#define SYMB_GEMM16S_ACLOBBERS "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15", "a16", "a17", "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31", "a32", "a33", "a34", "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46", "a47", "a48", "a49", "a50", "a51", "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61", "a62", "a63"

// ---- 256x128 tile: a wavefront owns 8x4 blocks, block (i, j) in a[4(4i+j) : 4(4i+j)+3].
// Main loop operands: %0-%3 A fragment lane offsets inside an A unit (32-k step 0 first / second
// read, step 1 first / second read); %4-%7 B fragment lane offsets inside a B unit (K-contiguous W:
// as for A in %4-%7; N-contiguous W: one per 16-column block); %8-%15 / %16-%19 global byte offsets
// of this lane's 8 A / 4 B loads per stage; %20,%21 global base of the A / B stage (64-bit SGPR);
// %22 byte stride of B between stages; %23 number of 64-k stages (>= 1); %24 LDS byte address of the
// dynamic segment + this wavefront's first load inside a unit (wave * 8192); %26 the stage to start from (GA, GB point to it); %25 as %24 for B (wave * 4096); the lane offsets of load j are 1024 (j % 4) lower, the bases 4096 lower than that.  LDS: units of
// 32 / 16 KiB, A at unit 0/1/2, B at unit 3 on.  Fixed registers: s80-s99, v116-v223 (fragment sets at
// v128 and v176), a0-a127.
#define SYMB_GEMM16T_LOOP_NT \
    "s_mov_b64 s[80:81], %20\n\t" \
    "s_mov_b64 s[82:83], %21\n\t" \
    "s_sub_u32 s84, %23, 3\n\t" \
    "s_mov_b32 s98, %26\n\t" \
    "s_mov_b32 s99, %26\n\t" \
    "s_sub_u32 s91, %23, 1\n\t" \
    "s_mul_i32 s94, s91, 128\n\t" \
    "s_mul_hi_u32 s95, s91, 128\n\t" \
    "s_sub_u32 s94, 0, s94\n\t" \
    "s_subb_u32 s95, 0, s95\n\t" \
    "s_mul_i32 s96, s91, %22\n\t" \
    "s_mul_hi_u32 s97, s91, %22\n\t" \
    "s_sub_u32 s96, 0, s96\n\t" \
    "s_subb_u32 s97, 0, s97\n\t" \
    "s_mov_b32 s85, 0\n\t" \
    "s_mov_b32 s86, 32768\n\t" \
    "s_mov_b32 s87, 65536\n\t" \
    "s_mov_b32 s88, 98304\n\t" \
    "s_mov_b32 s89, 114688\n\t" \
    "s_mov_b32 s92, 131072\n\t" \
    "s_mov_b32 s93, 147456\n\t" \
    "s_add_u32 s90, s85, %24\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %8, s[80:81] offset:0\n\t" \
    "global_load_lds_dwordx4 %9, s[80:81] offset:1024\n\t" \
    "global_load_lds_dwordx4 %10, s[80:81] offset:2048\n\t" \
    "global_load_lds_dwordx4 %11, s[80:81] offset:3072\n\t" \
    "s_add_u32 s90, s85, %24\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %12, s[80:81] offset:0\n\t" \
    "global_load_lds_dwordx4 %13, s[80:81] offset:1024\n\t" \
    "global_load_lds_dwordx4 %14, s[80:81] offset:2048\n\t" \
    "global_load_lds_dwordx4 %15, s[80:81] offset:3072\n\t" \
    "s_add_u32 s98, s98, 1\n\t" \
    "s_cmp_eq_u32 s98, %23\n\t" \
    "s_cselect_b32 s91, s94, 128\n\t" \
    "s_cselect_b32 s90, s95, 0\n\t" \
    "s_cselect_b32 s98, 0, s98\n\t" \
    "s_add_u32 s80, s80, s91\n\t" \
    "s_addc_u32 s81, s81, s90\n\t" \
    "s_add_u32 s90, s88, %25\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %16, s[82:83] offset:0\n\t" \
    "global_load_lds_dwordx4 %17, s[82:83] offset:1024\n\t" \
    "global_load_lds_dwordx4 %18, s[82:83] offset:2048\n\t" \
    "global_load_lds_dwordx4 %19, s[82:83] offset:3072\n\t" \
    "s_add_u32 s99, s99, 1\n\t" \
    "s_cmp_eq_u32 s99, %23\n\t" \
    "s_cselect_b32 s91, s96, %22\n\t" \
    "s_cselect_b32 s90, s97, 0\n\t" \
    "s_cselect_b32 s99, 0, s99\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, s90\n\t" \
    "s_add_u32 s90, s86, %24\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %8, s[80:81] offset:0\n\t" \
    "global_load_lds_dwordx4 %9, s[80:81] offset:1024\n\t" \
    "global_load_lds_dwordx4 %10, s[80:81] offset:2048\n\t" \
    "global_load_lds_dwordx4 %11, s[80:81] offset:3072\n\t" \
    "s_add_u32 s90, s86, %24\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %12, s[80:81] offset:0\n\t" \
    "global_load_lds_dwordx4 %13, s[80:81] offset:1024\n\t" \
    "global_load_lds_dwordx4 %14, s[80:81] offset:2048\n\t" \
    "global_load_lds_dwordx4 %15, s[80:81] offset:3072\n\t" \
    "s_add_u32 s98, s98, 1\n\t" \
    "s_cmp_eq_u32 s98, %23\n\t" \
    "s_cselect_b32 s91, s94, 128\n\t" \
    "s_cselect_b32 s90, s95, 0\n\t" \
    "s_cselect_b32 s98, 0, s98\n\t" \
    "s_add_u32 s80, s80, s91\n\t" \
    "s_addc_u32 s81, s81, s90\n\t" \
    "s_add_u32 s90, s89, %25\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %16, s[82:83] offset:0\n\t" \
    "global_load_lds_dwordx4 %17, s[82:83] offset:1024\n\t" \
    "global_load_lds_dwordx4 %18, s[82:83] offset:2048\n\t" \
    "global_load_lds_dwordx4 %19, s[82:83] offset:3072\n\t" \
    "s_add_u32 s99, s99, 1\n\t" \
    "s_cmp_eq_u32 s99, %23\n\t" \
    "s_cselect_b32 s91, s96, %22\n\t" \
    "s_cselect_b32 s90, s97, 0\n\t" \
    "s_cselect_b32 s99, 0, s99\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, s90\n\t" \
    "s_add_u32 s90, s87, %24\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %8, s[80:81] offset:0\n\t" \
    "global_load_lds_dwordx4 %9, s[80:81] offset:1024\n\t" \
    "global_load_lds_dwordx4 %10, s[80:81] offset:2048\n\t" \
    "global_load_lds_dwordx4 %11, s[80:81] offset:3072\n\t" \
    "s_add_u32 s90, s87, %24\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %12, s[80:81] offset:0\n\t" \
    "global_load_lds_dwordx4 %13, s[80:81] offset:1024\n\t" \
    "global_load_lds_dwordx4 %14, s[80:81] offset:2048\n\t" \
    "global_load_lds_dwordx4 %15, s[80:81] offset:3072\n\t" \
    "s_add_u32 s98, s98, 1\n\t" \
    "s_cmp_eq_u32 s98, %23\n\t" \
    "s_cselect_b32 s91, s94, 128\n\t" \
    "s_cselect_b32 s90, s95, 0\n\t" \
    "s_cselect_b32 s98, 0, s98\n\t" \
    "s_add_u32 s80, s80, s91\n\t" \
    "s_addc_u32 s81, s81, s90\n\t" \
    "s_add_u32 s90, s92, %25\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %16, s[82:83] offset:0\n\t" \
    "global_load_lds_dwordx4 %17, s[82:83] offset:1024\n\t" \
    "global_load_lds_dwordx4 %18, s[82:83] offset:2048\n\t" \
    "global_load_lds_dwordx4 %19, s[82:83] offset:3072\n\t" \
    "s_add_u32 s99, s99, 1\n\t" \
    "s_cmp_eq_u32 s99, %23\n\t" \
    "s_cselect_b32 s91, s96, %22\n\t" \
    "s_cselect_b32 s90, s97, 0\n\t" \
    "s_cselect_b32 s99, 0, s99\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, s90\n\t" \
    "v_accvgpr_write_b32 a0, 0\n\t" \
    "v_accvgpr_write_b32 a1, 0\n\t" \
    "v_accvgpr_write_b32 a2, 0\n\t" \
    "v_accvgpr_write_b32 a3, 0\n\t" \
    "v_accvgpr_write_b32 a4, 0\n\t" \
    "v_accvgpr_write_b32 a5, 0\n\t" \
    "v_accvgpr_write_b32 a6, 0\n\t" \
    "v_accvgpr_write_b32 a7, 0\n\t" \
    "v_accvgpr_write_b32 a8, 0\n\t" \
    "v_accvgpr_write_b32 a9, 0\n\t" \
    "v_accvgpr_write_b32 a10, 0\n\t" \
    "v_accvgpr_write_b32 a11, 0\n\t" \
    "v_accvgpr_write_b32 a12, 0\n\t" \
    "v_accvgpr_write_b32 a13, 0\n\t" \
    "v_accvgpr_write_b32 a14, 0\n\t" \
    "v_accvgpr_write_b32 a15, 0\n\t" \
    "v_accvgpr_write_b32 a16, 0\n\t" \
    "v_accvgpr_write_b32 a17, 0\n\t" \
    "v_accvgpr_write_b32 a18, 0\n\t" \
    "v_accvgpr_write_b32 a19, 0\n\t" \
    "v_accvgpr_write_b32 a20, 0\n\t" \
    "v_accvgpr_write_b32 a21, 0\n\t" \
    "v_accvgpr_write_b32 a22, 0\n\t" \
    "v_accvgpr_write_b32 a23, 0\n\t" \
    "v_accvgpr_write_b32 a24, 0\n\t" \
    "v_accvgpr_write_b32 a25, 0\n\t" \
    "v_accvgpr_write_b32 a26, 0\n\t" \
    "v_accvgpr_write_b32 a27, 0\n\t" \
    "v_accvgpr_write_b32 a28, 0\n\t" \
    "v_accvgpr_write_b32 a29, 0\n\t" \
    "v_accvgpr_write_b32 a30, 0\n\t" \
    "v_accvgpr_write_b32 a31, 0\n\t" \
    "v_accvgpr_write_b32 a32, 0\n\t" \
    "v_accvgpr_write_b32 a33, 0\n\t" \
    "v_accvgpr_write_b32 a34, 0\n\t" \
    "v_accvgpr_write_b32 a35, 0\n\t" \
    "v_accvgpr_write_b32 a36, 0\n\t" \
    "v_accvgpr_write_b32 a37, 0\n\t" \
    "v_accvgpr_write_b32 a38, 0\n\t" \
    "v_accvgpr_write_b32 a39, 0\n\t" \
    "v_accvgpr_write_b32 a40, 0\n\t" \
    "v_accvgpr_write_b32 a41, 0\n\t" \
    "v_accvgpr_write_b32 a42, 0\n\t" \
    "v_accvgpr_write_b32 a43, 0\n\t" \
    "v_accvgpr_write_b32 a44, 0\n\t" \
    "v_accvgpr_write_b32 a45, 0\n\t" \
    "v_accvgpr_write_b32 a46, 0\n\t" \
    "v_accvgpr_write_b32 a47, 0\n\t" \
    "v_accvgpr_write_b32 a48, 0\n\t" \
    "v_accvgpr_write_b32 a49, 0\n\t" \
    "v_accvgpr_write_b32 a50, 0\n\t" \
    "v_accvgpr_write_b32 a51, 0\n\t" \
    "v_accvgpr_write_b32 a52, 0\n\t" \
    "v_accvgpr_write_b32 a53, 0\n\t" \
    "v_accvgpr_write_b32 a54, 0\n\t" \
    "v_accvgpr_write_b32 a55, 0\n\t" \
    "v_accvgpr_write_b32 a56, 0\n\t" \
    "v_accvgpr_write_b32 a57, 0\n\t" \
    "v_accvgpr_write_b32 a58, 0\n\t" \
    "v_accvgpr_write_b32 a59, 0\n\t" \
    "v_accvgpr_write_b32 a60, 0\n\t" \
    "v_accvgpr_write_b32 a61, 0\n\t" \
    "v_accvgpr_write_b32 a62, 0\n\t" \
    "v_accvgpr_write_b32 a63, 0\n\t" \
    "v_accvgpr_write_b32 a64, 0\n\t" \
    "v_accvgpr_write_b32 a65, 0\n\t" \
    "v_accvgpr_write_b32 a66, 0\n\t" \
    "v_accvgpr_write_b32 a67, 0\n\t" \
    "v_accvgpr_write_b32 a68, 0\n\t" \
    "v_accvgpr_write_b32 a69, 0\n\t" \
    "v_accvgpr_write_b32 a70, 0\n\t" \
    "v_accvgpr_write_b32 a71, 0\n\t" \
    "v_accvgpr_write_b32 a72, 0\n\t" \
    "v_accvgpr_write_b32 a73, 0\n\t" \
    "v_accvgpr_write_b32 a74, 0\n\t" \
    "v_accvgpr_write_b32 a75, 0\n\t" \
    "v_accvgpr_write_b32 a76, 0\n\t" \
    "v_accvgpr_write_b32 a77, 0\n\t" \
    "v_accvgpr_write_b32 a78, 0\n\t" \
    "v_accvgpr_write_b32 a79, 0\n\t" \
    "v_accvgpr_write_b32 a80, 0\n\t" \
    "v_accvgpr_write_b32 a81, 0\n\t" \
    "v_accvgpr_write_b32 a82, 0\n\t" \
    "v_accvgpr_write_b32 a83, 0\n\t" \
    "v_accvgpr_write_b32 a84, 0\n\t" \
    "v_accvgpr_write_b32 a85, 0\n\t" \
    "v_accvgpr_write_b32 a86, 0\n\t" \
    "v_accvgpr_write_b32 a87, 0\n\t" \
    "v_accvgpr_write_b32 a88, 0\n\t" \
    "v_accvgpr_write_b32 a89, 0\n\t" \
    "v_accvgpr_write_b32 a90, 0\n\t" \
    "v_accvgpr_write_b32 a91, 0\n\t" \
    "v_accvgpr_write_b32 a92, 0\n\t" \
    "v_accvgpr_write_b32 a93, 0\n\t" \
    "v_accvgpr_write_b32 a94, 0\n\t" \
    "v_accvgpr_write_b32 a95, 0\n\t" \
    "v_accvgpr_write_b32 a96, 0\n\t" \
    "v_accvgpr_write_b32 a97, 0\n\t" \
    "v_accvgpr_write_b32 a98, 0\n\t" \
    "v_accvgpr_write_b32 a99, 0\n\t" \
    "v_accvgpr_write_b32 a100, 0\n\t" \
    "v_accvgpr_write_b32 a101, 0\n\t" \
    "v_accvgpr_write_b32 a102, 0\n\t" \
    "v_accvgpr_write_b32 a103, 0\n\t" \
    "v_accvgpr_write_b32 a104, 0\n\t" \
    "v_accvgpr_write_b32 a105, 0\n\t" \
    "v_accvgpr_write_b32 a106, 0\n\t" \
    "v_accvgpr_write_b32 a107, 0\n\t" \
    "v_accvgpr_write_b32 a108, 0\n\t" \
    "v_accvgpr_write_b32 a109, 0\n\t" \
    "v_accvgpr_write_b32 a110, 0\n\t" \
    "v_accvgpr_write_b32 a111, 0\n\t" \
    "v_accvgpr_write_b32 a112, 0\n\t" \
    "v_accvgpr_write_b32 a113, 0\n\t" \
    "v_accvgpr_write_b32 a114, 0\n\t" \
    "v_accvgpr_write_b32 a115, 0\n\t" \
    "v_accvgpr_write_b32 a116, 0\n\t" \
    "v_accvgpr_write_b32 a117, 0\n\t" \
    "v_accvgpr_write_b32 a118, 0\n\t" \
    "v_accvgpr_write_b32 a119, 0\n\t" \
    "v_accvgpr_write_b32 a120, 0\n\t" \
    "v_accvgpr_write_b32 a121, 0\n\t" \
    "v_accvgpr_write_b32 a122, 0\n\t" \
    "v_accvgpr_write_b32 a123, 0\n\t" \
    "v_accvgpr_write_b32 a124, 0\n\t" \
    "v_accvgpr_write_b32 a125, 0\n\t" \
    "v_accvgpr_write_b32 a126, 0\n\t" \
    "v_accvgpr_write_b32 a127, 0\n\t" \
    "s_nop 3\n\t" \
    "s_waitcnt vmcnt(24)\n\t" \
    "s_barrier\n\t" \
    "v_add_u32 v118, s88, %4\n\t" \
    "ds_read_b64 v[160:161], v118 offset:0\n\t" \
    "ds_read_b64 v[164:165], v118 offset:2048\n\t" \
    "ds_read_b64 v[168:169], v118 offset:4096\n\t" \
    "ds_read_b64 v[172:173], v118 offset:6144\n\t" \
    "v_add_u32 v119, s88, %5\n\t" \
    "ds_read_b64 v[162:163], v119 offset:0\n\t" \
    "ds_read_b64 v[166:167], v119 offset:2048\n\t" \
    "ds_read_b64 v[170:171], v119 offset:4096\n\t" \
    "ds_read_b64 v[174:175], v119 offset:6144\n\t" \
    "v_add_u32 v116, s85, %0\n\t" \
    "v_add_u32 v117, s85, %1\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "ds_read_b64 v[144:145], v116 offset:8192\n\t" \
    "ds_read_b64 v[146:147], v117 offset:8192\n\t" \
    "ds_read_b64 v[148:149], v116 offset:10240\n\t" \
    "ds_read_b64 v[150:151], v117 offset:10240\n\t" \
    "ds_read_b64 v[152:153], v116 offset:12288\n\t" \
    "ds_read_b64 v[154:155], v117 offset:12288\n\t" \
    "ds_read_b64 v[156:157], v116 offset:14336\n\t" \
    "ds_read_b64 v[158:159], v117 offset:14336\n\t" \
    "s_cmp_lt_u32 %23, 4\n\t" \
    "s_cbranch_scc1 2f\n\t" \
    "1:\n\t" \
    "s_waitcnt lgkmcnt(14)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v118, s88, %6\n\t" \
    "ds_read_b64 v[208:209], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "ds_read_b64 v[212:213], v118 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "ds_read_b64 v[216:217], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "ds_read_b64 v[220:221], v118 offset:6144\n\t" \
    "s_add_u32 s90, s93, %25\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[160:163], v[132:135], a[16:19]\n\t" \
    "global_load_lds_dwordx4 %16, s[82:83] offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[164:167], v[132:135], a[20:23]\n\t" \
    "v_add_u32 v119, s88, %7\n\t" \
    "ds_read_b64 v[210:211], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[168:171], v[132:135], a[24:27]\n\t" \
    "ds_read_b64 v[214:215], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[172:175], v[132:135], a[28:31]\n\t" \
    "ds_read_b64 v[218:219], v119 offset:4096\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[136:139], a[32:35]\n\t" \
    "ds_read_b64 v[222:223], v119 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[136:139], a[36:39]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[176:177], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[136:139], a[40:43]\n\t" \
    "ds_read_b64 v[178:179], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[136:139], a[44:47]\n\t" \
    "ds_read_b64 v[180:181], v116 offset:2048\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[160:163], v[140:143], a[48:51]\n\t" \
    "global_load_lds_dwordx4 %17, s[82:83] offset:1024\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[164:167], v[140:143], a[52:55]\n\t" \
    "ds_read_b64 v[182:183], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[168:171], v[140:143], a[56:59]\n\t" \
    "ds_read_b64 v[184:185], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[172:175], v[140:143], a[60:63]\n\t" \
    "ds_read_b64 v[186:187], v117 offset:4096\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[144:147], a[64:67]\n\t" \
    "ds_read_b64 v[188:189], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[144:147], a[68:71]\n\t" \
    "ds_read_b64 v[190:191], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[144:147], a[72:75]\n\t" \
    "ds_read_b64 v[192:193], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[144:147], a[76:79]\n\t" \
    "ds_read_b64 v[194:195], v117 offset:8192\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[160:163], v[148:151], a[80:83]\n\t" \
    "global_load_lds_dwordx4 %18, s[82:83] offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[164:167], v[148:151], a[84:87]\n\t" \
    "ds_read_b64 v[196:197], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[168:171], v[148:151], a[88:91]\n\t" \
    "ds_read_b64 v[198:199], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[172:175], v[148:151], a[92:95]\n\t" \
    "ds_read_b64 v[200:201], v116 offset:12288\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[152:155], a[96:99]\n\t" \
    "ds_read_b64 v[202:203], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[152:155], a[100:103]\n\t" \
    "ds_read_b64 v[204:205], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[152:155], a[104:107]\n\t" \
    "ds_read_b64 v[206:207], v117 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[152:155], a[108:111]\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[160:163], v[156:159], a[112:115]\n\t" \
    "global_load_lds_dwordx4 %19, s[82:83] offset:3072\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[164:167], v[156:159], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[168:171], v[156:159], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[172:175], v[156:159], a[124:127]\n\t" \
    "s_add_u32 s99, s99, 1\n\t" \
    "s_cmp_eq_u32 s99, %23\n\t" \
    "s_cselect_b32 s91, s96, %22\n\t" \
    "s_cselect_b32 s90, s97, 0\n\t" \
    "s_cselect_b32 s99, 0, s99\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, s90\n\t" \
    "s_waitcnt vmcnt(16) lgkmcnt(0)\n\t" \
    "s_barrier\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[208:211], v[176:179], a[0:3]\n\t" \
    "v_add_u32 v118, s89, %4\n\t" \
    "ds_read_b64 v[160:161], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[212:215], v[176:179], a[4:7]\n\t" \
    "ds_read_b64 v[164:165], v118 offset:2048\n\t" \
    "s_add_u32 s90, s85, %24\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[216:219], v[176:179], a[8:11]\n\t" \
    "global_load_lds_dwordx4 %8, s[80:81] offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[220:223], v[176:179], a[12:15]\n\t" \
    "ds_read_b64 v[168:169], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[208:211], v[180:183], a[16:19]\n\t" \
    "ds_read_b64 v[172:173], v118 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[212:215], v[180:183], a[20:23]\n\t" \
    "v_add_u32 v119, s89, %5\n\t" \
    "ds_read_b64 v[162:163], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[216:219], v[180:183], a[24:27]\n\t" \
    "global_load_lds_dwordx4 %9, s[80:81] offset:1024\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[220:223], v[180:183], a[28:31]\n\t" \
    "ds_read_b64 v[166:167], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[208:211], v[184:187], a[32:35]\n\t" \
    "ds_read_b64 v[170:171], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[212:215], v[184:187], a[36:39]\n\t" \
    "ds_read_b64 v[174:175], v119 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[216:219], v[184:187], a[40:43]\n\t" \
    "global_load_lds_dwordx4 %10, s[80:81] offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[220:223], v[184:187], a[44:47]\n\t" \
    "v_add_u32 v116, s86, %0\n\t" \
    "v_add_u32 v117, s86, %1\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[208:211], v[188:191], a[48:51]\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[212:215], v[188:191], a[52:55]\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[216:219], v[188:191], a[56:59]\n\t" \
    "global_load_lds_dwordx4 %11, s[80:81] offset:3072\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[220:223], v[188:191], a[60:63]\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[208:211], v[192:195], a[64:67]\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[212:215], v[192:195], a[68:71]\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "s_add_u32 s90, s85, %24\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[216:219], v[192:195], a[72:75]\n\t" \
    "global_load_lds_dwordx4 %12, s[80:81] offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[220:223], v[192:195], a[76:79]\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[208:211], v[196:199], a[80:83]\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[212:215], v[196:199], a[84:87]\n\t" \
    "ds_read_b64 v[144:145], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[216:219], v[196:199], a[88:91]\n\t" \
    "global_load_lds_dwordx4 %13, s[80:81] offset:1024\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[220:223], v[196:199], a[92:95]\n\t" \
    "ds_read_b64 v[146:147], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[208:211], v[200:203], a[96:99]\n\t" \
    "ds_read_b64 v[148:149], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[212:215], v[200:203], a[100:103]\n\t" \
    "ds_read_b64 v[150:151], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[216:219], v[200:203], a[104:107]\n\t" \
    "global_load_lds_dwordx4 %14, s[80:81] offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[220:223], v[200:203], a[108:111]\n\t" \
    "ds_read_b64 v[152:153], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[208:211], v[204:207], a[112:115]\n\t" \
    "ds_read_b64 v[154:155], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[212:215], v[204:207], a[116:119]\n\t" \
    "ds_read_b64 v[156:157], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[216:219], v[204:207], a[120:123]\n\t" \
    "global_load_lds_dwordx4 %15, s[80:81] offset:3072\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[220:223], v[204:207], a[124:127]\n\t" \
    "ds_read_b64 v[158:159], v117 offset:14336\n\t" \
    "s_add_u32 s98, s98, 1\n\t" \
    "s_cmp_eq_u32 s98, %23\n\t" \
    "s_cselect_b32 s91, s94, 128\n\t" \
    "s_cselect_b32 s90, s95, 0\n\t" \
    "s_cselect_b32 s98, 0, s98\n\t" \
    "s_add_u32 s80, s80, s91\n\t" \
    "s_addc_u32 s81, s81, s90\n\t" \
    "s_mov_b32 s90, s85\n\t" \
    "s_mov_b32 s85, s86\n\t" \
    "s_mov_b32 s86, s87\n\t" \
    "s_mov_b32 s87, s90\n\t" \
    "s_mov_b32 s90, s88\n\t" \
    "s_mov_b32 s88, s89\n\t" \
    "s_mov_b32 s89, s92\n\t" \
    "s_mov_b32 s92, s93\n\t" \
    "s_mov_b32 s93, s90\n\t" \
    "s_sub_u32 s84, s84, 1\n\t" \
    "s_cmp_lg_u32 s84, 0\n\t" \
    "s_cbranch_scc1 1b\n\t" \
    "2:\n\t" \
    "s_cmp_lt_u32 %23, 3\n\t" \
    "s_cbranch_scc1 3f\n\t" \
    "s_waitcnt lgkmcnt(14)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v118, s88, %6\n\t" \
    "ds_read_b64 v[208:209], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "ds_read_b64 v[212:213], v118 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "ds_read_b64 v[216:217], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "ds_read_b64 v[220:221], v118 offset:6144\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[160:163], v[132:135], a[16:19]\n\t" \
    "v_add_u32 v119, s88, %7\n\t" \
    "ds_read_b64 v[210:211], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[164:167], v[132:135], a[20:23]\n\t" \
    "ds_read_b64 v[214:215], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[168:171], v[132:135], a[24:27]\n\t" \
    "ds_read_b64 v[218:219], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[172:175], v[132:135], a[28:31]\n\t" \
    "ds_read_b64 v[222:223], v119 offset:6144\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[136:139], a[32:35]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[176:177], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[136:139], a[36:39]\n\t" \
    "ds_read_b64 v[178:179], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[136:139], a[40:43]\n\t" \
    "ds_read_b64 v[180:181], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[136:139], a[44:47]\n\t" \
    "ds_read_b64 v[182:183], v117 offset:2048\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[160:163], v[140:143], a[48:51]\n\t" \
    "ds_read_b64 v[184:185], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[164:167], v[140:143], a[52:55]\n\t" \
    "ds_read_b64 v[186:187], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[168:171], v[140:143], a[56:59]\n\t" \
    "ds_read_b64 v[188:189], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[172:175], v[140:143], a[60:63]\n\t" \
    "ds_read_b64 v[190:191], v117 offset:6144\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[144:147], a[64:67]\n\t" \
    "ds_read_b64 v[192:193], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[144:147], a[68:71]\n\t" \
    "ds_read_b64 v[194:195], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[144:147], a[72:75]\n\t" \
    "ds_read_b64 v[196:197], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[144:147], a[76:79]\n\t" \
    "ds_read_b64 v[198:199], v117 offset:10240\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[160:163], v[148:151], a[80:83]\n\t" \
    "ds_read_b64 v[200:201], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[164:167], v[148:151], a[84:87]\n\t" \
    "ds_read_b64 v[202:203], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[168:171], v[148:151], a[88:91]\n\t" \
    "ds_read_b64 v[204:205], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[172:175], v[148:151], a[92:95]\n\t" \
    "ds_read_b64 v[206:207], v117 offset:14336\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[152:155], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[152:155], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[152:155], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[152:155], a[108:111]\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[160:163], v[156:159], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[164:167], v[156:159], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[168:171], v[156:159], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[172:175], v[156:159], a[124:127]\n\t" \
    "s_waitcnt vmcnt(12) lgkmcnt(0)\n\t" \
    "s_barrier\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[208:211], v[176:179], a[0:3]\n\t" \
    "v_add_u32 v118, s89, %4\n\t" \
    "ds_read_b64 v[160:161], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[212:215], v[176:179], a[4:7]\n\t" \
    "ds_read_b64 v[164:165], v118 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[216:219], v[176:179], a[8:11]\n\t" \
    "ds_read_b64 v[168:169], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[220:223], v[176:179], a[12:15]\n\t" \
    "ds_read_b64 v[172:173], v118 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[208:211], v[180:183], a[16:19]\n\t" \
    "v_add_u32 v119, s89, %5\n\t" \
    "ds_read_b64 v[162:163], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[212:215], v[180:183], a[20:23]\n\t" \
    "ds_read_b64 v[166:167], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[216:219], v[180:183], a[24:27]\n\t" \
    "ds_read_b64 v[170:171], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[220:223], v[180:183], a[28:31]\n\t" \
    "ds_read_b64 v[174:175], v119 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[208:211], v[184:187], a[32:35]\n\t" \
    "v_add_u32 v116, s86, %0\n\t" \
    "v_add_u32 v117, s86, %1\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[212:215], v[184:187], a[36:39]\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[216:219], v[184:187], a[40:43]\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[220:223], v[184:187], a[44:47]\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[208:211], v[188:191], a[48:51]\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[212:215], v[188:191], a[52:55]\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[216:219], v[188:191], a[56:59]\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[220:223], v[188:191], a[60:63]\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[208:211], v[192:195], a[64:67]\n\t" \
    "ds_read_b64 v[144:145], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[212:215], v[192:195], a[68:71]\n\t" \
    "ds_read_b64 v[146:147], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[216:219], v[192:195], a[72:75]\n\t" \
    "ds_read_b64 v[148:149], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[220:223], v[192:195], a[76:79]\n\t" \
    "ds_read_b64 v[150:151], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[208:211], v[196:199], a[80:83]\n\t" \
    "ds_read_b64 v[152:153], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[212:215], v[196:199], a[84:87]\n\t" \
    "ds_read_b64 v[154:155], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[216:219], v[196:199], a[88:91]\n\t" \
    "ds_read_b64 v[156:157], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[220:223], v[196:199], a[92:95]\n\t" \
    "ds_read_b64 v[158:159], v117 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[208:211], v[200:203], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[212:215], v[200:203], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[216:219], v[200:203], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[220:223], v[200:203], a[108:111]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[208:211], v[204:207], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[212:215], v[204:207], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[216:219], v[204:207], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[220:223], v[204:207], a[124:127]\n\t" \
    "s_mov_b32 s90, s85\n\t" \
    "s_mov_b32 s85, s86\n\t" \
    "s_mov_b32 s86, s87\n\t" \
    "s_mov_b32 s87, s90\n\t" \
    "s_mov_b32 s90, s88\n\t" \
    "s_mov_b32 s88, s89\n\t" \
    "s_mov_b32 s89, s92\n\t" \
    "s_mov_b32 s92, s93\n\t" \
    "s_mov_b32 s93, s90\n\t" \
    "3:\n\t" \
    "s_cmp_lt_u32 %23, 2\n\t" \
    "s_cbranch_scc1 4f\n\t" \
    "s_waitcnt lgkmcnt(14)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v118, s88, %6\n\t" \
    "ds_read_b64 v[208:209], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "ds_read_b64 v[212:213], v118 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "ds_read_b64 v[216:217], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "ds_read_b64 v[220:221], v118 offset:6144\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[160:163], v[132:135], a[16:19]\n\t" \
    "v_add_u32 v119, s88, %7\n\t" \
    "ds_read_b64 v[210:211], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[164:167], v[132:135], a[20:23]\n\t" \
    "ds_read_b64 v[214:215], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[168:171], v[132:135], a[24:27]\n\t" \
    "ds_read_b64 v[218:219], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[172:175], v[132:135], a[28:31]\n\t" \
    "ds_read_b64 v[222:223], v119 offset:6144\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[136:139], a[32:35]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[176:177], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[136:139], a[36:39]\n\t" \
    "ds_read_b64 v[178:179], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[136:139], a[40:43]\n\t" \
    "ds_read_b64 v[180:181], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[136:139], a[44:47]\n\t" \
    "ds_read_b64 v[182:183], v117 offset:2048\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[160:163], v[140:143], a[48:51]\n\t" \
    "ds_read_b64 v[184:185], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[164:167], v[140:143], a[52:55]\n\t" \
    "ds_read_b64 v[186:187], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[168:171], v[140:143], a[56:59]\n\t" \
    "ds_read_b64 v[188:189], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[172:175], v[140:143], a[60:63]\n\t" \
    "ds_read_b64 v[190:191], v117 offset:6144\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[144:147], a[64:67]\n\t" \
    "ds_read_b64 v[192:193], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[144:147], a[68:71]\n\t" \
    "ds_read_b64 v[194:195], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[144:147], a[72:75]\n\t" \
    "ds_read_b64 v[196:197], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[144:147], a[76:79]\n\t" \
    "ds_read_b64 v[198:199], v117 offset:10240\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[160:163], v[148:151], a[80:83]\n\t" \
    "ds_read_b64 v[200:201], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[164:167], v[148:151], a[84:87]\n\t" \
    "ds_read_b64 v[202:203], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[168:171], v[148:151], a[88:91]\n\t" \
    "ds_read_b64 v[204:205], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[172:175], v[148:151], a[92:95]\n\t" \
    "ds_read_b64 v[206:207], v117 offset:14336\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[152:155], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[152:155], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[152:155], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[152:155], a[108:111]\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[160:163], v[156:159], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[164:167], v[156:159], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[168:171], v[156:159], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[172:175], v[156:159], a[124:127]\n\t" \
    "s_waitcnt vmcnt(0) lgkmcnt(0)\n\t" \
    "s_barrier\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[208:211], v[176:179], a[0:3]\n\t" \
    "v_add_u32 v118, s89, %4\n\t" \
    "ds_read_b64 v[160:161], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[212:215], v[176:179], a[4:7]\n\t" \
    "ds_read_b64 v[164:165], v118 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[216:219], v[176:179], a[8:11]\n\t" \
    "ds_read_b64 v[168:169], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[220:223], v[176:179], a[12:15]\n\t" \
    "ds_read_b64 v[172:173], v118 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[208:211], v[180:183], a[16:19]\n\t" \
    "v_add_u32 v119, s89, %5\n\t" \
    "ds_read_b64 v[162:163], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[212:215], v[180:183], a[20:23]\n\t" \
    "ds_read_b64 v[166:167], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[216:219], v[180:183], a[24:27]\n\t" \
    "ds_read_b64 v[170:171], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[220:223], v[180:183], a[28:31]\n\t" \
    "ds_read_b64 v[174:175], v119 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[208:211], v[184:187], a[32:35]\n\t" \
    "v_add_u32 v116, s86, %0\n\t" \
    "v_add_u32 v117, s86, %1\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[212:215], v[184:187], a[36:39]\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[216:219], v[184:187], a[40:43]\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[220:223], v[184:187], a[44:47]\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[208:211], v[188:191], a[48:51]\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[212:215], v[188:191], a[52:55]\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[216:219], v[188:191], a[56:59]\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[220:223], v[188:191], a[60:63]\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[208:211], v[192:195], a[64:67]\n\t" \
    "ds_read_b64 v[144:145], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[212:215], v[192:195], a[68:71]\n\t" \
    "ds_read_b64 v[146:147], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[216:219], v[192:195], a[72:75]\n\t" \
    "ds_read_b64 v[148:149], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[220:223], v[192:195], a[76:79]\n\t" \
    "ds_read_b64 v[150:151], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[208:211], v[196:199], a[80:83]\n\t" \
    "ds_read_b64 v[152:153], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[212:215], v[196:199], a[84:87]\n\t" \
    "ds_read_b64 v[154:155], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[216:219], v[196:199], a[88:91]\n\t" \
    "ds_read_b64 v[156:157], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[220:223], v[196:199], a[92:95]\n\t" \
    "ds_read_b64 v[158:159], v117 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[208:211], v[200:203], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[212:215], v[200:203], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[216:219], v[200:203], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[220:223], v[200:203], a[108:111]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[208:211], v[204:207], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[212:215], v[204:207], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[216:219], v[204:207], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[220:223], v[204:207], a[124:127]\n\t" \
    "s_mov_b32 s90, s85\n\t" \
    "s_mov_b32 s85, s86\n\t" \
    "s_mov_b32 s86, s87\n\t" \
    "s_mov_b32 s87, s90\n\t" \
    "s_mov_b32 s90, s88\n\t" \
    "s_mov_b32 s88, s89\n\t" \
    "s_mov_b32 s89, s92\n\t" \
    "s_mov_b32 s92, s93\n\t" \
    "s_mov_b32 s93, s90\n\t" \
    "4:\n\t" \
    "s_waitcnt lgkmcnt(14)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v118, s88, %6\n\t" \
    "ds_read_b64 v[208:209], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "ds_read_b64 v[212:213], v118 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "ds_read_b64 v[216:217], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "ds_read_b64 v[220:221], v118 offset:6144\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[160:163], v[132:135], a[16:19]\n\t" \
    "v_add_u32 v119, s88, %7\n\t" \
    "ds_read_b64 v[210:211], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[164:167], v[132:135], a[20:23]\n\t" \
    "ds_read_b64 v[214:215], v119 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[168:171], v[132:135], a[24:27]\n\t" \
    "ds_read_b64 v[218:219], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[172:175], v[132:135], a[28:31]\n\t" \
    "ds_read_b64 v[222:223], v119 offset:6144\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[136:139], a[32:35]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[176:177], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[136:139], a[36:39]\n\t" \
    "ds_read_b64 v[178:179], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[136:139], a[40:43]\n\t" \
    "ds_read_b64 v[180:181], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[136:139], a[44:47]\n\t" \
    "ds_read_b64 v[182:183], v117 offset:2048\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[160:163], v[140:143], a[48:51]\n\t" \
    "ds_read_b64 v[184:185], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[164:167], v[140:143], a[52:55]\n\t" \
    "ds_read_b64 v[186:187], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[168:171], v[140:143], a[56:59]\n\t" \
    "ds_read_b64 v[188:189], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[172:175], v[140:143], a[60:63]\n\t" \
    "ds_read_b64 v[190:191], v117 offset:6144\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[144:147], a[64:67]\n\t" \
    "ds_read_b64 v[192:193], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[144:147], a[68:71]\n\t" \
    "ds_read_b64 v[194:195], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[144:147], a[72:75]\n\t" \
    "ds_read_b64 v[196:197], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[144:147], a[76:79]\n\t" \
    "ds_read_b64 v[198:199], v117 offset:10240\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[160:163], v[148:151], a[80:83]\n\t" \
    "ds_read_b64 v[200:201], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[164:167], v[148:151], a[84:87]\n\t" \
    "ds_read_b64 v[202:203], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[168:171], v[148:151], a[88:91]\n\t" \
    "ds_read_b64 v[204:205], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[172:175], v[148:151], a[92:95]\n\t" \
    "ds_read_b64 v[206:207], v117 offset:14336\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[152:155], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[152:155], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[152:155], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[152:155], a[108:111]\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[160:163], v[156:159], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[164:167], v[156:159], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[168:171], v[156:159], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[172:175], v[156:159], a[124:127]\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[208:211], v[176:179], a[0:3]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[212:215], v[176:179], a[4:7]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[216:219], v[176:179], a[8:11]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[220:223], v[176:179], a[12:15]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[208:211], v[180:183], a[16:19]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[212:215], v[180:183], a[20:23]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[216:219], v[180:183], a[24:27]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[220:223], v[180:183], a[28:31]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[208:211], v[184:187], a[32:35]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[212:215], v[184:187], a[36:39]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[216:219], v[184:187], a[40:43]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[220:223], v[184:187], a[44:47]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[208:211], v[188:191], a[48:51]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[212:215], v[188:191], a[52:55]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[216:219], v[188:191], a[56:59]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[220:223], v[188:191], a[60:63]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[208:211], v[192:195], a[64:67]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[212:215], v[192:195], a[68:71]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[216:219], v[192:195], a[72:75]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[220:223], v[192:195], a[76:79]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[208:211], v[196:199], a[80:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[212:215], v[196:199], a[84:87]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[216:219], v[196:199], a[88:91]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[220:223], v[196:199], a[92:95]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[208:211], v[200:203], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[212:215], v[200:203], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[216:219], v[200:203], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[220:223], v[200:203], a[108:111]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[208:211], v[204:207], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[212:215], v[204:207], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[216:219], v[204:207], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[220:223], v[204:207], a[124:127]\n\t" \
    "s_waitcnt vmcnt(0)\n\t" \
    "s_nop 15\n\t" \
    "s_nop 7\n\t" \
    ""

#define SYMB_GEMM16T_LOOP_NN \
    "s_mov_b64 s[80:81], %20\n\t" \
    "s_mov_b64 s[82:83], %21\n\t" \
    "s_sub_u32 s84, %23, 3\n\t" \
    "s_mov_b32 s98, %26\n\t" \
    "s_mov_b32 s99, %26\n\t" \
    "s_sub_u32 s91, %23, 1\n\t" \
    "s_mul_i32 s94, s91, 128\n\t" \
    "s_mul_hi_u32 s95, s91, 128\n\t" \
    "s_sub_u32 s94, 0, s94\n\t" \
    "s_subb_u32 s95, 0, s95\n\t" \
    "s_mul_i32 s96, s91, %22\n\t" \
    "s_mul_hi_u32 s97, s91, %22\n\t" \
    "s_sub_u32 s96, 0, s96\n\t" \
    "s_subb_u32 s97, 0, s97\n\t" \
    "s_mov_b32 s85, 0\n\t" \
    "s_mov_b32 s86, 32768\n\t" \
    "s_mov_b32 s87, 65536\n\t" \
    "s_mov_b32 s88, 98304\n\t" \
    "s_mov_b32 s89, 114688\n\t" \
    "s_mov_b32 s92, 131072\n\t" \
    "s_mov_b32 s93, 147456\n\t" \
    "s_add_u32 s90, s85, %24\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %8, s[80:81] offset:0\n\t" \
    "global_load_lds_dwordx4 %9, s[80:81] offset:1024\n\t" \
    "global_load_lds_dwordx4 %10, s[80:81] offset:2048\n\t" \
    "global_load_lds_dwordx4 %11, s[80:81] offset:3072\n\t" \
    "s_add_u32 s90, s85, %24\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %12, s[80:81] offset:0\n\t" \
    "global_load_lds_dwordx4 %13, s[80:81] offset:1024\n\t" \
    "global_load_lds_dwordx4 %14, s[80:81] offset:2048\n\t" \
    "global_load_lds_dwordx4 %15, s[80:81] offset:3072\n\t" \
    "s_add_u32 s98, s98, 1\n\t" \
    "s_cmp_eq_u32 s98, %23\n\t" \
    "s_cselect_b32 s91, s94, 128\n\t" \
    "s_cselect_b32 s90, s95, 0\n\t" \
    "s_cselect_b32 s98, 0, s98\n\t" \
    "s_add_u32 s80, s80, s91\n\t" \
    "s_addc_u32 s81, s81, s90\n\t" \
    "s_add_u32 s90, s88, %25\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %16, s[82:83] offset:0\n\t" \
    "global_load_lds_dwordx4 %17, s[82:83] offset:1024\n\t" \
    "global_load_lds_dwordx4 %18, s[82:83] offset:2048\n\t" \
    "global_load_lds_dwordx4 %19, s[82:83] offset:3072\n\t" \
    "s_add_u32 s99, s99, 1\n\t" \
    "s_cmp_eq_u32 s99, %23\n\t" \
    "s_cselect_b32 s91, s96, %22\n\t" \
    "s_cselect_b32 s90, s97, 0\n\t" \
    "s_cselect_b32 s99, 0, s99\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, s90\n\t" \
    "s_add_u32 s90, s86, %24\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %8, s[80:81] offset:0\n\t" \
    "global_load_lds_dwordx4 %9, s[80:81] offset:1024\n\t" \
    "global_load_lds_dwordx4 %10, s[80:81] offset:2048\n\t" \
    "global_load_lds_dwordx4 %11, s[80:81] offset:3072\n\t" \
    "s_add_u32 s90, s86, %24\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %12, s[80:81] offset:0\n\t" \
    "global_load_lds_dwordx4 %13, s[80:81] offset:1024\n\t" \
    "global_load_lds_dwordx4 %14, s[80:81] offset:2048\n\t" \
    "global_load_lds_dwordx4 %15, s[80:81] offset:3072\n\t" \
    "s_add_u32 s98, s98, 1\n\t" \
    "s_cmp_eq_u32 s98, %23\n\t" \
    "s_cselect_b32 s91, s94, 128\n\t" \
    "s_cselect_b32 s90, s95, 0\n\t" \
    "s_cselect_b32 s98, 0, s98\n\t" \
    "s_add_u32 s80, s80, s91\n\t" \
    "s_addc_u32 s81, s81, s90\n\t" \
    "s_add_u32 s90, s89, %25\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %16, s[82:83] offset:0\n\t" \
    "global_load_lds_dwordx4 %17, s[82:83] offset:1024\n\t" \
    "global_load_lds_dwordx4 %18, s[82:83] offset:2048\n\t" \
    "global_load_lds_dwordx4 %19, s[82:83] offset:3072\n\t" \
    "s_add_u32 s99, s99, 1\n\t" \
    "s_cmp_eq_u32 s99, %23\n\t" \
    "s_cselect_b32 s91, s96, %22\n\t" \
    "s_cselect_b32 s90, s97, 0\n\t" \
    "s_cselect_b32 s99, 0, s99\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, s90\n\t" \
    "s_add_u32 s90, s87, %24\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %8, s[80:81] offset:0\n\t" \
    "global_load_lds_dwordx4 %9, s[80:81] offset:1024\n\t" \
    "global_load_lds_dwordx4 %10, s[80:81] offset:2048\n\t" \
    "global_load_lds_dwordx4 %11, s[80:81] offset:3072\n\t" \
    "s_add_u32 s90, s87, %24\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %12, s[80:81] offset:0\n\t" \
    "global_load_lds_dwordx4 %13, s[80:81] offset:1024\n\t" \
    "global_load_lds_dwordx4 %14, s[80:81] offset:2048\n\t" \
    "global_load_lds_dwordx4 %15, s[80:81] offset:3072\n\t" \
    "s_add_u32 s98, s98, 1\n\t" \
    "s_cmp_eq_u32 s98, %23\n\t" \
    "s_cselect_b32 s91, s94, 128\n\t" \
    "s_cselect_b32 s90, s95, 0\n\t" \
    "s_cselect_b32 s98, 0, s98\n\t" \
    "s_add_u32 s80, s80, s91\n\t" \
    "s_addc_u32 s81, s81, s90\n\t" \
    "s_add_u32 s90, s92, %25\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_nop 0\n\t" \
    "global_load_lds_dwordx4 %16, s[82:83] offset:0\n\t" \
    "global_load_lds_dwordx4 %17, s[82:83] offset:1024\n\t" \
    "global_load_lds_dwordx4 %18, s[82:83] offset:2048\n\t" \
    "global_load_lds_dwordx4 %19, s[82:83] offset:3072\n\t" \
    "s_add_u32 s99, s99, 1\n\t" \
    "s_cmp_eq_u32 s99, %23\n\t" \
    "s_cselect_b32 s91, s96, %22\n\t" \
    "s_cselect_b32 s90, s97, 0\n\t" \
    "s_cselect_b32 s99, 0, s99\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, s90\n\t" \
    "v_accvgpr_write_b32 a0, 0\n\t" \
    "v_accvgpr_write_b32 a1, 0\n\t" \
    "v_accvgpr_write_b32 a2, 0\n\t" \
    "v_accvgpr_write_b32 a3, 0\n\t" \
    "v_accvgpr_write_b32 a4, 0\n\t" \
    "v_accvgpr_write_b32 a5, 0\n\t" \
    "v_accvgpr_write_b32 a6, 0\n\t" \
    "v_accvgpr_write_b32 a7, 0\n\t" \
    "v_accvgpr_write_b32 a8, 0\n\t" \
    "v_accvgpr_write_b32 a9, 0\n\t" \
    "v_accvgpr_write_b32 a10, 0\n\t" \
    "v_accvgpr_write_b32 a11, 0\n\t" \
    "v_accvgpr_write_b32 a12, 0\n\t" \
    "v_accvgpr_write_b32 a13, 0\n\t" \
    "v_accvgpr_write_b32 a14, 0\n\t" \
    "v_accvgpr_write_b32 a15, 0\n\t" \
    "v_accvgpr_write_b32 a16, 0\n\t" \
    "v_accvgpr_write_b32 a17, 0\n\t" \
    "v_accvgpr_write_b32 a18, 0\n\t" \
    "v_accvgpr_write_b32 a19, 0\n\t" \
    "v_accvgpr_write_b32 a20, 0\n\t" \
    "v_accvgpr_write_b32 a21, 0\n\t" \
    "v_accvgpr_write_b32 a22, 0\n\t" \
    "v_accvgpr_write_b32 a23, 0\n\t" \
    "v_accvgpr_write_b32 a24, 0\n\t" \
    "v_accvgpr_write_b32 a25, 0\n\t" \
    "v_accvgpr_write_b32 a26, 0\n\t" \
    "v_accvgpr_write_b32 a27, 0\n\t" \
    "v_accvgpr_write_b32 a28, 0\n\t" \
    "v_accvgpr_write_b32 a29, 0\n\t" \
    "v_accvgpr_write_b32 a30, 0\n\t" \
    "v_accvgpr_write_b32 a31, 0\n\t" \
    "v_accvgpr_write_b32 a32, 0\n\t" \
    "v_accvgpr_write_b32 a33, 0\n\t" \
    "v_accvgpr_write_b32 a34, 0\n\t" \
    "v_accvgpr_write_b32 a35, 0\n\t" \
    "v_accvgpr_write_b32 a36, 0\n\t" \
    "v_accvgpr_write_b32 a37, 0\n\t" \
    "v_accvgpr_write_b32 a38, 0\n\t" \
    "v_accvgpr_write_b32 a39, 0\n\t" \
    "v_accvgpr_write_b32 a40, 0\n\t" \
    "v_accvgpr_write_b32 a41, 0\n\t" \
    "v_accvgpr_write_b32 a42, 0\n\t" \
    "v_accvgpr_write_b32 a43, 0\n\t" \
    "v_accvgpr_write_b32 a44, 0\n\t" \
    "v_accvgpr_write_b32 a45, 0\n\t" \
    "v_accvgpr_write_b32 a46, 0\n\t" \
    "v_accvgpr_write_b32 a47, 0\n\t" \
    "v_accvgpr_write_b32 a48, 0\n\t" \
    "v_accvgpr_write_b32 a49, 0\n\t" \
    "v_accvgpr_write_b32 a50, 0\n\t" \
    "v_accvgpr_write_b32 a51, 0\n\t" \
    "v_accvgpr_write_b32 a52, 0\n\t" \
    "v_accvgpr_write_b32 a53, 0\n\t" \
    "v_accvgpr_write_b32 a54, 0\n\t" \
    "v_accvgpr_write_b32 a55, 0\n\t" \
    "v_accvgpr_write_b32 a56, 0\n\t" \
    "v_accvgpr_write_b32 a57, 0\n\t" \
    "v_accvgpr_write_b32 a58, 0\n\t" \
    "v_accvgpr_write_b32 a59, 0\n\t" \
    "v_accvgpr_write_b32 a60, 0\n\t" \
    "v_accvgpr_write_b32 a61, 0\n\t" \
    "v_accvgpr_write_b32 a62, 0\n\t" \
    "v_accvgpr_write_b32 a63, 0\n\t" \
    "v_accvgpr_write_b32 a64, 0\n\t" \
    "v_accvgpr_write_b32 a65, 0\n\t" \
    "v_accvgpr_write_b32 a66, 0\n\t" \
    "v_accvgpr_write_b32 a67, 0\n\t" \
    "v_accvgpr_write_b32 a68, 0\n\t" \
    "v_accvgpr_write_b32 a69, 0\n\t" \
    "v_accvgpr_write_b32 a70, 0\n\t" \
    "v_accvgpr_write_b32 a71, 0\n\t" \
    "v_accvgpr_write_b32 a72, 0\n\t" \
    "v_accvgpr_write_b32 a73, 0\n\t" \
    "v_accvgpr_write_b32 a74, 0\n\t" \
    "v_accvgpr_write_b32 a75, 0\n\t" \
    "v_accvgpr_write_b32 a76, 0\n\t" \
    "v_accvgpr_write_b32 a77, 0\n\t" \
    "v_accvgpr_write_b32 a78, 0\n\t" \
    "v_accvgpr_write_b32 a79, 0\n\t" \
    "v_accvgpr_write_b32 a80, 0\n\t" \
    "v_accvgpr_write_b32 a81, 0\n\t" \
    "v_accvgpr_write_b32 a82, 0\n\t" \
    "v_accvgpr_write_b32 a83, 0\n\t" \
    "v_accvgpr_write_b32 a84, 0\n\t" \
    "v_accvgpr_write_b32 a85, 0\n\t" \
    "v_accvgpr_write_b32 a86, 0\n\t" \
    "v_accvgpr_write_b32 a87, 0\n\t" \
    "v_accvgpr_write_b32 a88, 0\n\t" \
    "v_accvgpr_write_b32 a89, 0\n\t" \
    "v_accvgpr_write_b32 a90, 0\n\t" \
    "v_accvgpr_write_b32 a91, 0\n\t" \
    "v_accvgpr_write_b32 a92, 0\n\t" \
    "v_accvgpr_write_b32 a93, 0\n\t" \
    "v_accvgpr_write_b32 a94, 0\n\t" \
    "v_accvgpr_write_b32 a95, 0\n\t" \
    "v_accvgpr_write_b32 a96, 0\n\t" \
    "v_accvgpr_write_b32 a97, 0\n\t" \
    "v_accvgpr_write_b32 a98, 0\n\t" \
    "v_accvgpr_write_b32 a99, 0\n\t" \
    "v_accvgpr_write_b32 a100, 0\n\t" \
    "v_accvgpr_write_b32 a101, 0\n\t" \
    "v_accvgpr_write_b32 a102, 0\n\t" \
    "v_accvgpr_write_b32 a103, 0\n\t" \
    "v_accvgpr_write_b32 a104, 0\n\t" \
    "v_accvgpr_write_b32 a105, 0\n\t" \
    "v_accvgpr_write_b32 a106, 0\n\t" \
    "v_accvgpr_write_b32 a107, 0\n\t" \
    "v_accvgpr_write_b32 a108, 0\n\t" \
    "v_accvgpr_write_b32 a109, 0\n\t" \
    "v_accvgpr_write_b32 a110, 0\n\t" \
    "v_accvgpr_write_b32 a111, 0\n\t" \
    "v_accvgpr_write_b32 a112, 0\n\t" \
    "v_accvgpr_write_b32 a113, 0\n\t" \
    "v_accvgpr_write_b32 a114, 0\n\t" \
    "v_accvgpr_write_b32 a115, 0\n\t" \
    "v_accvgpr_write_b32 a116, 0\n\t" \
    "v_accvgpr_write_b32 a117, 0\n\t" \
    "v_accvgpr_write_b32 a118, 0\n\t" \
    "v_accvgpr_write_b32 a119, 0\n\t" \
    "v_accvgpr_write_b32 a120, 0\n\t" \
    "v_accvgpr_write_b32 a121, 0\n\t" \
    "v_accvgpr_write_b32 a122, 0\n\t" \
    "v_accvgpr_write_b32 a123, 0\n\t" \
    "v_accvgpr_write_b32 a124, 0\n\t" \
    "v_accvgpr_write_b32 a125, 0\n\t" \
    "v_accvgpr_write_b32 a126, 0\n\t" \
    "v_accvgpr_write_b32 a127, 0\n\t" \
    "s_nop 3\n\t" \
    "s_waitcnt vmcnt(24)\n\t" \
    "s_barrier\n\t" \
    "v_add_u32 v118, s88, %4\n\t" \
    "ds_read_b64_tr_b16 v[160:161], v118 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[162:163], v118 offset:4096\n\t" \
    "v_add_u32 v119, s88, %5\n\t" \
    "ds_read_b64_tr_b16 v[164:165], v119 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[166:167], v119 offset:4096\n\t" \
    "v_add_u32 v120, s88, %6\n\t" \
    "ds_read_b64_tr_b16 v[168:169], v120 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[170:171], v120 offset:4096\n\t" \
    "v_add_u32 v121, s88, %7\n\t" \
    "ds_read_b64_tr_b16 v[172:173], v121 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[174:175], v121 offset:4096\n\t" \
    "v_add_u32 v116, s85, %0\n\t" \
    "v_add_u32 v117, s85, %1\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "ds_read_b64 v[144:145], v116 offset:8192\n\t" \
    "ds_read_b64 v[146:147], v117 offset:8192\n\t" \
    "ds_read_b64 v[148:149], v116 offset:10240\n\t" \
    "ds_read_b64 v[150:151], v117 offset:10240\n\t" \
    "ds_read_b64 v[152:153], v116 offset:12288\n\t" \
    "ds_read_b64 v[154:155], v117 offset:12288\n\t" \
    "ds_read_b64 v[156:157], v116 offset:14336\n\t" \
    "ds_read_b64 v[158:159], v117 offset:14336\n\t" \
    "s_cmp_lt_u32 %23, 4\n\t" \
    "s_cbranch_scc1 2f\n\t" \
    "1:\n\t" \
    "s_waitcnt lgkmcnt(14)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v118, s88, %4\n\t" \
    "ds_read_b64_tr_b16 v[208:209], v118 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "ds_read_b64_tr_b16 v[210:211], v118 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "v_add_u32 v119, s88, %5\n\t" \
    "ds_read_b64_tr_b16 v[212:213], v119 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "ds_read_b64_tr_b16 v[214:215], v119 offset:12288\n\t" \
    "s_add_u32 s90, s93, %25\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[160:163], v[132:135], a[16:19]\n\t" \
    "global_load_lds_dwordx4 %16, s[82:83] offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[164:167], v[132:135], a[20:23]\n\t" \
    "v_add_u32 v120, s88, %6\n\t" \
    "ds_read_b64_tr_b16 v[216:217], v120 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[168:171], v[132:135], a[24:27]\n\t" \
    "ds_read_b64_tr_b16 v[218:219], v120 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[172:175], v[132:135], a[28:31]\n\t" \
    "v_add_u32 v121, s88, %7\n\t" \
    "ds_read_b64_tr_b16 v[220:221], v121 offset:8192\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[136:139], a[32:35]\n\t" \
    "ds_read_b64_tr_b16 v[222:223], v121 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[136:139], a[36:39]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[176:177], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[136:139], a[40:43]\n\t" \
    "ds_read_b64 v[178:179], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[136:139], a[44:47]\n\t" \
    "ds_read_b64 v[180:181], v116 offset:2048\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[160:163], v[140:143], a[48:51]\n\t" \
    "global_load_lds_dwordx4 %17, s[82:83] offset:1024\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[164:167], v[140:143], a[52:55]\n\t" \
    "ds_read_b64 v[182:183], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[168:171], v[140:143], a[56:59]\n\t" \
    "ds_read_b64 v[184:185], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[172:175], v[140:143], a[60:63]\n\t" \
    "ds_read_b64 v[186:187], v117 offset:4096\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[144:147], a[64:67]\n\t" \
    "ds_read_b64 v[188:189], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[144:147], a[68:71]\n\t" \
    "ds_read_b64 v[190:191], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[144:147], a[72:75]\n\t" \
    "ds_read_b64 v[192:193], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[144:147], a[76:79]\n\t" \
    "ds_read_b64 v[194:195], v117 offset:8192\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[160:163], v[148:151], a[80:83]\n\t" \
    "global_load_lds_dwordx4 %18, s[82:83] offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[164:167], v[148:151], a[84:87]\n\t" \
    "ds_read_b64 v[196:197], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[168:171], v[148:151], a[88:91]\n\t" \
    "ds_read_b64 v[198:199], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[172:175], v[148:151], a[92:95]\n\t" \
    "ds_read_b64 v[200:201], v116 offset:12288\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[152:155], a[96:99]\n\t" \
    "ds_read_b64 v[202:203], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[152:155], a[100:103]\n\t" \
    "ds_read_b64 v[204:205], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[152:155], a[104:107]\n\t" \
    "ds_read_b64 v[206:207], v117 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[152:155], a[108:111]\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[160:163], v[156:159], a[112:115]\n\t" \
    "global_load_lds_dwordx4 %19, s[82:83] offset:3072\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[164:167], v[156:159], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[168:171], v[156:159], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[172:175], v[156:159], a[124:127]\n\t" \
    "s_add_u32 s99, s99, 1\n\t" \
    "s_cmp_eq_u32 s99, %23\n\t" \
    "s_cselect_b32 s91, s96, %22\n\t" \
    "s_cselect_b32 s90, s97, 0\n\t" \
    "s_cselect_b32 s99, 0, s99\n\t" \
    "s_add_u32 s82, s82, s91\n\t" \
    "s_addc_u32 s83, s83, s90\n\t" \
    "s_waitcnt vmcnt(16) lgkmcnt(0)\n\t" \
    "s_barrier\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[208:211], v[176:179], a[0:3]\n\t" \
    "v_add_u32 v118, s89, %4\n\t" \
    "ds_read_b64_tr_b16 v[160:161], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[212:215], v[176:179], a[4:7]\n\t" \
    "ds_read_b64_tr_b16 v[162:163], v118 offset:4096\n\t" \
    "s_add_u32 s90, s85, %24\n\t" \
    "s_add_u32 m0, s90, 0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[216:219], v[176:179], a[8:11]\n\t" \
    "global_load_lds_dwordx4 %8, s[80:81] offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[220:223], v[176:179], a[12:15]\n\t" \
    "v_add_u32 v119, s89, %5\n\t" \
    "ds_read_b64_tr_b16 v[164:165], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[208:211], v[180:183], a[16:19]\n\t" \
    "ds_read_b64_tr_b16 v[166:167], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[212:215], v[180:183], a[20:23]\n\t" \
    "v_add_u32 v120, s89, %6\n\t" \
    "ds_read_b64_tr_b16 v[168:169], v120 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[216:219], v[180:183], a[24:27]\n\t" \
    "global_load_lds_dwordx4 %9, s[80:81] offset:1024\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[220:223], v[180:183], a[28:31]\n\t" \
    "ds_read_b64_tr_b16 v[170:171], v120 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[208:211], v[184:187], a[32:35]\n\t" \
    "v_add_u32 v121, s89, %7\n\t" \
    "ds_read_b64_tr_b16 v[172:173], v121 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[212:215], v[184:187], a[36:39]\n\t" \
    "ds_read_b64_tr_b16 v[174:175], v121 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[216:219], v[184:187], a[40:43]\n\t" \
    "global_load_lds_dwordx4 %10, s[80:81] offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[220:223], v[184:187], a[44:47]\n\t" \
    "v_add_u32 v116, s86, %0\n\t" \
    "v_add_u32 v117, s86, %1\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[208:211], v[188:191], a[48:51]\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[212:215], v[188:191], a[52:55]\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[216:219], v[188:191], a[56:59]\n\t" \
    "global_load_lds_dwordx4 %11, s[80:81] offset:3072\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[220:223], v[188:191], a[60:63]\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[208:211], v[192:195], a[64:67]\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[212:215], v[192:195], a[68:71]\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "s_add_u32 s90, s85, %24\n\t" \
    "s_add_u32 m0, s90, 4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[216:219], v[192:195], a[72:75]\n\t" \
    "global_load_lds_dwordx4 %12, s[80:81] offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[220:223], v[192:195], a[76:79]\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[208:211], v[196:199], a[80:83]\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[212:215], v[196:199], a[84:87]\n\t" \
    "ds_read_b64 v[144:145], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[216:219], v[196:199], a[88:91]\n\t" \
    "global_load_lds_dwordx4 %13, s[80:81] offset:1024\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[220:223], v[196:199], a[92:95]\n\t" \
    "ds_read_b64 v[146:147], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[208:211], v[200:203], a[96:99]\n\t" \
    "ds_read_b64 v[148:149], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[212:215], v[200:203], a[100:103]\n\t" \
    "ds_read_b64 v[150:151], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[216:219], v[200:203], a[104:107]\n\t" \
    "global_load_lds_dwordx4 %14, s[80:81] offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[220:223], v[200:203], a[108:111]\n\t" \
    "ds_read_b64 v[152:153], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[208:211], v[204:207], a[112:115]\n\t" \
    "ds_read_b64 v[154:155], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[212:215], v[204:207], a[116:119]\n\t" \
    "ds_read_b64 v[156:157], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[216:219], v[204:207], a[120:123]\n\t" \
    "global_load_lds_dwordx4 %15, s[80:81] offset:3072\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[220:223], v[204:207], a[124:127]\n\t" \
    "ds_read_b64 v[158:159], v117 offset:14336\n\t" \
    "s_add_u32 s98, s98, 1\n\t" \
    "s_cmp_eq_u32 s98, %23\n\t" \
    "s_cselect_b32 s91, s94, 128\n\t" \
    "s_cselect_b32 s90, s95, 0\n\t" \
    "s_cselect_b32 s98, 0, s98\n\t" \
    "s_add_u32 s80, s80, s91\n\t" \
    "s_addc_u32 s81, s81, s90\n\t" \
    "s_mov_b32 s90, s85\n\t" \
    "s_mov_b32 s85, s86\n\t" \
    "s_mov_b32 s86, s87\n\t" \
    "s_mov_b32 s87, s90\n\t" \
    "s_mov_b32 s90, s88\n\t" \
    "s_mov_b32 s88, s89\n\t" \
    "s_mov_b32 s89, s92\n\t" \
    "s_mov_b32 s92, s93\n\t" \
    "s_mov_b32 s93, s90\n\t" \
    "s_sub_u32 s84, s84, 1\n\t" \
    "s_cmp_lg_u32 s84, 0\n\t" \
    "s_cbranch_scc1 1b\n\t" \
    "2:\n\t" \
    "s_cmp_lt_u32 %23, 3\n\t" \
    "s_cbranch_scc1 3f\n\t" \
    "s_waitcnt lgkmcnt(14)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v118, s88, %4\n\t" \
    "ds_read_b64_tr_b16 v[208:209], v118 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "ds_read_b64_tr_b16 v[210:211], v118 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "v_add_u32 v119, s88, %5\n\t" \
    "ds_read_b64_tr_b16 v[212:213], v119 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "ds_read_b64_tr_b16 v[214:215], v119 offset:12288\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[160:163], v[132:135], a[16:19]\n\t" \
    "v_add_u32 v120, s88, %6\n\t" \
    "ds_read_b64_tr_b16 v[216:217], v120 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[164:167], v[132:135], a[20:23]\n\t" \
    "ds_read_b64_tr_b16 v[218:219], v120 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[168:171], v[132:135], a[24:27]\n\t" \
    "v_add_u32 v121, s88, %7\n\t" \
    "ds_read_b64_tr_b16 v[220:221], v121 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[172:175], v[132:135], a[28:31]\n\t" \
    "ds_read_b64_tr_b16 v[222:223], v121 offset:12288\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[136:139], a[32:35]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[176:177], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[136:139], a[36:39]\n\t" \
    "ds_read_b64 v[178:179], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[136:139], a[40:43]\n\t" \
    "ds_read_b64 v[180:181], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[136:139], a[44:47]\n\t" \
    "ds_read_b64 v[182:183], v117 offset:2048\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[160:163], v[140:143], a[48:51]\n\t" \
    "ds_read_b64 v[184:185], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[164:167], v[140:143], a[52:55]\n\t" \
    "ds_read_b64 v[186:187], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[168:171], v[140:143], a[56:59]\n\t" \
    "ds_read_b64 v[188:189], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[172:175], v[140:143], a[60:63]\n\t" \
    "ds_read_b64 v[190:191], v117 offset:6144\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[144:147], a[64:67]\n\t" \
    "ds_read_b64 v[192:193], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[144:147], a[68:71]\n\t" \
    "ds_read_b64 v[194:195], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[144:147], a[72:75]\n\t" \
    "ds_read_b64 v[196:197], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[144:147], a[76:79]\n\t" \
    "ds_read_b64 v[198:199], v117 offset:10240\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[160:163], v[148:151], a[80:83]\n\t" \
    "ds_read_b64 v[200:201], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[164:167], v[148:151], a[84:87]\n\t" \
    "ds_read_b64 v[202:203], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[168:171], v[148:151], a[88:91]\n\t" \
    "ds_read_b64 v[204:205], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[172:175], v[148:151], a[92:95]\n\t" \
    "ds_read_b64 v[206:207], v117 offset:14336\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[152:155], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[152:155], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[152:155], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[152:155], a[108:111]\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[160:163], v[156:159], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[164:167], v[156:159], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[168:171], v[156:159], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[172:175], v[156:159], a[124:127]\n\t" \
    "s_waitcnt vmcnt(12) lgkmcnt(0)\n\t" \
    "s_barrier\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[208:211], v[176:179], a[0:3]\n\t" \
    "v_add_u32 v118, s89, %4\n\t" \
    "ds_read_b64_tr_b16 v[160:161], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[212:215], v[176:179], a[4:7]\n\t" \
    "ds_read_b64_tr_b16 v[162:163], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[216:219], v[176:179], a[8:11]\n\t" \
    "v_add_u32 v119, s89, %5\n\t" \
    "ds_read_b64_tr_b16 v[164:165], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[220:223], v[176:179], a[12:15]\n\t" \
    "ds_read_b64_tr_b16 v[166:167], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[208:211], v[180:183], a[16:19]\n\t" \
    "v_add_u32 v120, s89, %6\n\t" \
    "ds_read_b64_tr_b16 v[168:169], v120 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[212:215], v[180:183], a[20:23]\n\t" \
    "ds_read_b64_tr_b16 v[170:171], v120 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[216:219], v[180:183], a[24:27]\n\t" \
    "v_add_u32 v121, s89, %7\n\t" \
    "ds_read_b64_tr_b16 v[172:173], v121 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[220:223], v[180:183], a[28:31]\n\t" \
    "ds_read_b64_tr_b16 v[174:175], v121 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[208:211], v[184:187], a[32:35]\n\t" \
    "v_add_u32 v116, s86, %0\n\t" \
    "v_add_u32 v117, s86, %1\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[212:215], v[184:187], a[36:39]\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[216:219], v[184:187], a[40:43]\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[220:223], v[184:187], a[44:47]\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[208:211], v[188:191], a[48:51]\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[212:215], v[188:191], a[52:55]\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[216:219], v[188:191], a[56:59]\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[220:223], v[188:191], a[60:63]\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[208:211], v[192:195], a[64:67]\n\t" \
    "ds_read_b64 v[144:145], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[212:215], v[192:195], a[68:71]\n\t" \
    "ds_read_b64 v[146:147], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[216:219], v[192:195], a[72:75]\n\t" \
    "ds_read_b64 v[148:149], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[220:223], v[192:195], a[76:79]\n\t" \
    "ds_read_b64 v[150:151], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[208:211], v[196:199], a[80:83]\n\t" \
    "ds_read_b64 v[152:153], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[212:215], v[196:199], a[84:87]\n\t" \
    "ds_read_b64 v[154:155], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[216:219], v[196:199], a[88:91]\n\t" \
    "ds_read_b64 v[156:157], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[220:223], v[196:199], a[92:95]\n\t" \
    "ds_read_b64 v[158:159], v117 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[208:211], v[200:203], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[212:215], v[200:203], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[216:219], v[200:203], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[220:223], v[200:203], a[108:111]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[208:211], v[204:207], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[212:215], v[204:207], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[216:219], v[204:207], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[220:223], v[204:207], a[124:127]\n\t" \
    "s_mov_b32 s90, s85\n\t" \
    "s_mov_b32 s85, s86\n\t" \
    "s_mov_b32 s86, s87\n\t" \
    "s_mov_b32 s87, s90\n\t" \
    "s_mov_b32 s90, s88\n\t" \
    "s_mov_b32 s88, s89\n\t" \
    "s_mov_b32 s89, s92\n\t" \
    "s_mov_b32 s92, s93\n\t" \
    "s_mov_b32 s93, s90\n\t" \
    "3:\n\t" \
    "s_cmp_lt_u32 %23, 2\n\t" \
    "s_cbranch_scc1 4f\n\t" \
    "s_waitcnt lgkmcnt(14)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v118, s88, %4\n\t" \
    "ds_read_b64_tr_b16 v[208:209], v118 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "ds_read_b64_tr_b16 v[210:211], v118 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "v_add_u32 v119, s88, %5\n\t" \
    "ds_read_b64_tr_b16 v[212:213], v119 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "ds_read_b64_tr_b16 v[214:215], v119 offset:12288\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[160:163], v[132:135], a[16:19]\n\t" \
    "v_add_u32 v120, s88, %6\n\t" \
    "ds_read_b64_tr_b16 v[216:217], v120 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[164:167], v[132:135], a[20:23]\n\t" \
    "ds_read_b64_tr_b16 v[218:219], v120 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[168:171], v[132:135], a[24:27]\n\t" \
    "v_add_u32 v121, s88, %7\n\t" \
    "ds_read_b64_tr_b16 v[220:221], v121 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[172:175], v[132:135], a[28:31]\n\t" \
    "ds_read_b64_tr_b16 v[222:223], v121 offset:12288\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[136:139], a[32:35]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[176:177], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[136:139], a[36:39]\n\t" \
    "ds_read_b64 v[178:179], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[136:139], a[40:43]\n\t" \
    "ds_read_b64 v[180:181], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[136:139], a[44:47]\n\t" \
    "ds_read_b64 v[182:183], v117 offset:2048\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[160:163], v[140:143], a[48:51]\n\t" \
    "ds_read_b64 v[184:185], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[164:167], v[140:143], a[52:55]\n\t" \
    "ds_read_b64 v[186:187], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[168:171], v[140:143], a[56:59]\n\t" \
    "ds_read_b64 v[188:189], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[172:175], v[140:143], a[60:63]\n\t" \
    "ds_read_b64 v[190:191], v117 offset:6144\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[144:147], a[64:67]\n\t" \
    "ds_read_b64 v[192:193], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[144:147], a[68:71]\n\t" \
    "ds_read_b64 v[194:195], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[144:147], a[72:75]\n\t" \
    "ds_read_b64 v[196:197], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[144:147], a[76:79]\n\t" \
    "ds_read_b64 v[198:199], v117 offset:10240\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[160:163], v[148:151], a[80:83]\n\t" \
    "ds_read_b64 v[200:201], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[164:167], v[148:151], a[84:87]\n\t" \
    "ds_read_b64 v[202:203], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[168:171], v[148:151], a[88:91]\n\t" \
    "ds_read_b64 v[204:205], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[172:175], v[148:151], a[92:95]\n\t" \
    "ds_read_b64 v[206:207], v117 offset:14336\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[152:155], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[152:155], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[152:155], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[152:155], a[108:111]\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[160:163], v[156:159], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[164:167], v[156:159], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[168:171], v[156:159], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[172:175], v[156:159], a[124:127]\n\t" \
    "s_waitcnt vmcnt(0) lgkmcnt(0)\n\t" \
    "s_barrier\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[208:211], v[176:179], a[0:3]\n\t" \
    "v_add_u32 v118, s89, %4\n\t" \
    "ds_read_b64_tr_b16 v[160:161], v118 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[212:215], v[176:179], a[4:7]\n\t" \
    "ds_read_b64_tr_b16 v[162:163], v118 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[216:219], v[176:179], a[8:11]\n\t" \
    "v_add_u32 v119, s89, %5\n\t" \
    "ds_read_b64_tr_b16 v[164:165], v119 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[220:223], v[176:179], a[12:15]\n\t" \
    "ds_read_b64_tr_b16 v[166:167], v119 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[208:211], v[180:183], a[16:19]\n\t" \
    "v_add_u32 v120, s89, %6\n\t" \
    "ds_read_b64_tr_b16 v[168:169], v120 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[212:215], v[180:183], a[20:23]\n\t" \
    "ds_read_b64_tr_b16 v[170:171], v120 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[216:219], v[180:183], a[24:27]\n\t" \
    "v_add_u32 v121, s89, %7\n\t" \
    "ds_read_b64_tr_b16 v[172:173], v121 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[220:223], v[180:183], a[28:31]\n\t" \
    "ds_read_b64_tr_b16 v[174:175], v121 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[208:211], v[184:187], a[32:35]\n\t" \
    "v_add_u32 v116, s86, %0\n\t" \
    "v_add_u32 v117, s86, %1\n\t" \
    "ds_read_b64 v[128:129], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[212:215], v[184:187], a[36:39]\n\t" \
    "ds_read_b64 v[130:131], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[216:219], v[184:187], a[40:43]\n\t" \
    "ds_read_b64 v[132:133], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[220:223], v[184:187], a[44:47]\n\t" \
    "ds_read_b64 v[134:135], v117 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[208:211], v[188:191], a[48:51]\n\t" \
    "ds_read_b64 v[136:137], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[212:215], v[188:191], a[52:55]\n\t" \
    "ds_read_b64 v[138:139], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[216:219], v[188:191], a[56:59]\n\t" \
    "ds_read_b64 v[140:141], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[220:223], v[188:191], a[60:63]\n\t" \
    "ds_read_b64 v[142:143], v117 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[208:211], v[192:195], a[64:67]\n\t" \
    "ds_read_b64 v[144:145], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[212:215], v[192:195], a[68:71]\n\t" \
    "ds_read_b64 v[146:147], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[216:219], v[192:195], a[72:75]\n\t" \
    "ds_read_b64 v[148:149], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[220:223], v[192:195], a[76:79]\n\t" \
    "ds_read_b64 v[150:151], v117 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[208:211], v[196:199], a[80:83]\n\t" \
    "ds_read_b64 v[152:153], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[212:215], v[196:199], a[84:87]\n\t" \
    "ds_read_b64 v[154:155], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[216:219], v[196:199], a[88:91]\n\t" \
    "ds_read_b64 v[156:157], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[220:223], v[196:199], a[92:95]\n\t" \
    "ds_read_b64 v[158:159], v117 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[208:211], v[200:203], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[212:215], v[200:203], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[216:219], v[200:203], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[220:223], v[200:203], a[108:111]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[208:211], v[204:207], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[212:215], v[204:207], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[216:219], v[204:207], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[220:223], v[204:207], a[124:127]\n\t" \
    "s_mov_b32 s90, s85\n\t" \
    "s_mov_b32 s85, s86\n\t" \
    "s_mov_b32 s86, s87\n\t" \
    "s_mov_b32 s87, s90\n\t" \
    "s_mov_b32 s90, s88\n\t" \
    "s_mov_b32 s88, s89\n\t" \
    "s_mov_b32 s89, s92\n\t" \
    "s_mov_b32 s92, s93\n\t" \
    "s_mov_b32 s93, s90\n\t" \
    "4:\n\t" \
    "s_waitcnt lgkmcnt(14)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_add_u32 v118, s88, %4\n\t" \
    "ds_read_b64_tr_b16 v[208:209], v118 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "ds_read_b64_tr_b16 v[210:211], v118 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "v_add_u32 v119, s88, %5\n\t" \
    "ds_read_b64_tr_b16 v[212:213], v119 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "ds_read_b64_tr_b16 v[214:215], v119 offset:12288\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[160:163], v[132:135], a[16:19]\n\t" \
    "v_add_u32 v120, s88, %6\n\t" \
    "ds_read_b64_tr_b16 v[216:217], v120 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[164:167], v[132:135], a[20:23]\n\t" \
    "ds_read_b64_tr_b16 v[218:219], v120 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[168:171], v[132:135], a[24:27]\n\t" \
    "v_add_u32 v121, s88, %7\n\t" \
    "ds_read_b64_tr_b16 v[220:221], v121 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[172:175], v[132:135], a[28:31]\n\t" \
    "ds_read_b64_tr_b16 v[222:223], v121 offset:12288\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[136:139], a[32:35]\n\t" \
    "v_add_u32 v116, s85, %2\n\t" \
    "v_add_u32 v117, s85, %3\n\t" \
    "ds_read_b64 v[176:177], v116 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[136:139], a[36:39]\n\t" \
    "ds_read_b64 v[178:179], v117 offset:0\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[136:139], a[40:43]\n\t" \
    "ds_read_b64 v[180:181], v116 offset:2048\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[136:139], a[44:47]\n\t" \
    "ds_read_b64 v[182:183], v117 offset:2048\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[160:163], v[140:143], a[48:51]\n\t" \
    "ds_read_b64 v[184:185], v116 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[164:167], v[140:143], a[52:55]\n\t" \
    "ds_read_b64 v[186:187], v117 offset:4096\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[168:171], v[140:143], a[56:59]\n\t" \
    "ds_read_b64 v[188:189], v116 offset:6144\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[172:175], v[140:143], a[60:63]\n\t" \
    "ds_read_b64 v[190:191], v117 offset:6144\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[144:147], a[64:67]\n\t" \
    "ds_read_b64 v[192:193], v116 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[144:147], a[68:71]\n\t" \
    "ds_read_b64 v[194:195], v117 offset:8192\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[144:147], a[72:75]\n\t" \
    "ds_read_b64 v[196:197], v116 offset:10240\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[144:147], a[76:79]\n\t" \
    "ds_read_b64 v[198:199], v117 offset:10240\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[160:163], v[148:151], a[80:83]\n\t" \
    "ds_read_b64 v[200:201], v116 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[164:167], v[148:151], a[84:87]\n\t" \
    "ds_read_b64 v[202:203], v117 offset:12288\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[168:171], v[148:151], a[88:91]\n\t" \
    "ds_read_b64 v[204:205], v116 offset:14336\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[172:175], v[148:151], a[92:95]\n\t" \
    "ds_read_b64 v[206:207], v117 offset:14336\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[152:155], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[152:155], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[152:155], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[152:155], a[108:111]\n\t" \
    "s_waitcnt lgkmcnt(15)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[160:163], v[156:159], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[164:167], v[156:159], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[168:171], v[156:159], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[172:175], v[156:159], a[124:127]\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[208:211], v[176:179], a[0:3]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[212:215], v[176:179], a[4:7]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[216:219], v[176:179], a[8:11]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[220:223], v[176:179], a[12:15]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[208:211], v[180:183], a[16:19]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[212:215], v[180:183], a[20:23]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[216:219], v[180:183], a[24:27]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[220:223], v[180:183], a[28:31]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[208:211], v[184:187], a[32:35]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[212:215], v[184:187], a[36:39]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[216:219], v[184:187], a[40:43]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[220:223], v[184:187], a[44:47]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[208:211], v[188:191], a[48:51]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[212:215], v[188:191], a[52:55]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[216:219], v[188:191], a[56:59]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[220:223], v[188:191], a[60:63]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[208:211], v[192:195], a[64:67]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[212:215], v[192:195], a[68:71]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[216:219], v[192:195], a[72:75]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[220:223], v[192:195], a[76:79]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[208:211], v[196:199], a[80:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[212:215], v[196:199], a[84:87]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[216:219], v[196:199], a[88:91]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[220:223], v[196:199], a[92:95]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[208:211], v[200:203], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[212:215], v[200:203], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[216:219], v[200:203], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[220:223], v[200:203], a[108:111]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[208:211], v[204:207], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[212:215], v[204:207], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[216:219], v[204:207], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[220:223], v[204:207], a[124:127]\n\t" \
    "s_waitcnt vmcnt(0)\n\t" \
    "s_nop 15\n\t" \
    "s_nop 7\n\t" \
    ""

#define SYMB_GEMM16T_KSTEP32_NT \
    "s_cmp_eq_u32 %4, 0\n\t" \
    "s_cbranch_scc1 19f\n\t" \
    "ds_read_b64 v[160:161], %2 offset:0\n\t" \
    "ds_read_b64 v[164:165], %2 offset:2048\n\t" \
    "ds_read_b64 v[168:169], %2 offset:4096\n\t" \
    "ds_read_b64 v[172:173], %2 offset:6144\n\t" \
    "ds_read_b64 v[162:163], %3 offset:0\n\t" \
    "ds_read_b64 v[166:167], %3 offset:2048\n\t" \
    "ds_read_b64 v[170:171], %3 offset:4096\n\t" \
    "ds_read_b64 v[174:175], %3 offset:6144\n\t" \
    "s_bitcmp1_b32 %4, 0\n\t" \
    "s_cbranch_scc0 20f\n\t" \
    "ds_read_b64 v[128:129], %0 offset:0\n\t" \
    "ds_read_b64 v[130:131], %1 offset:0\n\t" \
    "20:\n\t" \
    "s_bitcmp1_b32 %4, 1\n\t" \
    "s_cbranch_scc0 21f\n\t" \
    "ds_read_b64 v[132:133], %0 offset:2048\n\t" \
    "ds_read_b64 v[134:135], %1 offset:2048\n\t" \
    "21:\n\t" \
    "s_bitcmp1_b32 %4, 2\n\t" \
    "s_cbranch_scc0 22f\n\t" \
    "ds_read_b64 v[136:137], %0 offset:4096\n\t" \
    "ds_read_b64 v[138:139], %1 offset:4096\n\t" \
    "22:\n\t" \
    "s_bitcmp1_b32 %4, 3\n\t" \
    "s_cbranch_scc0 23f\n\t" \
    "ds_read_b64 v[140:141], %0 offset:6144\n\t" \
    "ds_read_b64 v[142:143], %1 offset:6144\n\t" \
    "23:\n\t" \
    "s_bitcmp1_b32 %4, 4\n\t" \
    "s_cbranch_scc0 24f\n\t" \
    "ds_read_b64 v[144:145], %0 offset:8192\n\t" \
    "ds_read_b64 v[146:147], %1 offset:8192\n\t" \
    "24:\n\t" \
    "s_bitcmp1_b32 %4, 5\n\t" \
    "s_cbranch_scc0 25f\n\t" \
    "ds_read_b64 v[148:149], %0 offset:10240\n\t" \
    "ds_read_b64 v[150:151], %1 offset:10240\n\t" \
    "25:\n\t" \
    "s_bitcmp1_b32 %4, 6\n\t" \
    "s_cbranch_scc0 26f\n\t" \
    "ds_read_b64 v[152:153], %0 offset:12288\n\t" \
    "ds_read_b64 v[154:155], %1 offset:12288\n\t" \
    "26:\n\t" \
    "s_bitcmp1_b32 %4, 7\n\t" \
    "s_cbranch_scc0 27f\n\t" \
    "ds_read_b64 v[156:157], %0 offset:14336\n\t" \
    "ds_read_b64 v[158:159], %1 offset:14336\n\t" \
    "27:\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_bitcmp1_b32 %4, 0\n\t" \
    "s_cbranch_scc0 30f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "30:\n\t" \
    "s_bitcmp1_b32 %4, 1\n\t" \
    "s_cbranch_scc0 31f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[160:163], v[132:135], a[16:19]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[164:167], v[132:135], a[20:23]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[168:171], v[132:135], a[24:27]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[172:175], v[132:135], a[28:31]\n\t" \
    "31:\n\t" \
    "s_bitcmp1_b32 %4, 2\n\t" \
    "s_cbranch_scc0 32f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[136:139], a[32:35]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[136:139], a[36:39]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[136:139], a[40:43]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[136:139], a[44:47]\n\t" \
    "32:\n\t" \
    "s_bitcmp1_b32 %4, 3\n\t" \
    "s_cbranch_scc0 33f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[160:163], v[140:143], a[48:51]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[164:167], v[140:143], a[52:55]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[168:171], v[140:143], a[56:59]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[172:175], v[140:143], a[60:63]\n\t" \
    "33:\n\t" \
    "s_bitcmp1_b32 %4, 4\n\t" \
    "s_cbranch_scc0 34f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[144:147], a[64:67]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[144:147], a[68:71]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[144:147], a[72:75]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[144:147], a[76:79]\n\t" \
    "34:\n\t" \
    "s_bitcmp1_b32 %4, 5\n\t" \
    "s_cbranch_scc0 35f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[160:163], v[148:151], a[80:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[164:167], v[148:151], a[84:87]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[168:171], v[148:151], a[88:91]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[172:175], v[148:151], a[92:95]\n\t" \
    "35:\n\t" \
    "s_bitcmp1_b32 %4, 6\n\t" \
    "s_cbranch_scc0 36f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[152:155], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[152:155], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[152:155], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[152:155], a[108:111]\n\t" \
    "36:\n\t" \
    "s_bitcmp1_b32 %4, 7\n\t" \
    "s_cbranch_scc0 37f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[160:163], v[156:159], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[164:167], v[156:159], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[168:171], v[156:159], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[172:175], v[156:159], a[124:127]\n\t" \
    "37:\n\t" \
    "s_nop 15\n\t" \
    "s_nop 7\n\t" \
    "19:\n\t" \
    ""

#define SYMB_GEMM16T_KSTEP32_NN \
    "s_cmp_eq_u32 %6, 0\n\t" \
    "s_cbranch_scc1 19f\n\t" \
    "ds_read_b64_tr_b16 v[160:161], %2 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[162:163], %2 offset:4096\n\t" \
    "ds_read_b64_tr_b16 v[164:165], %3 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[166:167], %3 offset:4096\n\t" \
    "ds_read_b64_tr_b16 v[168:169], %4 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[170:171], %4 offset:4096\n\t" \
    "ds_read_b64_tr_b16 v[172:173], %5 offset:0\n\t" \
    "ds_read_b64_tr_b16 v[174:175], %5 offset:4096\n\t" \
    "s_bitcmp1_b32 %6, 0\n\t" \
    "s_cbranch_scc0 20f\n\t" \
    "ds_read_b64 v[128:129], %0 offset:0\n\t" \
    "ds_read_b64 v[130:131], %1 offset:0\n\t" \
    "20:\n\t" \
    "s_bitcmp1_b32 %6, 1\n\t" \
    "s_cbranch_scc0 21f\n\t" \
    "ds_read_b64 v[132:133], %0 offset:2048\n\t" \
    "ds_read_b64 v[134:135], %1 offset:2048\n\t" \
    "21:\n\t" \
    "s_bitcmp1_b32 %6, 2\n\t" \
    "s_cbranch_scc0 22f\n\t" \
    "ds_read_b64 v[136:137], %0 offset:4096\n\t" \
    "ds_read_b64 v[138:139], %1 offset:4096\n\t" \
    "22:\n\t" \
    "s_bitcmp1_b32 %6, 3\n\t" \
    "s_cbranch_scc0 23f\n\t" \
    "ds_read_b64 v[140:141], %0 offset:6144\n\t" \
    "ds_read_b64 v[142:143], %1 offset:6144\n\t" \
    "23:\n\t" \
    "s_bitcmp1_b32 %6, 4\n\t" \
    "s_cbranch_scc0 24f\n\t" \
    "ds_read_b64 v[144:145], %0 offset:8192\n\t" \
    "ds_read_b64 v[146:147], %1 offset:8192\n\t" \
    "24:\n\t" \
    "s_bitcmp1_b32 %6, 5\n\t" \
    "s_cbranch_scc0 25f\n\t" \
    "ds_read_b64 v[148:149], %0 offset:10240\n\t" \
    "ds_read_b64 v[150:151], %1 offset:10240\n\t" \
    "25:\n\t" \
    "s_bitcmp1_b32 %6, 6\n\t" \
    "s_cbranch_scc0 26f\n\t" \
    "ds_read_b64 v[152:153], %0 offset:12288\n\t" \
    "ds_read_b64 v[154:155], %1 offset:12288\n\t" \
    "26:\n\t" \
    "s_bitcmp1_b32 %6, 7\n\t" \
    "s_cbranch_scc0 27f\n\t" \
    "ds_read_b64 v[156:157], %0 offset:14336\n\t" \
    "ds_read_b64 v[158:159], %1 offset:14336\n\t" \
    "27:\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    "s_bitcmp1_b32 %6, 0\n\t" \
    "s_cbranch_scc0 30f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[0:3], v[160:163], v[128:131], a[0:3]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[4:7], v[164:167], v[128:131], a[4:7]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[8:11], v[168:171], v[128:131], a[8:11]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[12:15], v[172:175], v[128:131], a[12:15]\n\t" \
    "30:\n\t" \
    "s_bitcmp1_b32 %6, 1\n\t" \
    "s_cbranch_scc0 31f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[16:19], v[160:163], v[132:135], a[16:19]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[20:23], v[164:167], v[132:135], a[20:23]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[24:27], v[168:171], v[132:135], a[24:27]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[28:31], v[172:175], v[132:135], a[28:31]\n\t" \
    "31:\n\t" \
    "s_bitcmp1_b32 %6, 2\n\t" \
    "s_cbranch_scc0 32f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[32:35], v[160:163], v[136:139], a[32:35]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[36:39], v[164:167], v[136:139], a[36:39]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[40:43], v[168:171], v[136:139], a[40:43]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[44:47], v[172:175], v[136:139], a[44:47]\n\t" \
    "32:\n\t" \
    "s_bitcmp1_b32 %6, 3\n\t" \
    "s_cbranch_scc0 33f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[48:51], v[160:163], v[140:143], a[48:51]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[52:55], v[164:167], v[140:143], a[52:55]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[56:59], v[168:171], v[140:143], a[56:59]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[60:63], v[172:175], v[140:143], a[60:63]\n\t" \
    "33:\n\t" \
    "s_bitcmp1_b32 %6, 4\n\t" \
    "s_cbranch_scc0 34f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[64:67], v[160:163], v[144:147], a[64:67]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[68:71], v[164:167], v[144:147], a[68:71]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[72:75], v[168:171], v[144:147], a[72:75]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[76:79], v[172:175], v[144:147], a[76:79]\n\t" \
    "34:\n\t" \
    "s_bitcmp1_b32 %6, 5\n\t" \
    "s_cbranch_scc0 35f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[80:83], v[160:163], v[148:151], a[80:83]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[84:87], v[164:167], v[148:151], a[84:87]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[88:91], v[168:171], v[148:151], a[88:91]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[92:95], v[172:175], v[148:151], a[92:95]\n\t" \
    "35:\n\t" \
    "s_bitcmp1_b32 %6, 6\n\t" \
    "s_cbranch_scc0 36f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[96:99], v[160:163], v[152:155], a[96:99]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[100:103], v[164:167], v[152:155], a[100:103]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[104:107], v[168:171], v[152:155], a[104:107]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[108:111], v[172:175], v[152:155], a[108:111]\n\t" \
    "36:\n\t" \
    "s_bitcmp1_b32 %6, 7\n\t" \
    "s_cbranch_scc0 37f\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[112:115], v[160:163], v[156:159], a[112:115]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[116:119], v[164:167], v[156:159], a[116:119]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[120:123], v[168:171], v[156:159], a[120:123]\n\t" \
    "v_mfma_f32_16x16x32_bf16 a[124:127], v[172:175], v[156:159], a[124:127]\n\t" \
    "37:\n\t" \
    "s_nop 15\n\t" \
    "s_nop 7\n\t" \
    "19:\n\t" \
    ""

#define SYMB_GEMM16T_ZERO \
    "v_accvgpr_write_b32 a0, 0\n\t" \
    "v_accvgpr_write_b32 a1, 0\n\t" \
    "v_accvgpr_write_b32 a2, 0\n\t" \
    "v_accvgpr_write_b32 a3, 0\n\t" \
    "v_accvgpr_write_b32 a4, 0\n\t" \
    "v_accvgpr_write_b32 a5, 0\n\t" \
    "v_accvgpr_write_b32 a6, 0\n\t" \
    "v_accvgpr_write_b32 a7, 0\n\t" \
    "v_accvgpr_write_b32 a8, 0\n\t" \
    "v_accvgpr_write_b32 a9, 0\n\t" \
    "v_accvgpr_write_b32 a10, 0\n\t" \
    "v_accvgpr_write_b32 a11, 0\n\t" \
    "v_accvgpr_write_b32 a12, 0\n\t" \
    "v_accvgpr_write_b32 a13, 0\n\t" \
    "v_accvgpr_write_b32 a14, 0\n\t" \
    "v_accvgpr_write_b32 a15, 0\n\t" \
    "v_accvgpr_write_b32 a16, 0\n\t" \
    "v_accvgpr_write_b32 a17, 0\n\t" \
    "v_accvgpr_write_b32 a18, 0\n\t" \
    "v_accvgpr_write_b32 a19, 0\n\t" \
    "v_accvgpr_write_b32 a20, 0\n\t" \
    "v_accvgpr_write_b32 a21, 0\n\t" \
    "v_accvgpr_write_b32 a22, 0\n\t" \
    "v_accvgpr_write_b32 a23, 0\n\t" \
    "v_accvgpr_write_b32 a24, 0\n\t" \
    "v_accvgpr_write_b32 a25, 0\n\t" \
    "v_accvgpr_write_b32 a26, 0\n\t" \
    "v_accvgpr_write_b32 a27, 0\n\t" \
    "v_accvgpr_write_b32 a28, 0\n\t" \
    "v_accvgpr_write_b32 a29, 0\n\t" \
    "v_accvgpr_write_b32 a30, 0\n\t" \
    "v_accvgpr_write_b32 a31, 0\n\t" \
    "v_accvgpr_write_b32 a32, 0\n\t" \
    "v_accvgpr_write_b32 a33, 0\n\t" \
    "v_accvgpr_write_b32 a34, 0\n\t" \
    "v_accvgpr_write_b32 a35, 0\n\t" \
    "v_accvgpr_write_b32 a36, 0\n\t" \
    "v_accvgpr_write_b32 a37, 0\n\t" \
    "v_accvgpr_write_b32 a38, 0\n\t" \
    "v_accvgpr_write_b32 a39, 0\n\t" \
    "v_accvgpr_write_b32 a40, 0\n\t" \
    "v_accvgpr_write_b32 a41, 0\n\t" \
    "v_accvgpr_write_b32 a42, 0\n\t" \
    "v_accvgpr_write_b32 a43, 0\n\t" \
    "v_accvgpr_write_b32 a44, 0\n\t" \
    "v_accvgpr_write_b32 a45, 0\n\t" \
    "v_accvgpr_write_b32 a46, 0\n\t" \
    "v_accvgpr_write_b32 a47, 0\n\t" \
    "v_accvgpr_write_b32 a48, 0\n\t" \
    "v_accvgpr_write_b32 a49, 0\n\t" \
    "v_accvgpr_write_b32 a50, 0\n\t" \
    "v_accvgpr_write_b32 a51, 0\n\t" \
    "v_accvgpr_write_b32 a52, 0\n\t" \
    "v_accvgpr_write_b32 a53, 0\n\t" \
    "v_accvgpr_write_b32 a54, 0\n\t" \
    "v_accvgpr_write_b32 a55, 0\n\t" \
    "v_accvgpr_write_b32 a56, 0\n\t" \
    "v_accvgpr_write_b32 a57, 0\n\t" \
    "v_accvgpr_write_b32 a58, 0\n\t" \
    "v_accvgpr_write_b32 a59, 0\n\t" \
    "v_accvgpr_write_b32 a60, 0\n\t" \
    "v_accvgpr_write_b32 a61, 0\n\t" \
    "v_accvgpr_write_b32 a62, 0\n\t" \
    "v_accvgpr_write_b32 a63, 0\n\t" \
    "v_accvgpr_write_b32 a64, 0\n\t" \
    "v_accvgpr_write_b32 a65, 0\n\t" \
    "v_accvgpr_write_b32 a66, 0\n\t" \
    "v_accvgpr_write_b32 a67, 0\n\t" \
    "v_accvgpr_write_b32 a68, 0\n\t" \
    "v_accvgpr_write_b32 a69, 0\n\t" \
    "v_accvgpr_write_b32 a70, 0\n\t" \
    "v_accvgpr_write_b32 a71, 0\n\t" \
    "v_accvgpr_write_b32 a72, 0\n\t" \
    "v_accvgpr_write_b32 a73, 0\n\t" \
    "v_accvgpr_write_b32 a74, 0\n\t" \
    "v_accvgpr_write_b32 a75, 0\n\t" \
    "v_accvgpr_write_b32 a76, 0\n\t" \
    "v_accvgpr_write_b32 a77, 0\n\t" \
    "v_accvgpr_write_b32 a78, 0\n\t" \
    "v_accvgpr_write_b32 a79, 0\n\t" \
    "v_accvgpr_write_b32 a80, 0\n\t" \
    "v_accvgpr_write_b32 a81, 0\n\t" \
    "v_accvgpr_write_b32 a82, 0\n\t" \
    "v_accvgpr_write_b32 a83, 0\n\t" \
    "v_accvgpr_write_b32 a84, 0\n\t" \
    "v_accvgpr_write_b32 a85, 0\n\t" \
    "v_accvgpr_write_b32 a86, 0\n\t" \
    "v_accvgpr_write_b32 a87, 0\n\t" \
    "v_accvgpr_write_b32 a88, 0\n\t" \
    "v_accvgpr_write_b32 a89, 0\n\t" \
    "v_accvgpr_write_b32 a90, 0\n\t" \
    "v_accvgpr_write_b32 a91, 0\n\t" \
    "v_accvgpr_write_b32 a92, 0\n\t" \
    "v_accvgpr_write_b32 a93, 0\n\t" \
    "v_accvgpr_write_b32 a94, 0\n\t" \
    "v_accvgpr_write_b32 a95, 0\n\t" \
    "v_accvgpr_write_b32 a96, 0\n\t" \
    "v_accvgpr_write_b32 a97, 0\n\t" \
    "v_accvgpr_write_b32 a98, 0\n\t" \
    "v_accvgpr_write_b32 a99, 0\n\t" \
    "v_accvgpr_write_b32 a100, 0\n\t" \
    "v_accvgpr_write_b32 a101, 0\n\t" \
    "v_accvgpr_write_b32 a102, 0\n\t" \
    "v_accvgpr_write_b32 a103, 0\n\t" \
    "v_accvgpr_write_b32 a104, 0\n\t" \
    "v_accvgpr_write_b32 a105, 0\n\t" \
    "v_accvgpr_write_b32 a106, 0\n\t" \
    "v_accvgpr_write_b32 a107, 0\n\t" \
    "v_accvgpr_write_b32 a108, 0\n\t" \
    "v_accvgpr_write_b32 a109, 0\n\t" \
    "v_accvgpr_write_b32 a110, 0\n\t" \
    "v_accvgpr_write_b32 a111, 0\n\t" \
    "v_accvgpr_write_b32 a112, 0\n\t" \
    "v_accvgpr_write_b32 a113, 0\n\t" \
    "v_accvgpr_write_b32 a114, 0\n\t" \
    "v_accvgpr_write_b32 a115, 0\n\t" \
    "v_accvgpr_write_b32 a116, 0\n\t" \
    "v_accvgpr_write_b32 a117, 0\n\t" \
    "v_accvgpr_write_b32 a118, 0\n\t" \
    "v_accvgpr_write_b32 a119, 0\n\t" \
    "v_accvgpr_write_b32 a120, 0\n\t" \
    "v_accvgpr_write_b32 a121, 0\n\t" \
    "v_accvgpr_write_b32 a122, 0\n\t" \
    "v_accvgpr_write_b32 a123, 0\n\t" \
    "v_accvgpr_write_b32 a124, 0\n\t" \
    "v_accvgpr_write_b32 a125, 0\n\t" \
    "v_accvgpr_write_b32 a126, 0\n\t" \
    "v_accvgpr_write_b32 a127, 0\n\t" \
    "s_nop 3\n\t" \
    ""

#define SYMB_GEMM16T_STAGE_OUT \
    "v_accvgpr_read_b32 v128, a0\n\t" \
    "v_accvgpr_read_b32 v129, a1\n\t" \
    "v_accvgpr_read_b32 v130, a2\n\t" \
    "v_accvgpr_read_b32 v131, a3\n\t" \
    "v_cvt_pk_bf16_f32 v132, v128, v129\n\t" \
    "v_cvt_pk_bf16_f32 v133, v130, v131\n\t" \
    "ds_write_b64 %0, v[132:133] offset:0\n\t" \
    "v_accvgpr_read_b32 v134, a4\n\t" \
    "v_accvgpr_read_b32 v135, a5\n\t" \
    "v_accvgpr_read_b32 v136, a6\n\t" \
    "v_accvgpr_read_b32 v137, a7\n\t" \
    "v_cvt_pk_bf16_f32 v138, v134, v135\n\t" \
    "v_cvt_pk_bf16_f32 v139, v136, v137\n\t" \
    "ds_write_b64 %0, v[138:139] offset:32\n\t" \
    "v_accvgpr_read_b32 v140, a8\n\t" \
    "v_accvgpr_read_b32 v141, a9\n\t" \
    "v_accvgpr_read_b32 v142, a10\n\t" \
    "v_accvgpr_read_b32 v143, a11\n\t" \
    "v_cvt_pk_bf16_f32 v144, v140, v141\n\t" \
    "v_cvt_pk_bf16_f32 v145, v142, v143\n\t" \
    "ds_write_b64 %0, v[144:145] offset:64\n\t" \
    "v_accvgpr_read_b32 v146, a12\n\t" \
    "v_accvgpr_read_b32 v147, a13\n\t" \
    "v_accvgpr_read_b32 v148, a14\n\t" \
    "v_accvgpr_read_b32 v149, a15\n\t" \
    "v_cvt_pk_bf16_f32 v150, v146, v147\n\t" \
    "v_cvt_pk_bf16_f32 v151, v148, v149\n\t" \
    "ds_write_b64 %0, v[150:151] offset:96\n\t" \
    "v_accvgpr_read_b32 v152, a16\n\t" \
    "v_accvgpr_read_b32 v153, a17\n\t" \
    "v_accvgpr_read_b32 v154, a18\n\t" \
    "v_accvgpr_read_b32 v155, a19\n\t" \
    "v_cvt_pk_bf16_f32 v156, v152, v153\n\t" \
    "v_cvt_pk_bf16_f32 v157, v154, v155\n\t" \
    "ds_write_b64 %0, v[156:157] offset:4352\n\t" \
    "v_accvgpr_read_b32 v158, a20\n\t" \
    "v_accvgpr_read_b32 v159, a21\n\t" \
    "v_accvgpr_read_b32 v160, a22\n\t" \
    "v_accvgpr_read_b32 v161, a23\n\t" \
    "v_cvt_pk_bf16_f32 v162, v158, v159\n\t" \
    "v_cvt_pk_bf16_f32 v163, v160, v161\n\t" \
    "ds_write_b64 %0, v[162:163] offset:4384\n\t" \
    "v_accvgpr_read_b32 v164, a24\n\t" \
    "v_accvgpr_read_b32 v165, a25\n\t" \
    "v_accvgpr_read_b32 v166, a26\n\t" \
    "v_accvgpr_read_b32 v167, a27\n\t" \
    "v_cvt_pk_bf16_f32 v168, v164, v165\n\t" \
    "v_cvt_pk_bf16_f32 v169, v166, v167\n\t" \
    "ds_write_b64 %0, v[168:169] offset:4416\n\t" \
    "v_accvgpr_read_b32 v170, a28\n\t" \
    "v_accvgpr_read_b32 v171, a29\n\t" \
    "v_accvgpr_read_b32 v172, a30\n\t" \
    "v_accvgpr_read_b32 v173, a31\n\t" \
    "v_cvt_pk_bf16_f32 v174, v170, v171\n\t" \
    "v_cvt_pk_bf16_f32 v175, v172, v173\n\t" \
    "ds_write_b64 %0, v[174:175] offset:4448\n\t" \
    "v_accvgpr_read_b32 v128, a32\n\t" \
    "v_accvgpr_read_b32 v129, a33\n\t" \
    "v_accvgpr_read_b32 v130, a34\n\t" \
    "v_accvgpr_read_b32 v131, a35\n\t" \
    "v_cvt_pk_bf16_f32 v132, v128, v129\n\t" \
    "v_cvt_pk_bf16_f32 v133, v130, v131\n\t" \
    "ds_write_b64 %0, v[132:133] offset:8704\n\t" \
    "v_accvgpr_read_b32 v134, a36\n\t" \
    "v_accvgpr_read_b32 v135, a37\n\t" \
    "v_accvgpr_read_b32 v136, a38\n\t" \
    "v_accvgpr_read_b32 v137, a39\n\t" \
    "v_cvt_pk_bf16_f32 v138, v134, v135\n\t" \
    "v_cvt_pk_bf16_f32 v139, v136, v137\n\t" \
    "ds_write_b64 %0, v[138:139] offset:8736\n\t" \
    "v_accvgpr_read_b32 v140, a40\n\t" \
    "v_accvgpr_read_b32 v141, a41\n\t" \
    "v_accvgpr_read_b32 v142, a42\n\t" \
    "v_accvgpr_read_b32 v143, a43\n\t" \
    "v_cvt_pk_bf16_f32 v144, v140, v141\n\t" \
    "v_cvt_pk_bf16_f32 v145, v142, v143\n\t" \
    "ds_write_b64 %0, v[144:145] offset:8768\n\t" \
    "v_accvgpr_read_b32 v146, a44\n\t" \
    "v_accvgpr_read_b32 v147, a45\n\t" \
    "v_accvgpr_read_b32 v148, a46\n\t" \
    "v_accvgpr_read_b32 v149, a47\n\t" \
    "v_cvt_pk_bf16_f32 v150, v146, v147\n\t" \
    "v_cvt_pk_bf16_f32 v151, v148, v149\n\t" \
    "ds_write_b64 %0, v[150:151] offset:8800\n\t" \
    "v_accvgpr_read_b32 v152, a48\n\t" \
    "v_accvgpr_read_b32 v153, a49\n\t" \
    "v_accvgpr_read_b32 v154, a50\n\t" \
    "v_accvgpr_read_b32 v155, a51\n\t" \
    "v_cvt_pk_bf16_f32 v156, v152, v153\n\t" \
    "v_cvt_pk_bf16_f32 v157, v154, v155\n\t" \
    "ds_write_b64 %0, v[156:157] offset:13056\n\t" \
    "v_accvgpr_read_b32 v158, a52\n\t" \
    "v_accvgpr_read_b32 v159, a53\n\t" \
    "v_accvgpr_read_b32 v160, a54\n\t" \
    "v_accvgpr_read_b32 v161, a55\n\t" \
    "v_cvt_pk_bf16_f32 v162, v158, v159\n\t" \
    "v_cvt_pk_bf16_f32 v163, v160, v161\n\t" \
    "ds_write_b64 %0, v[162:163] offset:13088\n\t" \
    "v_accvgpr_read_b32 v164, a56\n\t" \
    "v_accvgpr_read_b32 v165, a57\n\t" \
    "v_accvgpr_read_b32 v166, a58\n\t" \
    "v_accvgpr_read_b32 v167, a59\n\t" \
    "v_cvt_pk_bf16_f32 v168, v164, v165\n\t" \
    "v_cvt_pk_bf16_f32 v169, v166, v167\n\t" \
    "ds_write_b64 %0, v[168:169] offset:13120\n\t" \
    "v_accvgpr_read_b32 v170, a60\n\t" \
    "v_accvgpr_read_b32 v171, a61\n\t" \
    "v_accvgpr_read_b32 v172, a62\n\t" \
    "v_accvgpr_read_b32 v173, a63\n\t" \
    "v_cvt_pk_bf16_f32 v174, v170, v171\n\t" \
    "v_cvt_pk_bf16_f32 v175, v172, v173\n\t" \
    "ds_write_b64 %0, v[174:175] offset:13152\n\t" \
    "v_accvgpr_read_b32 v128, a64\n\t" \
    "v_accvgpr_read_b32 v129, a65\n\t" \
    "v_accvgpr_read_b32 v130, a66\n\t" \
    "v_accvgpr_read_b32 v131, a67\n\t" \
    "v_cvt_pk_bf16_f32 v132, v128, v129\n\t" \
    "v_cvt_pk_bf16_f32 v133, v130, v131\n\t" \
    "ds_write_b64 %0, v[132:133] offset:17408\n\t" \
    "v_accvgpr_read_b32 v134, a68\n\t" \
    "v_accvgpr_read_b32 v135, a69\n\t" \
    "v_accvgpr_read_b32 v136, a70\n\t" \
    "v_accvgpr_read_b32 v137, a71\n\t" \
    "v_cvt_pk_bf16_f32 v138, v134, v135\n\t" \
    "v_cvt_pk_bf16_f32 v139, v136, v137\n\t" \
    "ds_write_b64 %0, v[138:139] offset:17440\n\t" \
    "v_accvgpr_read_b32 v140, a72\n\t" \
    "v_accvgpr_read_b32 v141, a73\n\t" \
    "v_accvgpr_read_b32 v142, a74\n\t" \
    "v_accvgpr_read_b32 v143, a75\n\t" \
    "v_cvt_pk_bf16_f32 v144, v140, v141\n\t" \
    "v_cvt_pk_bf16_f32 v145, v142, v143\n\t" \
    "ds_write_b64 %0, v[144:145] offset:17472\n\t" \
    "v_accvgpr_read_b32 v146, a76\n\t" \
    "v_accvgpr_read_b32 v147, a77\n\t" \
    "v_accvgpr_read_b32 v148, a78\n\t" \
    "v_accvgpr_read_b32 v149, a79\n\t" \
    "v_cvt_pk_bf16_f32 v150, v146, v147\n\t" \
    "v_cvt_pk_bf16_f32 v151, v148, v149\n\t" \
    "ds_write_b64 %0, v[150:151] offset:17504\n\t" \
    "v_accvgpr_read_b32 v152, a80\n\t" \
    "v_accvgpr_read_b32 v153, a81\n\t" \
    "v_accvgpr_read_b32 v154, a82\n\t" \
    "v_accvgpr_read_b32 v155, a83\n\t" \
    "v_cvt_pk_bf16_f32 v156, v152, v153\n\t" \
    "v_cvt_pk_bf16_f32 v157, v154, v155\n\t" \
    "ds_write_b64 %0, v[156:157] offset:21760\n\t" \
    "v_accvgpr_read_b32 v158, a84\n\t" \
    "v_accvgpr_read_b32 v159, a85\n\t" \
    "v_accvgpr_read_b32 v160, a86\n\t" \
    "v_accvgpr_read_b32 v161, a87\n\t" \
    "v_cvt_pk_bf16_f32 v162, v158, v159\n\t" \
    "v_cvt_pk_bf16_f32 v163, v160, v161\n\t" \
    "ds_write_b64 %0, v[162:163] offset:21792\n\t" \
    "v_accvgpr_read_b32 v164, a88\n\t" \
    "v_accvgpr_read_b32 v165, a89\n\t" \
    "v_accvgpr_read_b32 v166, a90\n\t" \
    "v_accvgpr_read_b32 v167, a91\n\t" \
    "v_cvt_pk_bf16_f32 v168, v164, v165\n\t" \
    "v_cvt_pk_bf16_f32 v169, v166, v167\n\t" \
    "ds_write_b64 %0, v[168:169] offset:21824\n\t" \
    "v_accvgpr_read_b32 v170, a92\n\t" \
    "v_accvgpr_read_b32 v171, a93\n\t" \
    "v_accvgpr_read_b32 v172, a94\n\t" \
    "v_accvgpr_read_b32 v173, a95\n\t" \
    "v_cvt_pk_bf16_f32 v174, v170, v171\n\t" \
    "v_cvt_pk_bf16_f32 v175, v172, v173\n\t" \
    "ds_write_b64 %0, v[174:175] offset:21856\n\t" \
    "v_accvgpr_read_b32 v128, a96\n\t" \
    "v_accvgpr_read_b32 v129, a97\n\t" \
    "v_accvgpr_read_b32 v130, a98\n\t" \
    "v_accvgpr_read_b32 v131, a99\n\t" \
    "v_cvt_pk_bf16_f32 v132, v128, v129\n\t" \
    "v_cvt_pk_bf16_f32 v133, v130, v131\n\t" \
    "ds_write_b64 %0, v[132:133] offset:26112\n\t" \
    "v_accvgpr_read_b32 v134, a100\n\t" \
    "v_accvgpr_read_b32 v135, a101\n\t" \
    "v_accvgpr_read_b32 v136, a102\n\t" \
    "v_accvgpr_read_b32 v137, a103\n\t" \
    "v_cvt_pk_bf16_f32 v138, v134, v135\n\t" \
    "v_cvt_pk_bf16_f32 v139, v136, v137\n\t" \
    "ds_write_b64 %0, v[138:139] offset:26144\n\t" \
    "v_accvgpr_read_b32 v140, a104\n\t" \
    "v_accvgpr_read_b32 v141, a105\n\t" \
    "v_accvgpr_read_b32 v142, a106\n\t" \
    "v_accvgpr_read_b32 v143, a107\n\t" \
    "v_cvt_pk_bf16_f32 v144, v140, v141\n\t" \
    "v_cvt_pk_bf16_f32 v145, v142, v143\n\t" \
    "ds_write_b64 %0, v[144:145] offset:26176\n\t" \
    "v_accvgpr_read_b32 v146, a108\n\t" \
    "v_accvgpr_read_b32 v147, a109\n\t" \
    "v_accvgpr_read_b32 v148, a110\n\t" \
    "v_accvgpr_read_b32 v149, a111\n\t" \
    "v_cvt_pk_bf16_f32 v150, v146, v147\n\t" \
    "v_cvt_pk_bf16_f32 v151, v148, v149\n\t" \
    "ds_write_b64 %0, v[150:151] offset:26208\n\t" \
    "v_accvgpr_read_b32 v152, a112\n\t" \
    "v_accvgpr_read_b32 v153, a113\n\t" \
    "v_accvgpr_read_b32 v154, a114\n\t" \
    "v_accvgpr_read_b32 v155, a115\n\t" \
    "v_cvt_pk_bf16_f32 v156, v152, v153\n\t" \
    "v_cvt_pk_bf16_f32 v157, v154, v155\n\t" \
    "ds_write_b64 %0, v[156:157] offset:30464\n\t" \
    "v_accvgpr_read_b32 v158, a116\n\t" \
    "v_accvgpr_read_b32 v159, a117\n\t" \
    "v_accvgpr_read_b32 v160, a118\n\t" \
    "v_accvgpr_read_b32 v161, a119\n\t" \
    "v_cvt_pk_bf16_f32 v162, v158, v159\n\t" \
    "v_cvt_pk_bf16_f32 v163, v160, v161\n\t" \
    "ds_write_b64 %0, v[162:163] offset:30496\n\t" \
    "v_accvgpr_read_b32 v164, a120\n\t" \
    "v_accvgpr_read_b32 v165, a121\n\t" \
    "v_accvgpr_read_b32 v166, a122\n\t" \
    "v_accvgpr_read_b32 v167, a123\n\t" \
    "v_cvt_pk_bf16_f32 v168, v164, v165\n\t" \
    "v_cvt_pk_bf16_f32 v169, v166, v167\n\t" \
    "ds_write_b64 %0, v[168:169] offset:30528\n\t" \
    "v_accvgpr_read_b32 v170, a124\n\t" \
    "v_accvgpr_read_b32 v171, a125\n\t" \
    "v_accvgpr_read_b32 v172, a126\n\t" \
    "v_accvgpr_read_b32 v173, a127\n\t" \
    "v_cvt_pk_bf16_f32 v174, v170, v171\n\t" \
    "v_cvt_pk_bf16_f32 v175, v172, v173\n\t" \
    "ds_write_b64 %0, v[174:175] offset:30560\n\t" \
    "s_waitcnt lgkmcnt(0)\n\t" \
    ""

#define SYMB_GEMM16T_STORE_PARTIAL \
    "v_mov_b32 v116, %0\n\t" \
    "global_store_dwordx4 v116, a[0:3], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[4:7], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[8:11], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[12:15], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[16:19], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[20:23], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[24:27], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[28:31], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[32:35], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[36:39], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[40:43], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[44:47], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[48:51], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[52:55], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[56:59], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[60:63], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[64:67], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[68:71], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[72:75], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[76:79], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[80:83], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[84:87], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[88:91], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[92:95], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[96:99], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[100:103], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[104:107], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[108:111], %1 offset:3072\n\t" \
    "v_add_u32 v116, 4096, v116\n\t" \
    "global_store_dwordx4 v116, a[112:115], %1 offset:0\n\t" \
    "global_store_dwordx4 v116, a[116:119], %1 offset:1024\n\t" \
    "global_store_dwordx4 v116, a[120:123], %1 offset:2048\n\t" \
    "global_store_dwordx4 v116, a[124:127], %1 offset:3072\n\t" \
    "s_waitcnt vmcnt(0)\n\t" \
    ""

#define SYMB_GEMM16T_VCLOBBERS "v116", "v117", "v118", "v119", "v120", "v121", "v122", "v123", "v124", "v125", "v126", "v127", "v128", "v129", "v130", "v131", "v132", "v133", "v134", "v135", "v136", "v137", "v138", "v139", "v140", "v141", "v142", "v143", "v144", "v145", "v146", "v147", "v148", "v149", "v150", "v151", "v152", "v153", "v154", "v155", "v156", "v157", "v158", "v159", "v160", "v161", "v162", "v163", "v164", "v165", "v166", "v167", "v168", "v169", "v170", "v171", "v172", "v173", "v174", "v175", "v176", "v177", "v178", "v179", "v180", "v181", "v182", "v183", "v184", "v185", "v186", "v187", "v188", "v189", "v190", "v191", "v192", "v193", "v194", "v195", "v196", "v197", "v198", "v199", "v200", "v201", "v202", "v203", "v204", "v205", "v206", "v207", "v208", "v209", "v210", "v211", "v212", "v213", "v214", "v215", "v216", "v217", "v218", "v219", "v220", "v221", "v222", "v223"
#define SYMB_GEMM16T_ACLOBBERS "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15", "a16", "a17", "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31", "a32", "a33", "a34", "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46", "a47", "a48", "a49", "a50", "a51", "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61", "a62", "a63", "a64", "a65", "a66", "a67", "a68", "a69", "a70", "a71", "a72", "a73", "a74", "a75", "a76", "a77", "a78", "a79", "a80", "a81", "a82", "a83", "a84", "a85", "a86", "a87", "a88", "a89", "a90", "a91", "a92", "a93", "a94", "a95", "a96", "a97", "a98", "a99", "a100", "a101", "a102", "a103", "a104", "a105", "a106", "a107", "a108", "a109", "a110", "a111", "a112", "a113", "a114", "a115", "a116", "a117", "a118", "a119", "a120", "a121", "a122", "a123", "a124", "a125", "a126", "a127"

#define SYMB_GEMM16_SCLOBBERS "s80", "s81", "s82", "s83", "s84", "s85", "s86", "s87", "s88", "s89", "s90", "s91"
#define SYMB_GEMM16T_SCLOBBERS "s80", "s81", "s82", "s83", "s84", "s85", "s86", "s87", "s88", "s89", "s90", "s91", "s92", "s93", "s94", "s95", "s96", "s97", "s98", "s99"
