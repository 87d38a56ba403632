// The main loop of the 256 x 256 tile (TileLarge in gemm_tile.hpp) as one block of assembly per pair of
// operand layouts, and why it is one.
//
// Four waves, one per SIMD, each with 128 x 128 of the tile (in four pieces of 64 x 64): the 512 registers of a lane are
// 256 accumulators (a[0:255]), the fragments of both halves of both operands (v[128:255]) and what the compiler
// keeps (v[0:127]).  Against eight waves of 128 x 64 a third of the reads from LDS is gone, but nothing is left to
// cover a wave's own waits: the reads of the next fragments and the copies of later K tiles have to stand
// between the MFMAs, counted, in an order that no compiler keeps (and it puts a wait for ALL copies before a
// transposing read).  All loads to registers are waited for inside the block.
//
// A = rows (m) and B = columns (n) of the tile in halves of 128; fragments FA0, FA1 (halves of A) at v128, v160 and FX, FY
// (halves of B, which swap roles from one K tile to the next) at v192, v224.  K tile k, in LDS stage k & 1:
//     part  multiplies             reads             copies (after the barrier that ends their last read)
//     0     A1 B0 of k - 1         B0 of k -> FX     A1 of k + 1
//     1     A0 B0                  B1     -> FY      A0 of k + 2                        barrier
//     2     A0 B1                  A1     -> FA1     B0 of k + 2
//     3     A1 B1                  A0 of k + 1       B1 of k + 2                        barrier
// Copies are issued in the order in which they are needed, four instructions per half tile; at either barrier the
// halves that the next two parts read are those before the last four: at most 16 outstanding.  A barrier after
// every part (24 outstanding) measured 1.2 % less.  Copies past the last K tile are issued all
// the same, from an empty buffer, so that the counts stay what they are.
//
// Measured, TFLOP/s (8192 x 32768 x 2048 and, dHidden, 2048 x 32768 x 8192; no result stored, one card), the loop of eight
// waves in two groups before it / this one: A transposed 1428 / 1610, both transposed 1395 / 1600, neither 1570 / 1610.
// It keeps the matrix pipes 91 to 93 % busy; what bounds all four products alike is the card's power limit, which
// takes the clock down to 1.75 GHz (copies of zeros: 2000 to 2200 at 2.38 GHz; without copies 1820 to 1930; without
// reads from LDS either 2100 to 2280).  v_mfma_f32_32x32x16_bf16 in the same loop draws more power: 1360 to 1440.
// Whole calls, us, before / after: 777 x 2048 x 151936 1822 / 1748, 4096 rows 6992 / 6558, 32768 rows 62430 / 59570.
#ifndef ULORL_GEMM_LOOP_HPP
#define ULORL_GEMM_LOOP_HPP

// Scalar registers of the block: s[40:43], s[44:47] buffer descriptors of A and B, s48 K tiles left to multiply, s49 K tiles
// left to copy, s52, s53 the offset along k of a K_ROWS operand, s[54:56], s[57:59] the offsets of copy instructions 1 to 3 of
// a K_COLS one.
// v94 and v95 are the offsets of a K_ROWS operand's copies.
// Operands: sw = LDS address of the stages + 1024 x wave; r<op>0.. LDS read addresses; v<op>.. byte offsets of a
// lane's copies; K_ROWS: g<op>, h<op> bytes from one copy instruction to the next and from half 0 to half 1; K_COLS:
// s<op>1..3 offsets of copy instruction 1..3, t<op>l/h bytes from one K tile to the next.

// One MFMA of a part, number n (0..31) of it: block (i, j) of piece (I0 / 4, J0 / 4).
#define UL_MFMA_IJ(FA, FB, I0, J0, KS, I, J)                                                                   \
    "v_mfma_f32_16x16x32_bf16 a[((" I0 "+" I ")*8+" J0 "+" J ")*4:((" I0 "+" I ")*8+" J0 "+" J ")*4+3], "        \
    "v[" FA "+(" KS ")*16+(" I ")*4:" FA "+(" KS ")*16+(" I ")*4+3], "                                           \
    "v[" FB "+(" KS ")*16+(" J ")*4:" FB "+(" KS ")*16+(" J ")*4+3], "
#define UL_ACC(I0, J0, I, J) "a[((" I0 "+" I ")*8+" J0 "+" J ")*4:((" I0 "+" I ")*8+" J0 "+" J ")*4+3]\n"
#define UL_MFMA(FA, FB, I0, J0) \
    UL_MFMA_IJ(FA, FB, I0, J0, "n/16", "(n%%16)/4", "n%%4") UL_ACC(I0, J0, "(n%%16)/4", "n%%4")
// The same with the accumulators' first values 0 (part 1 to 3 of the first K tile).
#define UL_MFMA_NEW(FA, FB, I0, J0)                                                                            \
    ".if n<16\n" UL_MFMA_IJ(FA, FB, I0, J0, "n/16", "(n%%16)/4", "n%%4") "0\n.else\n" UL_MFMA(FA, FB, I0, J0) ".endif\n"
// Column blocks one after the other, for a part that ends after j1 of them.
#define UL_MFMA_COLS(FA, FB, I0, J0) \
    UL_MFMA_IJ(FA, FB, I0, J0, "(n%%8)/4", "n%%4", "n/8") UL_ACC(I0, J0, "n%%4", "n/8")
#define UL_MFMA_COLS_NEW(FA, FB, I0, J0)                                                                       \
    ".if (n%%8)<4\n" UL_MFMA_IJ(FA, FB, I0, J0, "(n%%8)/4", "n%%4", "n/8") "0\n.else\n" UL_MFMA_COLS(FA, FB, I0, J0) ".endif\n"

// Fragment reads of one half into DST: K_ROWS eight, after every other of the first 16 MFMAs; K_COLS sixteen.
#define UL_READ_ROWS(X, DST, OFF)                                                                              \
    ".if (n<8)&&(n%%2==1)\nds_read_b128 v[" DST "+(n/2)*4:" DST "+(n/2)*4+3], %[r" X "0] offset:" OFF "+((n/2)%%4)*2048\n.endif\n" \
    ".if (n>=8)&&(n<16)&&(n%%2==1)\nds_read_b128 v[" DST "+(n/2)*4:" DST "+(n/2)*4+3], %[r" X "1] offset:" OFF "+((n/2)%%4)*2048\n.endif\n"
#define UL_READ_COLS_BLOCK(X, DST, OFF, B)                                                                     \
    ".if (n<16)&&((n%%8)/2==" B ")\nds_read_b64_tr_b16 v[" DST "+((n/8)*4+" B ")*4+(n%%2)*2:" DST "+((n/8)*4+" B ")*4+(n%%2)*2+1], " \
    "%[r" X B "] offset:" OFF "+(n/8)*8192+(n%%2)*1024\n.endif\n"
#define UL_READ_COLS(X, DST, OFF)                                                                              \
    UL_READ_COLS_BLOCK(X, DST, OFF, "0") UL_READ_COLS_BLOCK(X, DST, OFF, "1") UL_READ_COLS_BLOCK(X, DST, OFF, "2") UL_READ_COLS_BLOCK(X, DST, OFF, "3")
// Half 1 of B has read addresses of its own where its width varies (K_ROWS).
#define UL_READ1_ROWS(DST, OFF) UL_READ_ROWS("y", DST, OFF)
#define UL_READ1_COLS(DST, OFF) UL_READ_COLS("b", DST, OFF)

// This wave's four instructions of one half tile's copy, J after MFMA 18 + 3 J.  gfx9 parts need an instruction between a
// scalar write of m0 and the copy that takes its LDS address from there, and the compiler looks for that outside of
// assembly only: whatever expands a copy for n and n + 1 puts one between them.
#define UL_COPY_AT(J) "(" UL_COPY_FIRST "+3*" J ")"
#define UL_COPY_ONE(LDS, J, LOAD)                                                                              \
    ".if n==" UL_COPY_AT(J) "\ns_add_u32 m0, %[sw], " LDS "+" J "*4096\n.endif\n"                             \
    ".if n==" UL_COPY_AT(J) "+1\n" LOAD " offen lds\n.endif\n"
#define UL_COPY_FIRST "17"
#define UL_RSRC_a "s[40:43], "
#define UL_RSRC_b "s[44:47], "
#define UL_KOFF_a "s52"
#define UL_KOFF_b "s53"
#define UL_COFF_a1 "s54"
#define UL_COFF_a2 "s55"
#define UL_COFF_a3 "s56"
#define UL_COFF_b1 "s57"
#define UL_COFF_b2 "s58"
#define UL_COFF_b3 "s59"
#define UL_ROW_a "v94"
#define UL_ROW_b "v95"
#define UL_FIRST_ROW_0(XS, X) "v_mov_b32 " UL_ROW_##X ", %[v" XS "]\n"
#define UL_FIRST_ROW_1(XS, X) "v_add_u32 " UL_ROW_##X ", %[h" XS "], %[v" XS "]\n"
#define UL_NEXT_ROW(XS, X, J) ".if n==" UL_COPY_AT(J) "\nv_add_u32 " UL_ROW_##X ", %[g" XS "], " UL_ROW_##X "\n.endif\n"
#define UL_COPY_ROWS(XS, X, H, LDS)                                                                            \
    ".if n==" UL_COPY_AT("0") "\n" UL_FIRST_ROW_##H(XS, X) ".endif\n"                                          \
    UL_COPY_ONE(LDS, "0", "buffer_load_dwordx4 " UL_ROW_##X ", " UL_RSRC_##X UL_KOFF_##X) UL_NEXT_ROW(XS, X, "1") \
    UL_COPY_ONE(LDS, "1", "buffer_load_dwordx4 " UL_ROW_##X ", " UL_RSRC_##X UL_KOFF_##X) UL_NEXT_ROW(XS, X, "2") \
    UL_COPY_ONE(LDS, "2", "buffer_load_dwordx4 " UL_ROW_##X ", " UL_RSRC_##X UL_KOFF_##X) UL_NEXT_ROW(XS, X, "3") \
    UL_COPY_ONE(LDS, "3", "buffer_load_dwordx4 " UL_ROW_##X ", " UL_RSRC_##X UL_KOFF_##X)
#define UL_COPY_COLS(XS, X, H, LDS)                                                                            \
    UL_COPY_ONE(LDS, "0", "buffer_load_dwordx4 %[v" XS #H "], " UL_RSRC_##X "0")                                  \
    UL_COPY_ONE(LDS, "1", "buffer_load_dwordx4 %[v" XS #H "], " UL_RSRC_##X UL_COFF_##X##1)                        \
    UL_COPY_ONE(LDS, "2", "buffer_load_dwordx4 %[v" XS #H "], " UL_RSRC_##X UL_COFF_##X##2)                        \
    UL_COPY_ONE(LDS, "3", "buffer_load_dwordx4 %[v" XS #H "], " UL_RSRC_##X UL_COFF_##X##3)
// The copy cursor of one operand to the next K tile.
#define UL_NEXT_ROWS_a "s_add_u32 s52, s52, 128\n"
#define UL_NEXT_ROWS_b "s_add_u32 s53, s53, 128\n"
#define UL_NEXT_COLS_a "s_add_u32 s40, s40, %[tal]\ns_addc_u32 s41, s41, %[tah]\n"
#define UL_NEXT_COLS_b "s_add_u32 s44, s44, %[tbl]\ns_addc_u32 s45, s45, %[tbh]\n"
// One K tile fewer to copy.  If none is left, the buffers are empty from now on (and nothing is added to a lane's offset).
#define UL_END_ROWS_a "s_cselect_b32 s52, s52, 0\n"
#define UL_END_ROWS_b "s_cselect_b32 s53, s53, 0\n"
#define UL_END_COLS_a "s_cselect_b32 s54, %[sa1], 0\ns_cselect_b32 s55, %[sa2], 0\ns_cselect_b32 s56, %[sa3], 0\n"
#define UL_END_COLS_b "s_cselect_b32 s57, %[sb1], 0\ns_cselect_b32 s58, %[sb2], 0\ns_cselect_b32 s59, %[sb3], 0\n"
#define UL_COPIES_LEFT(LA, LB)                                                                                 \
    "s_cmp_gt_i32 s49, 0\ns_cselect_b32 s42, %[ea], 0\ns_cselect_b32 s46, %[eb], 0\n"                          \
    UL_END_##LA##_a UL_END_##LB##_b "s_sub_u32 s49, s49, 1\n"

#define UL_REPEAT(BODY) ".set n,0\n.rept 32\n" BODY ".set n,n+1\n.endr\n"
#define UL_ONLY_COPY(C)                                                                                        \
    UL_REPEAT(C ".if (n==" UL_COPY_AT("0") ")||(n==" UL_COPY_AT("1") ")||(n==" UL_COPY_AT("2") ")||(n==" UL_COPY_AT("3") ")\ns_nop 0\n.endif\n")
#define UL_READS_DONE "s_waitcnt lgkmcnt(0)\n"
#define UL_BARRIER "s_waitcnt vmcnt(16) lgkmcnt(0)\ns_barrier\n"
// A part over j1 column blocks: it leaves after the last one.  Reads and copies stand in the first block's eight MFMAs, two steps
// of each after an MFMA.  A read stands between the two steps of the copies (either layout has one at every odd n below
// 16), so that a write of m0 in the first is not followed at once by its copy.
#define UL_SHORT_PART(M, RD, CP)                                                                               \
    ".set n,0\n.rept 8\n" M ".set m,n\n.set n,2*m\n" RD ".set n," UL_COPY_FIRST "+2*m-2\n" CP                    \
    ".set n,2*m+1\n" RD ".set n," UL_COPY_FIRST "+2*m-1\n" CP ".set n,m+1\n.endr\n"                              \
    ".rept 3\ns_cmp_le_u32 %[j1], n/8\ns_cbranch_scc1 5f\n.rept 8\n" M ".set n,n+1\n.endr\n.endr\n5:\n"

// Byte offsets of the halves in LDS: A half h of stage s at 32768 s + 16384 h, B 65536 further (its read addresses include that).
#define UL_PART0(LA, LB, FX, FY, S, T) \
    UL_REPEAT(UL_MFMA("160", FY, "4", "0") UL_READ_##LB("b", FX, S) UL_COPY_##LA("a", a, 1, T "+16384")) UL_NEXT_##LA##_a UL_COPIES_LEFT(LA, LB) UL_READS_DONE
#define UL_PART1(M, LA, LB, FX, FY, S) \
    UL_REPEAT(M("128", FX, "0", "0") UL_READ1_##LB(FY, S "+16384") UL_COPY_##LA("a", a, 0, S)) UL_BARRIER
#define UL_PART2(M, LA, LB, FX, FY, S) \
    UL_REPEAT(M("128", FY, "0", "4") UL_READ_##LA("a", "160", S "+16384") UL_COPY_##LB("b", b, 0, S "+65536")) UL_READS_DONE
#define UL_PART3(M, LA, LB, FX, FY, S, T) \
    UL_REPEAT(M("160", FY, "4", "4") UL_READ_##LA("a", "128", T) UL_COPY_##LB("b", b, 1, S "+65536+16384")) UL_NEXT_##LB##_b UL_BARRIER
#define UL_PART2S(M, LA, LB, FX, FY, S) \
    UL_SHORT_PART(M("128", FY, "0", "4"), UL_READ_##LA("a", "160", S "+16384"), UL_COPY_##LB("b", b, 0, S "+65536")) UL_READS_DONE
#define UL_PART3S(M, LA, LB, FX, FY, S, T) \
    UL_SHORT_PART(M("160", FY, "4", "4"), UL_READ_##LA("a", "128", T), UL_COPY_##LB("b", b, 1, S "+65536+16384")) UL_NEXT_##LB##_b UL_BARRIER

#define UL_TILE(LA, LB, FX, FY, S, T)                                                                          \
    UL_PART0(LA, LB, FX, FY, S, T) UL_PART1(UL_MFMA, LA, LB, FX, FY, S)                                          \
    UL_PART2(UL_MFMA, LA, LB, FX, FY, S) UL_PART3(UL_MFMA, LA, LB, FX, FY, S, T)
#define UL_TILES(LA, LB, FX, FY, S, T)                                                                         \
    UL_PART0(LA, LB, FX, FY, S, T) UL_PART1(UL_MFMA, LA, LB, FX, FY, S)                                          \
    UL_PART2S(UL_MFMA_COLS, LA, LB, FX, FY, S) UL_PART3S(UL_MFMA_COLS, LA, LB, FX, FY, S, T)
#define UL_LEAVE_AFTER_LAST(WHERE) "s_sub_u32 s48, s48, 1\ns_cmp_eq_u32 s48, 0\ns_cbranch_scc1 " WHERE "\n"

// First copies: all of K tile 0 and, if there is one, K tile 1 but for half 1 of A.
#define UL_BEGIN(LA, LB)                                                                                       \
    "s_mov_b64 s[40:41], %[pa]\ns_mov_b32 s42, %[ea]\ns_mov_b32 s43, 0x20000\n"                                 \
    "s_mov_b64 s[44:45], %[pb]\ns_mov_b32 s46, %[eb]\ns_mov_b32 s47, 0x20000\n"                                 \
    "s_mov_b32 s49, %[kt]\ns_mov_b32 s52, 0\ns_mov_b32 s53, 0\n" UL_COPIES_LEFT(LA, LB)                       \
    UL_ONLY_COPY(UL_COPY_##LA("a", a, 0, "0")) UL_ONLY_COPY(UL_COPY_##LB("b", b, 0, "65536"))               \
    UL_ONLY_COPY(UL_COPY_##LB("b", b, 1, "65536+16384")) UL_ONLY_COPY(UL_COPY_##LA("a", a, 1, "16384"))     \
    UL_NEXT_##LA##_a UL_NEXT_##LB##_b UL_COPIES_LEFT(LA, LB)                                                           \
    UL_ONLY_COPY(UL_COPY_##LA("a", a, 0, "32768")) UL_ONLY_COPY(UL_COPY_##LB("b", b, 0, "65536+32768"))     \
    UL_ONLY_COPY(UL_COPY_##LB("b", b, 1, "65536+16384+32768"))

// The rest.  The accumulators of piece (1, 0), whose first MFMAs stand in the loop, are cleared during the first reads.
// pa, pb: the cursors where UL_BEGIN left them, but for B's, which is one K tile further.
#define UL_MAIN(LA, LB)                                                                                        \
    "s_mov_b64 s[40:41], %[pa]\ns_mov_b32 s42, %[ea]\ns_mov_b32 s43, 0x20000\n"                                 \
    "s_mov_b64 s[44:45], %[pb]\ns_mov_b32 s46, %[eb]\ns_mov_b32 s47, 0x20000\n"                                 \
    "s_mov_b32 s48, %[kt]\ns_sub_u32 s49, %[kt], 1\ns_mov_b32 s52, 128\ns_mov_b32 s53, 256\n"                    \
    UL_COPIES_LEFT(LA, LB)                                                                                             \
    UL_BARRIER                                                                                                 \
    UL_REPEAT(UL_READ_##LA("a", "128", "0")) UL_REPEAT(UL_READ_##LB("b", "192", "0"))                           \
    UL_ONLY_COPY(UL_COPY_##LA("a", a, 1, "32768+16384")) UL_NEXT_##LA##_a UL_COPIES_LEFT(LA, LB)                      \
    ".set n,0\n.rept 64\nv_accvgpr_write_b32 a[(4+n/16)*32+n%%16], 0\n.set n,n+1\n.endr\n"                       \
    "s_waitcnt lgkmcnt(0)\ns_barrier\n"                                                                        \
    "s_cmp_lt_u32 %[j1], 4\ns_cbranch_scc1 11f\n"                                                              \
    UL_PART1(UL_MFMA_NEW, LA, LB, "192", "224", "0") UL_PART2(UL_MFMA_NEW, LA, LB, "192", "224", "0")           \
    UL_PART3(UL_MFMA_NEW, LA, LB, "192", "224", "0", "32768")                                                  \
    "1:\n" UL_LEAVE_AFTER_LAST("2f") UL_TILE(LA, LB, "224", "192", "32768", "0")                                \
    UL_LEAVE_AFTER_LAST("3f") UL_TILE(LA, LB, "192", "224", "0", "32768") "s_branch 1b\n"                       \
    "11:\n"                                                                                                    \
    UL_PART1(UL_MFMA_NEW, LA, LB, "192", "224", "0") UL_PART2S(UL_MFMA_COLS_NEW, LA, LB, "192", "224", "0")     \
    UL_PART3S(UL_MFMA_COLS_NEW, LA, LB, "192", "224", "0", "32768")                                            \
    "12:\n" UL_LEAVE_AFTER_LAST("2f") UL_TILES(LA, LB, "224", "192", "32768", "0")                              \
    UL_LEAVE_AFTER_LAST("3f") UL_TILES(LA, LB, "192", "224", "0", "32768") "s_branch 12b\n"                     \
    "2:\n" UL_REPEAT(UL_MFMA("160", "192", "4", "0")) "s_branch 4f\n"                                          \
    "3:\n" UL_REPEAT(UL_MFMA("160", "224", "4", "0"))                                                          \
    "4:\ns_waitcnt vmcnt(0)\ns_barrier\ns_nop 15\ns_nop 15\n"

// Operands of the blocks for `this` of a TileLarge.
#define UL_IN [sw] "s"(lds_base + 1024u * wave), [kt] "s"(kt), [ea] "s"(a.extent), [eb] "s"(b.extent)
#define UL_IN_COPY_ROWS_A [va] "v"(a.voff[0]), [ga] "s"((uint32_t)a.row_step), [ha] "s"((uint32_t)(4 * a.row_step))
#define UL_IN_COPY_ROWS_B [vb] "v"(b.voff[0]), [gb] "s"((uint32_t)b.row_step), [hb] "s"((uint32_t)(4 * b.row_step))
#define UL_IN_COPY_COLS_A [va0] "v"(a.voff[0]), [va1] "v"(a.voff[1]), [sa1] "s"((uint32_t)a.row_step), [sa2] "s"((uint32_t)(2 * a.row_step)), \
        [sa3] "s"((uint32_t)(3 * a.row_step)), [tal] "s"((uint32_t)a.step), [tah] "s"((uint32_t)(a.step >> 32))
#define UL_IN_COPY_COLS_B [vb0] "v"(b.voff[0]), [vb1] "v"(b.voff[1]), [sb1] "s"((uint32_t)b.row_step), [sb2] "s"((uint32_t)(2 * b.row_step)), \
        [sb3] "s"((uint32_t)(3 * b.row_step)), [tbl] "s"((uint32_t)b.step), [tbh] "s"((uint32_t)(b.step >> 32))
#define UL_IN_READ_ROWS_A [ra0] "v"(lds_base + a.roff[0]), [ra1] "v"(lds_base + a.roff[1])
#define UL_IN_READ_COLS_A UL_IN_READ_ROWS_A, [ra2] "v"(lds_base + a.roff[2]), [ra3] "v"(lds_base + a.roff[3])
#define UL_IN_READ_ROWS_B [rb0] "v"(lds_base + 65536u + b.roff[0]), [rb1] "v"(lds_base + 65536u + b.roff[1]), \
        [ry0] "v"(lds_base + 65536u + b.roff[0] + y_shift), [ry1] "v"(lds_base + 65536u + b.roff[1] + y_shift)
#define UL_IN_READ_COLS_B [rb0] "v"(lds_base + 65536u + b.roff[0]), [rb1] "v"(lds_base + 65536u + b.roff[1]), \
        [rb2] "v"(lds_base + 65536u + b.roff[2]), [rb3] "v"(lds_base + 65536u + b.roff[3])
#define UL_CLOBBERS "memory", "scc", "vcc", "m0", "s40", "s41", "s42", "s43", "s44", "s45", "s46", "s47", "s48", "s49", "s52", "s53", \
        "s54", "s55", "s56", "s57", "s58", "s59", "v94", "v95"
// Eight values of the caller in registers that the block does not write.
#define UL_KEPT(X, r0, r1, r2, r3, r4, r5, r6, r7)                                                             \
    "{v" #r0 "}"(X[0]), "{v" #r1 "}"(X[1]), "{v" #r2 "}"(X[2]), "{v" #r3 "}"(X[3]),                              \
    "{v" #r4 "}"(X[4]), "{v" #r5 "}"(X[5]), "{v" #r6 "}"(X[6]), "{v" #r7 "}"(X[7])
// Accumulator block (i, j) is a[32 i + 4 j : 32 i + 4 j + 3]: X(i, j, first, last).
#define UL_BLOCKS(X) \
    X(0, 0, 0, 3) X(0, 1, 4, 7) X(0, 2, 8, 11) X(0, 3, 12, 15) X(0, 4, 16, 19) X(0, 5, 20, 23) X(0, 6, 24, 27) X(0, 7, 28, 31) \
    X(1, 0, 32, 35) X(1, 1, 36, 39) X(1, 2, 40, 43) X(1, 3, 44, 47) X(1, 4, 48, 51) X(1, 5, 52, 55) X(1, 6, 56, 59) X(1, 7, 60, 63) \
    X(2, 0, 64, 67) X(2, 1, 68, 71) X(2, 2, 72, 75) X(2, 3, 76, 79) X(2, 4, 80, 83) X(2, 5, 84, 87) X(2, 6, 88, 91) X(2, 7, 92, 95) \
    X(3, 0, 96, 99) X(3, 1, 100, 103) X(3, 2, 104, 107) X(3, 3, 108, 111) X(3, 4, 112, 115) X(3, 5, 116, 119) X(3, 6, 120, 123) X(3, 7, 124, 127) \
    X(4, 0, 128, 131) X(4, 1, 132, 135) X(4, 2, 136, 139) X(4, 3, 140, 143) X(4, 4, 144, 147) X(4, 5, 148, 151) X(4, 6, 152, 155) X(4, 7, 156, 159) \
    X(5, 0, 160, 163) X(5, 1, 164, 167) X(5, 2, 168, 171) X(5, 3, 172, 175) X(5, 4, 176, 179) X(5, 5, 180, 183) X(5, 6, 184, 187) X(5, 7, 188, 191) \
    X(6, 0, 192, 195) X(6, 1, 196, 199) X(6, 2, 200, 203) X(6, 3, 204, 207) X(6, 4, 208, 211) X(6, 5, 212, 215) X(6, 6, 216, 219) X(6, 7, 220, 223) \
    X(7, 0, 224, 227) X(7, 1, 228, 231) X(7, 2, 232, 235) X(7, 3, 236, 239) X(7, 4, 240, 243) X(7, 5, 244, 247) X(7, 6, 248, 251) X(7, 7, 252, 255)
#define UL_OUT(i, j, lo, hi) "={a[" #lo ":" #hi "]}"(acc[i][j]),
// The four values of block (I, J) into x.  The compiler would move all accumulators out at once where they are used.
#define UL_TAKE(i, j, lo, hi)                                                                                  \
    if constexpr (I == i && J == j)                                                                            \
        asm volatile("v_accvgpr_read_b32 %0, a[" #lo "]\nv_accvgpr_read_b32 %1, a[" #lo "+1]\n"                 \
                     "v_accvgpr_read_b32 %2, a[" #lo "+2]\nv_accvgpr_read_b32 %3, a[" #lo "+3]"                  \
                     : "=v"(x[0]), "=v"(x[1]), "=v"(x[2]), "=v"(x[3]) : "{a[" #lo ":" #hi "]}"(acc[i][j]));
// z = accumulator number p (4 i + r; -1: none) of column block J, skipped where no lane of the wave has one.
#define UL_PICK(j, A0, A1, B0, B1, C0, C1, D0, D1, E0, E1, F0, F1, G0, G1, H0, H1)                              \
    if constexpr (J == j)                                                                                      \
        asm volatile("v_cmp_le_i32 vcc, 0, %1\ns_cbranch_vccz 7f\n.set n,0\n.rept 32\n"                        \
                     "v_accvgpr_read_b32 %2, a[(n/4)*32+" #j "*4+n%%4]\nv_cmp_eq_u32 vcc, n, %1\n"              \
                     "v_cndmask_b32 %0, %0, %2, vcc\n.set n,n+1\n.endr\n7:"                                    \
                     : "+v"(z), "+v"(p), "=&v"(t)                                                              \
                     : "{a[" #A0 ":" #A1 "]}"(acc[0][j]), "{a[" #B0 ":" #B1 "]}"(acc[1][j]), "{a[" #C0 ":" #C1 "]}"(acc[2][j]), \
                       "{a[" #D0 ":" #D1 "]}"(acc[3][j]), "{a[" #E0 ":" #E1 "]}"(acc[4][j]), "{a[" #F0 ":" #F1 "]}"(acc[5][j]), \
                       "{a[" #G0 ":" #G1 "]}"(acc[6][j]), "{a[" #H0 ":" #H1 "]}"(acc[7][j])                     \
                     : "vcc");
#define UL_COLUMNS(X)                                                                                          \
    X(0, 0, 3, 32, 35, 64, 67, 96, 99, 128, 131, 160, 163, 192, 195, 224, 227) \
    X(1, 4, 7, 36, 39, 68, 71, 100, 103, 132, 135, 164, 167, 196, 199, 228, 231) \
    X(2, 8, 11, 40, 43, 72, 75, 104, 107, 136, 139, 168, 171, 200, 203, 232, 235) \
    X(3, 12, 15, 44, 47, 76, 79, 108, 111, 140, 143, 172, 175, 204, 207, 236, 239) \
    X(4, 16, 19, 48, 51, 80, 83, 112, 115, 144, 147, 176, 179, 208, 211, 240, 243) \
    X(5, 20, 23, 52, 55, 84, 87, 116, 119, 148, 151, 180, 183, 212, 215, 244, 247) \
    X(6, 24, 27, 56, 59, 88, 91, 120, 123, 152, 155, 184, 187, 216, 219, 248, 251) \
    X(7, 28, 31, 60, 63, 92, 95, 124, 127, 156, 159, 188, 191, 220, 223, 252, 255)

#endif
