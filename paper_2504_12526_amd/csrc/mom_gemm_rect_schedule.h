// The stage schedule of the rectangular GEMM tiles (mom_gemm_rect.hip.inc), as data that the kernel and a host program
// (tests/rect_schedule_check.cpp) ask.  Plain C++17, no HIP types.
//
// A stage is 64 K-elements of both operand tiles: MB 16-row token blocks and NB 16-row weight blocks per wavefront, MB x NB
// pairs of MFMAs (K-half 0, then K-half 1 into the same accumulator block).  The operand with more blocks is the OUTER one:
// a row of the stage is one outer block by all inner ones, an outer block's two fragments are free once its row is done and
// take those of the next stage there, and the inner fragments are double-buffered by stage parity: 8 outer + 16 inner
// registers per lane.  Each operand has its own LDS ring: stage T of operand op lives in slot T % slots(op).
#ifndef MOM_GEMM_RECT_SCHEDULE_H
#define MOM_GEMM_RECT_SCHEDULE_H

#if defined(__HIPCC__)
#define MOM_RECT_FN __host__ __device__ constexpr
#else
#define MOM_RECT_FN constexpr
#endif

namespace momk {
namespace rect {

enum Operand { TOK = 0, WGT = 1, NONE = 2 };

MOM_RECT_FN int blocks(int MB, int NB, int op) { return op == TOK ? MB : NB; }
MOM_RECT_FN int outer(int MB, int NB) { return NB > MB ? WGT : TOK; }
MOM_RECT_FN int outer_blocks(int MB, int NB) { return blocks(MB, NB, outer(MB, NB)); }
MOM_RECT_FN int inner_blocks(int MB, int NB) { return blocks(MB, NB, 1 - outer(MB, NB)); }

// Ring slots of an operand; a tile row of a stage is 128 bytes, and LDS holds 1280 of them.  Three of each where they fit:
// then both tiles of the stage two ahead are in flight at the stage barrier.  Else three of one operand, of the larger
// one where that fits (a CU has 256 rows in flight at most, and the three-slot tile is what is in flight there).
constexpr int kLdsRows = 1280;
MOM_RECT_FN int slots(int MB, int NB, int op) {
    const int tm = 32 * MB, tn = 32 * NB;
    if (3 * (tm + tn) <= kLdsRows) return 3;
    const int large = tn > tm ? WGT : TOK;
    const int l = tn > tm ? tn : tm, s = tn > tm ? tm : tn;
    const int three = 3 * l + 2 * s <= kLdsRows ? large : 1 - large;
    return op == three ? 3 : 2;
}
MOM_RECT_FN int ring_rows(int MB, int NB) { return slots(MB, NB, TOK) * 32 * MB + slots(MB, NB, WGT) * 32 * NB; }
MOM_RECT_FN int period(int, int) { return 6; }       // stages after which slots and buffer parity repeat

// The stage barrier (s_waitcnt for own ring loads and LDS reads, then s_barrier) sits in front of row 1 of stage T.  Behind
// it stage T+1 is in LDS whole, and the slots of stage T are free: their last fragments were read in row 0.
MOM_RECT_FN int barrier_row() { return 1; }

// Ring loads: those of a stage are spread evenly over its pairs from row 1 on and row 0 of the next stage, the loads of the
// operand with fewer slots first (they are due first).  Operand op of stage T + slots(op) goes into the slot of stage T.
MOM_RECT_FN int first_operand(int MB, int NB) { return slots(MB, NB, TOK) < slots(MB, NB, WGT) ? TOK : WGT; }
struct Load { int op, index; };
MOM_RECT_FN Load load_number(int MB, int NB, int j) {
    const int f = first_operand(MB, NB), n = blocks(MB, NB, f);
    return j < n ? Load{f, j} : Load{1 - f, j - n};
}
MOM_RECT_FN Load ring_load(int MB, int NB, int row, int pair) {
    const int OB = outer_blocks(MB, NB), IB = inner_blocks(MB, NB), P = OB * IB, L = MB + NB;
    const int p = (row + OB - 1) % OB * IB + pair;
    const int j = (p * L + P - 1) / P;
    if (j >= L || j * P / L != p) return {NONE, 0};
    return load_number(MB, NB, j);
}
// The first ring load of a stage that is issued in row 0 of the next one.
MOM_RECT_FN int first_load_of_row_0(int MB, int NB) {
    const int OB = outer_blocks(MB, NB), IB = inner_blocks(MB, NB), P = OB * IB, L = MB + NB;
    int j = 0;
    while (j < L && j * P / L < (OB - 1) * IB) ++j;
    return j;
}
// ... and this many of the youngest ring loads may be in flight behind the barrier: those of operands with three slots.
MOM_RECT_FN int barrier_loads_in_flight(int MB, int NB) {
    return (slots(MB, NB, TOK) == 3 ? MB : 0) + (slots(MB, NB, WGT) == 3 ? NB : 0);
}

// Position A of a pair (between its MFMAs), pair 0 of a row: the outer block that takes the next stage's fragments (ahead 1);
// row 0: the last block of the stage itself (ahead 0).
struct OuterRead { int block, ahead; };
MOM_RECT_FN OuterRead outer_read(int MB, int NB, int row) {
    return row == 0 ? OuterRead{outer_blocks(MB, NB) - 1, 0} : OuterRead{row - 1, 1};
}
// Position A of pair (row, pair): the inner fragments [begin, end) of stage T + 1 (fragment q: K-half q % 2 of block q / 2),
// spread evenly over the rows from row 1 on, behind the first MFMAs of pairs 1, 2, ... of a row (smeared over all pairs:
// 1 % slower at 8192 rows, 256 x 256 tiles).
struct InnerReads { int begin, end; };
MOM_RECT_FN InnerReads inner_reads(int MB, int NB, int row, int pair) {
    const int OB = outer_blocks(MB, NB), IB = inner_blocks(MB, NB), R = 2 * IB;
    if (row < 1 || pair < 1) return {0, 0};
    const int b = ((row - 1) * R + OB - 2) / (OB - 1), e = (row * R + OB - 2) / (OB - 1);      // of this row
    const int from = b + pair - 1, to = pair == IB - 1 ? e : from + 1;
    return {from, to < e ? to : e};
}

// Prologue: whole tiles in this order; of the last, what row 0 of stage 0 does not load.  The wait that follows lets all loads
// behind those of stage 0 stay in flight.
struct PrologueTile { int op, stage; };
MOM_RECT_FN int prologue_tiles(int MB, int NB) { return slots(MB, NB, TOK) + slots(MB, NB, WGT); }
MOM_RECT_FN PrologueTile prologue_tile(int MB, int NB, int i) {
    const int f = first_operand(MB, NB);
    if (i == 4 && slots(MB, NB, f) == 2) return {1 - f, 2};
    return {i % 2 ? 1 - f : f, i / 2};
}
MOM_RECT_FN int prologue_loads(int MB, int NB) {
    return slots(MB, NB, TOK) * MB + slots(MB, NB, WGT) * NB - (MB + NB - first_load_of_row_0(MB, NB));
}
MOM_RECT_FN int prologue_loads_in_flight(int MB, int NB) { return prologue_loads(MB, NB) - (MB + NB); }

}  // namespace rect
}  // namespace momk

#endif  // MOM_GEMM_RECT_SCHEDULE_H
