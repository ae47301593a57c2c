// Host-side check of the stage schedule of the rectangular GEMM tiles (csrc/mom_gemm_rect_schedule.h): walks a prologue and
// many stages as one wavefront executes them (mom_gemm_rect.hip.inc) and checks, for every tile form,
//   1. every tile of every stage is loaded block by block exactly once, with the operand pointer at its stage;
//   2. a fragment is read only behind a barrier whose s_waitcnt covered the loads of its tile (they complete in order);
//   3. a ring slot is loaded into only behind a barrier that follows the last read of what it held;
//   4. at every MFMA both operand registers hold the stage being multiplied.
#include <cstdio>
#include <map>
#include <tuple>
#include <vector>

#include "mom_gemm_forms.h"
#include "mom_gemm_rect_schedule.h"

namespace re = momk::rect;
typedef std::tuple<int, int, int> Key;

static int check(int MB, int NB) {
    const int OUT = re::outer(MB, NB), OB = re::outer_blocks(MB, NB), IB = re::inner_blocks(MB, NB), STAGES = 24;
    int slots[2] = {re::slots(MB, NB, 0), re::slots(MB, NB, 1)}, ptr[2] = {0, 0}, bad = 0;
    auto fail = [&](const char* what, int a = 0, int b = 0, int c = 0) {
        if (!bad++) std::printf("%d x %d: %s (%d, %d, %d)\n", 32 * MB, 32 * NB, what, a, b, c);
    };
    if (re::ring_rows(MB, NB) > re::kLdsRows) fail("LDS");
    if (slots[0] < 2 || slots[1] < 2 || 6 % slots[0] || 6 % slots[1] || re::period(MB, NB) != 6) fail("slots do not repeat");
    int issued = 0, landed = 0, barrier = 0;                 // ring loads; number of the last barrier
    std::map<Key, int> load;                                 // (operand, stage, block) -> number of its load
    std::map<std::pair<int, int>, int> holds, last_read;     // (operand, slot) -> stage; barrier that preceded the last read
    std::map<Key, int> reg;                                  // fragment register -> stage
    auto dma = [&](int op, int i, int slot) {
        const int stage = ptr[op];
        if (i < 0 || i >= re::blocks(MB, NB, op)) return fail("index of a ring load", op, i);
        if (slot != stage % slots[op]) fail("slot of a ring load", op, stage, slot);
        if (!load.insert({Key(op, stage, i), issued++}).second) fail("block loaded twice", op, stage, i);
        auto& h = holds[{op, slot}];
        auto r = last_read.find({op, slot});
        if (h != stage && r != last_read.end() && r->second >= barrier) fail("slot overwritten while it may be read", op, stage, slot);
        if (h != stage && stage >= slots[op] && h != stage - slots[op]) fail("stage left out", op, stage, h);
        h = stage;
    };
    auto frag = [&](int op, int kh, int block, int stage, int buf) {
        const int slot = stage % slots[op];
        if (block < 0 || block >= re::blocks(MB, NB, op)) return fail("fragment block", op, block);
        if (holds[{op, slot}] != stage) fail("slot holds another stage", op, stage, slot);
        for (int i = 0; i < re::blocks(MB, NB, op); ++i) {
            auto l = load.find(Key(op, stage, i));
            if (l == load.end() || l->second >= landed) return fail("fragment read before its tile has landed", op, stage, i);
        }
        last_read[{op, slot}] = barrier;
        reg[Key(op * 4 + kh * 2 + buf, block, 0)] = stage;
    };
    auto use = [&](int op, int kh, int block, int stage, int buf) {
        if (reg[Key(op * 4 + kh * 2 + buf, block, 0)] != stage) fail("operand register holds another stage", op, block, stage);
    };
    for (auto& s : {0, 1}) for (int i = 0; i < 3; ++i) holds[{s, i}] = -1;
    int n = 0;
    for (int t = 0; t < re::prologue_tiles(MB, NB); ++t) {
        const re::PrologueTile p = re::prologue_tile(MB, NB, t);
        ptr[p.op] = p.stage;
        for (int i = 0; i < re::blocks(MB, NB, p.op); ++i)
            if (n < re::prologue_loads(MB, NB)) { dma(p.op, i, p.stage); ++n; }
    }
    ptr[0] = slots[0] - 1; ptr[1] = slots[1] - 1;
    landed = issued - re::prologue_loads_in_flight(MB, NB);
    ++barrier;
    for (int kh = 0; kh < 2; ++kh) {
        for (int i = 0; i < IB; ++i) frag(1 - OUT, kh, i, 0, 0);
        for (int o = 0; o + 1 < OB; ++o) frag(OUT, kh, o, 0, 0);
    }
    int in_flight_max = 0;
    for (int T = 0; T < STAGES; ++T)
        for (int row = 0; row < OB; ++row) {
            if (row == re::barrier_row()) {
                landed = issued - re::barrier_loads_in_flight(MB, NB);
                ++barrier;
                ptr[0] = T + slots[0]; ptr[1] = T + slots[1];
            }
            for (int i = 0; i < IB; ++i) {
                for (int kh = 0; kh < 2; ++kh) {
                    use(OUT, kh, row, T, 0);
                    use(1 - OUT, kh, i, T, T % 2);
                    if (kh) continue;
                    const re::OuterRead r = re::outer_read(MB, NB, row);
                    // (both K-halves' registers of the block are free once its row is done)
                    if (i == 0) {
                        if (r.block == row && OB > 1) fail("outer fragment refilled in its own row", row);
                        for (int k = 0; k < 2; ++k) frag(OUT, k, r.block, T + r.ahead, 0);
                    }
                    const re::InnerReads q = re::inner_reads(MB, NB, row, i);
                    for (int k = q.begin; k < q.end; ++k) frag(1 - OUT, k % 2, k / 2, T + 1, (T + 1) % 2);
                }
                const re::Load l = re::ring_load(MB, NB, row, i);
                if (l.op != re::NONE) dma(l.op, l.index, (row == 0 ? T + 5 : T) % slots[l.op]);
            }
            if (issued - landed > in_flight_max) in_flight_max = issued - landed;
        }
    for (int op = 0; op < 2; ++op)
        for (int T = 0; T < STAGES; ++T)
            for (int i = 0; i < re::blocks(MB, NB, op); ++i)
                if (!load.count(Key(op, T, i))) fail("block never loaded", op, T, i);
    if (re::prologue_loads_in_flight(MB, NB) > 63 || re::barrier_loads_in_flight(MB, NB) > 63) fail("s_waitcnt counts to 63");
    return bad;
}

int main() {
    int bad = 0, forms = 0;
#define RECT(TM, TN) bad += check(TM / 32, TN / 32); ++forms;
    MOM_RECT_FORMS_DOWN(RECT)
    MOM_RECT_FORMS_GATEUP(RECT)
    std::printf("%d forms: %s\n", forms, bad ? "FAILED" : "ok");
    return bad != 0;
}
