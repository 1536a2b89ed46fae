// The scalar path's hot loop: threaded code for the instructions that make up
// almost all of a cartridge's work, written as one block of gfx950 assembly.
//
// What it computes: the same instructions, in the same order, as run_fast's
// full dispatch (interp.hip) -- the wave's group of lanes stands at one place,
// so program counter, cycle and row-log position are scalars and only A, X, Y,
// the flags, RAM, TIA registers and log stores are per lane.
//
// What bounds it: the latency of one wave's instruction stream (at most one
// wave per SIMD runs, and each pass depends on the one before).  On gfx950 an
// instruction issues every 4 cycles, a taken branch to another cache line
// costs 40-80 (instruction fetch), a scalar load that hits 40, an LDS read 60.
// A compiled loop takes several far branches per pass (compare chain, skipped
// cases, back edge: 471 cycles a pass on the plain step); here a handler ends
// by jumping straight to the next instruction's handler, so a pass has one.
//
// How it is laid out:
//  * a predecoded word (k_predecode) holds its handler's slot: handler address
//    = block base + (word & 0x7F80), 128-byte slots;
//  * every handler loads the next instruction's word as early as it can, does
//    its work while the load is in flight, waits once, and jumps.  An LDS read
//    nothing in the handler needs is issued after that wait and lands while
//    the next handler starts (whose own wait comes before it touches A, X, Y
//    or the flags);
//  * one scalar (ACC) counts the cycle inside the scanline in its top 7 bits,
//    biased so that passing cycle 75 carries out, and the instructions run in
//    the rest: one addition does both, and its carry selects the line-change
//    code instead of the handler (s_cselect, no branch).  The frame's cycle
//    cap is a line boundary, so it is checked only there;
//  * flags are kept unpacked: nz (Z: low byte is 0; N: bit 7 or 8), carry 0/1,
//    overflow in bit 7;
//  * lines, rows and the cap are one counter: L = lines left until the cap,
//    and the frame row of the current line is 286 - L.
//
// It stops before an instruction it does not cover (any word whose slot is
// HOT_REAL), a branch whose lanes part, a store whose effect falls on the next
// line or finds its log row full, and after a WSYNC when the group is not the
// whole wave.  Decimal mode is off in every lane on entry and nothing here
// turns it on.
//
// Every wait that a load needs is inside the block, in the handler that uses
// the value or before the block's end.
#pragma once

namespace vcs {

// Slots, and the opcode each runs (HOT_REAL: the word carries it).  Zero-page
// operands are RAM; a store to a TIA register that is kept as is, or to GRP0 /
// GRP1 (with the delayed copies), has three slots for its length; HOT_WSYNC
// and HOT_ST_NOP (nothing emulated changes) stand for a store of A, X or Y; the
// *_X branches cross a page when taken.
constexpr uint32_t HOT_REAL = 0, HOT_STA_TIA = 1, HOT_STA_GRP0 = 4, HOT_STA_GRP1 = 7, HOT_STX_TIA = 10, HOT_STX_GRP0 = 11, HOT_STX_GRP1 = 12, HOT_STY_TIA = 13, HOT_STY_GRP0 = 14, HOT_STY_GRP1 = 15,
                   HOT_WSYNC = 16, HOT_ST_NOP = 17, HOT_BPL_X = 18, HOT_BMI_X = 19, HOT_BVC_X = 20, HOT_BVS_X = 21, HOT_BCC_X = 22, HOT_BCS_X = 23, HOT_BNE_X = 24, HOT_BEQ_X = 25;
constexpr uint32_t kHotSlots = 84;
constexpr uint8_t kHotSlotOp[kHotSlots] = {
    0x00, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x86, 0x86, 0x86, 0x84, 0x84, 0x84,
    0x85, 0x85, 0x10, 0x30, 0x50, 0x70, 0x90, 0xB0, 0xD0, 0xF0, 0x05, 0x06, 0x09, 0x0A, 0x10, 0x18,
    0x24, 0x25, 0x26, 0x29, 0x2A, 0x30, 0x38, 0x45, 0x46, 0x49, 0x4A, 0x4C, 0x50, 0x65, 0x66, 0x69,
    0x6A, 0x70, 0x84, 0x85, 0x86, 0x88, 0x8A, 0x90, 0x98, 0xA0, 0xA2, 0xA4, 0xA5, 0xA6, 0xA8, 0xA9,
    0xAA, 0xB0, 0xB8, 0xC0, 0xC4, 0xC5, 0xC6, 0xC8, 0xC9, 0xCA, 0xD0, 0xD8, 0xE0, 0xE4, 0xE5, 0xE6,
    0xE8, 0xE9, 0xEA, 0xF0,
};
// The slot that runs opcode `op` without a page-crossing branch or a TIA store
// (HOT_REAL: none).
constexpr uint32_t hot_slot(uint32_t op) {
    for (uint32_t s = HOT_BEQ_X + 1; s < kHotSlots; ++s)
        if (kHotSlotOp[s] == op) return s;
    return HOT_REAL;
}

// ACC: cycle in the line + 52 in the top 7 bits, instructions below
constexpr uint32_t kAccBias = 52, kAccShift = 25, kAccCount = (1u << kAccShift) - 1;

// what ended the block
constexpr uint32_t HOT_EXIT_NEXT = 0;     // before the instruction at PO
constexpr uint32_t HOT_EXIT_LINE = 1;     // after a WSYNC: a partial group stops, or the cap is reached

#define HL_ORG(slot) ".org .Lhb%= + 128*" #slot "\n"
// advance to the next instruction and load its word
#define HL_FETCH(len)                         \
    "s_add_u32 s72, s72, 4*" #len "\n"        \
    "s_load_dword s74, s[70:71], s72\n"
#define HL_WAIT "s_waitcnt lgkmcnt(0)\n"
// the next handler's address (after the wait)
#define HL_TGT                                \
    "s_and_b32 s76, s74, 0x7f80\n"            \
    "s_add_u32 s76, s76, s78\n"
// count the instruction and its cycles, go on (to the line change on carry)
#define HL_GO(cyc)                                    \
    "s_add_u32 s73, s73, (" #cyc "<<25)+1\n"          \
    "s_cselect_b32 s76, s79, s76\n"                   \
    "s_setpc_b64 s[76:77]\n"
#define HL_B1_7 "s_bfe_u32 s87, s74, 0x70010\n"       // zero-page RAM offset
#define HL_B1_8 "s_bfe_u32 s87, s74, 0x80010\n"       // immediate
#define HL_RAMADDR "v_add_u32 v122, s87, %[ram]\n"

// implied: `work` after the wait
#define HL_IMP(slot, work) HL_ORG(slot) HL_FETCH(1) HL_WAIT work HL_TGT HL_GO(2)
// immediate: operand in s87
#define HL_IMM(slot, work) HL_ORG(slot) HL_B1_8 HL_FETCH(2) HL_WAIT work HL_TGT HL_GO(2)
// zero-page read whose result the handler needs: operand in v123
#define HL_ZPR(slot, work)                                                                        \
    HL_ORG(slot) HL_B1_7 HL_RAMADDR "ds_read_u8 v123, v122\n" HL_FETCH(2) HL_WAIT work HL_TGT HL_GO(3)
// zero-page load: lands in the register and nz during the next handler
#define HL_ZPL(slot, reg)                                                                         \
    HL_ORG(slot) HL_B1_7 HL_FETCH(2) HL_RAMADDR HL_WAIT                                           \
    "ds_read_u8 " reg ", v122\n"                                                                  \
    "ds_read_u8 %[nz], v122\n" HL_TGT HL_GO(3)
#define HL_ZPS(slot, reg)                                                                         \
    HL_ORG(slot) HL_B1_7 HL_FETCH(2) HL_RAMADDR HL_WAIT "ds_write_b8 v122, " reg "\n" HL_TGT HL_GO(3)
// read-modify-write of zero-page RAM: `work` takes v123 to the new value there
#define HL_ZPM(slot, work)                                                                        \
    HL_ORG(slot) HL_B1_7 HL_RAMADDR "ds_read_u8 v123, v122\n" HL_FETCH(2) HL_WAIT work            \
    "ds_write_b8 v122, v123\n" HL_TGT HL_GO(5)

#define HL_BIT                                             \
    "v_lshlrev_b32 %[v], 1, v123\n"                        \
    "v_and_b32 %[nz], %[a], v123\n"                        \
    "v_and_b32 v124, 0x80, v123\n"                         \
    "v_lshl_or_b32 %[nz], v124, 1, %[nz]\n"
// absolute jump (the target lies in the cartridge window; pc bits 12-15 kept apart)
#define HL_JMP(slot)                                       \
    HL_ORG(slot)                                           \
    "s_lshr_b32 s87, s74, 16\n"                            \
    "s_and_b32 s93, s87, 0xf000\n"                         \
    "s_and_b32 s87, s87, 0xfff\n"                          \
    "s_lshl2_add_u32 s72, s87, s68\n"                      \
    "s_load_dword s74, s[70:71], s72\n" HL_WAIT HL_TGT HL_GO(3)
// WSYNC: on to the next line's start; a write at the line's last cycles, whose
// stall ends a line later, is left to the full dispatch
#define HL_SYNC(slot)                                      \
    HL_ORG(slot)                                           \
    "s_add_u32 s87, s73, 2<<25\n"                          \
    "s_cbranch_scc1 .Lout%=\n" HL_FETCH(2)                 \
    "s_and_b32 s73, s73, 0x1ffffff\n"                      \
    "s_add_u32 s73, s73, (52<<25)+1\n"                     \
    "s_sub_u32 s80, s80, 1\n"                              \
    "s_cmp_le_u32 s80, s81\n"                              \
    "s_cbranch_scc1 .Lsync%=\n" HL_WAIT HL_TGT             \
    "s_setpc_b64 s[76:77]\n"

#define HL_NZ(reg) "v_mov_b32 %[nz], " reg "\n"
// arithmetic on A and operand `m` (a register or s87)
#define HL_AND(m) "v_and_b32 %[a], " m ", %[a]\n" HL_NZ("%[a]")
#define HL_ORA(m) "v_or_b32 %[a], " m ", %[a]\n" HL_NZ("%[a]")
#define HL_EOR(m) "v_xor_b32 %[a], " m ", %[a]\n" HL_NZ("%[a]")
// sum = A + m + C; overflow (A ^ sum) & (m ^ sum) (one three-input boolean)
#define HL_ADC(m)                                          \
    "v_add3_u32 v124, %[a], " m ", %[c]\n"                 \
    "v_bitop3_b32 %[v], %[a], " m ", v124 bitop3:0x42\n"   \
    "v_lshrrev_b32 %[c], 8, v124\n"                        \
    "v_and_b32 %[a], 0xff, v124\n" HL_NZ("%[a]")
// r - m: carry is no borrow
#define HL_CMP(r, m)                                       \
    "v_sub_u32 v124, " r ", " m "\n"                       \
    "v_ashrrev_i32 %[c], 31, v124\n"                       \
    "v_add_u32 %[c], 1, %[c]\n"                            \
    "v_and_b32 %[nz], 0xff, v124\n"
#define HL_CMP_S(r)                                        \
    "v_subrev_u32 v124, s87, " r "\n"                      \
    "v_ashrrev_i32 %[c], 31, v124\n"                       \
    "v_add_u32 %[c], 1, %[c]\n"                            \
    "v_and_b32 %[nz], 0xff, v124\n"
#define HL_INC(r)                                          \
    "v_add_u32 v124, 1, " r "\n"                           \
    "v_and_b32 " r ", 0xff, v124\n" HL_NZ(r)
#define HL_DEC(r)                                          \
    "v_add_u32 v124, -1, " r "\n"                          \
    "v_and_b32 " r ", 0xff, v124\n" HL_NZ(r)
#define HL_ASL(r)                                          \
    "v_lshlrev_b32 v124, 1, " r "\n"                       \
    "v_lshrrev_b32 %[c], 8, v124\n"                        \
    "v_and_b32 " r ", 0xff, v124\n" HL_NZ(r)
#define HL_LSR(r)                                          \
    "v_and_b32 %[c], 1, " r "\n"                           \
    "v_lshrrev_b32 " r ", 1, " r "\n" HL_NZ(r)
#define HL_ROL(r)                                          \
    "v_lshl_or_b32 v124, " r ", 1, %[c]\n"                 \
    "v_lshrrev_b32 %[c], 8, v124\n"                        \
    "v_and_b32 " r ", 0xff, v124\n" HL_NZ(r)
#define HL_ROR(r)                                          \
    "v_lshl_or_b32 v124, %[c], 8, " r "\n"                 \
    "v_and_b32 %[c], 1, " r "\n"                           \
    "v_lshrrev_b32 " r ", 1, v124\n" HL_NZ(r)

// branch: `test` sets vcc in the lanes that take it; taken: cycles' ACC step
// in scalar `tk`.  Both successors' words are loaded before the test is known.
#define HL_BR(slot, test, tk)                              \
    HL_ORG(slot)                                           \
    "s_add_u32 s89, s72, 8\n"                              \
    "s_bfe_i32 s87, s74, 0x80010\n"                        \
    "s_load_dword s74, s[70:71], s89\n"                    \
    "s_lshl2_add_u32 s88, s87, s89\n"                      \
    "s_load_dword s95, s[70:71], s88\n"                    \
    HL_WAIT test                                           \
    "s_cmp_eq_u64 vcc, exec\n"                             \
    "s_cselect_b32 s72, s88, s89\n"                        \
    "s_cselect_b32 s74, s95, s74\n"                        \
    "s_cselect_b32 s87, " tk ", (2<<25)+1\n"               \
    "s_cselect_b64 s[96:97], exec, 0\n"                    \
    "s_cmp_lg_u64 vcc, s[96:97]\n"                         \
    "s_cbranch_scc1 .Lpart%=\n" HL_TGT                     \
    "s_add_u32 s73, s73, s87\n"                            \
    "s_cselect_b32 s76, s79, s76\n"                        \
    "s_setpc_b64 s[76:77]\n"
#define HL_T_NE(mask, src) "v_and_b32 v122, " mask ", " src "\nv_cmp_ne_u32 vcc, 0, v122\n"
#define HL_T_EQ(mask, src) "v_and_b32 v122, " mask ", " src "\nv_cmp_eq_u32 vcc, 0, v122\n"

// TIA register store of v125: count it (a store that ends past the line's end
// is left to the full dispatch), log it in the open row, then `write`.
// s87: register code.  v[120:121]: address of the log entry.
#define HL_TIA_BODY(id, write)                             \
    "s_add_u32 s73, s73, (3<<25)+1\n"                      \
    "s_cbranch_scc1 .Lundo%=\n"                            \
    "s_cmp_eq_u32 s86, 0\n"                                \
    "s_cbranch_scc1 .Lreg" id "%=\n"                       \
    "s_lshr_b32 s88, s73, 25\n"                            \
    "s_sub_u32 s89, 287, s80\n"                            \
    "s_cmp_lg_u32 s89, s75\n"                              \
    "s_cbranch_scc1 .Lrow" id "%=\n"                       \
    ".Lent" id "%=:\n"                                     \
    "s_cmp_ge_u32 s90, s92\n"                              \
    "s_cbranch_scc1 .Lundo%=\n"                            \
    "s_mul_i32 s88, s88, 3\n"                              \
    "s_lshl_b32 s89, s87, 8\n"                             \
    "s_sub_u32 s88, s88, 224\n"                            \
    "s_or_b32 s88, s88, s89\n"                             \
    "v_lshl_add_u64 v[120:121], s[90:91], 2, %[log]\n"     \
    "v_lshl_or_b32 v123, v125, 16, s88\n"                  \
    "global_store_dword v[120:121], v123, off\n"           \
    "s_add_u32 s90, s90, 1\n"                              \
    ".Lreg" id "%=:\n" write HL_TGT                        \
    "s_setpc_b64 s[76:77]\n"                               \
    ".Lrow" id "%=:\n"                                     \
    "s_swappc_b64 s[96:97], s[64:65]\n"                  \
    "s_cbranch_scc0 .Lent" id "%=\n"                       \
    "s_branch .Lreg" id "%=\n"
#define HL_W_TIA "v_add_u32 v122, s87, %[tia]\nds_write_b8 v122, v125\n"
// GRP0 10, GRP1 11, delayed copies 16 / 17, flags 23, ENABL 34 / delayed 35
#define HL_W_GRP0                                          \
    "ds_read_u8 v122, %[tia] offset:11\n"                  \
    "ds_write_b8 %[tia], v125 offset:10\n" HL_WAIT         \
    "ds_write_b8 %[tia], v122 offset:17\n"
#define HL_W_GRP1                                          \
    "ds_read_u8 v122, %[tia] offset:10\n"                  \
    "ds_read_u8 v123, %[tia] offset:34\n"                  \
    "ds_read_u8 v124, %[tia] offset:23\n"                  \
    "ds_write_b8 %[tia], v125 offset:11\n" HL_WAIT         \
    "ds_write_b8 %[tia], v122 offset:16\n"                 \
    "ds_write_b8 %[tia], v123 offset:35\n"                 \
    "v_and_b32 v122, 4, v124\n"                            \
    "v_and_b32 v124, -9, v124\n"                           \
    "v_lshl_or_b32 v124, v122, 1, v124\n"                  \
    "ds_write_b8 %[tia], v124 offset:23\n"
#define HL_TIA(slot, id, write)                            \
    HL_ORG(slot)                                           \
    "s_and_b32 s87, s74, 31\n" HL_FETCH(2) HL_WAIT         \
    "v_mov_b32 v125, %[a]\n"                               \
    ".Lbody" id "%=:\n" HL_TIA_BODY(id, write)
#define HL_TIA_XY(slot, id, reg)                           \
    HL_ORG(slot)                                           \
    "s_and_b32 s87, s74, 31\n" HL_FETCH(2) HL_WAIT         \
    "v_mov_b32 v125, " reg "\n"                            \
    "s_branch .Lbody" id "%=\n"

// Scalars of a run, in the registers the block uses.
struct HotRegs {
    uint32_t po;         // byte offset of the instruction's word in the ROM's table (bank and pc)
    uint32_t acc;        // ACC
    uint32_t lines;      // lines until the cap
    uint32_t orow;       // open row + 1 (0 = none)
    uint32_t pos;        // next entry's dword in the frame's log
    uint32_t obase;      // the open row's first entry's dword
    uint32_t pchi;       // pc bits 12-15
    uint32_t why;        // HOT_EXIT_*
};

// Runs the block for the lanes in exec.  ram, tia: LDS addresses; log: the
// lane's row log (used only when logon); table: the ROM's predecoded words;
// bankpo: the bank's first word's byte offset; partial: all ones when the run
// must stop at the next WSYNC, else 0.
__device__ __forceinline__ void hot_loop(HotRegs& H, uint64_t table, uint32_t bankpo, uint32_t partial,
                                         uint32_t logon, uint32_t& a, uint32_t& x, uint32_t& y, uint32_t& nz,
                                         uint32_t& c, uint32_t& v, uint32_t ram, uint32_t tia, uint64_t log) {
    static_assert(kSnapArea == 1696 * 4 && kCountMask == 31 && kFrameEntries == 5280 && kRows == 210 &&
                      kFirstRow == 34 && kSnapBytes == 32,
                  "the block's constants");
    static_assert(R_GRP0 == 10 && R_GRP1 == 11 && R_GRP0_OLD == 16 && R_GRP1_OLD == 17 && R_FLAGS == 23 &&
                      R_ENABL == 34 && R_ENABL_OLD == 35,
                  "the block's register offsets");
    asm volatile(
        // --- entry: block base, line-change and row addresses, constants
        "s_getpc_b64 s[76:77]\n"
        ".Lpc%=:\n"
        "s_load_dword s74, s[70:71], s72\n"
        // (the block must lie in one 4 GB half: a handler's address is a 32-bit sum)
        "s_add_u32 s88, s76, .Lhb%=-.Lpc%=+0x8000\n"
        "s_cbranch_scc1 .Lout%=\n"
        "s_add_u32 s78, s76, .Lhb%=-.Lpc%=\n"
        "s_add_u32 s79, s76, .Lline%=-.Lpc%=\n"
        "s_add_u32 s64, s76, .Lsnap%=-.Lpc%=\n"
        "s_mov_b32 s65, s77\n"
        "s_mov_b32 s91, 0\n"
        "s_mov_b32 s67, 0\n"
        "s_mov_b32 s98, (3<<25)+1\n"
        "s_mov_b32 s99, (4<<25)+1\n"
        "s_add_u32 s92, s85, 31\n"                 // the open row's entries end here
        "s_min_u32 s92, s92, 1696+5280\n"
        "s_cmp_eq_u32 s82, 0\n"                    // s75: open row + 1, matching no row when none is open
        "s_cselect_b32 s75, 0x7fffffff, s82\n"
        HL_WAIT HL_TGT
        "s_setpc_b64 s[76:77]\n"
        // --- leaving
        ".Lundo%=:\n"                              // a 2-byte, 3-cycle store was fetched past and counted: take it back
        HL_WAIT
        "s_sub_u32 s73, s73, (3<<25)+1\n"
        "s_sub_u32 s72, s72, 8\n"
        "s_branch .Lout%=\n"
        ".Lpart%=:\n"                              // the lanes part at the branch
        "s_sub_u32 s72, s89, 8\n"
        ".Lout%=:\n"
        "s_mov_b32 s92, 0\n"
        "s_branch .Lend%=\n"
        ".Lsync%=:\n"
        "s_mov_b32 s92, 1\n"
        "s_branch .Lend%=\n"
        // --- line change without a WSYNC: ACC's cycle has wrapped past the bias
        ".Lline%=:\n"
        "s_add_u32 s73, s73, 52<<25\n"
        "s_sub_u32 s80, s80, 1\n"
        "s_cmp_eq_u32 s80, 0\n"
        "s_cbranch_scc1 .Lout%=\n"
        HL_WAIT HL_TGT
        "s_setpc_b64 s[76:77]\n"
        // --- rows reached by a TIA store at cycle s88 - 52 of the line whose row + 1 is s89:
        // snapshots of the rows before it (its own too when it lands in the visible
        // part).  SCC = 0 on return: its entry goes into the open row.
        ".Lsnap%=:\n"
        "s_cmp_ge_u32 s88, 75\n"                   // visible: 3 (cycle + 1) >= 68
        "s_cselect_b32 s94, 0, 1\n"
        "s_sub_u32 s95, s89, s94\n"                // rows to have open, at most 210
        "s_min_i32 s95, s95, 210\n"
        "s_cmp_ge_i32 s82, s95\n"
        "s_cbranch_scc1 .Lopen%=\n"
        "ds_read2_b32 v[112:113], %[tia] offset0:0 offset1:1\n"
        "ds_read2_b32 v[114:115], %[tia] offset0:2 offset1:3\n"
        "ds_read2_b32 v[116:117], %[tia] offset0:4 offset1:5\n"
        "ds_read2_b32 v[118:119], %[tia] offset0:6 offset1:7\n"
        "s_lshl_b32 s66, s82, 5\n"                 // the open row's end
        "s_cmp_eq_u32 s90, s85\n"                  // the open row's entry count (none: nothing to store)
        "s_cbranch_scc1 .Lcnt%=\n"
        "s_sub_u32 s85, s90, s85\n"
        "v_mov_b32 v123, s85\n"
        "v_lshl_add_u64 v[120:121], s[66:67], 0, %[log]\n"
        "global_store_byte v[120:121], v123, off offset:-17\n"
        ".Lcnt%=:\n"
        "s_mov_b32 s85, s90\n"
        "s_add_u32 s92, s85, 31\n"
        "s_min_u32 s92, s92, 1696+5280\n"
        "s_sub_u32 s84, s85, 1696\n"
        "s_waitcnt lgkmcnt(0)\n"
        "v_and_b32 v115, 0xffffff, v115\n"
        "v_and_b32 v119, 0xffff0000, v119\n"
        "v_or_b32 v119, s84, v119\n"
        ".Lsrow%=:\n"
        "v_lshl_add_u64 v[120:121], s[66:67], 0, %[log]\n"   // (its shift goes to 4)
        "global_store_dwordx4 v[120:121], v[112:115], off\n"
        "global_store_dwordx4 v[120:121], v[116:119], off offset:16\n"
        "s_add_u32 s66, s66, 32\n"
        "s_add_u32 s82, s82, 1\n"
        "s_cmp_lt_i32 s82, s95\n"
        "s_cbranch_scc1 .Lsrow%=\n"
        "s_mov_b32 s75, s82\n"
        ".Lopen%=:\n"
        "s_sub_u32 s95, s89, 1\n"                  // not in the visible part of a frame row: no entry
        "s_cmp_ge_u32 s95, 210\n"
        "s_cselect_b32 s95, 1, s94\n"
        "s_cmp_lg_u32 s95, 0\n"
        "s_setpc_b64 s[96:97]\n"
        // --- handlers
        ".p2align 7\n"
        ".Lhb%=:\n"
        HL_ORG(0) "s_branch .Lout%=\n"   // HOT_REAL
        HL_TIA(1, "t", HL_W_TIA)   // STA_TIA
        HL_TIA(4, "g", HL_W_GRP0)   // STA_GRP0
        HL_TIA(7, "h", HL_W_GRP1)   // STA_GRP1
        HL_TIA_XY(10, "t", "%[x]")   // STX_TIA
        HL_TIA_XY(11, "g", "%[x]")   // STX_GRP0
        HL_TIA_XY(12, "h", "%[x]")   // STX_GRP1
        HL_TIA_XY(13, "t", "%[y]")   // STY_TIA
        HL_TIA_XY(14, "g", "%[y]")   // STY_GRP0
        HL_TIA_XY(15, "h", "%[y]")   // STY_GRP1
        HL_SYNC(16)   // WSYNC
        HL_ORG(17) HL_FETCH(2) HL_WAIT HL_TGT HL_GO(3)   // ST_NOP
        HL_BR(18, HL_T_EQ("0x180", "%[nz]"), "s99")   // BPL_X
        HL_BR(19, HL_T_NE("0x180", "%[nz]"), "s99")   // BMI_X
        HL_BR(20, HL_T_EQ("0x80", "%[v]"), "s99")   // BVC_X
        HL_BR(21, HL_T_NE("0x80", "%[v]"), "s99")   // BVS_X
        HL_BR(22, "v_cmp_eq_u32 vcc, 0, %[c]\n", "s99")   // BCC_X
        HL_BR(23, "v_cmp_ne_u32 vcc, 0, %[c]\n", "s99")   // BCS_X
        HL_BR(24, HL_T_NE("0xff", "%[nz]"), "s99")   // BNE_X
        HL_BR(25, HL_T_EQ("0xff", "%[nz]"), "s99")   // BEQ_X
        HL_ZPR(26, HL_ORA("v123"))   // $05
        HL_ZPM(27, HL_ASL("v123"))   // $06
        HL_IMM(28, HL_ORA("s87"))   // $09
        HL_IMP(29, HL_ASL("%[a]"))   // $0A
        HL_BR(30, HL_T_EQ("0x180", "%[nz]"), "s98")   // $10
        HL_IMP(31, "v_mov_b32 %[c], 0\n")   // $18
        HL_ZPR(32, HL_BIT)   // $24
        HL_ZPR(33, HL_AND("v123"))   // $25
        HL_ZPM(34, HL_ROL("v123"))   // $26
        HL_IMM(35, HL_AND("s87"))   // $29
        HL_IMP(36, HL_ROL("%[a]"))   // $2A
        HL_BR(37, HL_T_NE("0x180", "%[nz]"), "s98")   // $30
        HL_IMP(38, "v_mov_b32 %[c], 1\n")   // $38
        HL_ZPR(39, HL_EOR("v123"))   // $45
        HL_ZPM(40, HL_LSR("v123"))   // $46
        HL_IMM(41, HL_EOR("s87"))   // $49
        HL_IMP(42, HL_LSR("%[a]"))   // $4A
        HL_JMP(43)   // $4C
        HL_BR(44, HL_T_EQ("0x80", "%[v]"), "s98")   // $50
        HL_ZPR(45, HL_ADC("v123"))   // $65
        HL_ZPM(46, HL_ROR("v123"))   // $66
        HL_IMM(47, HL_ADC("s87"))   // $69
        HL_IMP(48, HL_ROR("%[a]"))   // $6A
        HL_BR(49, HL_T_NE("0x80", "%[v]"), "s98")   // $70
        HL_ZPS(50, "%[y]")   // $84
        HL_ZPS(51, "%[a]")   // $85
        HL_ZPS(52, "%[x]")   // $86
        HL_IMP(53, HL_DEC("%[y]"))   // $88
        HL_IMP(54, "v_mov_b32 %[a], %[x]\n" HL_NZ("%[x]"))   // $8A
        HL_BR(55, "v_cmp_eq_u32 vcc, 0, %[c]\n", "s98")   // $90
        HL_IMP(56, "v_mov_b32 %[a], %[y]\n" HL_NZ("%[y]"))   // $98
        HL_IMM(57, "v_mov_b32 %[y], s87\nv_mov_b32 %[nz], s87\n")   // $A0
        HL_IMM(58, "v_mov_b32 %[x], s87\nv_mov_b32 %[nz], s87\n")   // $A2
        HL_ZPL(59, "%[y]")   // $A4
        HL_ZPL(60, "%[a]")   // $A5
        HL_ZPL(61, "%[x]")   // $A6
        HL_IMP(62, "v_mov_b32 %[y], %[a]\n" HL_NZ("%[a]"))   // $A8
        HL_IMM(63, "v_mov_b32 %[a], s87\nv_mov_b32 %[nz], s87\n")   // $A9
        HL_IMP(64, "v_mov_b32 %[x], %[a]\n" HL_NZ("%[a]"))   // $AA
        HL_BR(65, "v_cmp_ne_u32 vcc, 0, %[c]\n", "s98")   // $B0
        HL_IMP(66, "v_mov_b32 %[v], 0\n")   // $B8
        HL_IMM(67, HL_CMP_S("%[y]"))   // $C0
        HL_ZPR(68, HL_CMP("%[y]", "v123"))   // $C4
        HL_ZPR(69, HL_CMP("%[a]", "v123"))   // $C5
        HL_ZPM(70, HL_DEC("v123"))   // $C6
        HL_IMP(71, HL_INC("%[y]"))   // $C8
        HL_IMM(72, HL_CMP_S("%[a]"))   // $C9
        HL_IMP(73, HL_DEC("%[x]"))   // $CA
        HL_BR(74, HL_T_NE("0xff", "%[nz]"), "s98")   // $D0
        HL_IMP(75, "")   // $D8
        HL_IMM(76, HL_CMP_S("%[x]"))   // $E0
        HL_ZPR(77, HL_CMP("%[x]", "v123"))   // $E4
        HL_ZPR(78, "v_xor_b32 v123, 0xff, v123\n" HL_ADC("v123"))   // $E5
        HL_ZPM(79, HL_INC("v123"))   // $E6
        HL_IMP(80, HL_INC("%[x]"))   // $E8
        HL_IMM(81, "s_xor_b32 s87, s87, 0xff\n" HL_ADC("s87"))   // $E9
        HL_IMP(82, "")   // $EA
        HL_BR(83, HL_T_EQ("0xff", "%[nz]"), "s98")   // $F0
        ".Lend%=:\n"
        HL_WAIT
        : "+{s72}"(H.po), "+{s73}"(H.acc), "+{s80}"(H.lines), "+{s82}"(H.orow), "+{s90}"(H.pos), "+{s85}"(H.obase),
          "+{s93}"(H.pchi), "={s92}"(H.why), [a] "+v"(a), [x] "+v"(x), [y] "+v"(y), [nz] "+v"(nz), [c] "+v"(c),
          [v] "+v"(v)
        : "{s[70:71]}"(table), "{s68}"(bankpo), "{s81}"(partial), "{s86}"(logon), [ram] "v"(ram),
          [tia] "v"(tia), [log] "v"(log)
        : "memory", "scc", "vcc", "s74", "s75", "s76", "s77", "s78", "s79", "s66", "s67", "s84", "s87", "s88", "s89", "s91",
          "s94", "s95", "s96", "s97", "s98", "s99", "s64", "s65", "v112", "v113", "v114", "v115", "v116", "v117",
          "v118", "v119", "v120", "v121", "v122", "v123", "v124", "v125");
}

}  // namespace vcs
