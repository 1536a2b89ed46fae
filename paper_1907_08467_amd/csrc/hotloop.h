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
// operands are RAM; a store of A to a TIA register that is kept as is has a
// slot per register (hot_tia_slot), one of X or Y takes the register's code
// from the word; GRP0 / GRP1 stores also update the delayed copies; HOT_WSYNC
// and HOT_ST_NOP (nothing emulated changes) stand for a store of A, X or Y; the
// *_X branches cross a page when taken.  Long handlers have several slots.
constexpr uint32_t HOT_REAL = 0, HOT_STA_TIA = 1,
                   HOT_STA_GRP0 = 14, HOT_STA_GRP1 = 16, HOT_STX_TIA = 19, HOT_STX_GRP0 = 20, HOT_STX_GRP1 = 21, HOT_STY_TIA = 22, HOT_STY_GRP0 = 23, HOT_STY_GRP1 = 24,
                   HOT_WSYNC = 27, HOT_ST_NOP = 28, HOT_BPL_X = 29, kHotPlain = 37;
constexpr uint32_t kHotSlots = 95;
constexpr uint8_t kHotSlotOp[kHotSlots] = {
    0x00, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85,
    0x85, 0x85, 0x85, 0x86, 0x86, 0x86, 0x84, 0x84, 0x84, 0x00, 0x00, 0x85, 0x85, 0x10, 0x30, 0x50,
    0x70, 0x90, 0xB0, 0xD0, 0xF0, 0x05, 0x06, 0x09, 0x0A, 0x10, 0x18, 0x24, 0x25, 0x26, 0x29, 0x2A,
    0x30, 0x38, 0x45, 0x46, 0x49, 0x4A, 0x4C, 0x50, 0x65, 0x66, 0x69, 0x6A, 0x70, 0x84, 0x85, 0x86,
    0x88, 0x8A, 0x90, 0x98, 0xA0, 0xA2, 0xA4, 0xA5, 0xA6, 0xA8, 0xA9, 0xAA, 0xB0, 0xB8, 0xC0, 0xC4,
    0xC5, 0xC6, 0xC8, 0xC9, 0xCA, 0xD0, 0xD8, 0xE0, 0xE4, 0xE5, 0xE6, 0xE8, 0xE9, 0xEA, 0xF0,
};
// The slot that runs opcode `op` without a page-crossing branch or a TIA store
// (HOT_REAL: none).
constexpr uint32_t hot_slot(uint32_t op) {
    for (uint32_t s = kHotPlain; s < kHotSlots; ++s)
        if (kHotSlotOp[s] == op) return s;
    return HOT_REAL;
}
// The slot of a store of A to the TIA register with code `code` (R_COLUP0 ..
// R_PF2, R_VBLANK, R_NUSIZ0, R_NUSIZ1)
__host__ __device__ constexpr uint32_t hot_tia_slot(uint32_t code) {
    return HOT_STA_TIA + (code <= R_PF2 ? code : code == R_VBLANK ? 10 : code - R_NUSIZ0 + 11);
}

// ACC: cycle in the line + 52 in the top 7 bits, instructions below
constexpr uint32_t kAccBias = 52, kAccShift = 25, kAccCount = (1u << kAccShift) - 1;

// what ended the block
constexpr uint32_t HOT_EXIT_NEXT = 0;     // before the instruction at PO
constexpr uint32_t HOT_EXIT_LINE = 1;     // after a WSYNC: a partial group stops, or the cap is reached

#define HL_ORG(B, slot) ".org " B "%= + 128*" #slot "\n"
#define HL_WAIT "s_waitcnt lgkmcnt(0)\n"
// the next handler's address, from its word `n` (s76 + the instruction's length)
#define HL_TGT(n)                             \
    "s_and_b32 s74, " n ", 0x7f80\n"          \
    "s_add_u32 s74, s74, s84\n"
// advance to the next instruction, load its word and those behind it
#define HL_FETCH(len)                         \
    "s_add_u32 s72, s72, 4*" #len "\n"        \
    "s_load_dwordx4 s[76:79], s[70:71], s72\n"
// count the instruction and its cycles, go on (to the line change on carry)
#define HL_ACC(cyc)                           \
    "s_add_u32 s73, s73, (" #cyc "<<25)+1\n"  \
    "s_cselect_b32 s74, s85, s74\n"
#define HL_JUMP "s_setpc_b64 s[74:75]\n"
#define HL_GO(cyc) HL_ACC(cyc) HL_JUMP
#define HL_B1_7 "s_bfe_u32 s86, s76, 0x70010\n"       // zero-page RAM offset
#define HL_B1_8 "s_bfe_u32 s86, s76, 0x80010\n"       // immediate
#define HL_RAMADDR "v_add_u32 v122, s86, %[ram]\n"

// implied
#define HL_IMP(B, slot, work) HL_ORG(B, slot) HL_WAIT HL_TGT("s77") HL_FETCH(1) work HL_GO(2)
// immediate: operand in s86
#define HL_IMM(B, slot, work) HL_ORG(B, slot) HL_WAIT HL_B1_8 HL_TGT("s78") HL_FETCH(2) work HL_GO(2)
// zero-page read whose result the handler needs: operand in v123
#define HL_ZPR(B, slot, work)                                                                      \
    HL_ORG(B, slot) HL_WAIT HL_B1_7 HL_RAMADDR "ds_read_u8 v123, v122\n" HL_TGT("s78") HL_FETCH(2) \
    HL_ACC(3) HL_WAIT work HL_JUMP
// zero-page load: lands in the register and nz before the next handler's wait ends
#define HL_ZPL(B, slot, reg)                                                                       \
    HL_ORG(B, slot) HL_WAIT HL_B1_7 HL_RAMADDR "ds_read_u8 " reg ", v122\n"                        \
    "ds_read_u8 %[nz], v122\n" HL_TGT("s78") HL_FETCH(2) HL_GO(3)
#define HL_ZPS(B, slot, reg)                                                                       \
    HL_ORG(B, slot) HL_WAIT HL_B1_7 HL_RAMADDR "ds_write_b8 v122, " reg "\n" HL_TGT("s78") HL_FETCH(2) HL_GO(3)
// read-modify-write of zero-page RAM: `work` takes v123 to the new value there
#define HL_ZPM(B, slot, work)                                                                      \
    HL_ORG(B, slot) HL_WAIT HL_B1_7 HL_RAMADDR "ds_read_u8 v123, v122\n" HL_TGT("s78") HL_FETCH(2) \
    HL_ACC(5) HL_WAIT work "ds_write_b8 v122, v123\n" HL_JUMP

#define HL_NZ(reg) "v_mov_b32 %[nz], " reg "\n"
#define HL_LDI(reg) "v_mov_b32 " reg ", s86\nv_mov_b32 %[nz], s86\n"
// arithmetic on A and operand `m` (a register or s86)
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
    "v_subrev_u32 v124, s86, " r "\n"                      \
    "v_ashrrev_i32 %[c], 31, v124\n"                       \
    "v_add_u32 %[c], 1, %[c]\n"                            \
    "v_and_b32 %[nz], 0xff, v124\n"
#define HL_BIT                                             \
    "v_lshlrev_b32 %[v], 1, v123\n"                        \
    "v_and_b32 %[nz], %[a], v123\n"                        \
    "v_and_b32 v124, 0x80, v123\n"                         \
    "v_lshl_or_b32 %[nz], v124, 1, %[nz]\n"
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
#define HL_BR(B, slot, test, tk)                           \
    HL_ORG(B, slot) HL_WAIT                                \
    "s_bfe_i32 s86, s76, 0x80010\n"                        \
    "s_add_u32 s88, s72, 8\n"                              \
    "s_lshl2_add_u32 s89, s86, s88\n"                      \
    "s_load_dwordx4 s[60:63], s[70:71], s89\n"             \
    "s_load_dwordx4 s[76:79], s[70:71], s88\n" test        \
    "s_cmp_eq_u64 vcc, exec\n"                             \
    "s_cselect_b32 s72, s89, s88\n"                        \
    "s_cselect_b32 s87, " tk ", (2<<25)+1\n"               \
    "s_cselect_b64 s[96:97], exec, 0\n"                    \
    "s_cmp_lg_u64 vcc, s[96:97]\n"                         \
    "s_cbranch_scc1 .Lpart%=\n"                            \
    "s_cmp_eq_u64 s[96:97], exec\n" HL_WAIT                \
    "s_cselect_b64 s[76:77], s[60:61], s[76:77]\n"         \
    "s_cselect_b64 s[78:79], s[62:63], s[78:79]\n"         \
    HL_TGT("s76")                                          \
    "s_add_u32 s73, s73, s87\n"                            \
    "s_cselect_b32 s74, s85, s74\n" HL_JUMP
#define HL_T_NE(mask, src) "v_and_b32 v122, " mask ", " src "\nv_cmp_ne_u32 vcc, 0, v122\n"
#define HL_T_EQ(mask, src) "v_and_b32 v122, " mask ", " src "\nv_cmp_eq_u32 vcc, 0, v122\n"

// absolute jump (the target lies in the cartridge window; pc bits 12-15 kept apart)
#define HL_JMP(B, slot)                                    \
    HL_ORG(B, slot) HL_WAIT                                \
    "s_lshr_b32 s86, s76, 16\n"                            \
    "s_and_b32 s93, s86, 0xf000\n"                         \
    "s_and_b32 s86, s86, 0xfff\n"                          \
    "s_lshl2_add_u32 s72, s86, s68\n"                      \
    "s_load_dwordx4 s[76:79], s[70:71], s72\n" HL_WAIT HL_TGT("s76") HL_GO(3)

// WSYNC: on to the next line's start.  Left (.Lsync) when the run stops there
// or a write at the line's last cycles stalls a line longer.
#define HL_SYNC(B, slot)                                   \
    HL_ORG(B, slot) HL_WAIT HL_TGT("s78") HL_FETCH(2)      \
    "s_sub_u32 s80, s80, 1\n"                              \
    "s_add_u32 s87, s73, 2<<25\n"                          \
    "s_cselect_b32 s86, 0, s80\n"                          \
    "s_cmp_le_u32 s86, s81\n"                              \
    "s_cbranch_scc1 .Lsync%=\n"                            \
    "s_and_b32 s73, s73, 0x1ffffff\n"                      \
    "s_add_u32 s73, s73, (52<<25)+1\n" HL_JUMP

// TIA register stores (2 bytes, 3 cycles).  `val`: the stored register.
//
// Logged: the entry goes into the open row when that is the line's row and the
// line has not ended (s87 = the line's number, or -1 past its end, against the
// open row's); else .Lsnap opens rows first, or leaves the store to the full
// dispatch.  `code8`: the entry's register code << 8 less 3 * 52 + 68.
#define HL_LOGGED(id, val, code8, write)                   \
    "s_add_u32 s73, s73, (3<<25)+1\n"                      \
    "s_cselect_b32 s87, -1, s80\n"                         \
    "s_lshr_b32 s88, s73, 25\n"                            \
    "s_cmp_lg_u32 s87, s83\n"                              \
    "v_lshl_add_u64 v[120:121], s[90:91], 2, %[log]\n"     \
    "s_cbranch_scc1 .Lrow" id "%=\n"                       \
    ".Lent" id "%=:\n"                                     \
    "s_mul_i32 s87, s88, 3\n"                              \
    "s_add_u32 s90, s90, 1\n"                              \
    "s_add_u32 s87, s87, " code8 "\n"                      \
    "v_lshl_or_b32 v123, " val ", 16, s87\n"               \
    "global_store_dword v[120:121], v123, off\n"           \
    ".Lreg" id "%=:\n" write HL_JUMP                       \
    ".Lrow" id "%=:\n"                                     \
    "s_swappc_b64 s[96:97], s[64:65]\n"                    \
    "s_cbranch_scc0 .Lent" id "%=\n"                       \
    "s_branch .Lreg" id "%=\n"
#define HL_TIA_LOG(B, slot, code)                          \
    HL_ORG(B, slot) HL_WAIT HL_TGT("s78") HL_FETCH(2)      \
    HL_LOGGED("t" #code, "%[a]", #code "*256-224", "ds_write_b8 %[tia], %[a] offset:" #code "\n")
#define HL_TIA_NOLOG(B, slot, code)                        \
    HL_ORG(B, slot) HL_WAIT "ds_write_b8 %[tia], %[a] offset:" #code "\n" HL_TGT("s78") HL_FETCH(2) HL_GO(3)
// X or Y (moved to v125), and GRP0 / GRP1 of any register: the slot moves the
// value and joins the body.
#define HL_XY_(B, slot, reg, body)                         \
    HL_ORG(B, slot) HL_WAIT                                \
    "v_mov_b32 v125, " reg "\n"                            \
    "s_branch " body "%=\n"
#define HL_TIAX_LOG(B, slot)                               \
    HL_ORG(B, slot) ".Lbtl%=:\n"                            \
    "s_and_b32 s86, s76, 31\n" HL_TGT("s78") HL_FETCH(2)   \
    "v_add_u32 v122, s86, %[tia]\n"                        \
    "s_lshl_b32 s86, s86, 8\n"                             \
    "s_sub_u32 s86, s86, 224\n"                            \
    HL_LOGGED("x", "v125", "s86", "ds_write_b8 v122, v125\n")
#define HL_TIAX_NOLOG(B, slot)                             \
    HL_ORG(B, slot) ".Lbtu%=:\n"                            \
    "s_and_b32 s86, s76, 31\n"                             \
    "v_add_u32 v122, s86, %[tia]\n"                        \
    "ds_write_b8 v122, v125\n" HL_TGT("s78") HL_FETCH(2) HL_GO(3)
// GRP0 10, GRP1 11, delayed copies 16 / 17, flags 23, ENABL 34 / delayed 35
#define HL_GRP0_READ "ds_read_u8 v122, %[tia] offset:11\n"
#define HL_GRP0_WRITE                                      \
    HL_WAIT "ds_write_b8 %[tia], v125 offset:10\n"         \
    "ds_write_b8 %[tia], v122 offset:17\n"
#define HL_GRP1_READ                                       \
    "ds_read_u8 v122, %[tia] offset:10\n"                  \
    "ds_read_u8 v126, %[tia] offset:34\n"                  \
    "ds_read_u8 v124, %[tia] offset:23\n"
#define HL_GRP1_WRITE                                      \
    HL_WAIT "ds_write_b8 %[tia], v125 offset:11\n"         \
    "ds_write_b8 %[tia], v122 offset:16\n"                 \
    "ds_write_b8 %[tia], v126 offset:35\n"                 \
    "v_and_b32 v122, 4, v124\n"                            \
    "v_and_b32 v124, -9, v124\n"                           \
    "v_lshl_or_b32 v124, v122, 1, v124\n"                  \
    "ds_write_b8 %[tia], v124 offset:23\n"
#define HL_GRP0_LOG(B, slot)                               \
    HL_ORG(B, slot) HL_WAIT "v_mov_b32 v125, %[a]\n"       \
    ".Lbgl%=:\n" HL_GRP0_READ HL_TGT("s78") HL_FETCH(2)     \
    HL_LOGGED("g", "v125", "10*256-224", HL_GRP0_WRITE)
#define HL_GRP0_NOLOG(B, slot)                             \
    HL_ORG(B, slot) HL_WAIT "v_mov_b32 v125, %[a]\n"       \
    ".Lbgu%=:\n" HL_GRP0_READ HL_TGT("s78") HL_FETCH(2)     \
    HL_ACC(3) HL_GRP0_WRITE HL_JUMP
#define HL_GRP1_LOG(B, slot)                               \
    HL_ORG(B, slot) HL_WAIT "v_mov_b32 v125, %[a]\n"       \
    ".Lbhl%=:\n" HL_GRP1_READ HL_TGT("s78") HL_FETCH(2)     \
    HL_LOGGED("h", "v125", "11*256-224", HL_GRP1_WRITE)
#define HL_GRP1_NOLOG(B, slot)                             \
    HL_ORG(B, slot) HL_WAIT "v_mov_b32 v125, %[a]\n"       \
    ".Lbhu%=:\n" HL_GRP1_READ HL_TGT("s78") HL_FETCH(2)     \
    HL_ACC(3) HL_GRP1_WRITE HL_JUMP
#define HL_XY_LOG(B, slot, reg, body) HL_XY_(B, slot, reg, ".Lb" body "l")
#define HL_XY_NOLOG(B, slot, reg, body) HL_XY_(B, slot, reg, ".Lb" body "u")

// Every handler of one of the two blocks (frames whose writes are logged, and
// the others: dispatch by block spares each TIA store the question).
#define HL_BLOCK(B, TIA, TIAX, GRP0, GRP1, HL_XY) \
    HL_ORG(B, 0) "s_branch .Lout%=\n"                                                                /* HOT_REAL */ \
    TIA(B, 1, 0)                                                                                     /* STA COLUP0 */ \
    TIA(B, 2, 1)                                                                                     /* STA COLUP1 */ \
    TIA(B, 3, 2)                                                                                     /* STA COLUPF */ \
    TIA(B, 4, 3)                                                                                     /* STA COLUBK */ \
    TIA(B, 5, 4)                                                                                     /* STA CTRLPF */ \
    TIA(B, 6, 5)                                                                                     /* STA REFP0 */ \
    TIA(B, 7, 6)                                                                                     /* STA REFP1 */ \
    TIA(B, 8, 7)                                                                                     /* STA PF0 */ \
    TIA(B, 9, 8)                                                                                     /* STA PF1 */ \
    TIA(B, 10, 9)                                                                                    /* STA PF2 */ \
    TIA(B, 11, 14)                                                                                   /* STA VBLANK */ \
    TIA(B, 12, 18)                                                                                   /* STA NUSIZ0 */ \
    TIA(B, 13, 19)                                                                                   /* STA NUSIZ1 */ \
    GRP0(B, 14)                                                                                      /* STA GRP0 */ \
    GRP1(B, 16)                                                                                      /* STA GRP1 */ \
    HL_XY(B, 19, "%[x]", "t")                                                                        /* STX to a TIA register */ \
    HL_XY(B, 20, "%[x]", "g")                                                                        /* STX GRP0 */ \
    HL_XY(B, 21, "%[x]", "h")                                                                        /* STX GRP1 */ \
    HL_XY(B, 22, "%[y]", "t")                                                                        /* STY to a TIA register */ \
    HL_XY(B, 23, "%[y]", "g")                                                                        /* STY GRP0 */ \
    HL_XY(B, 24, "%[y]", "h")                                                                        /* STY GRP1 */ \
    TIAX(B, 25)                                                                                      /* the body of the two stores to a TIA register */ \
    HL_SYNC(B, 27)                                                                                   /* WSYNC */ \
    HL_ORG(B, 28) HL_WAIT HL_TGT("s78") HL_FETCH(2) HL_GO(3)                                         /* store without effect */ \
    HL_BR(B, 29, HL_T_EQ("0x180", "%[nz]"), "s99")                                                   /* BPL across a page */ \
    HL_BR(B, 30, HL_T_NE("0x180", "%[nz]"), "s99")                                                   /* BMI across a page */ \
    HL_BR(B, 31, HL_T_EQ("0x80", "%[v]"), "s99")                                                     /* BVC across a page */ \
    HL_BR(B, 32, HL_T_NE("0x80", "%[v]"), "s99")                                                     /* BVS across a page */ \
    HL_BR(B, 33, "v_cmp_eq_u32 vcc, 0, %[c]\n", "s99")                                               /* BCC across a page */ \
    HL_BR(B, 34, "v_cmp_ne_u32 vcc, 0, %[c]\n", "s99")                                               /* BCS across a page */ \
    HL_BR(B, 35, HL_T_NE("0xff", "%[nz]"), "s99")                                                    /* BNE across a page */ \
    HL_BR(B, 36, HL_T_EQ("0xff", "%[nz]"), "s99")                                                    /* BEQ across a page */ \
    HL_ZPR(B, 37, HL_ORA("v123"))                                                                    /* $05 */ \
    HL_ZPM(B, 38, HL_ASL("v123"))                                                                    /* $06 */ \
    HL_IMM(B, 39, HL_ORA("s86"))                                                                     /* $09 */ \
    HL_IMP(B, 40, HL_ASL("%[a]"))                                                                    /* $0A */ \
    HL_BR(B, 41, HL_T_EQ("0x180", "%[nz]"), "s98")                                                   /* $10 */ \
    HL_IMP(B, 42, "v_mov_b32 %[c], 0\n")                                                             /* $18 */ \
    HL_ZPR(B, 43, HL_BIT)                                                                            /* $24 */ \
    HL_ZPR(B, 44, HL_AND("v123"))                                                                    /* $25 */ \
    HL_ZPM(B, 45, HL_ROL("v123"))                                                                    /* $26 */ \
    HL_IMM(B, 46, HL_AND("s86"))                                                                     /* $29 */ \
    HL_IMP(B, 47, HL_ROL("%[a]"))                                                                    /* $2A */ \
    HL_BR(B, 48, HL_T_NE("0x180", "%[nz]"), "s98")                                                   /* $30 */ \
    HL_IMP(B, 49, "v_mov_b32 %[c], 1\n")                                                             /* $38 */ \
    HL_ZPR(B, 50, HL_EOR("v123"))                                                                    /* $45 */ \
    HL_ZPM(B, 51, HL_LSR("v123"))                                                                    /* $46 */ \
    HL_IMM(B, 52, HL_EOR("s86"))                                                                     /* $49 */ \
    HL_IMP(B, 53, HL_LSR("%[a]"))                                                                    /* $4A */ \
    HL_JMP(B, 54)                                                                                    /* $4C */ \
    HL_BR(B, 55, HL_T_EQ("0x80", "%[v]"), "s98")                                                     /* $50 */ \
    HL_ZPR(B, 56, HL_ADC("v123"))                                                                    /* $65 */ \
    HL_ZPM(B, 57, HL_ROR("v123"))                                                                    /* $66 */ \
    HL_IMM(B, 58, HL_ADC("s86"))                                                                     /* $69 */ \
    HL_IMP(B, 59, HL_ROR("%[a]"))                                                                    /* $6A */ \
    HL_BR(B, 60, HL_T_NE("0x80", "%[v]"), "s98")                                                     /* $70 */ \
    HL_ZPS(B, 61, "%[y]")                                                                            /* $84 */ \
    HL_ZPS(B, 62, "%[a]")                                                                            /* $85 */ \
    HL_ZPS(B, 63, "%[x]")                                                                            /* $86 */ \
    HL_IMP(B, 64, HL_DEC("%[y]"))                                                                    /* $88 */ \
    HL_IMP(B, 65, "v_mov_b32 %[a], %[x]\n" HL_NZ("%[x]"))                                            /* $8A */ \
    HL_BR(B, 66, "v_cmp_eq_u32 vcc, 0, %[c]\n", "s98")                                               /* $90 */ \
    HL_IMP(B, 67, "v_mov_b32 %[a], %[y]\n" HL_NZ("%[y]"))                                            /* $98 */ \
    HL_IMM(B, 68, HL_LDI("%[y]"))                                                                    /* $A0 */ \
    HL_IMM(B, 69, HL_LDI("%[x]"))                                                                    /* $A2 */ \
    HL_ZPL(B, 70, "%[y]")                                                                            /* $A4 */ \
    HL_ZPL(B, 71, "%[a]")                                                                            /* $A5 */ \
    HL_ZPL(B, 72, "%[x]")                                                                            /* $A6 */ \
    HL_IMP(B, 73, "v_mov_b32 %[y], %[a]\n" HL_NZ("%[a]"))                                            /* $A8 */ \
    HL_IMM(B, 74, HL_LDI("%[a]"))                                                                    /* $A9 */ \
    HL_IMP(B, 75, "v_mov_b32 %[x], %[a]\n" HL_NZ("%[a]"))                                            /* $AA */ \
    HL_BR(B, 76, "v_cmp_ne_u32 vcc, 0, %[c]\n", "s98")                                               /* $B0 */ \
    HL_IMP(B, 77, "v_mov_b32 %[v], 0\n")                                                             /* $B8 */ \
    HL_IMM(B, 78, HL_CMP_S("%[y]"))                                                                  /* $C0 */ \
    HL_ZPR(B, 79, HL_CMP("%[y]", "v123"))                                                            /* $C4 */ \
    HL_ZPR(B, 80, HL_CMP("%[a]", "v123"))                                                            /* $C5 */ \
    HL_ZPM(B, 81, HL_DEC("v123"))                                                                    /* $C6 */ \
    HL_IMP(B, 82, HL_INC("%[y]"))                                                                    /* $C8 */ \
    HL_IMM(B, 83, HL_CMP_S("%[a]"))                                                                  /* $C9 */ \
    HL_IMP(B, 84, HL_DEC("%[x]"))                                                                    /* $CA */ \
    HL_BR(B, 85, HL_T_NE("0xff", "%[nz]"), "s98")                                                    /* $D0 */ \
    HL_IMP(B, 86, "")                                                                                /* $D8 */ \
    HL_IMM(B, 87, HL_CMP_S("%[x]"))                                                                  /* $E0 */ \
    HL_ZPR(B, 88, HL_CMP("%[x]", "v123"))                                                            /* $E4 */ \
    HL_ZPR(B, 89, "v_xor_b32 v123, 0xff, v123\n" HL_ADC("v123"))                                     /* $E5 */ \
    HL_ZPM(B, 90, HL_INC("v123"))                                                                    /* $E6 */ \
    HL_IMP(B, 91, HL_INC("%[x]"))                                                                    /* $E8 */ \
    HL_IMM(B, 92, "s_xor_b32 s86, s86, 0xff\n" HL_ADC("s86"))                                        /* $E9 */ \
    HL_IMP(B, 93, "")                                                                                /* $EA */ \
    HL_BR(B, 94, HL_T_EQ("0xff", "%[nz]"), "s98")                                                    /* $F0 */

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
        "s_getpc_b64 s[74:75]\n"
        ".Lpc%=:\n"
        "s_load_dwordx4 s[76:79], s[70:71], s72\n"
        // (the blocks must lie in one 4 GB half: a handler's address is a 32-bit sum)
        "s_add_u32 s88, s74, .Lhu%=-.Lpc%=+0x8000\n"
        "s_cbranch_scc1 .Lout%=\n"
        "s_add_u32 s84, s74, .Lhb%=-.Lpc%=\n"
        "s_add_u32 s88, s74, .Lhu%=-.Lpc%=\n"
        "s_cmp_eq_u32 s59, 0\n"
        "s_cselect_b32 s84, s88, s84\n"
        "s_add_u32 s85, s74, .Lline%=-.Lpc%=\n"
        "s_add_u32 s64, s74, .Lsnap%=-.Lpc%=\n"
        "s_mov_b32 s65, s75\n"
        "s_mov_b32 s91, 0\n"
        "s_mov_b32 s67, 0\n"
        "s_mov_b32 s98, (3<<25)+1\n"
        "s_mov_b32 s99, (4<<25)+1\n"
        // s83: lines left in the open row's line; -2 (no line's) when none is open
        // or its entries might not all fit (.Lsnap then leaves the store)
        "s_sub_u32 s83, 287, s82\n"
        "s_cmp_eq_u32 s82, 0\n"
        "s_cselect_b32 s83, -2, s83\n"
        "s_cmp_gt_u32 s69, 1696+5280-31\n"
        "s_cselect_b32 s83, -2, s83\n"
        HL_WAIT HL_TGT("s76") HL_JUMP
        // --- leaving
        ".Lundo%=:\n"                              // a 2-byte, 3-cycle store was fetched past and counted: take it back
        "s_sub_u32 s73, s73, (3<<25)+1\n"
        "s_sub_u32 s72, s72, 8\n"
        "s_branch .Lout%=\n"
        ".Lpart%=:\n"                              // the lanes part at the branch
        "s_sub_u32 s72, s88, 8\n"
        ".Lout%=:\n"
        "s_mov_b32 s92, 0\n"
        "s_branch .Lend%=\n"
        ".Lsync%=:\n"
        "s_add_u32 s87, s73, 2<<25\n"
        "s_cbranch_scc1 .Lsync2%=\n"
        "s_and_b32 s73, s73, 0x1ffffff\n"
        "s_add_u32 s73, s73, (52<<25)+1\n"
        "s_mov_b32 s92, 1\n"
        "s_branch .Lend%=\n"
        ".Lsync2%=:\n"
        "s_add_u32 s80, s80, 1\n"
        "s_sub_u32 s72, s72, 8\n"
        "s_branch .Lout%=\n"
        // --- line change without a WSYNC: ACC's cycle has wrapped past the bias
        ".Lline%=:\n"
        "s_add_u32 s73, s73, 52<<25\n"
        "s_sub_u32 s80, s80, 1\n"
        "s_cmp_eq_u32 s80, 0\n"
        "s_cbranch_scc1 .Lout%=\n"
        HL_WAIT HL_TGT("s76") HL_JUMP
        // --- a logged TIA store at cycle s88 - 52 of its line, which is not the open row's
        // (s87 = -1: past the line's end): snapshots of the rows before it, and its own
        // when it lands in the visible part.  SCC = 0 on return: its entry goes into the open row.
        ".Lsnap%=:\n"
        "s_cmp_eq_u32 s87, -1\n"
        "s_cbranch_scc1 .Lundo%=\n"
        "s_sub_u32 s89, 287, s80\n"                // the line's row + 1
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
        "s_cmp_eq_u32 s90, s69\n"                  // the open row's entry count (none: nothing to store)
        "v_lshl_add_u64 v[120:121], s[66:67], 0, %[log]\n"   // (its shift goes to 4)
        "s_cbranch_scc1 .Lcnt%=\n"
        "s_sub_u32 s69, s90, s69\n"
        "v_mov_b32 v123, s69\n"
        "global_store_byte v[120:121], v123, off offset:-17\n"
        "s_mov_b32 s69, s90\n"
        ".Lcnt%=:\n"
        "s_sub_u32 s87, s69, 1696\n"
        HL_WAIT
        "v_and_b32 v115, 0xffffff, v115\n"
        "v_and_b32 v119, 0xffff0000, v119\n"
        "v_or_b32 v119, s87, v119\n"
        ".Lsrow%=:\n"
        "global_store_dwordx4 v[120:121], v[112:115], off\n"
        "global_store_dwordx4 v[120:121], v[116:119], off offset:16\n"
        "s_add_u32 s66, s66, 32\n"
        "s_add_u32 s82, s82, 1\n"
        "s_cmp_lt_i32 s82, s95\n"
        "v_lshl_add_u64 v[120:121], s[66:67], 0, %[log]\n"
        "s_cbranch_scc1 .Lsrow%=\n"
        "s_sub_u32 s83, 287, s82\n"
        ".Lopen%=:\n"
        "s_cmp_gt_u32 s69, 1696+5280-31\n"         // a row's entries might not fit
        "s_cbranch_scc1 .Lundo%=\n"
        "v_lshl_add_u64 v[120:121], s[90:91], 2, %[log]\n"
        "s_sub_u32 s95, s89, 1\n"                  // not in the visible part of a frame row: no entry
        "s_cmp_ge_u32 s95, 210\n"
        "s_cselect_b32 s95, 1, s94\n"
        "s_cmp_lg_u32 s95, 0\n"
        "s_setpc_b64 s[96:97]\n"
        // --- handlers
        ".p2align 7\n"
        ".Lhb%=:\n"
        HL_BLOCK(".Lhb", HL_TIA_LOG, HL_TIAX_LOG, HL_GRP0_LOG, HL_GRP1_LOG, HL_XY_LOG)
        ".p2align 7\n"
        ".Lhu%=:\n"
        HL_BLOCK(".Lhu", HL_TIA_NOLOG, HL_TIAX_NOLOG, HL_GRP0_NOLOG, HL_GRP1_NOLOG, HL_XY_NOLOG)
        ".Lend%=:\n"
        HL_WAIT
        : "+{s72}"(H.po), "+{s73}"(H.acc), "+{s80}"(H.lines), "+{s82}"(H.orow), "+{s90}"(H.pos), "+{s69}"(H.obase),
          "+{s93}"(H.pchi), "={s92}"(H.why), [a] "+v"(a), [x] "+v"(x), [y] "+v"(y), [nz] "+v"(nz), [c] "+v"(c),
          [v] "+v"(v)
        : "{s[70:71]}"(table), "{s68}"(bankpo), "{s81}"(partial), "{s59}"(logon), [ram] "v"(ram), [tia] "v"(tia),
          [log] "v"(log)
        : "memory", "scc", "vcc", "s60", "s61", "s62", "s63", "s64", "s65", "s66", "s67", "s74", "s75", "s76", "s77",
          "s78", "s79", "s83", "s84", "s85", "s86", "s87", "s88", "s89", "s91", "s94", "s95", "s96", "s97", "s98",
          "s99", "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119", "v120", "v121", "v122", "v123",
          "v124", "v125", "v126");
}

}  // namespace vcs
