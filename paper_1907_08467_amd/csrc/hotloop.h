// The scalar path's hot loop: threaded code for the instructions that make up
// almost all of a cartridge's work, written as one block of gfx950 assembly.
//
// What it computes: the same instructions, in the same order in every lane, as
// the full dispatch (run_cold, interp.hip) -- a group of lanes that stands at
// one place shares program counter, cycle and row-log position as scalars, and
// only A, X, Y, the flags, RAM, TIA registers and log stores are per lane.
//
// What bounds it: the latency of one wave's instruction stream (at most one
// wave per SIMD runs, and each pass depends on the one before).  On gfx950 an
// instruction issues every 4 cycles, a taken branch to another cache line
// costs 50-100 (instruction fetch), a scalar load that hits 40, an LDS read 60,
// a comparison's way to the scalar unit 24-32, v_readlane 28.
// A compiled loop takes several far branches per pass (compare chain, skipped
// cases, back edge: 471 cycles a pass on the step of 4,096 envs of one 4 KB
// cartridge, k_interp 2.62 ms); here a handler ends by jumping straight to the
// next instruction's handler, so a pass has one: 157 cycles, 0.87 ms.
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
// HOT_REAL), one whose lanes a handler cannot take together (an index out of RAM
// or plain ROM, a page crossed by some, a return to different places, a slice
// that differs, the stack outside RAM), a store whose effect falls on the next
// line or finds its log row full, and at the frame's cycle cap.  The way out and
// back costs some 2,000 cycles.
//
// Where it was loaded across a 4 GB boundary its 32-bit jumps would miss: it then
// does nothing, and every instruction runs per lane (the step's count of
// instructions on the wave-uniform path is 0).
//
// Every wait that a load needs is inside the block, in the handler that uses
// the value or before the block's end.
#pragma once

namespace vcs {

// Slots, and the opcode each runs (HOT_REAL: the word carries it).  Zero-page
// operands are RAM; a store of A to a TIA register that is kept as is has a
// pair of slots per register (hot_tia_slot), one of X or Y takes the register's code
// from the word; GRP0 / GRP1 stores also update the delayed copies; HOT_FLAG + i
// is a store of A to ENAM0, ENAM1, ENABL, VDELP0, VDELP1, VDELBL (two slots
// each); HOT_XR_* and HOT_XW access Superchip RAM through its read and write
// port; HOT_ABS is LDA from a linearly mapped cartridge, HOT_HS the same from a
// bank hotspot (the new bank in the word's low bits); HOT_HMP + 2 r + i is a
// store of A, X, Y (r) to HMP0 / HMP1 (i), HOT_HMM + i one of A to HMM0, HMM1,
// HMBL, HOT_HMCLR one of any register to HMCLR (the class: which << 5), HOT_VSYNC one of A to VSYNC (left to
// the full dispatch when a lane sets bit 1), HOT_INPT4 and HOT_SWCHA_* read the
// joystick; HOT_WSYNC and HOT_ST_NOP (nothing emulated changes) stand for a store
// of A, X or Y; the *_X branches (HOT_BPL_X + condition) cross a page when taken.
// HOT_RESP / HOT_RESM are a store of any register to RESPx / RESMx, RESBL (the
// class: the register's code | which store << 5); HOT_FLAG_X / _Y + i the flags
// above from X or Y; HOT_3F + r a store that selects a 3F slice; HOT_E0 LDA from
// an E0 hotspot; HOT_HS_ST a store to a linear scheme's (the class: the bank |
// which store << 5); HOT_A_TIA + 3 r + i an absolute store of register r to a TIA
// register kept as is (i = 0), GRP0 or GRP1; the others are named for operation
// and mode.  Long handlers have several slots (the opcode of the later ones: 0).
constexpr uint32_t HOT_REAL = 0, HOT_STA_TIA = 1,
                   HOT_STA_GRP0 = 27, HOT_STA_GRP1 = 30, HOT_STX_TIA = 33, HOT_STX_GRP0 = 34, HOT_STX_GRP1 = 35,
                   HOT_STY_TIA = 36, HOT_STY_GRP0 = 37, HOT_STY_GRP1 = 38, HOT_FLAG = 41, HOT_XR_LDA = 53,
                   HOT_XR_ADC = 54, HOT_XR_AND = 55, HOT_XR_EOR = 56, HOT_XR_ORA = 57, HOT_XW = 58,
                   HOT_ABS = 59, HOT_HS = 60, HOT_HMP = 61, HOT_VSYNC = 67, HOT_INPT4 = 68,
                   HOT_SWCHA_LDA = 69, HOT_SWCHA_EOR = 70, HOT_WSYNC = 71, HOT_ST_NOP = 72, HOT_BPL_X = 73,
                   kHotPlain = 81,
                   HOT_JSR = 147, HOT_RESP = 149, HOT_RESM = 150, HOT_FLAG_X = 151, HOT_FLAG_Y = 157, HOT_3F = 163,
                   HOT_E0 = 166, HOT_HS_ST = 168, HOT_Z_CONST = 169, HOT_Z_INPT4 = 170, HOT_A_CONST = 171,
                   HOT_A_SWCHA = 172, HOT_A_INTIM = 173, HOT_A_ROM = 175, HOT_A_RAM = 177, HOT_ZX = 178,
                   HOT_ZY = 179, HOT_ZX_RMW = 180, HOT_AX_ROM = 181, HOT_AY_ROM = 183, HOT_AX_RAM = 185,
                   HOT_AY_RAM = 186, HOT_IY_ROM = 187, HOT_A_RMW = 189, HOT_SEG = 190, HOT_SEG_X = 191, HOT_SEG_Y = 192,
                   HOT_STA_ZX = 193, HOT_STY_ZX = 194, HOT_STX_ZY = 195, HOT_STA_AX = 196, HOT_STA_AY = 197,
                   HOT_STA_A = 198, HOT_STX_A = 199, HOT_STY_A = 200, HOT_A_TIA = 201, HOT_PHP = 210, HOT_PLP = 212,
                   HOT_HMM = 214, HOT_HMCLR = 217;
// The two-step reads: HOT_Z_CONST .. HOT_SEG_Y fetch the operand (the word's
// class: the operation's number, and for the constants which one << 5) and go
// on to the operation, slot kHotWork + its number.
constexpr uint32_t kHotWork = 218, kHotWorks = 18;
enum : uint32_t { HW_LDA, HW_LDX, HW_LDY, HW_AND, HW_ORA, HW_EOR, HW_CMP, HW_CPX, HW_CPY, HW_BIT, HW_ADC, HW_SBC,
                  HW_ASL, HW_ROL, HW_LSR, HW_ROR, HW_DEC, HW_INC, HW_NONE };
constexpr uint32_t kHotSlots = kHotWork + kHotWorks;
constexpr uint8_t kHotSlotOp[kHotSlots] = {
    0x00, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85,
    0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85,
    0x85, 0x86, 0x86, 0x86, 0x84, 0x84, 0x84, 0x00, 0x00, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85, 0x85,
    0x85, 0x85, 0x85, 0x85, 0x85, 0xAD, 0x6D, 0x2D, 0x4D, 0x0D, 0x8D, 0xAD, 0xAD, 0x85, 0x85, 0x86,
    0x86, 0x84, 0x84, 0x85, 0xA5, 0xAD, 0x4D, 0x85, 0x85, 0x10, 0x30, 0x50, 0x70, 0x90, 0xB0, 0xD0,
    0xF0, 0x05, 0x06, 0x09, 0x0A, 0x10, 0x18, 0x24, 0x25, 0x26, 0x29, 0x2A, 0x30, 0x38, 0x45, 0x46,
    0x49, 0x4A, 0x4C, 0x50, 0x65, 0x66, 0x69, 0x6A, 0x70, 0x84, 0x85, 0x86, 0x88, 0x8A, 0x90, 0x98,
    0xA0, 0xA2, 0xA4, 0xA5, 0xA6, 0xA8, 0xA9, 0xAA, 0xB0, 0xB8, 0xC0, 0xC4, 0xC5, 0xC6, 0xC8, 0xC9,
    0xCA, 0xD0, 0xD8, 0xE0, 0xE4, 0xE5, 0xE6, 0xE8, 0xE9, 0xEA, 0xF0, 0xF8, 0x48, 0x68, 0xBA, 0x9A,
    0x60, 0x00, 0x00, 0x20, 0x00, 0x85, 0x85, 0x86, 0x86, 0x86, 0x86, 0x86, 0x86, 0x84, 0x84, 0x84,
    0x84, 0x84, 0x84, 0x85, 0x86, 0x84, 0xAD, 0x00, 0x8D, 0xA5, 0xA5, 0xAD, 0xAD, 0xAD, 0x00, 0xAD,
    0x00, 0xAD, 0xB5, 0xB6, 0x16, 0xBD, 0x00, 0xB9, 0x00, 0xBD, 0xB9, 0xB1, 0x00, 0x0E, 0xAD, 0xBD,
    0xB9, 0x95, 0x94, 0x96, 0x9D, 0x99, 0x8D, 0x8E, 0x8C, 0x8D, 0x8D, 0x8D, 0x8E, 0x8E, 0x8E, 0x8C,
    0x8C, 0x8C, 0x08, 0x00, 0x28, 0x00, 0x85, 0x85, 0x85, 0x85, 0x00, 0x00, 0x00, 0x00, 0x00, 0x00,
    0x00, 0x00, 0x00, 0x00, 0x00, 0x00, 0x00, 0x00, 0x00, 0x00, 0x00, 0x00,
};
// The slot that runs opcode `op` without a page-crossing branch or a TIA store
// (HOT_REAL: none).
constexpr uint32_t hot_slot(uint32_t op) {
    for (uint32_t s = kHotPlain; op && s < HOT_JSR; ++s)
        if (kHotSlotOp[s] == op) return s;
    return HOT_REAL;
}
// The slot of a store of A to the TIA register with code `code` (R_COLUP0 ..
// R_PF2, R_VBLANK, R_NUSIZ0, R_NUSIZ1)
__host__ __device__ constexpr uint32_t hot_tia_slot(uint32_t code) {
    return HOT_STA_TIA + 2 * (code <= R_PF2 ? code : code == R_VBLANK ? 10 : code - R_NUSIZ0 + 11);
}

// ACC: cycle in the line + 52 in the top 7 bits, instructions below
constexpr uint32_t kAccBias = 52, kAccShift = 25, kAccCount = (1u << kAccShift) - 1;

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
#define HL_IMM_(work) HL_B1_8 HL_TGT("s78") HL_FETCH(2) work HL_GO(2)
#define HL_IMM(B, slot, work) HL_ORG(B, slot) HL_WAIT HL_IMM_(work)
#define HL_IMMD(B, slot, work) HL_ORG(B, slot) HL_WAIT HL_B1_8 HL_TGT("s78") HL_FETCH(2) HL_ACC(2) work HL_JUMP
// zero-page read whose result the handler needs: operand in v123
#define HL_ZPR_(test, work)                                                                              \
    HL_B1_7 HL_RAMADDR "ds_read_u8 v123, v122\n" HL_TGT("s78") HL_FETCH(2) HL_ACC(3) test HL_WAIT work HL_JUMP
#define HL_ZPR(B, slot, work) HL_ORG(B, slot) HL_WAIT HL_ZPR_("", work)
// ADC, SBC: whether a lane is in decimal mode is found out while the operand comes
#define HL_ZPRD(B, slot, to, work) HL_ORG(B, slot) HL_WAIT HL_ZPR_(HL_BIN(to), work)
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
#define HL_LDV "v_mov_b32 %[a], v123\nv_mov_b32 %[nz], v123\n"
#define HL_LDI(reg) "v_mov_b32 " reg ", s86\nv_mov_b32 %[nz], s86\n"
// ADC and SBC of a group with a lane in decimal mode (s[50:51]) go on at `to`
#define HL_BIN(to)                                         \
    "s_and_b64 s[96:97], s[50:51], exec\n"                 \
    "s_cbranch_scc1 " to "%=\n"
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
#define HL_ADCV HL_BIN(".Ldadc") HL_ADC("v123")
#define HL_ADCI HL_BIN(".Ldadci") HL_ADC("s86")
#define HL_SBCV HL_BIN(".Ldsbc") "v_xor_b32 v123, 0xff, v123\n" HL_ADC("v123")
#define HL_SBCI HL_BIN(".Ldsbci") "s_xor_b32 s86, s86, 0xff\n" HL_ADC("s86")
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

// branch: `test` sets vcc in the lanes that take it, for the ACC step in s98 (3
// cycles) or s99 (4).  Both successors' words are loaded before the test is known.
#define HL_BR(B, slot, test, tk)                           \
    HL_ORG(B, slot) HL_WAIT                                \
    "s_bfe_i32 s86, s76, 0x80010\n"                        \
    "s_add_u32 s88, s72, 8\n"                              \
    "s_lshl2_add_u32 s89, s86, s88\n"                      \
    "s_load_dwordx4 s[60:63], s[70:71], s89\n"             \
    "s_load_dwordx4 s[76:79], s[70:71], s88\n" test        \
    "s_cmp_eq_u64 vcc, exec\n"                             \
    "s_cselect_b32 s72, s89, s88\n"                        \
    "s_cselect_b32 s87, s9" tk ", (2<<25)+1\n"             \
    "s_cselect_b64 s[96:97], exec, 0\n"                    \
    "s_cmp_lg_u64 vcc, s[96:97]\n"                         \
    "s_cbranch_scc1 .Lpart" tk "_%=\n"                      \
    "s_cmp_eq_u64 s[96:97], exec\n" HL_WAIT                \
    "s_cselect_b64 s[76:77], s[60:61], s[76:77]\n"         \
    "s_cselect_b64 s[78:79], s[62:63], s[78:79]\n"         \
    HL_TGT("s76")                                          \
    "s_add_u32 s73, s73, s87\n"                            \
    "s_cselect_b32 s74, s85, s74\n" HL_JUMP
#define HL_T_NE(mask, src) "v_and_b32 v122, " mask ", " src "\nv_cmp_ne_u32 vcc, 0, v122\n"
#define HL_T_EQ(mask, src) "v_and_b32 v122, " mask ", " src "\nv_cmp_eq_u32 vcc, 0, v122\n"

// absolute jump (the target lies in the cartridge window; one that changes pc
// bits 12-15, kept in KEY, is left to the full dispatch)
#define HL_JMP(B, slot)                                    \
    HL_ORG(B, slot) HL_WAIT                                \
    "s_xor_b32 s86, s76, s59\n"                            \
    "s_lshr_b32 s86, s86, 28\n"                            \
    "s_cbranch_scc1 .Lout%=\n"                             \
    "s_bfe_u32 s86, s76, 0xc0010\n"                        \
    "s_and_b32 s72, s72, 0xffffc000\n"                     \
    "s_lshl2_add_u32 s72, s86, s72\n"                      \
    "s_load_dwordx4 s[76:79], s[70:71], s72\n" HL_WAIT HL_TGT("s76") HL_GO(3)

// LDA absolute from the tile's cartridge s[40:41] (linear: bank << 12 | offset)
#define HL_ABSBYTE                                         \
    "s_and_b32 s87, s86, -4\n"                             \
    "s_load_dword s94, s[40:41], s87\n"                    \
    "s_lshl_b32 s86, s86, 3\n" HL_WAIT                     \
    "s_lshr_b32 s94, s94, s86\n"                           \
    "s_and_b32 s86, s94, 0xff\n" HL_LDI("%[a]")
#define HL_ABS(B, slot)                                    \
    HL_ORG(B, slot) HL_WAIT                                \
    "s_lshr_b32 s87, s72, 14\n"                            \
    "s_bfe_u32 s86, s76, 0xc0010\n"                        \
    "s_lshl_b32 s87, s87, 12\n"                            \
    "s_or_b32 s86, s86, s87\n" HL_TGT("s79") HL_FETCH(3)   \
    HL_ABSBYTE HL_GO(4)
#define HL_HS(B, slot)                                     \
    HL_ORG(B, slot) HL_WAIT                                \
    "s_and_b32 s87, s76, 7\n"                              \
    "s_bfe_u32 s86, s76, 0xc0010\n"                        \
    "s_lshl_b32 s88, s87, 14\n"                            \
    "s_lshl_b32 s87, s87, 12\n"                            \
    "s_add_u32 s72, s72, 12\n"                             \
    "s_and_b32 s72, s72, 0x3fff\n"                         \
    "s_or_b32 s72, s72, s88\n"                             \
    "s_or_b32 s86, s86, s87\n"                             \
    "s_load_dwordx4 s[76:79], s[70:71], s72\n" HL_ABSBYTE HL_TGT("s76") HL_GO(4)
// motion registers and VSYNC: no log entry, kept per lane
#define HL_HMP(B, slot, reg, hmp) HL_ORG(B, slot) HL_WAIT HL_TGT("s78") HL_FETCH(2) "v_mov_b32 " hmp ", " reg "\n" HL_GO(3)
#define HL_HMM(B, slot, reg) HL_ORG(B, slot) HL_WAIT "ds_write_b8 %[tia], %[a] offset:" #reg "\n" HL_TGT("s78") HL_FETCH(2) HL_GO(3)
#define HL_HMCLR(B, slot)                                  \
    HL_ORG(B, slot) HL_WAIT                                \
    "v_mov_b32 v122, 0\n"                                  \
    "v_mov_b32 %[hmp0], 0\n"                               \
    "v_mov_b32 %[hmp1], 0\n"                               \
    "ds_write_b8 %[tia], v122 offset:41\n"                 \
    "ds_write_b8 %[tia], v122 offset:42\n"                 \
    "ds_write_b8 %[tia], v122 offset:43\n" HL_TGT("s78") HL_FETCH(2) HL_GO(3)
#define HL_VSYNC(B, slot)                                  \
    HL_ORG(B, slot) HL_WAIT                                \
    "v_and_b32 v122, 2, %[a]\n"                            \
    "v_cmp_ne_u32 vcc, 0, v122\n"                          \
    "s_cbranch_vccnz .Lout%=\n" HL_TGT("s78") HL_FETCH(2)  \
    "v_mov_b32 %[vsync], %[a]\n" HL_GO(3)
// the joystick, held per lane for the frame
#define HL_LDR(reg) "v_mov_b32 %[a], " reg "\nv_mov_b32 %[nz], " reg "\n"
#define HL_IN(B, slot, len, next, cyc, work) HL_ORG(B, slot) HL_WAIT HL_TGT(next) HL_FETCH(len) work HL_GO(cyc)
// Superchip RAM of the lane's env, in HBM: operand in v123 (the wait includes
// the log stores before it)
#define HL_XADDR                                           \
    "s_bfe_u32 s66, s76, 0x70010\n"                        \
    "v_lshl_add_u64 v[120:121], s[66:67], 0, %[xram]\n"
#define HL_XR_(work)                                       \
    HL_XADDR "global_load_ubyte v123, v[120:121], off\n" HL_TGT("s79") HL_FETCH(3) HL_ACC(4)        \
    "s_waitcnt vmcnt(0)\n" work HL_JUMP
#define HL_XR(B, slot, work) HL_ORG(B, slot) HL_WAIT HL_XR_(work)
#define HL_XW(B, slot)                                     \
    HL_ORG(B, slot) HL_WAIT HL_XADDR                       \
    "global_store_byte v[120:121], %[a], off\n" HL_TGT("s79") HL_FETCH(3) HL_GO(4)

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
// line has not ended (the line's number, or -1 past its end, against the open
// row's); before the visible part it only changes the register when the row
// before is open (about half the stores of the plain workload).  Else .Lsnap
// opens rows first, or leaves the store to the full dispatch.  `code8`: the entry's register code << 8 less 3 * 52 + 68.  Where
// the entry goes is per lane: lanes whose earlier writes fell on different
// sides of a line's visible part have logged different numbers of entries, and
// still run as one group.
#define HL_LOGGED(id, val, code8, write)                   \
    "s_add_u32 s73, s73, (3<<25)+1\n"                      \
    "s_cselect_b32 s87, -9, s80\n"                         \
    "s_lshr_b32 s88, s73, 25\n"                            \
    "s_cmp_lt_u32 s88, 75\n"                               \
    "s_cbranch_scc1 .Lhbl" id "_%=\n"                       \
    "s_cmp_lg_u32 s87, s83\n"                              \
    "s_mul_i32 s87, s88, 3\n"                              \
    "s_cbranch_scc1 .Lrow" id "_%=\n"                       \
    ".Lent" id "_%=:\n"                                     \
    "s_add_u32 s87, s87, " code8 "\n"                      \
    "v_lshl_or_b32 v123, " val ", 16, s87\n"               \
    "global_store_dword v[100:101], v123, off\n"           \
    "v_lshl_add_u64 v[100:101], 1, 2, v[100:101]\n"        \
    ".Lreg" id "_%=:\n" write HL_JUMP                       \
    ".Lhbl" id "_%=:\n"                                     \
    "s_add_u32 s87, s87, 1\n"                              \
    "s_cmp_lg_u32 s87, s83\n"                              \
    "s_cbranch_scc1 .Lrow" id "_%=\n" write HL_JUMP         \
    ".Lrow" id "_%=:\n"                                     \
    "s_swappc_b64 s[96:97], s[64:65]\n"                    \
    "s_cbranch_scc0 .Lent" id "_%=\n"                       \
    "s_branch .Lreg" id "_%=\n"
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
// ENAMx, ENABL (bit 1), VDELx (bit 0): bit k of the flags byte and the full byte 32 + k
#define HL_FLAG_(slot, B, k, bit, body)                    \
    HL_ORG(B, slot) HL_WAIT "v_mov_b32 v126, %[a]\n"       \
    ".Lbf" #k body "%=:\n"                                 \
    "ds_read_u8 v124, %[tia] offset:23\n"                  \
    "v_bfe_u32 v122, v126, " #bit ", 1\n" HL_TGT("s78") HL_FETCH(2) HL_WAIT \
    "v_and_b32 v124, ~(1<<" #k "), v124\n"                 \
    "v_lshl_or_b32 v125, v122, " #k ", v124\n"
#define HL_FLAG_WRITE(k)                                   \
    "ds_write_b8 %[tia], v125 offset:23\n"                 \
    "ds_write_b8 %[tia], v126 offset:32+" #k "\n"
#define HL_FLAG_LOG(B, slot, k, bit)                       \
    HL_FLAG_(slot, B, k, bit, "l") HL_LOGGED("f" #k, "v125", "23*256-224", HL_FLAG_WRITE(k))
#define HL_FLAG_NOLOG(B, slot, k, bit) HL_FLAG_(slot, B, k, bit, "u") HL_FLAG_WRITE(k) HL_GO(3)
// the same of X or Y
#define HL_FLAG_XY(B, slot, reg, k, body) HL_ORG(B, slot) HL_WAIT "v_mov_b32 v126, " reg "\ns_branch .Lbf" #k body "%=\n"
#define HL_FLAGS_XY(B, body)                                                                                   \
    HL_FLAG_XY(B, 151, "%[x]", 0, body) HL_FLAG_XY(B, 152, "%[x]", 1, body) HL_FLAG_XY(B, 153, "%[x]", 2, body) \
    HL_FLAG_XY(B, 154, "%[x]", 4, body) HL_FLAG_XY(B, 155, "%[x]", 5, body) HL_FLAG_XY(B, 156, "%[x]", 6, body) \
    HL_FLAG_XY(B, 157, "%[y]", 0, body) HL_FLAG_XY(B, 158, "%[y]", 1, body) HL_FLAG_XY(B, 159, "%[y]", 2, body) \
    HL_FLAG_XY(B, 160, "%[y]", 4, body) HL_FLAG_XY(B, 161, "%[y]", 5, body) HL_FLAG_XY(B, 162, "%[y]", 6, body)
// RESPx, RESMx, RESBL (of any register): the position is the beam's + `delay`
// in the visible part, delay - 2 before it; then as a register store
#define HL_RES(B, slot, delay, body)                       \
    HL_ORG(B, slot) HL_WAIT                                \
    "s_add_u32 s88, s73, 3<<25\n"                          \
    "s_lshr_b32 s88, s88, 25\n"                            \
    "s_mul_i32 s87, s88, 3\n"                              \
    "s_sub_u32 s87, s87, 3*52+68-" #delay "\n"             \
    "s_sub_u32 s86, s87, 160\n"                            \
    "s_cselect_b32 s87, s87, s86\n"                        \
    "s_cmp_lt_u32 s88, 75\n"                               \
    "s_cselect_b32 s87, " #delay "-2, s87\n"               \
    "v_mov_b32 v125, s87\n"                                \
    "s_branch .Lbt" body "%=\n"
#define HL_RES_LOG(B, slot, delay) HL_RES(B, slot, delay, "l")
#define HL_RES_NOLOG(B, slot, delay) HL_RES(B, slot, delay, "u")
#define HL_FXY_LOG(B) HL_FLAGS_XY(B, "l")
#define HL_FXY_NOLOG(B) HL_FLAGS_XY(B, "u")

// The stack, while it stays in RAM in every lane (a push at $80 or above, a
// pull from below $FF); a return whose lanes or window part is left too.
#define HL_PUSHADDR "v_and_b32 v122, 0x7f, %[sp]\nv_add_u32 v122, v122, %[ram]\n"
#define HL_PHA(B, slot)                                    \
    HL_ORG(B, slot) HL_WAIT                                \
    "v_cmp_gt_u32 vcc, 0x80, %[sp]\n" HL_PUSHADDR          \
    "s_cbranch_vccnz .Lout%=\n" HL_TGT("s77") HL_FETCH(1)  \
    "ds_write_b8 v122, %[a]\n"                             \
    "v_add_u32 %[sp], -1, %[sp]\n" HL_GO(3)
#define HL_PLA(B, slot)                                    \
    HL_ORG(B, slot) HL_WAIT                                \
    "v_add_u32 v122, 0xffffff81, %[sp]\n"                  \
    "v_cmp_lt_u32 vcc, 0x7f, v122\n"                       \
    "v_add_u32 v122, v122, %[ram]\n"                       \
    "s_cbranch_vccnz .Lout%=\n" HL_TGT("s77") HL_FETCH(1)  \
    "ds_read_u8 %[a], v122\n"                              \
    "ds_read_u8 %[nz], v122\n"                             \
    "v_add_u32 %[sp], 1, %[sp]\n" HL_GO(4)
#define HL_JSR(B, slot)                                    \
    HL_ORG(B, slot) HL_WAIT                                \
    "s_xor_b32 s86, s76, s59\n"                            \
    "s_lshr_b32 s86, s86, 28\n"                            \
    "s_cbranch_scc1 .Lout%=\n"                             \
    "v_cmp_gt_u32 vcc, 0x81, %[sp]\n" HL_PUSHADDR          \
    "s_cbranch_vccnz .Lout%=\n"                            \
    "s_lshr_b32 s87, s72, 2\n"                             \
    "s_and_b32 s87, s87, 0xfff\n"                          \
    "s_lshr_b32 s88, s59, 28\n"                            \
    "s_lshl_b32 s88, s88, 12\n"                            \
    "s_bfe_u32 s86, s76, 0xc0010\n"                        \
    "s_and_b32 s72, s72, 0xffffc000\n"                     \
    "s_lshl2_add_u32 s72, s86, s72\n"                      \
    "s_load_dwordx4 s[76:79], s[70:71], s72\n"             \
    "s_add_u32 s87, s87, 2\n"                              \
    "s_or_b32 s87, s87, s88\n"                             \
    "s_lshr_b32 s88, s87, 8\n"                             \
    "v_mov_b32 v123, s88\n"                                \
    "v_mov_b32 v124, s87\n"                                \
    "ds_write_b8 v122, v123\n"                             \
    "v_add_u32 v122, -1, v122\n"                           \
    "ds_write_b8 v122, v124\n"                             \
    "v_add_u32 %[sp], -2, %[sp]\n" HL_WAIT HL_TGT("s76") HL_GO(6)
#define HL_RTS(B, slot)                                    \
    HL_ORG(B, slot) HL_WAIT                                \
    "v_add_u32 v122, 0xffffff81, %[sp]\n"                  \
    "v_cmp_lt_u32 vcc, 0x7e, v122\n"                       \
    "v_add_u32 v122, v122, %[ram]\n"                       \
    "s_cbranch_vccnz .Lout%=\n"                            \
    "ds_read_u8 v123, v122\n"                              \
    "ds_read_u8 v124, v122 offset:1\n" HL_WAIT             \
    "v_lshl_or_b32 v123, v124, 8, v123\n"                  \
    "v_add_u32 v123, 1, v123\n"                            \
    "v_and_b32 v123, 0xffff, v123\n"                       \
    "s_nop 1\n"                                            \
    "v_readfirstlane_b32 s86, v123\n"                      \
    "s_lshr_b32 s88, s59, 28\n"                            \
    "s_lshr_b32 s87, s86, 12\n"                            \
    "s_cmp_lg_u32 s87, s88\n"                              \
    "v_cmp_ne_u32 vcc, s86, v123\n"                        \
    "s_cbranch_scc1 .Lout%=\n"                             \
    "s_and_b32 s86, s86, 0xfff\n"                          \
    "s_cbranch_vccnz .Lout%=\n"                            \
    "s_cmp_gt_u32 s86, 0xffc\n"                            \
    "s_cbranch_scc1 .Lout%=\n"                             \
    "s_and_b32 s72, s72, 0xffffc000\n"                     \
    "s_lshl2_add_u32 s72, s86, s72\n"                      \
    "s_load_dwordx4 s[76:79], s[70:71], s72\n"             \
    "v_add_u32 %[sp], 2, %[sp]\n" HL_WAIT HL_TGT("s76") HL_GO(6)

#define HL_PHP(B, slot)                                    \
    HL_ORG(B, slot) HL_WAIT                                \
    "v_cmp_gt_u32 vcc, 0x80, %[sp]\n" HL_PUSHADDR          \
    "s_cbranch_vccnz .Lout%=\n" HL_TGT("s77") HL_FETCH(1)  \
    "v_and_b32 v124, 0x180, %[nz]\n"                       \
    "v_cmp_ne_u32 vcc, 0, v124\n"                          \
    "v_and_b32 v123, 4, %[p]\n"                            \
    "v_or_b32 v123, 0x30, v123\n"                          \
    "v_mov_b32 v125, 0x80\n"                               \
    "v_cndmask_b32 v125, 0, v125, vcc\n"                   \
    "v_and_b32 v124, 0xff, %[nz]\n"                        \
    "v_cmp_eq_u32 vcc, 0, v124\n"                          \
    "v_or3_b32 v123, v123, v125, %[c]\n"                   \
    "v_mov_b32 v125, 2\n"                                  \
    "v_mov_b32 v124, 8\n"                                  \
    "v_cndmask_b32 v125, 0, v125, vcc\n"                   \
    "v_cndmask_b32 v124, 0, v124, s[50:51]\n"              \
    "v_or3_b32 v123, v123, v125, v124\n"                   \
    "v_bfe_u32 v124, %[v], 7, 1\n"                         \
    "v_lshl_or_b32 v123, v124, 6, v123\n"                  \
    "ds_write_b8 v122, v123\n"                             \
    "v_add_u32 %[sp], -1, %[sp]\n" HL_GO(3)
#define HL_PLP(B, slot)                                    \
    HL_ORG(B, slot) HL_WAIT                                \
    "v_add_u32 v122, 0xffffff81, %[sp]\n"                  \
    "v_cmp_lt_u32 vcc, 0x7f, v122\n"                       \
    "v_add_u32 v122, v122, %[ram]\n"                       \
    "s_cbranch_vccnz .Lout%=\n"                            \
    "ds_read_u8 v123, v122\n" HL_TGT("s77") HL_FETCH(1)    \
    "v_add_u32 %[sp], 1, %[sp]\n" HL_ACC(4) HL_WAIT        \
    "v_and_b32 v124, 0xef, v123\n"                         \
    "v_or_b32 %[p], 0x20, v124\n"                          \
    "v_and_b32 %[c], 1, v123\n"                            \
    "v_lshlrev_b32 %[v], 1, v123\n"                        \
    "v_and_b32 v124, 0x80, v123\n"                         \
    "v_bfe_u32 v125, v123, 1, 1\n"                         \
    "v_xor_b32 v125, 1, v125\n"                            \
    "v_lshl_or_b32 %[nz], v124, 1, v125\n"                 \
    "v_and_b32 v124, 8, v123\n"                            \
    "v_cmp_ne_u32 vcc, 0, v124\n"                          \
    "s_andn2_b64 s[50:51], s[50:51], exec\n"               \
    "s_or_b64 s[50:51], s[50:51], vcc\n" HL_JUMP

// Absolute stores: to RAM; to a TIA register that the zero-page form logs, as
// that form a cycle and a byte later (left first when it would be: at the
// line's end, or when a row's entries might not fit)
#define HL_ASTO(B, slot, reg)                              \
    HL_ORG(B, slot) HL_WAIT HL_B1_7 HL_RAMADDR "ds_write_b8 v122, " reg "\n" HL_TGT("s79") HL_FETCH(3) HL_GO(4)
#define HL_ATIA(B, slot, reg, body)                        \
    HL_ORG(B, slot) HL_WAIT                                \
    "v_sub_u32 v122, v100, %[log0]\n"                      \
    "v_lshrrev_b32 v122, 2, v122\n"                        \
    "v_cmp_lt_u32 vcc, s69, v122\n"                        \
    "s_add_u32 s87, s73, 4<<25\n"                          \
    "s_cbranch_scc1 .Lout%=\n"                             \
    "s_bitcmp1_b32 s59, 27\n"                              \
    "s_cselect_b64 vcc, vcc, 0\n"                          \
    "s_cbranch_vccnz .Lout%=\n"                            \
    "s_add_u32 s73, s73, 1<<25\n"                          \
    "s_add_u32 s72, s72, 4\n"                              \
    "s_mov_b32 s78, s79\n"                                 \
    "v_mov_b32 v125, " reg "\n"                            \
    "s_branch .Lb" body "%=\n"
#define HL_ATIAS(B, l)                                                                                            \
    HL_ATIA(B, 201, "%[a]", "t" l) HL_ATIA(B, 202, "%[a]", "g" l) HL_ATIA(B, 203, "%[a]", "h" l)                 \
    HL_ATIA(B, 204, "%[x]", "t" l) HL_ATIA(B, 205, "%[x]", "g" l) HL_ATIA(B, 206, "%[x]", "h" l)                 \
    HL_ATIA(B, 207, "%[y]", "t" l) HL_ATIA(B, 208, "%[y]", "g" l) HL_ATIA(B, 209, "%[y]", "h" l)
#define HL_ATIA_LOG(B) HL_ATIAS(B, "l")
#define HL_ATIA_NOLOG(B) HL_ATIAS(B, "u")

// 3F: a store to $00-$3F selects a slice (mask: the class), the same in every lane
#define HL_3F(B, slot, reg)                                \
    HL_ORG(B, slot) HL_WAIT                                \
    "s_and_b32 s86, s76, 0x7f\n"                           \
    "v_and_b32 v122, s86, " reg "\n"                       \
    "s_branch .Lslice%=\n"
// LDA from an E0 hotspot ($1FE0-$1FF7: slice number in bits 0-2, segment in
// 3-4), whose byte lies in the last slice
#define HL_E0(B, slot)                                     \
    HL_ORG(B, slot) HL_WAIT HL_B1_8                        \
    "s_bfe_u32 s87, s86, 0x20003\n"                        \
    "s_mul_i32 s87, s87, 3\n"                              \
    "s_add_u32 s87, s87, 14\n"                             \
    "s_lshl_b32 s88, 7, s87\n"                             \
    "s_and_b32 s89, s86, 7\n"                              \
    "s_lshl_b32 s89, s89, s87\n"                           \
    "s_add_u32 s72, s72, 12\n"                             \
    "s_andn2_b32 s72, s72, s88\n"                          \
    "s_or_b32 s72, s72, s89\n"                             \
    "s_load_dwordx4 s[76:79], s[70:71], s72\n"             \
    "s_or_b32 s86, s86, 0x1f00\n" HL_ABSBYTE HL_TGT("s76") HL_GO(4)
// a store to a bank hotspot of a linear scheme (the new bank in the class)
#define HL_HS_ST(B, slot)                                  \
    HL_ORG(B, slot) HL_WAIT                                \
    "s_and_b32 s87, s76, 7\n"                              \
    "s_lshl_b32 s87, s87, 14\n"                            \
    "s_add_u32 s72, s72, 12\n"                             \
    "s_and_b32 s72, s72, 0x3fff\n"                         \
    "s_or_b32 s72, s72, s87\n"                             \
    "s_load_dwordx4 s[76:79], s[70:71], s72\n" HL_WAIT HL_TGT("s76") HL_GO(4)

// Two-step reads: the operand to v123, then on to the operation's slot (HL_OP,
// taken from the word before the next one is loaded).
#define HL_OP                                              \
    "s_and_b32 s90, s76, 31\n"                             \
    "s_lshl_b32 s90, s90, 7\n"                             \
    "s_add_u32 s90, s90, s84\n"                            \
    "s_add_u32 s90, s90, 128*218\n"
#define HL_DO "s_setpc_b64 s[90:91]\n"
#define HL_WORK(B, slot, work) HL_ORG(B, slot) work HL_JUMP
// constants: 0, $80, $0B (SWCHB)
#define HL_CONST                                           \
    "s_bfe_u32 s87, s76, 0x20005\n"                        \
    "s_lshl_b32 s87, s87, 3\n"                             \
    "s_lshr_b32 s86, 0x0b8000, s87\n"                      \
    "s_and_b32 s86, s86, 0xff\n"                           \
    "v_mov_b32 v123, s86\n"
#define HL_ZIN(B, slot, get) HL_ORG(B, slot) HL_WAIT get HL_OP HL_TGT("s78") HL_FETCH(2) HL_ACC(3) HL_DO
#define HL_AIN(B, slot, get) HL_ORG(B, slot) HL_WAIT get HL_OP HL_TGT("s79") HL_FETCH(3) HL_ACC(4) HL_DO
#define HL_AROM(B, slot)                                   \
    HL_ORG(B, slot) HL_WAIT                                \
    "s_lshr_b32 s87, s72, 14\n"                            \
    "s_bfe_u32 s86, s76, 0xc0010\n"                        \
    "s_lshl_b32 s87, s87, 12\n"                            \
    "s_or_b32 s86, s86, s87\n" HL_OP HL_TGT("s79") HL_FETCH(3) HL_ACC(4) \
    "s_and_b32 s87, s86, -4\n"                             \
    "s_load_dword s94, s[40:41], s87\n"                    \
    "s_lshl_b32 s86, s86, 3\n" HL_WAIT                     \
    "s_lshr_b32 s94, s94, s86\n"                           \
    "s_and_b32 s86, s94, 0xff\n"                           \
    "v_mov_b32 v123, s86\n" HL_DO
#define HL_ARAM(B, slot)                                   \
    HL_ORG(B, slot) HL_WAIT HL_B1_7 HL_RAMADDR "ds_read_u8 v123, v122\n"   \
    HL_OP HL_TGT("s79") HL_FETCH(3) HL_ACC(4) HL_WAIT HL_DO
// INTIM: cycles since the timer was written are the lane's `tm` + the access
// cycle (76 lines + the cycle in the line, from the base line)
#define HL_INTIM(B, slot)                                  \
    HL_ORG(B, slot) HL_WAIT                                \
    "s_bfe_i32 s86, s59, 0x1b0000\n"                       \
    "s_sub_u32 s86, s86, s80\n"                            \
    "s_mul_i32 s86, s86, 76\n"                             \
    "s_lshr_b32 s87, s73, 25\n"                            \
    "s_add_u32 s86, s86, s87\n"                            \
    "s_add_u32 s86, s86, 76*320-52+3\n"                    \
    HL_OP HL_TGT("s79") HL_FETCH(3)                        \
    "v_add_u32 v122, s86, %[tm]\n"                         \
    "v_add_u32 v124, 1, %[tv]\n"                           \
    "v_lshlrev_b32 v124, %[tsh], v124\n"                   \
    "v_sub_u32 v124, v122, v124\n"                         \
    "v_cmp_gt_i32 vcc, 0, v124\n"                          \
    "v_sub_u32 v124, 0xff, v124\n"                         \
    "v_ashrrev_i32 v123, %[tsh], v122\n"                   \
    "v_sub_u32 v123, %[tv], v123\n"                        \
    "v_cndmask_b32 v123, v124, v123, vcc\n"                \
    "v_and_b32 v123, 0xff, v123\n" HL_ACC(4) HL_DO
// indexed by a register: the address in RAM in every lane, or left.  Zero page
// (wraps in it), and absolute with a zero-page base (does not).
#define HL_ZIDX(idx)                                       \
    HL_B1_8                                                \
    "v_add_u32 v122, s86, " idx "\n"                       \
    "v_and_b32 v122, 0xff, v122\n" HL_INRAM
#define HL_AIDX(idx)                                       \
    HL_B1_8                                                \
    "v_add_u32 v122, s86, " idx "\n" HL_INRAM
#define HL_INRAM                                           \
    "v_add_u32 v122, 0xffffff80, v122\n"                   \
    "v_cmp_lt_u32 vcc, 0x7f, v122\n"                       \
    "v_add_u32 v122, v122, %[ram]\n"                       \
    "s_cbranch_vccnz .Lout%=\n"
#define HL_RIDX(B, slot, addr, len, next, cyc)             \
    HL_ORG(B, slot) HL_WAIT addr "ds_read_u8 v123, v122\n" \
    HL_OP HL_TGT(next) HL_FETCH(len) HL_ACC(cyc) HL_WAIT HL_DO
#define HL_SIDX(B, slot, addr, reg, len, next, cyc)        \
    HL_ORG(B, slot) HL_WAIT addr "ds_write_b8 v122, " reg "\n" HL_TGT(next) HL_FETCH(len) HL_GO(cyc)
// ... in a linear cartridge: every lane in the bank's plain ROM (offsets s92 ..
// s92 + s42 - 1: no hotspot, no Superchip RAM), and all or none across a page.
// s39: the LDS copy, or -1: read from HBM (the wait includes the log stores before it)
#define HL_AXROM(B, slot, idx)                             \
    HL_ORG(B, slot) HL_WAIT HL_B1_8                        \
    "s_bfe_u32 s87, s76, 0xc0010\n"                        \
    "v_add_u32 v122, s87, " idx "\n"                       \
    "v_add_u32 v124, s86, " idx "\n"                       \
    HL_INROM(4, ".Lhbm") HL_ROM_GO("s79", 3) HL_WAIT HL_DO
// (v122: the offset in the bank, v124: above $FF across a page)
#define HL_INROM(cyc, hbm)                                 \
    "v_subrev_u32 v123, s92, v122\n"                       \
    "v_cmp_le_u32 s[96:97], s42, v123\n" HL_CROSS(cyc)     \
    "s_lshr_b32 s87, s72, 14\n"                            \
    "s_lshl_b32 s87, s87, 12\n" HL_ROMBYTE(hbm)
#define HL_CROSS(cyc)                                      \
    "v_cmp_lt_u32 vcc, 0xff, v124\n"                       \
    "s_cmp_lg_u64 s[96:97], 0\n"                           \
    "s_cbranch_scc1 .Lout%=\n"                             \
    "s_mov_b32 s88, (" #cyc "<<25)+1\n"                    \
    "s_cmp_eq_u64 vcc, exec\n"                             \
    "s_cselect_b32 s88, ((" #cyc "+1)<<25)+1, s88\n"       \
    "s_cselect_b64 s[96:97], exec, 0\n"                    \
    "s_cmp_lg_u64 vcc, s[96:97]\n"                         \
    "s_cbranch_scc1 .Lout%=\n"
#define HL_ROMBYTE(hbm)                                    \
    "v_add_u32 v122, s87, v122\n"                          \
    "s_cmp_eq_u32 s39, -1\n"                               \
    "s_cbranch_scc1 " hbm "%=\n"                           \
    "v_add_u32 v122, s39, v122\n"                          \
    "ds_read_u8 v123, v122\n"
#define HL_ROM_GO(next, len)                               \
    HL_OP HL_TGT(next) HL_FETCH(len)                       \
    "s_add_u32 s73, s73, s88\n"                            \
    "s_cselect_b32 s74, s85, s74\n"
// ... in an E0 or 3F cartridge: v125, the index, added inside the segment or half
#define HL_SEG(B, slot, idx) HL_ORG(B, slot) HL_WAIT "v_mov_b32 v125, " idx "\ns_branch .Lseg%=\n"
// (zp),Y: the pointer in RAM, per lane
#define HL_IYROM(B, slot)                                  \
    HL_ORG(B, slot) HL_WAIT HL_B1_7 HL_RAMADDR             \
    "ds_read_u8 v124, v122\n"                              \
    "ds_read_u8 v123, v122 offset:1\n" HL_WAIT             \
    "v_add_u32 v124, v124, %[y]\n"                         \
    "v_lshl_add_u32 v122, v123, 8, v124\n"                 \
    "v_and_b32 v122, 0x1fff, v122\n"                       \
    "v_add_u32 v122, 0xfffff000, v122\n"                   \
    HL_INROM(5, ".Lhbmy") HL_ROM_GO("s78", 2) HL_WAIT HL_DO
#define HL_XY_LOG(B, slot, reg, body) HL_XY_(B, slot, reg, ".Lb" body "l")
#define HL_XY_NOLOG(B, slot, reg, body) HL_XY_(B, slot, reg, ".Lb" body "u")

// Every handler of one of the two blocks (frames whose writes are logged, and
// the others: dispatch by block spares each TIA store the question).
#define HL_BLOCK(B, TIA, TIAX, GRP0, GRP1, HL_XY, FLAG, RES, FXY, ATIA) \
    HL_ORG(B, 0) "s_branch .Lout%=\n"                                                                /* HOT_REAL */ \
    TIA(B, 1, 0)                                                                                     /* STA COLUP0 */ \
    TIA(B, 3, 1)                                                                                     /* STA COLUP1 */ \
    TIA(B, 5, 2)                                                                                     /* STA COLUPF */ \
    TIA(B, 7, 3)                                                                                     /* STA COLUBK */ \
    TIA(B, 9, 4)                                                                                     /* STA CTRLPF */ \
    TIA(B, 11, 5)                                                                                    /* STA REFP0 */ \
    TIA(B, 13, 6)                                                                                    /* STA REFP1 */ \
    TIA(B, 15, 7)                                                                                    /* STA PF0 */ \
    TIA(B, 17, 8)                                                                                    /* STA PF1 */ \
    TIA(B, 19, 9)                                                                                    /* STA PF2 */ \
    TIA(B, 21, 14)                                                                                   /* STA VBLANK */ \
    TIA(B, 23, 18)                                                                                   /* STA NUSIZ0 */ \
    TIA(B, 25, 19)                                                                                   /* STA NUSIZ1 */ \
    GRP0(B, 27)                                                                                      /* STA GRP0 */ \
    GRP1(B, 30)                                                                                      /* STA GRP1 */ \
    HL_XY(B, 33, "%[x]", "t")                                                                        /* STX to a TIA register */ \
    HL_XY(B, 34, "%[x]", "g")                                                                        /* STX GRP0 */ \
    HL_XY(B, 35, "%[x]", "h")                                                                        /* STX GRP1 */ \
    HL_XY(B, 36, "%[y]", "t")                                                                        /* STY to a TIA register */ \
    HL_XY(B, 37, "%[y]", "g")                                                                        /* STY GRP0 */ \
    HL_XY(B, 38, "%[y]", "h")                                                                        /* STY GRP1 */ \
    TIAX(B, 39)                                                                                      /* the body of the two stores to a TIA register */ \
    FLAG(B, 41, 0, 1)                                                                                /* STA ENAM0 */ \
    FLAG(B, 43, 1, 1)                                                                                /* STA ENAM1 */ \
    FLAG(B, 45, 2, 1)                                                                                /* STA ENABL */ \
    FLAG(B, 47, 4, 0)                                                                                /* STA VDELP0 */ \
    FLAG(B, 49, 5, 0)                                                                                /* STA VDELP1 */ \
    FLAG(B, 51, 6, 0)                                                                                /* STA VDELBL */ \
    HL_XR(B, 53, HL_LDV)                                                                             /* LDA from Superchip RAM */ \
    HL_XR(B, 54, HL_ADCV)                                                                             /* ADC from Superchip RAM */ \
    HL_XR(B, 55, HL_AND("v123"))                                                                     /* AND from Superchip RAM */ \
    HL_XR(B, 56, HL_EOR("v123"))                                                                     /* EOR from Superchip RAM */ \
    HL_XR(B, 57, HL_ORA("v123"))                                                                     /* ORA from Superchip RAM */ \
    HL_XW(B, 58)                                                                                     /* STA to Superchip RAM */ \
    HL_ABS(B, 59)                                                                                    /* LDA from the cartridge */ \
    HL_HS(B, 60)                                                                                     /* LDA from a bank hotspot */ \
    HL_HMP(B, 61, "%[a]", "%[hmp0]")                                                                 /* STA HMP0 */ \
    HL_HMP(B, 62, "%[a]", "%[hmp1]")                                                                 /* STA HMP1 */ \
    HL_HMP(B, 63, "%[x]", "%[hmp0]")                                                                 /* STX HMP0 */ \
    HL_HMP(B, 64, "%[x]", "%[hmp1]")                                                                 /* STX HMP1 */ \
    HL_HMP(B, 65, "%[y]", "%[hmp0]")                                                                 /* STY HMP0 */ \
    HL_HMP(B, 66, "%[y]", "%[hmp1]")                                                                 /* STY HMP1 */ \
    HL_VSYNC(B, 67)                                                                                  /* STA VSYNC without bit 1 */ \
    HL_IN(B, 68, 2, "s78", 3, HL_LDR("%[inpt4]"))                                                    /* LDA INPT4 */ \
    HL_IN(B, 69, 3, "s79", 4, HL_LDR("%[swcha]"))                                                    /* LDA SWCHA */ \
    HL_IN(B, 70, 3, "s79", 4, HL_EOR("%[swcha]"))                                                    /* EOR SWCHA */ \
    HL_SYNC(B, 71)                                                                                   /* WSYNC */ \
    HL_ORG(B, 72) HL_WAIT HL_TGT("s78") HL_FETCH(2) HL_GO(3)                                         /* store without effect */ \
    HL_BR(B, 73, HL_T_EQ("0x180", "%[nz]"), "9")                                                     /* BPL across a page */ \
    HL_BR(B, 74, HL_T_NE("0x180", "%[nz]"), "9")                                                     /* BMI across a page */ \
    HL_BR(B, 75, HL_T_EQ("0x80", "%[v]"), "9")                                                       /* BVC across a page */ \
    HL_BR(B, 76, HL_T_NE("0x80", "%[v]"), "9")                                                       /* BVS across a page */ \
    HL_BR(B, 77, "v_cmp_eq_u32 vcc, 0, %[c]\n", "9")                                                 /* BCC across a page */ \
    HL_BR(B, 78, "v_cmp_ne_u32 vcc, 0, %[c]\n", "9")                                                 /* BCS across a page */ \
    HL_BR(B, 79, HL_T_NE("0xff", "%[nz]"), "9")                                                      /* BNE across a page */ \
    HL_BR(B, 80, HL_T_EQ("0xff", "%[nz]"), "9")                                                      /* BEQ across a page */ \
    HL_ZPR(B, 81, HL_ORA("v123"))                                                                    /* $05 */ \
    HL_ZPM(B, 82, HL_ASL("v123"))                                                                    /* $06 */ \
    HL_IMM(B, 83, HL_ORA("s86"))                                                                     /* $09 */ \
    HL_IMP(B, 84, HL_ASL("%[a]"))                                                                    /* $0A */ \
    HL_BR(B, 85, HL_T_EQ("0x180", "%[nz]"), "8")                                                     /* $10 */ \
    HL_IMP(B, 86, "v_mov_b32 %[c], 0\n")                                                             /* $18 */ \
    HL_ZPR(B, 87, HL_BIT)                                                                            /* $24 */ \
    HL_ZPR(B, 88, HL_AND("v123"))                                                                    /* $25 */ \
    HL_ZPM(B, 89, HL_ROL("v123"))                                                                    /* $26 */ \
    HL_IMM(B, 90, HL_AND("s86"))                                                                     /* $29 */ \
    HL_IMP(B, 91, HL_ROL("%[a]"))                                                                    /* $2A */ \
    HL_BR(B, 92, HL_T_NE("0x180", "%[nz]"), "8")                                                     /* $30 */ \
    HL_IMP(B, 93, "v_mov_b32 %[c], 1\n")                                                             /* $38 */ \
    HL_ZPR(B, 94, HL_EOR("v123"))                                                                    /* $45 */ \
    HL_ZPM(B, 95, HL_LSR("v123"))                                                                    /* $46 */ \
    HL_IMM(B, 96, HL_EOR("s86"))                                                                     /* $49 */ \
    HL_IMP(B, 97, HL_LSR("%[a]"))                                                                    /* $4A */ \
    HL_JMP(B, 98)                                                                                    /* $4C */ \
    HL_BR(B, 99, HL_T_EQ("0x80", "%[v]"), "8")                                                       /* $50 */ \
    HL_ZPRD(B, 100, ".Ldadc", HL_ADC("v123"))                                                        /* $65 */ \
    HL_ZPM(B, 101, HL_ROR("v123"))                                                                   /* $66 */ \
    HL_IMMD(B, 102, HL_ADCI)                                                                         /* $69 */ \
    HL_IMP(B, 103, HL_ROR("%[a]"))                                                                   /* $6A */ \
    HL_BR(B, 104, HL_T_NE("0x80", "%[v]"), "8")                                                      /* $70 */ \
    HL_ZPS(B, 105, "%[y]")                                                                           /* $84 */ \
    HL_ZPS(B, 106, "%[a]")                                                                           /* $85 */ \
    HL_ZPS(B, 107, "%[x]")                                                                           /* $86 */ \
    HL_IMP(B, 108, HL_DEC("%[y]"))                                                                   /* $88 */ \
    HL_IMP(B, 109, "v_mov_b32 %[a], %[x]\n" HL_NZ("%[x]"))                                           /* $8A */ \
    HL_BR(B, 110, "v_cmp_eq_u32 vcc, 0, %[c]\n", "8")                                                /* $90 */ \
    HL_IMP(B, 111, "v_mov_b32 %[a], %[y]\n" HL_NZ("%[y]"))                                           /* $98 */ \
    HL_IMM(B, 112, HL_LDI("%[y]"))                                                                   /* $A0 */ \
    HL_IMM(B, 113, HL_LDI("%[x]"))                                                                   /* $A2 */ \
    HL_ZPL(B, 114, "%[y]")                                                                           /* $A4 */ \
    HL_ZPL(B, 115, "%[a]")                                                                           /* $A5 */ \
    HL_ZPL(B, 116, "%[x]")                                                                           /* $A6 */ \
    HL_IMP(B, 117, "v_mov_b32 %[y], %[a]\n" HL_NZ("%[a]"))                                           /* $A8 */ \
    HL_IMM(B, 118, HL_LDI("%[a]"))                                                                   /* $A9 */ \
    HL_IMP(B, 119, "v_mov_b32 %[x], %[a]\n" HL_NZ("%[a]"))                                           /* $AA */ \
    HL_BR(B, 120, "v_cmp_ne_u32 vcc, 0, %[c]\n", "8")                                                /* $B0 */ \
    HL_IMP(B, 121, "v_mov_b32 %[v], 0\n")                                                            /* $B8 */ \
    HL_IMM(B, 122, HL_CMP_S("%[y]"))                                                                 /* $C0 */ \
    HL_ZPR(B, 123, HL_CMP("%[y]", "v123"))                                                           /* $C4 */ \
    HL_ZPR(B, 124, HL_CMP("%[a]", "v123"))                                                           /* $C5 */ \
    HL_ZPM(B, 125, HL_DEC("v123"))                                                                   /* $C6 */ \
    HL_IMP(B, 126, HL_INC("%[y]"))                                                                   /* $C8 */ \
    HL_IMM(B, 127, HL_CMP_S("%[a]"))                                                                 /* $C9 */ \
    HL_IMP(B, 128, HL_DEC("%[x]"))                                                                   /* $CA */ \
    HL_BR(B, 129, HL_T_NE("0xff", "%[nz]"), "8")                                                     /* $D0 */ \
    HL_IMP(B, 130, "s_andn2_b64 s[50:51], s[50:51], exec\n")                                         /* $D8 */ \
    HL_IMM(B, 131, HL_CMP_S("%[x]"))                                                                 /* $E0 */ \
    HL_ZPR(B, 132, HL_CMP("%[x]", "v123"))                                                           /* $E4 */ \
    HL_ZPRD(B, 133, ".Ldsbc", "v_xor_b32 v123, 0xff, v123\n" HL_ADC("v123"))                         /* $E5 */ \
    HL_ZPM(B, 134, HL_INC("v123"))                                                                   /* $E6 */ \
    HL_IMP(B, 135, HL_INC("%[x]"))                                                                   /* $E8 */ \
    HL_IMMD(B, 136, HL_SBCI)                                                                         /* $E9 */ \
    HL_IMP(B, 137, "")                                                                               /* $EA */ \
    HL_BR(B, 138, HL_T_EQ("0xff", "%[nz]"), "8")                                                     /* $F0 */ \
    HL_IMP(B, 139, "s_or_b64 s[50:51], s[50:51], exec\n")                                            /* $F8 */ \
    HL_PHA(B, 140)                                                                                   /* $48 */ \
    HL_PLA(B, 141)                                                                                   /* $68 */ \
    HL_IMP(B, 142, "v_mov_b32 %[x], %[sp]\n" HL_NZ("%[sp]"))                                         /* $BA */ \
    HL_IMP(B, 143, "v_mov_b32 %[sp], %[x]\n")                                                        /* $9A */ \
    HL_RTS(B, 144)                                                                                   /* $60 */ \
    HL_JSR(B, 147)                                                                                   /* $20 */ \
    RES(B, 149, 5)                                                                                   /* RESP0, RESP1 */ \
    RES(B, 150, 4)                                                                                   /* RESM0, RESM1, RESBL */ \
    FXY(B)                                                                                           /* STX, STY to ENAM0 .. VDELBL */ \
    HL_3F(B, 163, "%[a]")                                                                            /* STA selecting a 3F slice */ \
    HL_3F(B, 164, "%[x]")                                                                            /* STX selecting one */ \
    HL_3F(B, 165, "%[y]")                                                                            /* STY selecting one */ \
    HL_E0(B, 166)                                                                                    /* LDA from an E0 hotspot */ \
    HL_HS_ST(B, 168)                                                                                 /* store to a bank hotspot */ \
    HL_ZIN(B, 169, HL_CONST)                                                                         /* a constant TIA read, zero page */ \
    HL_ZIN(B, 170, "v_mov_b32 v123, %[inpt4]\n")                                                     /* INPT4 */ \
    HL_AIN(B, 171, HL_CONST)                                                                         /* a constant read, absolute */ \
    HL_AIN(B, 172, "v_mov_b32 v123, %[swcha]\n")                                                     /* SWCHA */ \
    HL_INTIM(B, 173)                                                                                 /* INTIM */ \
    HL_AROM(B, 175)                                                                                  /* the cartridge, absolute */ \
    HL_ARAM(B, 177)                                                                                  /* RAM, absolute */ \
    HL_RIDX(B, 178, HL_ZIDX("%[x]"), 2, "s78", 4)                                                    /* zero page, X */ \
    HL_RIDX(B, 179, HL_ZIDX("%[y]"), 2, "s78", 4)                                                    /* zero page, Y */ \
    HL_RIDX(B, 180, HL_ZIDX("%[x]"), 2, "s78", 6)                                                    /* read-modify-write of it */ \
    HL_AXROM(B, 181, "%[x]")                                                                         /* the cartridge, absolute, X */ \
    HL_AXROM(B, 183, "%[y]")                                                                         /* the cartridge, absolute, Y */ \
    HL_RIDX(B, 185, HL_AIDX("%[x]"), 3, "s79", 4)                                                    /* RAM, absolute, X */ \
    HL_RIDX(B, 186, HL_AIDX("%[y]"), 3, "s79", 4)                                                    /* RAM, absolute, Y */ \
    HL_IYROM(B, 187)                                                                                 /* the cartridge through a pointer, Y */ \
    HL_RIDX(B, 189, HL_B1_7 HL_RAMADDR, 3, "s79", 6)                                                 /* read-modify-write of RAM, absolute */ \
    HL_SEG(B, 190, "0")                                                                              /* an E0 or 3F cartridge, absolute */ \
    HL_SEG(B, 191, "%[x]")                                                                           /* absolute, X */ \
    HL_SEG(B, 192, "%[y]")                                                                           /* absolute, Y */ \
    HL_SIDX(B, 193, HL_ZIDX("%[x]"), "%[a]", 2, "s78", 4)                                            /* $95 */ \
    HL_SIDX(B, 194, HL_ZIDX("%[x]"), "%[y]", 2, "s78", 4)                                            /* $94 */ \
    HL_SIDX(B, 195, HL_ZIDX("%[y]"), "%[x]", 2, "s78", 4)                                            /* $96 */ \
    HL_SIDX(B, 196, HL_AIDX("%[x]"), "%[a]", 3, "s79", 5)                                            /* $9D */ \
    HL_SIDX(B, 197, HL_AIDX("%[y]"), "%[a]", 3, "s79", 5)                                            /* $99 */ \
    HL_ASTO(B, 198, "%[a]")                                                                          /* $8D to RAM */ \
    HL_ASTO(B, 199, "%[x]")                                                                          /* $8E */ \
    HL_ASTO(B, 200, "%[y]")                                                                          /* $8C */ \
    ATIA(B)                                                                                          /* absolute stores to TIA registers */ \
    HL_PHP(B, 210)                                                                                   /* $08 */ \
    HL_PLP(B, 212)                                                                                   /* $28 */ \
    HL_HMM(B, 214, 41)                                                                               /* STA HMM0 */ \
    HL_HMM(B, 215, 42)                                                                               /* STA HMM1 */ \
    HL_HMM(B, 216, 43)                                                                               /* STA HMBL */ \
    HL_HMCLR(B, 217)                                                                                 /* HMCLR */ \
    HL_WORK(B, 218, HL_LDV)                                                                          /* LDA */ \
    HL_WORK(B, 219, "v_mov_b32 %[x], v123\n" HL_NZ("v123"))                                          /* LDX */ \
    HL_WORK(B, 220, "v_mov_b32 %[y], v123\n" HL_NZ("v123"))                                          /* LDY */ \
    HL_WORK(B, 221, HL_AND("v123"))                                                                  /* AND */ \
    HL_WORK(B, 222, HL_ORA("v123"))                                                                  /* ORA */ \
    HL_WORK(B, 223, HL_EOR("v123"))                                                                  /* EOR */ \
    HL_WORK(B, 224, HL_CMP("%[a]", "v123"))                                                          /* CMP */ \
    HL_WORK(B, 225, HL_CMP("%[x]", "v123"))                                                          /* CPX */ \
    HL_WORK(B, 226, HL_CMP("%[y]", "v123"))                                                          /* CPY */ \
    HL_WORK(B, 227, HL_BIT)                                                                          /* BIT */ \
    HL_WORK(B, 228, HL_ADCV)                                                                         /* ADC */ \
    HL_WORK(B, 229, HL_SBCV)                                                                         /* SBC */ \
    HL_WORK(B, 230, HL_ASL("v123") "ds_write_b8 v122, v123\n")                                       /* ASL */ \
    HL_WORK(B, 231, HL_ROL("v123") "ds_write_b8 v122, v123\n")                                       /* ROL */ \
    HL_WORK(B, 232, HL_LSR("v123") "ds_write_b8 v122, v123\n")                                       /* LSR */ \
    HL_WORK(B, 233, HL_ROR("v123") "ds_write_b8 v122, v123\n")                                       /* ROR */ \
    HL_WORK(B, 234, HL_DEC("v123") "ds_write_b8 v122, v123\n")                                       /* DEC */ \
    HL_WORK(B, 235, HL_INC("v123") "ds_write_b8 v122, v123\n")                                       /* INC */

// Fold the current group's instruction count into its lanes' counts and the
// wave's passes (exec: the group).
#define HL_FOLD(extra)                                     \
    "s_and_b32 s86, s73, 0x1ffffff\n"                      \
    "s_and_b32 s73, s73, 0xfe000000\n" extra               \
    "s_add_u32 s57, s57, s86\n"                            \
    "v_add_u32 %[ic], s86, %[ic]\n"
// The group's place in time: its lines left less the frame's first line (more
// is earlier; lanes of one wave may be in different frames)
#define HL_TIME                                            \
    "s_bfe_i32 s86, s59, 0x1b0000\n"                       \
    "s_sub_u32 s86, s80, s86\n"
#define HL_LINES                                           \
    "s_bfe_i32 s86, s59, 0x1b0000\n"                       \
    "s_add_u32 s80, s80, s86\n"
// Put the current group, its count folded, into a free lane of the table.
#define HL_PUT HL_TIME                                     \
    "s_ff0_i32_b64 s93, s[54:55]\n"                        \
    "s_bitset1_b64 s[54:55], s93\n"                        \
    "s_mov_b32 m0, s93\n"                                  \
    "s_nop 0\n"                                            \
    "v_writelane_b32 v102, s52, m0\n"                      \
    "v_writelane_b32 v103, s53, m0\n"                      \
    "v_writelane_b32 v104, s72, m0\n"                      \
    "v_writelane_b32 v105, s73, m0\n"                      \
    "v_writelane_b32 v106, s86, m0\n"                      \
    "v_writelane_b32 v107, s82, m0\n"                      \
    "v_writelane_b32 v108, s59, m0\n"
// Lanes whose fields equal the current group's: vcc
#define HL_SAME(po, acc, lines, of, orow, key)                 \
    "v_xor_b32 v122, s72, " po "\n"                        \
    "v_xor_b32 v123, s73, " acc "\n"                       \
    "v_xor_b32 v124, " lines ", " of "\n"                     \
    "v_or3_b32 v122, v122, v123, v124\n"                   \
    "v_xor_b32 v123, s82, " orow "\n"                      \
    "v_xor_b32 v124, s59, " key "\n"                       \
    "v_or3_b32 v122, v122, v123, v124\n"                   \
    "v_cmp_eq_u32 vcc, 0, v122\n"
#define HL_TOLANES                                         \
    "v_mov_b32 %[po], s72\n"                               \
    "v_mov_b32 %[acc], s73\n"                              \
    "v_mov_b32 %[lines], s80\n"                            \
    "v_mov_b32 %[orow], s82\n"

// Where a lane stands, as the block keeps it.
struct HotLane {
    uint32_t po;         // byte offset of its instruction's word in the ROM's table (virtual bank and
                         // pc), or kHotNone: the block does not run it
    uint32_t acc;        // ACC, count 0
    uint32_t lines;      // lines until the frame's cap
    uint32_t orow;       // open row + 1 (0 = none)
    uint32_t key;        // pc bits 12-15 << 28 | frame logged << 27 | frame line (27 bits)
    uint64_t lp;         // where the next entry goes (not part of the place)
    uint32_t obase;      // the open row's first entry, in dwords from the log's start (nor this)
};
// The lane's timer: cycles of the base line's start after the one that the last
// write is visible at, its value and log2 interval.
struct HotTimer {
    uint32_t tm, tv, tshift;
};
// The cartridge: its LDS copy's address or -1; linear schemes: the bank offsets
// that are plain ROM; E0: span 0; 3F: span 1, first the fixed half's ROM offset.
struct HotRom {
    uint32_t lds, first, span;
};
constexpr uint32_t kHotNone = 0xFFFFFFFFu;
constexpr uint32_t kHotLogged = 1u << 27;

// Runs the wave's lanes in `lanes` until a group of them meets an instruction
// the block does not run; returns that group (0: the block cannot run where it
// was loaded, nothing done).  Call it with every lane of the
// wave in exec.  table: the ROM's predecoded words; rom: the cartridge in HBM
// (linear schemes); ram, tia: LDS addresses of the lane's RAM and TIA
// registers; log, xram: its row log and Superchip RAM; ic: instructions run
// (added to); passes, rounds: of the wave (added to).
//
// Groups.  Lanes that stand at one place (HotLane fields po to key equal) run as
// one group: exec is the group, its place is in scalars.  The other groups wait
// in a table, one group per lane of v102-v108 (its lanes, then its place), bit k
// of s[54:55] for table lane k.  A branch whose lanes part puts the lanes that
// do not take it into the table and goes on with the others; a group that
// reaches a WSYNC while others wait joins the waiting group at the same place,
// or waits itself, and the group at the earliest line runs next -- so
// groups that part in a scanline meet again at the next line's start.  All of
// it stays in registers: a switch costs about 40 instructions, where leaving
// the block and forming a group from per-lane state took some 2,000 cycles.
__device__ __forceinline__ uint64_t hot_wave(uint64_t lanes, uint64_t table, uint64_t rom, HotLane& H, uint32_t& a,
                                             uint32_t& x, uint32_t& y, uint32_t& p, uint32_t& nz, uint32_t& c,
                                             uint32_t& v, uint32_t& hmp0, uint32_t& hmp1, uint32_t& vsync,
                                             uint32_t inpt4, uint32_t swcha, uint32_t& ic, uint32_t& passes, uint32_t& rounds,
                                             uint32_t ram, uint32_t tia, uint64_t log, uint64_t xram, uint32_t& sp,
                                             const HotTimer& T, const HotRom& R) {
    static_assert(kSnapArea == 1696 * 4 && kCountMask == 31 && kFrameEntries == 5280 && kRows == 210 &&
                      kFirstRow == 34 && kSnapBytes == 32,
                  "the block's constants");
    static_assert(R_GRP0 == 10 && R_GRP1 == 11 && R_GRP0_OLD == 16 && R_GRP1_OLD == 17 && R_FLAGS == 23 &&
                      R_ENAM0 == 32 && R_ENABL == 34 && R_ENABL_OLD == 35 && R_VDELBL == 38,
                  "the block's register offsets");
    static_assert(kHotWork == 218 && R_HMM0 == 41 && HW_INC == kHotWorks - 1 && (HW_NONE | 3 << 5) < 128 && kHotSlots * 128 < 0x8000,
                  "the block's slots");
    asm volatile(
        // --- entry: block bases, line-change and row addresses, constants
        "s_mov_b64 s[44:45], exec\n"
        "s_mov_b32 s43, m0\n"
        "s_mov_b64 exec, -1\n"
        "s_mov_b64 s[54:55], 0\n"
        "s_getpc_b64 s[74:75]\n"
        ".Lpc%=:\n"
        "v_and_b32 v122, 8, %[p]\n"
        "v_cmp_ne_u32 s[50:51], 0, v122\n"         // lanes in decimal mode
        // (the blocks must lie in one 4 GB half: a handler's address is a 32-bit sum)
        "s_add_u32 s88, s74, .Lhu%=-.Lpc%=+0x8000\n"
        "s_cbranch_scc1 .Lnone%=\n"
        "s_add_u32 s46, s74, .Lhb%=-.Lpc%=\n"
        "s_add_u32 s47, s74, .Lhu%=-.Lpc%=\n"
        "s_add_u32 s85, s74, .Lline%=-.Lpc%=\n"
        "s_add_u32 s64, s74, .Lsnap%=-.Lpc%=\n"
        "s_mov_b32 s65, s75\n"
        "s_mov_b32 s91, s75\n"
        "s_mov_b32 s67, 0\n"
        "s_movk_i32 s68, 1696\n"
        "s_movk_i32 s69, 1696+5280-31\n"
        "s_mov_b32 s98, (3<<25)+1\n"
        "s_mov_b32 s99, (4<<25)+1\n"
        "s_mov_b32 s56, 0x7fffffff\n"             // no group picked yet
        // --- groups of the lanes in s[48:49]
        ".Lform%=:\n"
        "s_ff1_i32_b64 s93, s[48:49]\n"
        "s_nop 3\n"
        "v_readlane_b32 s72, %[po], s93\n"
        "v_readlane_b32 s73, %[acc], s93\n"
        "v_readlane_b32 s80, %[lines], s93\n"
        "v_readlane_b32 s82, %[orow], s93\n"
        "v_readlane_b32 s59, %[key], s93\n"
        HL_SAME("%[po]", "%[acc]", "s80", "%[lines]", "%[orow]", "%[key]")
        "s_and_b64 s[52:53], vcc, s[48:49]\n"
        "s_andn2_b64 s[48:49], s[48:49], s[52:53]\n"
        "s_cbranch_scc1 .Lforw%=\n"
        "s_cmp_lg_u64 s[54:55], 0\n"
        "s_cbranch_scc0 .Lrun%=\n"                 // one group, none waiting
        ".Lforw%=:\n"
        HL_PUT
        "s_cmp_lg_u64 s[48:49], 0\n"
        "s_cbranch_scc1 .Lform%=\n"
        // --- the next group: the earliest (s56: the last one's time)
        ".Lpick%=:\n"
        "v_cmp_eq_u32 vcc, s56, v106\n"
        "s_and_b64 s[60:61], vcc, s[54:55]\n"
        "s_cbranch_scc1 .Lgot%=\n"
        "s_sub_u32 s56, s56, 1\n"                 // (none waits at s56, so none before s56 - 1)
        "v_cmp_eq_u32 vcc, s56, v106\n"
        "s_and_b64 s[60:61], vcc, s[54:55]\n"
        "s_cbranch_scc1 .Lgot%=\n"
        "s_mov_b64 s[88:89], s[54:55]\n"
        "s_mov_b32 s56, 0x80000000\n"
        ".Lscan%=:\n"
        "s_ff1_i32_b64 s93, s[88:89]\n"
        "s_bitset0_b64 s[88:89], s93\n"
        "s_nop 3\n"
        "v_readlane_b32 s86, v106, s93\n"
        "s_max_i32 s56, s56, s86\n"
        "s_cmp_lg_u64 s[88:89], 0\n"
        "s_cbranch_scc1 .Lscan%=\n"
        "s_branch .Lpick%=\n"
        ".Lgot%=:\n"
        "s_ff1_i32_b64 s93, s[60:61]\n"
        "s_bitset0_b64 s[54:55], s93\n"
        "s_nop 3\n"
        "v_readlane_b32 s72, v104, s93\n"
        "v_readlane_b32 s52, v102, s93\n"
        "v_readlane_b32 s53, v103, s93\n"
        "v_readlane_b32 s73, v105, s93\n"
        "v_readlane_b32 s80, v106, s93\n"
        "v_readlane_b32 s82, v107, s93\n"
        "v_readlane_b32 s59, v108, s93\n"
        HL_LINES
        ".Lrun%=:\n"
        "s_add_u32 s58, s58, 1\n"
        "s_mov_b64 exec, s[52:53]\n"
        "s_cmp_eq_u32 s72, -1\n"                   // not run here
        "s_cbranch_scc1 .Lout%=\n"
        "s_load_dwordx4 s[76:79], s[70:71], s72\n"
        "s_cmp_eq_u32 s80, 0\n"                    // at the cap
        "s_cbranch_scc1 .Lout%=\n"
        "s_cmp_lg_u64 s[54:55], 0\n"               // stop at the next WSYNC while others wait
        "s_cselect_b32 s81, -1, 0\n"
        "s_bitcmp1_b32 s59, 27\n"
        "s_cselect_b32 s84, s46, s47\n"
        // s83: lines left in the open row's line; -2 (no line's) when none is open
        "s_sub_u32 s83, 287, s82\n"
        "s_cmp_eq_u32 s82, 0\n"
        "s_cselect_b32 s83, -2, s83\n"
        HL_WAIT HL_TGT("s76") HL_JUMP
        // --- lanes part at a branch (vcc: taken): the others wait
        ".Lpart8_%=:\n"
        "s_mov_b32 s94, 3<<25\n"
        "s_branch .Lpart%=\n"
        ".Lpart9_%=:\n"
        "s_mov_b32 s94, 4<<25\n"
        ".Lpart%=:\n"
        HL_WAIT
        HL_FOLD("s_add_u32 s86, s86, 1\n")
        "s_mov_b32 s95, s73\n"
        "s_mov_b32 s66, s80\n"
        "s_andn2_b64 s[52:53], exec, vcc\n"
        "s_mov_b32 s72, s88\n"
        "s_add_u32 s73, s95, 2<<25\n"
        "s_cbranch_scc0 .Lpn%=\n"
        "s_add_u32 s73, s73, 52<<25\n"             // into the next line
        "s_sub_u32 s80, s80, 1\n"
        ".Lpn%=:\n"
        HL_PUT
        "s_mov_b64 s[52:53], vcc\n"
        "s_mov_b64 exec, vcc\n"
        "s_mov_b32 s72, s89\n"
        "s_mov_b32 s80, s66\n"
        "s_mov_b32 s81, -1\n"
        "s_add_u32 s73, s95, s94\n"
        "s_cbranch_scc0 .Lpt%=\n"
        "s_add_u32 s73, s73, 52<<25\n"
        "s_sub_u32 s80, s80, 1\n"
        "s_cmp_eq_u32 s80, 0\n"
        "s_cbranch_scc1 .Lout%=\n"
        ".Lpt%=:\n"
        "s_add_u32 s58, s58, 1\n"
        "s_mov_b64 s[76:77], s[60:61]\n"
        "s_mov_b64 s[78:79], s[62:63]\n" HL_TGT("s76") HL_JUMP
        // --- a WSYNC that is not simply the next line (s80 counted down, not yet ACC)
        ".Lsync%=:\n"
        HL_WAIT
        "s_add_u32 s87, s73, 2<<25\n"
        "s_cbranch_scc1 .Lstall%=\n"
        "s_and_b32 s73, s73, 0x1ffffff\n"
        "s_add_u32 s73, s73, (52<<25)+1\n"
        "s_cmp_eq_u32 s80, 0\n"
        "s_cbranch_scc1 .Lout%=\n"                 // the cap
        // others wait: join the one at this place, or wait too
        HL_FOLD("")
        "s_mov_b64 exec, -1\n"
        HL_TIME HL_SAME("v104", "v105", "s86", "v106", "v107", "v108")
        "s_and_b64 s[60:61], vcc, s[54:55]\n"
        "s_cbranch_scc1 .Ljoin%=\n"
        HL_PUT
        "s_branch .Lpick%=\n"
        ".Ljoin%=:\n"
        "s_ff1_i32_b64 s93, s[60:61]\n"
        "s_nop 3\n"
        "v_readlane_b32 s86, v102, s93\n"
        "v_readlane_b32 s87, v103, s93\n"
        "s_mov_b32 m0, s93\n"
        "s_or_b32 s86, s86, s52\n"
        "s_or_b32 s87, s87, s53\n"
        "v_writelane_b32 v102, s86, m0\n"
        "v_writelane_b32 v103, s87, m0\n"
        "s_branch .Lpick%=\n"
        ".Lstall%=:\n"                             // a write at the line's end stalls a line longer
        "s_add_u32 s80, s80, 1\n"
        "s_sub_u32 s72, s72, 8\n"
        "s_branch .Lout%=\n"
        // --- leaving: every group's place back to its lanes
        ".Lnone%=:\n"
        "s_mov_b64 s[48:49], 0\n"
        "s_branch .Lend%=\n"
        ".Lundo%=:\n"                              // a 2-byte, 3-cycle store was fetched past and counted: take it back
        "s_sub_u32 s73, s73, (3<<25)+1\n"
        "s_sub_u32 s72, s72, 8\n"
        ".Lout%=:\n"
        HL_WAIT
        HL_FOLD("")
        HL_TOLANES
        "s_mov_b64 s[48:49], s[52:53]\n"
        ".Lflush%=:\n"
        "s_cmp_eq_u64 s[54:55], 0\n"
        "s_cbranch_scc1 .Lend%=\n"
        "s_ff1_i32_b64 s93, s[54:55]\n"
        "s_bitset0_b64 s[54:55], s93\n"
        "s_nop 3\n"
        "v_readlane_b32 s52, v102, s93\n"
        "v_readlane_b32 s53, v103, s93\n"
        "v_readlane_b32 s72, v104, s93\n"
        "v_readlane_b32 s73, v105, s93\n"
        "v_readlane_b32 s80, v106, s93\n"
        "v_readlane_b32 s82, v107, s93\n"
        "v_readlane_b32 s59, v108, s93\n"
        "s_mov_b64 exec, s[52:53]\n"
        HL_LINES
        HL_TOLANES
        "s_branch .Lflush%=\n"
        // --- line change without a WSYNC: ACC's cycle has wrapped past the bias
        ".Lline%=:\n"
        "s_add_u32 s73, s73, 52<<25\n"
        "s_sub_u32 s80, s80, 1\n"
        "s_cmp_eq_u32 s80, 0\n"
        "s_cbranch_scc1 .Lout%=\n"
        HL_WAIT HL_TGT("s76") HL_JUMP
        // --- a logged TIA store at cycle s88 - 52 of its line, which is not the open row's
        // (s88 < 52: past the line's end): snapshots of the rows before it, and its own
        // when it lands in the visible part.  SCC = 0 on return: its entry goes into the open row.
        ".Lsnap%=:\n"
        "s_cmp_lt_u32 s88, 52\n"
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
        "v_sub_u32 v111, v100, %[log0]\n"        // entries so far: the open row's count, the new row's first
        "v_lshrrev_b32 v111, 2, v111\n"
        "v_lshl_add_u64 v[120:121], s[66:67], 0, %[log]\n"   // (its shift goes to 4)
        "v_sub_u32 v123, v111, %[obase]\n"
        "v_mov_b32 %[obase], v111\n"
        "v_subrev_u32 v111, s68, v111\n"
        "s_cmp_eq_u32 s82, 0\n"
        "s_cbranch_scc1 .Lcnt%=\n"
        "global_store_byte v[120:121], v123, off offset:-17\n"
        ".Lcnt%=:\n"
        HL_WAIT
        "v_and_b32 v115, 0xffffff, v115\n"
        "v_and_b32 v119, 0xffff0000, v119\n"
        "v_or_b32 v119, v111, v119\n"
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
        "v_cmp_lt_u32 vcc, s69, %[obase]\n"        // a row's entries might not fit
        "s_sub_u32 s95, s89, 1\n"                  // not in the visible part of a frame row: no entry
        "s_cmp_ge_u32 s95, 210\n"
        "s_cselect_b32 s95, 1, s94\n"
        "s_mul_i32 s87, s88, 3\n"
        "s_cbranch_vccnz .Lundo%=\n"
        "s_cmp_lg_u32 s95, 0\n"
        "s_setpc_b64 s[96:97]\n"
        // --- an indexed cartridge read without an LDS copy
        ".Lhbm%=:\n"
        "global_load_ubyte v123, v122, s[40:41]\n" HL_ROM_GO("s79", 3)
        "s_waitcnt vmcnt(0)\n" HL_DO
        ".Lhbmy%=:\n"
        "global_load_ubyte v123, v122, s[40:41]\n" HL_ROM_GO("s78", 2)
        "s_waitcnt vmcnt(0)\n" HL_DO
        // --- an E0 (s42: 0) or 3F cartridge read at the word's address + v125: in the
        // segment of 1 KB (below E0's hotspots in the last) or half of 2 KB it begins in
        ".Lseg%=:\n"
        "s_bfe_u32 s86, s76, 0x80010\n"
        "s_bfe_u32 s89, s76, 0xc0010\n"
        "s_lshr_b32 s87, s72, 14\n"
        "s_cmp_lg_u32 s42, 0\n"
        "s_cbranch_scc1 .Lhalf%=\n"
        "s_lshr_b32 s88, s89, 10\n"
        "s_mul_i32 s60, s88, 3\n"
        "s_lshr_b32 s87, s87, s60\n"
        "s_and_b32 s87, s87, 7\n"
        "s_movk_i32 s61, 0x400\n"
        "s_cmp_eq_u32 s88, 3\n"
        "s_cselect_b32 s87, 7, s87\n"
        "s_cselect_b32 s61, 0x3e0, s61\n"
        "s_lshl_b32 s87, s87, 10\n"
        "s_and_b32 s89, s89, 0x3ff\n"
        "s_branch .Lsegc%=\n"
        ".Lhalf%=:\n"
        "s_lshl_b32 s87, s87, 11\n"
        "s_bitcmp1_b32 s89, 11\n"
        "s_cselect_b32 s87, s92, s87\n"
        "s_and_b32 s89, s89, 0x7ff\n"
        "s_movk_i32 s61, 0x800\n"
        ".Lsegc%=:\n"
        "v_add_u32 v122, s89, v125\n"
        "v_add_u32 v124, s86, v125\n"
        "v_cmp_le_u32 s[96:97], s61, v122\n" HL_CROSS(4)
        HL_ROMBYTE(".Lhbm") HL_ROM_GO("s79", 3) HL_WAIT HL_DO
        // --- a 3F slice (v122), if the same in every lane
        ".Lslice%=:\n"
        "s_nop 0\n"
        "v_readfirstlane_b32 s87, v122\n"
        "s_lshl_b32 s88, s87, 14\n"
        "s_nop 1\n"
        "v_cmp_ne_u32 vcc, s87, v122\n"
        "s_cbranch_vccnz .Lout%=\n"
        "s_add_u32 s72, s72, 8\n"
        "s_and_b32 s72, s72, 0x3fff\n"
        "s_or_b32 s72, s72, s88\n"
        "s_load_dwordx4 s[76:79], s[70:71], s72\n" HL_WAIT HL_TGT("s76") HL_GO(3)
        // --- ADC of groups with lanes in decimal mode (do_adc): operand in v123, or s86.
        // v124: the binary sum, v116 its low byte, v120 its overflow
        ".Ldadci%=:\n"
        "v_mov_b32 v123, s86\n"
        ".Ldadc%=:\n" HL_WAIT
        "v_add3_u32 v124, %[a], v123, %[c]\n"
        "v_bitop3_b32 v120, %[a], v123, v124 bitop3:0x42\n"
        "v_and_b32 v116, 0xff, v124\n"
        "v_and_b32 v122, 15, %[a]\n"
        "v_and_b32 v125, 15, v123\n"
        "v_add3_u32 v122, v122, v125, %[c]\n"     // the low digits
        "v_cmp_lt_u32 vcc, 9, v122\n"
        "v_add_u32 v125, 6, v122\n"
        "v_and_b32 v125, 15, v125\n"
        "v_or_b32 v125, 16, v125\n"
        "v_cndmask_b32 v122, v122, v125, vcc\n"
        "v_and_b32 v125, 0xf0, %[a]\n"
        "v_and_b32 v126, 0xf0, v123\n"
        "v_bfe_i32 v118, v125, 0, 8\n"
        "v_bfe_i32 v119, v126, 0, 8\n"
        "v_add3_u32 v119, v118, v119, v122\n"     // the signed sum: N, V
        "v_add3_u32 v125, v125, v126, v122\n"
        "v_cmp_lt_u32 vcc, 0x9f, v125\n"
        "v_add_u32 v126, 0x60, v125\n"
        "v_add_u32 v117, 0x80, v119\n"
        "v_cndmask_b32 v125, v125, v126, vcc\n"
        "v_lshrrev_b32 v118, 8, v125\n"
        "v_min_u32 v118, 1, v118\n"
        "v_and_b32 v117, 0xffffff00, v117\n"
        "v_min_u32 v117, 0x80, v117\n"
        "v_min_u32 v115, 1, v116\n"               // Z by the binary sum
        "v_and_b32 v119, 0x80, v119\n"
        "v_lshl_or_b32 v115, v119, 1, v115\n"
        "v_and_b32 v125, 0xff, v125\n"
        "v_lshrrev_b32 v124, 8, v124\n"
        "v_cndmask_b32 %[a], v116, v125, s[50:51]\n"
        "v_cndmask_b32 %[c], v124, v118, s[50:51]\n"
        "v_cndmask_b32 %[v], v120, v117, s[50:51]\n"
        "v_cndmask_b32 %[nz], v116, v115, s[50:51]\n" HL_JUMP
        // --- SBC of such groups (do_sbc): all flags by the binary difference
        ".Ldsbci%=:\n"
        "v_mov_b32 v123, s86\n"
        ".Ldsbc%=:\n" HL_WAIT
        "v_xor_b32 v126, 0xff, v123\n"
        "v_add3_u32 v124, %[a], v126, %[c]\n"
        "v_bitop3_b32 %[v], %[a], v126, v124 bitop3:0x42\n"
        "v_and_b32 v122, 15, %[a]\n"
        "v_and_b32 v125, 15, v123\n"
        "v_sub_u32 v122, v122, v125\n"
        "v_add3_u32 v122, v122, %[c], -1\n"
        "v_cmp_gt_i32 vcc, 0, v122\n"
        "v_add_u32 v125, -6, v122\n"
        "v_and_b32 v125, 15, v125\n"
        "v_add_u32 v125, -16, v125\n"
        "v_cndmask_b32 v122, v122, v125, vcc\n"
        "v_and_b32 v125, 0xf0, %[a]\n"
        "v_and_b32 v117, 0xf0, v123\n"
        "v_sub_u32 v125, v125, v117\n"
        "v_add_u32 v125, v125, v122\n"
        "v_cmp_gt_i32 vcc, 0, v125\n"
        "v_add_u32 v117, 0xffffffa0, v125\n"
        "v_and_b32 %[nz], 0xff, v124\n"
        "v_cndmask_b32 v125, v125, v117, vcc\n"
        "v_and_b32 v125, 0xff, v125\n"
        "v_lshrrev_b32 %[c], 8, v124\n"
        "v_cndmask_b32 %[a], %[nz], v125, s[50:51]\n" HL_JUMP
        // --- handlers
        ".p2align 7\n"
        ".Lhb%=:\n"
        HL_BLOCK(".Lhb", HL_TIA_LOG, HL_TIAX_LOG, HL_GRP0_LOG, HL_GRP1_LOG, HL_XY_LOG, HL_FLAG_LOG, HL_RES_LOG, HL_FXY_LOG,
                 HL_ATIA_LOG)
        ".p2align 7\n"
        ".Lhu%=:\n"
        HL_BLOCK(".Lhu", HL_TIA_NOLOG, HL_TIAX_NOLOG, HL_GRP0_NOLOG, HL_GRP1_NOLOG, HL_XY_NOLOG, HL_FLAG_NOLOG, HL_RES_NOLOG,
                 HL_FXY_NOLOG, HL_ATIA_NOLOG)
        ".Lend%=:\n"
        "s_mov_b64 exec, s[44:45]\n"
        "s_mov_b32 m0, s43\n"
        "v_mov_b32 v122, 8\n"
        "v_and_b32 %[p], ~8, %[p]\n"
        "v_cndmask_b32 v122, 0, v122, s[50:51]\n"
        "v_or_b32 %[p], %[p], v122\n"
        : "+{s[48:49]}"(lanes), "+{s57}"(passes), "+{s58}"(rounds), [po] "+v"(H.po), [acc] "+v"(H.acc),
          [lines] "+v"(H.lines), [orow] "+v"(H.orow), "+{v[100:101]}"(H.lp), [obase] "+v"(H.obase), [a] "+v"(a),
          [x] "+v"(x), [y] "+v"(y), [p] "+v"(p), [nz] "+v"(nz), [c] "+v"(c), [v] "+v"(v), [hmp0] "+v"(hmp0),
          [hmp1] "+v"(hmp1), [vsync] "+v"(vsync), [ic] "+v"(ic), [sp] "+v"(sp)
        : "{s[70:71]}"(table), "{s[40:41]}"(rom), "{s39}"(R.lds), "{s42}"(R.span), "{s92}"(R.first),
          [tm] "v"(T.tm), [tv] "v"(T.tv), [tsh] "v"(T.tshift), [key] "v"(H.key), [inpt4] "v"(inpt4), [swcha] "v"(swcha), [ram] "v"(ram), [tia] "v"(tia), [log] "v"(log),
          [log0] "v"((uint32_t)log), [xram] "v"(xram)
        : "memory", "scc", "vcc", "s43", "s44", "s45", "s46", "s47", "s50", "s51", "s52", "s53", "s54", "s55", "s56",
          "s59", "s60", "s61", "s62", "s63", "s64", "s65", "s66", "s67", "s68", "s69", "s72", "s73", "s74", "s75",
          "s76", "s77", "s78", "s79", "s80", "s81", "s82", "s83", "s84", "s85", "s86", "s87", "s88", "s89", "s90", "s91", "s93",
          "s94", "s95", "s96", "s97", "s98", "s99", "v102", "v103", "v104", "v105", "v106", "v107", "v108", "v111", "v112",
          "v113", "v114", "v115", "v116", "v117", "v118", "v119", "v120", "v121", "v122", "v123", "v124", "v125",
          "v126");
    return lanes;
}

}  // namespace vcs
