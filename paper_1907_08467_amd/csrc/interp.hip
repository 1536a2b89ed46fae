// 6507 interpreter kernel: one lane per env, one wave per ROM-homogeneous tile.
//
// What it computes (paper, Section 3): the "Atari CPU kernel" -- each env's
// CPU runs the cartridge code, updates its 128 B of RAM and the CPU state, and
// passes every TIA register write on to the renderer instead of drawing.
// Here the TIA writes go into a row log (vcs_device.h) only for the frames
// that will be rendered (all frames, or the last two of the step).
//
// Machine conventions (the paper gives none; the public 6502/TIA/RIOT
// definitions plus these readings):
//  * bus: a = addr & $1FFF; a & $1000 cartridge, else a & $80 == 0 TIA,
//    else a & $200 == 0 RAM[a & $7F], else RIOT;
//  * an instruction that starts at cycle t and lasts n cycles performs all its
//    data accesses at cycle t+n-1; opcode/operand fetches happen at t and have
//    no side effects; RMW writes once; no dummy reads;
//  * a TIA write at cycle c takes effect at colour clock 3(c+1); WSYNC written
//    at c resumes the CPU at 76*(c/76+1); a frame ends after the instruction
//    that turns VSYNC bit 1 on; 320 scanlines without that end the frame
//    (FRAME_CAP), as does an undocumented opcode (ILLEGAL);
//  * RIOT timer in closed form: after TIMnT <- v written at cycle w, a read at
//    t sees e = t-w-1: INTIM = v - e/n while e < (v+1)n, then
//    ($FF - (e - (v+1)n)) & $FF with TIMINT bit 7 set;
//  * decimal ADC/SBC follow the NMOS behaviour described by B. Clark
//    ("Decimal Mode", 6502.org, Appendix A).
//
// Dispatch: the running lanes at one place (bank, pc, cycle, frame line) form a
// group, which the hot loop (hotloop.h) runs as threaded code with its control
// state in scalars, one group after the other in order of emulated time; groups
// part at data-dependent branches and meet again there.  An instruction the hot
// loop does not cover goes through the full scalar dispatch (run_cold), which
// goes on to the next one that the loop covers.  What that refuses --
// undocumented opcodes, indirect jumps and stores, latch reads, timer writes,
// HMOVE, lanes that disagree about a bank, code outside the cartridge window --
// goes through the per-lane path: the wave executes one opcode at a time for all
// lanes that share it (readfirstlane + compare), so the opcode's decode word is
// a scalar and the addressing-mode and operation switches of the one generic
// executor are scalar branches; TIA writes are queued during the pass and
// applied in one shared block afterwards.
#include "tia_draw.h"
#include "hotloop.h"

namespace vcs {

enum Mn : int {
    ADC, AND, ASL, BCC, BCS, BEQ, BIT, BMI, BNE, BPL, BRK, BVC, BVS, CLC, CLD, CLI, CLV, CMP,
    CPX, CPY, DEC, DEX, DEY, EOR, INC, INX, INY, JMP, JSR, LDA, LDX, LDY, LSR, NOP, ORA, PHA,
    PHP, PLA, PLP, ROL, ROR, RTI, RTS, SBC, SEC, SED, SEI, STA, STX, STY, TAX, TAY, TSX, TXA,
    TXS, TYA,
    SLO, RLA, SRE, RRA, SAX, LAX, DCP, ISC, ANC, ALR, ARR, SBX, LAS,   // undocumented, stable
    ILL
};
enum Md : int { IMP, ACC, IMM, ZP, ZPX, ZPY, ABS, ABX, ABY, IZX, IZY, IND, REL };

struct OpInfo {
    int mn, md, cyc;
    bool pen;   // +1 cycle on an indexed page cross
};

// Decode of the documented opcodes from their aaabbbcc structure.
constexpr OpInfo decode_doc(int op) {
    const int a = op >> 5, b = (op >> 2) & 7, cc = op & 3;
    OpInfo ill{ILL, IMP, 2, false};
    if (cc == 1) {
        const int mns[8] = {ORA, AND, EOR, ADC, STA, LDA, CMP, SBC};
        const int mds[8] = {IZX, ZP, IMM, ABS, IZY, ZPX, ABY, ABX};
        const int rd_cyc[8] = {6, 3, 2, 4, 5, 4, 4, 4};
        const int st_cyc[8] = {6, 3, 0, 4, 6, 4, 5, 5};
        if (mns[a] == STA) {
            if (b == 2) return ill;
            return OpInfo{STA, mds[b], st_cyc[b], false};
        }
        return OpInfo{mns[a], mds[b], rd_cyc[b], b == 4 || b == 6 || b == 7};
    }
    if (cc == 2) {
        const int mns[8] = {ASL, ROL, LSR, ROR, STX, LDX, DEC, INC};
        const int mn = mns[a];
        const bool rmw = (a < 4) || (a >= 6);
        switch (b) {
        case 0: return a == 5 ? OpInfo{LDX, IMM, 2, false} : ill;
        case 1: return OpInfo{mn, ZP, rmw ? 5 : 3, false};
        case 2:
            if (a < 4) return OpInfo{mn, ACC, 2, false};
            if (a == 4) return OpInfo{TXA, IMP, 2, false};
            if (a == 5) return OpInfo{TAX, IMP, 2, false};
            if (a == 6) return OpInfo{DEX, IMP, 2, false};
            return OpInfo{NOP, IMP, 2, false};
        case 3: return OpInfo{mn, ABS, rmw ? 6 : 4, false};
        case 5: return OpInfo{mn, (a == 4 || a == 5) ? ZPY : ZPX, rmw ? 6 : 4, false};
        case 6:
            if (a == 4) return OpInfo{TXS, IMP, 2, false};
            if (a == 5) return OpInfo{TSX, IMP, 2, false};
            return ill;
        case 7:
            if (a == 4) return ill;
            if (a == 5) return OpInfo{LDX, ABY, 4, true};
            return OpInfo{mn, ABX, 7, false};
        default: return ill;
        }
    }
    if (cc == 0) {
        if (b == 4) {
            const int br[8] = {BPL, BMI, BVC, BVS, BCC, BCS, BNE, BEQ};
            return OpInfo{br[a], REL, 2, false};
        }
        if (b == 6) {
            const int fl[8] = {CLC, SEC, CLI, SEI, TYA, CLV, CLD, SED};
            return OpInfo{fl[a], IMP, 2, false};
        }
        if (b == 2) {
            const int st[8] = {PHP, PLP, PHA, PLA, DEY, TAY, INY, INX};
            const int cy[8] = {3, 4, 3, 4, 2, 2, 2, 2};
            return OpInfo{st[a], IMP, cy[a], false};
        }
        if (b == 0) {
            switch (a) {
            case 0: return OpInfo{BRK, IMP, 7, false};
            case 1: return OpInfo{JSR, ABS, 6, false};
            case 2: return OpInfo{RTI, IMP, 6, false};
            case 3: return OpInfo{RTS, IMP, 6, false};
            case 5: return OpInfo{LDY, IMM, 2, false};
            case 6: return OpInfo{CPY, IMM, 2, false};
            case 7: return OpInfo{CPX, IMM, 2, false};
            default: return ill;
            }
        }
        const int mns[8] = {ILL, BIT, JMP, JMP, STY, LDY, CPY, CPX};
        if (b == 1) return (a == 1 || a >= 4) ? OpInfo{mns[a], ZP, 3, false} : ill;
        if (b == 3) {
            if (a == 0) return ill;
            if (a == 2) return OpInfo{JMP, ABS, 3, false};
            if (a == 3) return OpInfo{JMP, IND, 5, false};
            return OpInfo{mns[a], ABS, 4, false};
        }
        if (b == 5) return (a == 4 || a == 5) ? OpInfo{mns[a], ZPX, 4, false} : ill;
        if (b == 7) return a == 5 ? OpInfo{LDY, ABX, 4, true} : ill;
        return ill;
    }
    return ill;
}

// Decode of every opcode: the documented ones, then the stable undocumented
// ones (NMOS unintended-opcode matrix); JAMs and the unstable ANE, LXA, SHA,
// SHX, SHY, TAS stay ILL.
constexpr OpInfo decode(int op) {
    const OpInfo d = decode_doc(op);
    if (d.mn != ILL) return d;
    const int a = op >> 5, b = (op >> 2) & 7, cc = op & 3;
    OpInfo ill{ILL, IMP, 2, false};
    if (cc == 3) {
        const int combo[8] = {SLO, RLA, SRE, RRA, SAX, LAX, DCP, ISC};
        const int mn = combo[a];
        if (b == 2) {                               // immediate column
            const int imm[8] = {ANC, ANC, ALR, ARR, ILL, ILL, SBX, SBC};
            return imm[a] == ILL ? ill : OpInfo{imm[a], IMM, 2, false};
        }
        if (mn == SAX) {
            switch (b) {
            case 0: return OpInfo{SAX, IZX, 6, false};
            case 1: return OpInfo{SAX, ZP, 3, false};
            case 3: return OpInfo{SAX, ABS, 4, false};
            case 5: return OpInfo{SAX, ZPY, 4, false};
            default: return ill;                    // SHA, TAS, SHA: unstable
            }
        }
        if (mn == LAX) {
            switch (b) {
            case 0: return OpInfo{LAX, IZX, 6, false};
            case 1: return OpInfo{LAX, ZP, 3, false};
            case 3: return OpInfo{LAX, ABS, 4, false};
            case 4: return OpInfo{LAX, IZY, 5, true};
            case 5: return OpInfo{LAX, ZPY, 4, false};
            case 6: return OpInfo{LAS, ABY, 4, true};
            default: return OpInfo{LAX, ABY, 4, true};
            }
        }
        const int mds[8] = {IZX, ZP, IMM, ABS, IZY, ZPX, ABY, ABX};
        const int cyc[8] = {8, 5, 2, 6, 8, 6, 7, 7};
        return OpInfo{mn, mds[b], cyc[b], false};
    }
    // NOPs of every width; the rest of the undocumented cc = 0, 1, 2 opcodes
    // are JAMs or unstable
    if (b == 0 && (op == 0x80 || op == 0x82 || op == 0xC2 || op == 0xE2)) return OpInfo{NOP, IMM, 2, false};
    if (op == 0x89) return OpInfo{NOP, IMM, 2, false};
    if (cc == 0 && b == 1 && (a == 0 || a == 2 || a == 3)) return OpInfo{NOP, ZP, 3, false};
    if (op == 0x0C) return OpInfo{NOP, ABS, 4, false};
    if (cc == 0 && b == 5 && a != 4 && a != 5) return OpInfo{NOP, ZPX, 4, false};
    if (cc == 0 && b == 7 && a != 4 && a != 5) return OpInfo{NOP, ABX, 4, true};
    if (cc == 2 && b == 6 && a != 4 && a != 5) return OpInfo{NOP, IMP, 2, false};
    return ill;
}

constexpr bool combo_mn(int mn) {
    return mn == SLO || mn == RLA || mn == SRE || mn == RRA || mn == DCP || mn == ISC;
}

constexpr int op_len(int md) {
    return (md == IMP || md == ACC) ? 1 : (md == ABS || md == ABX || md == ABY || md == IND) ? 3 : 2;
}

// status flags
constexpr uint32_t FC = 0x01, FZ = 0x02, FI = 0x04, FD = 0x08, FB = 0x10, FU = 0x20, FV = 0x40, FN = 0x80;
// per-instruction events
constexpr uint32_t EV_WSYNC = 1, EV_VSYNC = 2;

// Joystick of the 18 actions (ALE order): actions 2..9 and 10..17 are the
// directions UP, RIGHT, LEFT, DOWN, UPRIGHT, UPLEFT, DOWNRIGHT, DOWNLEFT;
// their pressed bits in SWCHA's high nibble (D7 right, D6 left, D5 down,
// D4 up) are packed one byte per direction; 1 and 10..17 hold fire.
constexpr uint64_t kDirBits = 0x60A0509020408010ull;
__device__ __forceinline__ uint32_t joy_pressed(uint32_t a) {
    const uint32_t dir = a >= 10 ? a - 8 : a;
    return dir >= 2 ? (uint32_t)(kDirBits >> (8 * (dir - 2))) & 0xF0u : 0u;
}
__device__ __forceinline__ bool fire_pressed(uint32_t a) { return a == 1 || a >= 10; }

// Predecoded words, read through the scalar cache: they never change while a
// kernel runs (the constant address space says so; the compiler could not
// tell past the hot loop's assembly).
typedef const __attribute__((address_space(4))) uint32_t* PreWords;

struct Wave {                 // per-workgroup (uniform) data
    const uint8_t* rom;       // the tile's cartridge: its LDS copy, or its HBM slot
    uint8_t* ram;             // LDS, kRamStride bytes per lane
    uint8_t* tia;             // LDS, kTiaStride bytes per lane
    uint32_t ram_lds, tia_lds;   // their LDS addresses
    PreWords pre;             // the tile ROM's predecoded words
    CartMap cm;               // its cartridge mapping
    uint32_t track;           // collision latches tracked
};

__device__ __forceinline__ uint32_t cm_kind(const Wave& W) { return W.cm.a & 3; }
__device__ __forceinline__ uint32_t cm_sc(const Wave& W) { return (W.cm.a >> 2) & 1; }
__device__ __forceinline__ uint32_t cm_tf_mask(const Wave& W) { return W.cm.b >> 16; }
__device__ __forceinline__ uint32_t rom_off(const Wave& W, uint32_t bank, uint32_t a) {
    return cart_rom_off(W.cm.a & 3, W.cm.b & 0xFFFF, bank, a);
}
__device__ __forceinline__ uint32_t hotspot(const Wave& W, uint32_t bank, uint32_t a) {
    return cart_hotspot(W.cm.a & 3, W.cm.a >> 8, (W.cm.a >> 4) & 15, bank, a);
}
constexpr int kRamStride = 132;   // 33 dwords: bank-conflict free for equal offsets
constexpr int kTiaStride = 52;    // 13 dwords (R[0..47] + 1): bank-conflict free

struct Cpu {
    uint32_t a, x, y, sp, p, pc, bank;
    uint64_t base;            // absolute cycle of the start of the lane's base line
    uint32_t cyc;             // cycles since `base`
    int32_t fl;               // scanline of the frame's start write, relative to the base line
    uint32_t cap;             // an instruction starting at or after this cycle ends the frame
    uint32_t swcha, inpt4;
    uint32_t vsync, hmp0, hmp1;
    int64_t tbase;            // absolute
    uint32_t tv, tshift;
    uint32_t ev, err;
    uint32_t ac;              // access cycle of the current instruction
    uint32_t tqr0, tqr1, tqr2;     // queued TIA writes: register (scalar when the address is)
    uint32_t tqv0, tqv1, tqv2;     //   and value
    uint32_t tqm;                  //   and the mask of used slots
    uint32_t ram_off, tia_off;
    uint8_t* log;             // current frame's row log, or nullptr
    uint8_t* xram;            // the env's Superchip RAM (in its DevEnv)
    uint32_t slot, slots;     // its slot; slots completed so far
    int32_t open_row;
    uint32_t open_cnt;        // entries logged in the open row
    uint32_t open_base;       // stream index of the open row's first entry
    uint32_t icount;
    uint32_t ucount;          // instructions executed in wave-uniform mode
    int32_t hmb_line;         // line (relative to the base line) an early HMOVE blanked, or -1
    uint32_t cx;              // collision latches (bit 2r+1 / 2r = D7 / D6 of CX register r)
    int32_t cx_row, cx_x;     // the frame's pixels before (row, x) are in cx
    int32_t cx_need;          // >= 0: a latch read needs the pixels through this clock scanned first
    int32_t ptr_memo;         // >= 0: the (zp,X) address / (zp),Y base of the instruction being run
                              // again, fixed by the run that had scanned through its fetch cycle
    uint32_t log_scratch;     // the row log is the collision scratch copy, not a rendered frame
};

__device__ __forceinline__ uint32_t nz(uint32_t p, uint32_t v) {
    return (p & ~(FN | FZ)) | (v & FN) | (v == 0 ? FZ : 0);
}

// Position of colour clock `clk` (relative to the base line) in the frame's
// rows: (row, first pixel after it)
__device__ __forceinline__ bool cx_scanned(const Cpu& c, int32_t clk) {
    const int32_t line = clk / 228, h = clk % 228;
    const int32_t row = line - c.fl - kFirstRow;
    if (row < 0) return true;
    if (row >= kRows) return c.cx_row >= kRows;
    const int32_t x = h >= 68 ? h - 68 + 1 : 0;
    return c.cx_row > row || (c.cx_row == row && c.cx_x >= x);
}

// TIA data read of address a by an access that sees the beam through clock
// `through`.  A latch read (tracked) whose pixels are not all scanned yet
// records that need and reads 0; the per-lane dispatch then scans the row
// log and runs the instruction again.
__device__ __forceinline__ uint32_t tia_read(Cpu& c, const Wave& W, uint32_t a, int32_t through) {
    const uint32_t r = a & 0x0F;
    if (W.track && r < 8) {
        if (!cx_scanned(c, through)) c.cx_need = through;
        return ((c.cx >> (2 * r)) & 3) << 6;
    }
    return r == 0x0C ? c.inpt4 : (r == 0x0D ? 0x80u : 0u);      // untracked latches read 0 here too
}
// The same for an instruction fetch (kernel loop), whose caller has scanned
// the latches through the fetch cycle's pixels first.
__device__ __forceinline__ uint32_t tia_peek(const Cpu& c, const Wave& W, uint32_t a) {
    const uint32_t r = a & 0x0F;
    if (W.track && r < 8) return ((c.cx >> (2 * r)) & 3) << 6;
    return r == 0x0C ? c.inpt4 : (r == 0x0D ? 0x80u : 0u);
}

__device__ __forceinline__ uint32_t riot_read(const Cpu& c, const Wave& W, uint32_t a, uint32_t t) {
    if (!(a & 4)) {
        const uint32_t r = a & 3;
        return r == 0 ? c.swcha : (r == 2 ? 0x0Bu : 0u);
    }
    const int64_t e = (int64_t)(c.base + t) - c.tbase;
    const int64_t lim = (int64_t)(c.tv + 1) << c.tshift;
    // both outcomes computed and masked: no per-lane branch
    const uint32_t m = 0u - (uint32_t)(e >= lim);
    if (a & 1) return m & 0x80u;
    const uint32_t after = (uint32_t)(0xFF - (e - lim)) & 0xFF;
    const uint32_t before = (uint32_t)(c.tv - (uint32_t)(e >> c.tshift)) & 0xFF;
    return (after & m) | (before & ~m);
}

// Superchip RAM window: cartridge offsets $000-$0FF (write port below $080)
__device__ __forceinline__ bool sc_window(const Wave& W, uint32_t a) { return cm_sc(W) && !(a & 0xF00); }

// data read at cycle t (side effects: bank hotspots)
__device__ __forceinline__ uint32_t rd(Cpu& c, const Wave& W, uint32_t addr, uint32_t t) {
    const uint32_t a = addr & 0x1FFF;
    if (a & 0x1000) {
        c.bank = hotspot(W, c.bank, a);
        if (sc_window(W, a)) return (a & 0x80) ? (uint32_t)c.xram[a & 0x7F] : 0u;   // the write port reads 0
        return W.rom[rom_off(W, c.bank, a)];
    }
    if (!(a & 0x80)) return tia_read(c, W, a, 3 * (int32_t)t + 2);   // the access cycle's own pixels too
    if (!(a & 0x200)) return W.ram[c.ram_off + (a & 0x7F)];
    return riot_read(c, W, a, t);
}

// instruction fetch at cycle t, without side effects; the cartridge area
// shows ROM even in the Superchip RAM window
__device__ __forceinline__ uint32_t peek(const Cpu& c, const Wave& W, uint32_t addr, uint32_t t) {
    const uint32_t a = addr & 0x1FFF;
    if (a & 0x1000) return W.rom[rom_off(W, c.bank, a)];
    if (!(a & 0x80)) return tia_peek(c, W, a);
    if (!(a & 0x200)) return W.ram[c.ram_off + (a & 0x7F)];
    return riot_read(c, W, a, t);
}

// zero-page pointer byte, fetched with the instruction at its first cycle:
// RAM, or a TIA read register (a latch read sees the pixels through
// `through`, like a data read)
__device__ __forceinline__ uint32_t zp_fetch(Cpu& c, const Wave& W, uint32_t z, int32_t through) {
    return (z & 0x80) ? (uint32_t)W.ram[c.ram_off + (z & 0x7F)] : tia_read(c, W, z, through);
}

// data write at cycle t; TIA writes are queued in slot K of the instruction
template <int K>
__device__ __forceinline__ void wr(Cpu& c, const Wave& W, uint32_t addr, uint32_t v, uint32_t t) {
    const uint32_t a = addr & 0x1FFF;
    if (a & 0x1000) {
        c.bank = hotspot(W, c.bank, a);
        if (sc_window(W, a) && !(a & 0x80)) c.xram[a & 0x7F] = (uint8_t)v;   // writes to the read port do nothing
    } else if (!(a & 0x80)) {
        if (cm_kind(W) == CART_3F && a <= 0x3F) c.bank = v & cm_tf_mask(W);   // 3F: selects the lower slice
        if (K == 0) { c.tqr0 = a & 0x3F; c.tqv0 = v & 0xFF; }
        if (K == 1) { c.tqr1 = a & 0x3F; c.tqv1 = v & 0xFF; }
        if (K == 2) { c.tqr2 = a & 0x3F; c.tqv2 = v & 0xFF; }
        c.tqm |= 1u << K;
    } else if (!(a & 0x200)) {
        W.ram[c.ram_off + (a & 0x7F)] = (uint8_t)v;
    } else if ((a & 0x14) == 0x14) {     // TIM1T / TIM8T / TIM64T / T1024T
        c.tv = v & 0xFF;
        c.tshift = (0x0A060300u >> (8 * (a & 3))) & 0xFF;   // intervals 1, 8, 64, 1024
        c.tbase = (int64_t)(c.base + t) + 1;
    }
}

template <int K>
__device__ __forceinline__ void push(Cpu& c, const Wave& W, uint32_t v, uint32_t t) {
    wr<K>(c, W, 0x100 | c.sp, v, t);
    c.sp = (c.sp - 1) & 0xFF;
}
__device__ __forceinline__ uint32_t pull(Cpu& c, const Wave& W, uint32_t t) {
    c.sp = (c.sp + 1) & 0xFF;
    return rd(c, W, 0x100 | c.sp, t);
}

__device__ __forceinline__ int32_t sext8(uint32_t v) { return (int32_t)(int8_t)(uint8_t)v; }

__device__ __forceinline__ void do_adc(Cpu& c, uint32_t v) {
    const uint32_t cin = c.p & FC;
    const uint32_t bin = c.a + v + cin;
    if (!(c.p & FD)) {
        const uint32_t ovf = (c.a ^ bin) & (v ^ bin) & 0x80;
        c.p = (c.p & ~(FC | FV)) | (bin > 0xFF ? FC : 0) | (ovf ? FV : 0);
        c.a = bin & 0xFF;
        c.p = nz(c.p, c.a);
        return;
    }
    int32_t lo = (int32_t)((c.a & 0x0F) + (v & 0x0F) + cin);
    if (lo > 9) lo = ((lo + 6) & 0x0F) + 0x10;
    int32_t s = (int32_t)(c.a & 0xF0) + (int32_t)(v & 0xF0) + lo;
    const int32_t ss = sext8(c.a & 0xF0) + sext8(v & 0xF0) + lo;
    if (s >= 0xA0) s += 0x60;
    c.p &= ~(FC | FV | FN | FZ);
    c.p |= (s >= 0x100 ? FC : 0) | ((ss < -128 || ss > 127) ? FV : 0) | (ss & 0x80 ? FN : 0) |
           ((bin & 0xFF) == 0 ? FZ : 0);
    c.a = (uint32_t)s & 0xFF;
}

__device__ __forceinline__ void do_sbc(Cpu& c, uint32_t v) {
    const uint32_t cin = c.p & FC;
    const uint32_t inv = (~v) & 0xFF;
    const uint32_t bin = c.a + inv + cin;
    const uint32_t ovf = (c.a ^ bin) & (inv ^ bin) & 0x80;
    uint32_t res = bin & 0xFF;
    if (c.p & FD) {
        int32_t lo = (int32_t)(c.a & 0x0F) - (int32_t)(v & 0x0F) + (int32_t)cin - 1;
        if (lo < 0) lo = ((lo - 6) & 0x0F) - 0x10;
        int32_t s = (int32_t)(c.a & 0xF0) - (int32_t)(v & 0xF0) + lo;
        if (s < 0) s -= 0x60;
        res = (uint32_t)s & 0xFF;
    }
    c.p = (c.p & ~(FC | FV)) | (bin > 0xFF ? FC : 0) | (ovf ? FV : 0);
    c.p = nz(c.p, bin & 0xFF);
    c.a = res;
}

__device__ __forceinline__ void do_cmp(Cpu& c, uint32_t r, uint32_t v) {
    c.p = (c.p & ~FC) | (r >= v ? FC : 0);
    c.p = nz(c.p, (r - v) & 0xFF);
}

// ARR: (A AND operand) rotated right through C.  Binary: N, Z of the result,
// C = bit 6, V = bit 6 ^ bit 5.  Decimal (NMOS): N = the old C, Z and V from
// the rotate (V: bit 6 changed), then BCD fix-ups of each nibble decided on
// the unrotated value, the high one also giving C.
__device__ __forceinline__ void do_arr(Cpu& c, uint32_t v) {
    const uint32_t t = c.a & v;
    const uint32_t cin = c.p & FC;
    uint32_t r = (t >> 1) | (cin << 7);
    if (!(c.p & FD)) {
        c.p = nz(c.p & ~(FC | FV), r) | ((r >> 6) & 1) | ((((r >> 6) ^ (r >> 5)) & 1) ? FV : 0);
        c.a = r;
        return;
    }
    uint32_t p = c.p & ~(FN | FZ | FV | FC);
    p |= (cin ? FN : 0) | (r == 0 ? FZ : 0) | (((t ^ r) & 0x40) ? FV : 0);
    if ((t & 0x0F) + (t & 0x01) > 5) r = (r & 0xF0) | ((r + 6) & 0x0F);
    if ((t & 0xF0) + (t & 0x10) > 0x50) {
        r = (r + 0x60) & 0xFF;
        p |= FC;
    }
    c.p = p;
    c.a = r;
}

// Decode word of an opcode: mode | mnemonic << 4 | base cycles << 11 |
// page penalty << 15 | length << 16 | reads operand << 18 | writes to ea << 19.
constexpr uint32_t DW_CYC = 11, DW_PEN = 15, DW_LEN = 16, DW_RD = 18, DW_WR = 19;
constexpr uint32_t encode(int op) {
    const OpInfo I = decode(op);
    const bool rmw = I.mn == ASL || I.mn == LSR || I.mn == ROL || I.mn == ROR || I.mn == INC || I.mn == DEC ||
                     combo_mn(I.mn);
    const bool mem = I.md != IMP && I.md != ACC && I.md != REL && I.md != IMM;
    const bool reads = (I.mn == LDA || I.mn == LDX || I.mn == LDY || I.mn == ADC || I.mn == SBC || I.mn == AND ||
                        I.mn == ORA || I.mn == EOR || I.mn == CMP || I.mn == CPX || I.mn == CPY || I.mn == BIT ||
                        I.mn == LAX || I.mn == LAS || I.mn == NOP || rmw) && mem;
    const bool writes = (I.mn == STA || I.mn == STX || I.mn == STY || I.mn == SAX || rmw) && mem;
    return (uint32_t)I.md | ((uint32_t)I.mn << 4) | ((uint32_t)I.cyc << DW_CYC) | ((uint32_t)I.pen << DW_PEN) |
           ((uint32_t)op_len(I.md) << DW_LEN) | ((uint32_t)reads << DW_RD) | ((uint32_t)writes << DW_WR);
}
struct DecodeTable {
    uint32_t w[256];
    constexpr DecodeTable() : w() {
        for (int i = 0; i < 256; ++i) w[i] = encode(i);
    }
};
__constant__ DecodeTable kDecode = DecodeTable();

// Execute one instruction with decode word `d` (wave-uniform) for the lanes
// that fetched it.  Sets c.ac, c.pc, c.cyc (before a WSYNC stall) and queues
// TIA writes.
__device__ __forceinline__ void exec_generic(uint32_t d, Cpu& c, const Wave& W, uint32_t b1, uint32_t b2) {
    const uint32_t md = d & 15, mn = (d >> 4) & 127;
    uint32_t n = (d >> DW_CYC) & 15;
    if (mn == ILL) {
        c.err |= ERR_ILLEGAL;
        return;
    }
    uint32_t ea = 0;
    switch (md) {
    case ZP: ea = b1; break;
    case ZPX: ea = (b1 + c.x) & 0xFF; break;
    case ZPY: ea = (b1 + c.y) & 0xFF; break;
    case ABS: case IND: ea = b1 | (b2 << 8); break;
    case ABX: case ABY: {
        const uint32_t base = b1 | (b2 << 8);
        ea = (base + (md == ABX ? c.x : c.y)) & 0xFFFF;
        if ((d >> DW_PEN) & 1) n += ((base ^ ea) & 0xFF00) ? 1 : 0;
        break;
    }
    case IZX: {
        if (c.ptr_memo >= 0) {
            ea = (uint32_t)c.ptr_memo;
        } else {
            const uint32_t z = (b1 + c.x) & 0xFF;
            const int32_t th = 3 * (int32_t)c.cyc + 2;
            ea = zp_fetch(c, W, z, th) | (zp_fetch(c, W, (z + 1) & 0xFF, th) << 8);
            if (W.track && c.cx_need < 0) c.ptr_memo = (int32_t)ea;   // its latches are final
        }
        break;
    }
    case IZY: {
        uint32_t base;
        if (c.ptr_memo >= 0) {
            base = (uint32_t)c.ptr_memo;
        } else {
            const int32_t th = 3 * (int32_t)c.cyc + 2;
            base = zp_fetch(c, W, b1, th) | (zp_fetch(c, W, (b1 + 1) & 0xFF, th) << 8);
            if (W.track && c.cx_need < 0) c.ptr_memo = (int32_t)base;
        }
        ea = (base + c.y) & 0xFFFF;
        if ((d >> DW_PEN) & 1) n += ((base ^ ea) & 0xFF00) ? 1 : 0;
        break;
    }
    default: break;
    }
    // a pointer taken from latches not scanned yet names no address: stop
    // before any access (the caller scans the log and runs it again).  A
    // pointer that was read keeps its value for the runs that follow (a data
    // access later in the instruction may need the scan carried further,
    // past the pixels the pointer fetch saw).
    if (W.track && c.cx_need >= 0) return;
    const uint32_t next = (c.pc + ((d >> DW_LEN) & 3)) & 0xFFFF;
    uint32_t npc = next;
    if (md == REL) {
        bool taken;
        switch (mn) {
        case BPL: taken = !(c.p & FN); break;
        case BMI: taken = (c.p & FN) != 0; break;
        case BVC: taken = !(c.p & FV); break;
        case BVS: taken = (c.p & FV) != 0; break;
        case BCC: taken = !(c.p & FC); break;
        case BCS: taken = (c.p & FC) != 0; break;
        case BNE: taken = !(c.p & FZ); break;
        default: taken = (c.p & FZ) != 0; break;
        }
        if (taken) {
            const uint32_t tgt = (next + (uint32_t)sext8(b1)) & 0xFFFF;
            n += 1 + (((tgt ^ next) & 0xFF00) ? 1 : 0);
            npc = tgt;
        }
    }
    const uint32_t t = c.cyc + n - 1;     // access cycle
    c.ac = t;
    uint32_t v = b1;                      // operand (immediate, or read below)
    if ((d >> DW_RD) & 1) v = rd(c, W, ea, t);
    uint32_t res = 0;                     // value written to ea when (d >> 17) & 1
    switch (mn) {
    case LDA: c.a = v; c.p = nz(c.p, v); break;
    case LDX: c.x = v; c.p = nz(c.p, v); break;
    case LDY: c.y = v; c.p = nz(c.p, v); break;
    case STA: res = c.a; break;
    case STX: res = c.x; break;
    case STY: res = c.y; break;
    case ADC: do_adc(c, v); break;
    case SBC: do_sbc(c, v); break;
    case AND: c.a &= v; c.p = nz(c.p, c.a); break;
    case ORA: c.a |= v; c.p = nz(c.p, c.a); break;
    case EOR: c.a ^= v; c.p = nz(c.p, c.a); break;
    case CMP: do_cmp(c, c.a, v); break;
    case CPX: do_cmp(c, c.x, v); break;
    case CPY: do_cmp(c, c.y, v); break;
    case BIT: c.p = (c.p & ~(FN | FV | FZ)) | (v & (FN | FV)) | ((c.a & v) == 0 ? FZ : 0); break;
    case ASL: case LSR: case ROL: case ROR: case INC: case DEC: {
        const uint32_t x = md == ACC ? c.a : v;
        const uint32_t ci = c.p & FC;
        uint32_t r, co = ci;
        if (mn == ASL) { r = (x << 1) & 0xFF; co = x >> 7; }
        else if (mn == LSR) { r = x >> 1; co = x & 1; }
        else if (mn == ROL) { r = ((x << 1) | ci) & 0xFF; co = x >> 7; }
        else if (mn == ROR) { r = (x >> 1) | (ci << 7); co = x & 1; }
        else if (mn == INC) { r = (x + 1) & 0xFF; }
        else { r = (x - 1) & 0xFF; }
        c.p = nz((c.p & ~FC) | co, r);
        if (md == ACC) c.a = r;
        res = r;
        break;
    }
    case SLO: case RLA: case SRE: case RRA: case DCP: case ISC: {
        // the shift / rotate / count half; the ALU half follows the write
        const uint32_t ci = c.p & FC;
        uint32_t r, co = ci;
        if (mn == SLO) { r = (v << 1) & 0xFF; co = v >> 7; }
        else if (mn == RLA) { r = ((v << 1) | ci) & 0xFF; co = v >> 7; }
        else if (mn == SRE) { r = v >> 1; co = v & 1; }
        else if (mn == RRA) { r = (v >> 1) | (ci << 7); co = v & 1; }
        else if (mn == DCP) { r = (v - 1) & 0xFF; }
        else { r = (v + 1) & 0xFF; }
        c.p = (c.p & ~FC) | co;
        res = r;
        break;
    }
    case SAX: res = c.a & c.x; break;
    case LAX: c.a = c.x = v; c.p = nz(c.p, v); break;
    case LAS: c.sp &= v; c.a = c.x = c.sp; c.p = nz(c.p, c.a); break;
    case ANC: c.a &= v; c.p = nz(c.p, c.a); c.p = (c.p & ~FC) | (c.a >> 7); break;
    case ALR: c.a &= v; c.p = (c.p & ~FC) | (c.a & 1); c.a >>= 1; c.p = nz(c.p, c.a); break;
    case SBX: {
        const uint32_t t0 = c.a & c.x;
        c.p = (c.p & ~FC) | (t0 >= v ? FC : 0);
        c.x = (t0 - v) & 0xFF;
        c.p = nz(c.p, c.x);
        break;
    }
    case ARR: do_arr(c, v); break;
    case INX: c.x = (c.x + 1) & 0xFF; c.p = nz(c.p, c.x); break;
    case INY: c.y = (c.y + 1) & 0xFF; c.p = nz(c.p, c.y); break;
    case DEX: c.x = (c.x - 1) & 0xFF; c.p = nz(c.p, c.x); break;
    case DEY: c.y = (c.y - 1) & 0xFF; c.p = nz(c.p, c.y); break;
    case TAX: c.x = c.a; c.p = nz(c.p, c.x); break;
    case TAY: c.y = c.a; c.p = nz(c.p, c.y); break;
    case TXA: c.a = c.x; c.p = nz(c.p, c.a); break;
    case TYA: c.a = c.y; c.p = nz(c.p, c.a); break;
    case TSX: c.x = c.sp; c.p = nz(c.p, c.x); break;
    case TXS: c.sp = c.x; break;
    case CLC: c.p &= ~FC; break;
    case SEC: c.p |= FC; break;
    case CLI: c.p &= ~FI; break;
    case SEI: c.p |= FI; break;
    case CLV: c.p &= ~FV; break;
    case CLD: c.p &= ~FD; break;
    case SED: c.p |= FD; break;
    case PHA: push<0>(c, W, c.a, t); break;
    case PHP: push<0>(c, W, c.p | FB | FU, t); break;
    case PLA: c.a = pull(c, W, t); c.p = nz(c.p, c.a); break;
    case PLP: c.p = (pull(c, W, t) & ~FB) | FU; break;
    case JMP:
        if (md == ABS) {
            npc = ea;
        } else {                          // the pointer's high byte stays in its page
            const uint32_t lo = rd(c, W, ea, t);
            const uint32_t hi = rd(c, W, (ea & 0xFF00) | ((ea + 1) & 0xFF), t);
            npc = lo | (hi << 8);
        }
        break;
    case JSR: {
        const uint32_t ret = (next - 1) & 0xFFFF;
        push<0>(c, W, ret >> 8, t);
        push<1>(c, W, ret & 0xFF, t);
        npc = ea;
        break;
    }
    case RTS: {
        const uint32_t lo = pull(c, W, t);
        const uint32_t hi = pull(c, W, t);
        npc = ((lo | (hi << 8)) + 1) & 0xFFFF;
        break;
    }
    case RTI: {
        c.p = (pull(c, W, t) & ~FB) | FU;
        const uint32_t lo = pull(c, W, t);
        const uint32_t hi = pull(c, W, t);
        npc = lo | (hi << 8);
        break;
    }
    case BRK: {
        const uint32_t ret = (c.pc + 2) & 0xFFFF;
        push<0>(c, W, ret >> 8, t);
        push<1>(c, W, ret & 0xFF, t);
        push<2>(c, W, c.p | FB | FU, t);
        c.p |= FI;
        const uint32_t lo = rd(c, W, 0xFFFE, t);
        const uint32_t hi = rd(c, W, 0xFFFF, t);
        npc = lo | (hi << 8);
        break;
    }
    default: break;                       // NOP, branches
    }
    if ((d >> DW_WR) & 1) wr<0>(c, W, ea, res, t);
    if (mn == RRA) do_adc(c, res);        // the ALU half of the undocumented pairs,
    else if (mn == ISC) do_sbc(c, res);   // after the write of their shifted /
    else if (mn == DCP) do_cmp(c, c.a, res);   // counted operand
    else if (mn == SLO) { c.a |= res; c.p = nz(c.p, c.a); }
    else if (mn == RLA) { c.a &= res; c.p = nz(c.p, c.a); }
    else if (mn == SRE) { c.a ^= res; c.p = nz(c.p, c.a); }
    c.pc = npc;
    c.cyc = t + 1;
}

// ------------------------------------------------------------ row log

__device__ __forceinline__ void log_finalize(Cpu& c) {
    if (c.open_row >= 0 && c.open_cnt) c.log[c.open_row * kSnapBytes + 15] = (uint8_t)c.open_cnt;
}

// Take the snapshots of every row up to `target` (inclusive) from the
// registers as they are now; the new rows' entries start where the open
// row's end.
__device__ __forceinline__ void log_advance(Cpu& c, const Wave& W, int32_t target) {
    if (target > kRows - 1) target = kRows - 1;
    while (c.open_row < target) {
        log_finalize(c);
        c.open_row++;
        c.open_base += c.open_cnt;
        c.open_cnt = 0;
        const uint32_t* s = reinterpret_cast<const uint32_t*>(W.tia + c.tia_off);
        uint4* d = reinterpret_cast<uint4*>(c.log + c.open_row * kSnapBytes);
        d[0] = make_uint4(s[0], s[1], s[2], s[3] & 0x00FFFFFFu);
        d[1] = make_uint4(s[4], s[5], s[6], (s[7] & 0xFFFF0000u) | c.open_base);
    }
}

// The entry of a write in the open row.  Every write logs at most one entry
// and a row's count stays within its bound, so the guard (an error bit
// instead of a truncated row) is never expected to fire.
__device__ __forceinline__ void log_entry(Cpu& c, int32_t row, uint32_t x, uint32_t code, uint32_t v0, uint32_t v1) {
    if (row < 0 || row >= kRows) return;
    if (c.open_cnt >= kCountMask || c.open_base + c.open_cnt >= (uint32_t)kFrameEntries) {
        c.err |= ERR_LOG;
        return;
    }
    *reinterpret_cast<uint32_t*>(c.log + kSnapArea + 4 * (c.open_base + c.open_cnt)) =
        x | (code << 8) | (v0 << 16) | (v1 << 24);
    c.open_cnt++;
}

// A render-visible event with effect at colour clock 3(t+1): bring the
// snapshots up to date; if it lands in a row's visible part, log it there.
__device__ __forceinline__ void log_event(Cpu& c, const Wave& W, uint32_t t, uint32_t code, uint32_t v0,
                                          uint32_t v1) {
    const uint32_t ln = (t + 1) / 76;
    const uint32_t h = 3 * (t + 1 - 76 * ln);
    const int32_t row = (int32_t)ln - c.fl - kFirstRow;
    log_advance(c, W, h >= 68 ? row : row - 1);
    if (h >= 68) log_entry(c, row, h - 68, code, v0, v1);
}

// the frame ends with its last cycle at t: rows after it are outside
__device__ __forceinline__ void log_close(Cpu& c, const Wave& W, uint32_t t) {
    log_event(c, W, t, R_END, 0, 0);
    log_finalize(c);
    for (int32_t r = c.open_row + 1; r < kRows; ++r) {
        uint4* d = reinterpret_cast<uint4*>(c.log + r * kSnapBytes);
        d[0] = make_uint4(0, 0, 0, kRowOutside << 24);
        d[1] = make_uint4(0, 0, 0, 0);
    }
    c.log = nullptr;
    if (!c.log_scratch) c.slots |= 1u << c.slot;
}

// ------------------------------------------------------------ collisions

// The latches are found by scanning pixels out of the row log, only when a
// latch is read, when an instruction is fetched from a latch, and at the end of
// a frame.  Every row's record holds its whole starting state, so the rows of a
// scan are independent: the lanes that need one post a job each, and all
// threads of the block (the wave that emulates and the helper waves that wait
// for it at a barrier) share the jobs' rows.  A wave scanning its own envs' rows,
// one lane per env, took 6.2 M of the 8.7 M cycles of a 4-frame step of a tile
// of 64 envs with all objects in motion, on a chip of whose SIMDs 4,096 such
// envs use 1 in 16; shared by 8 waves, 0.8 M of 3.6 M.
struct CxJob {
    uint64_t log;             // the env's row log
    int32_t row, x;           // scanned so far: the frame's pixels before (row, x)
    int32_t row_end, x_end;   // to scan: up to there
    int32_t open_row;         // the row still being logged, and its entries so far
    uint32_t open_cnt;
    uint32_t cx;              // the latch bits found
    uint32_t pad;
};

constexpr uint32_t kCxPre = 8;

// The share of thread tid, of n_threads, of m jobs (1 <= m <= 64 <= n_threads):
// each job's rows are cut into as many runs as leave every thread at most one.
// Neighbouring threads take the same run of different jobs: envs of one ROM
// mostly log the same registers at the same pixels of a row, so a wave's lanes
// draw the same objects anew at the same time (lanes on different rows of one
// env took 3 times as long).
__device__ __forceinline__ void cx_scan_rows(CxJob* jobs, uint32_t m, uint32_t tid, uint32_t n_threads) {
    const uint32_t runs = n_threads / m, run = tid / m;
    if (run >= runs) return;
    CxJob& J = jobs[tid - run * m];
    const uint8_t* log = (const uint8_t*)J.log;
    const int32_t first = J.row, row_end = J.row_end;
    const int32_t stop = row_end + (J.x_end > 0 ? 1 : 0);
    const int32_t per = (int32_t)(((uint32_t)(stop - first) + runs - 1) / runs);
    int32_t r = first + (int32_t)run * per;
    const int32_t end = min(r + per, stop);
    if (r >= end) return;
    // Rows are read ahead, the record two rows and the first kCxPre entries one
    // row before they are needed: 8 waves on a compute unit do not hide one
    // round trip to memory per entry (a tenth of a scan's time).  As in the
    // renderer, the words past a row's last entry are inside the log.
    const uint32_t* stream = reinterpret_cast<const uint32_t*>(log + kSnapArea);
    auto record = [&](int32_t row, uint4& a, uint4& b) {
        const uint4* rec = reinterpret_cast<const uint4*>(log + row * kSnapBytes);
        a = rec[0];
        b = rec[1];
    };
    auto entries = [&](const uint4& b, uint32_t (&q)[kCxPre]) {
#pragma unroll
        for (uint32_t i = 0; i < kCxPre; ++i) q[i] = stream[(b.w & 0xFFFF) + i];
    };
    uint4 na, nb, na2 = make_uint4(0, 0, 0, 0), nb2 = na2;
    uint32_t nq[kCxPre];
    record(r, na, nb);
    if (r + 1 < end) record(r + 1, na2, nb2);
    entries(nb, nq);
    // the last whole row scanned: a whole row with the same snapshot and the
    // same writes draws the same pixels (unless an HMOVE blank falls on one of
    // the two), so its latch bits are already found
    uint4 pa = make_uint4(0, 0, 0, 0), pb = pa;
    uint32_t pq[kCxPre] = {};
    uint32_t pcnt = ~0u, cx = 0;
    RowObjects O;
    row_objects_none(O);
    for (; r < end; ++r) {
        const uint32_t xs = r == first ? (uint32_t)J.x : 0u, xe = r < row_end ? 160u : (uint32_t)J.x_end;
        const uint4 sa = na, sb = nb;
        uint32_t q[kCxPre];
#pragma unroll
        for (uint32_t i = 0; i < kCxPre; ++i) q[i] = nq[i];
        const uint32_t cnt = r == J.open_row ? J.open_cnt : ((sa.w >> 24) & kCountMask);
        const uint32_t* ents = stream + (sb.w & 0xFFFF);
        if (r + 1 < end) {
            na = na2;
            nb = nb2;
            entries(nb, nq);
            if (r + 2 < end) record(r + 2, na2, nb2);
        }
        const bool whole = xs == 0 && xe == 160;
        if (whole && cnt == pcnt && cnt <= kCxPre) {
            const uint32_t hmb = (sb.z >> 8) & 0xFF;
            bool same = sa.x == pa.x && sa.y == pa.y && sa.z == pa.z && ((sa.w ^ pa.w) & 0x80FFFFFFu) == 0 &&
                        sb.x == pb.x && sb.y == pb.y && sb.z == pb.z && ((sb.w ^ pb.w) & 0xFFFF0000u) == 0 &&
                        hmb != (uint32_t)r && hmb != (uint32_t)r + 1;
#pragma unroll
            for (uint32_t i = 0; i < kCxPre; ++i) same = same && (i >= cnt || q[i] == pq[i]);
            if (same) continue;
        }
        pcnt = whole ? cnt : ~0u;
        pa = sa;
        pb = sb;
#pragma unroll
        for (uint32_t i = 0; i < kCxPre; ++i) pq[i] = q[i];
        Regs R;
        unpack(R, sa, sb);
        uint32_t ei = 0, cur = xs;           // q[0]: the next write, if ei < cnt
        while (cur < xe) {
            // writes in effect here; colours, wherever they are, move no object
            while (ei < cnt && ((q[0] & 0xFF) <= cur || ((q[0] >> 8) & 0xFF) <= R_COLUBK)) {
                apply(R, q[0]);
                ++ei;
#pragma unroll
                for (uint32_t i = 0; i + 1 < kCxPre; ++i) q[i] = q[i + 1];
                q[kCxPre - 1] = ei + (kCxPre - 1) < cnt ? ents[ei + (kCxPre - 1)] : 0u;
            }
            const uint32_t nx = ei < cnt ? min(q[0] & 0xFF, xe) : xe;
            if (!(R.outside || (rb<R_VBLANK>(R) & 2))) {
                row_objects(O, R);
                cx |= row_collisions(O, rb<R_HMB>(R) == (uint32_t)r + 1 ? max(cur, 8u) : cur, nx);
            }
            cur = nx;
        }
    }
    if (cx) atomicOr(&J.cx, cx);
}

// The emulating wave's own share: a call, so that the scan's registers are not
// added to those of the emulation (which then spills some around it).
__device__ __attribute__((noinline)) void cx_scan_share(CxJob* jobs, uint32_t m, uint32_t n_threads) {
    cx_scan_rows(jobs, m, threadIdx.x, n_threads);
}

// Who scans: nobody, every wave of the block, or the helper waves alone.
enum : int { TRACK_NONE = 0, TRACK_ALL = 1, TRACK_HELPERS = 2 };

// Scan for the lanes with `scan` up to (row_end, x_end).  Called by the whole
// emulating wave; `jobs` has a place per lane, *n_jobs is the helpers' word.
template <int TRACK>
__device__ __forceinline__ void cx_scan(Cpu& c, CxJob* jobs, uint32_t* n_jobs, bool scan, int32_t row_end,
                                        int32_t x_end) {
    if (row_end >= kRows) {
        row_end = kRows;
        x_end = 0;
    }
    if (x_end >= 160) {
        ++row_end;
        x_end = 0;
    }
    const bool work = scan && (c.cx_row < row_end || (c.cx_row == row_end && c.cx_x < x_end));
    const uint64_t mask = __builtin_amdgcn_ballot_w64(work);
    if (mask == 0) return;
    const uint32_t m = (uint32_t)__builtin_popcountll(mask);
    const uint32_t place = (uint32_t)__builtin_popcountll(mask & ((1ull << (threadIdx.x & 63)) - 1));
    if (work) jobs[place] = CxJob{(uint64_t)c.log, c.cx_row, c.cx_x, row_end, x_end, c.open_row, c.open_cnt, 0u, 0u};
    *n_jobs = m;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the log's stores, the hot loop's too
    __syncthreads();
    if constexpr (TRACK == TRACK_ALL) cx_scan_share(jobs, m, blockDim.x);
    __syncthreads();
    if (work) {
        c.cx |= jobs[place].cx;
        c.cx_row = row_end;
        c.cx_x = x_end;
    }
}

// Scan the pixels through colour clock `through` (relative to the base line)
// into the latches, for the lanes with `scan`; the rows the beam has reached
// get their snapshots first (as the next logged write would take them).
template <int TRACK>
__device__ __forceinline__ void cx_catch_up(Cpu& c, const Wave& W, CxJob* jobs, uint32_t* n_jobs, bool scan,
                                            int32_t through) {
    const int32_t line = through / 228, h = through % 228;
    const int32_t row = line - c.fl - kFirstRow;
    scan = scan && row >= 0;
    if (scan) log_advance(c, W, h >= 68 ? row : row - 1);
    cx_scan<TRACK>(c, jobs, n_jobs, scan, row, h >= 68 ? h - 68 + 1 : 0);
}

// Position a RESPx (players, +5) or RESMx / RESBL (+4) write at cycle t sets.
__device__ __forceinline__ uint32_t reset_pos(uint32_t t, uint32_t delay) {
    const uint32_t h = 3 * ((t + 1) % 76);
    return h < 68 ? delay - 2 : (h - 68 + delay) % 160;
}

// Full-byte register k (R[32 + k]) shows in R_FLAGS bit k (R_FLAGS2 bit 0
// for k = 8): ENAM0, ENAM1, ENABL, ENABL (delayed), RESMP0, RESMP1 by D1,
// VDELP0, VDELP1, VDELBL by D0.  The flags byte a write of v makes:
__device__ __forceinline__ uint32_t flags_after(const uint8_t* R, uint32_t k, uint32_t v) {
    const uint32_t bit = (k >= 4 && k <= 6) ? (v & 1) : ((v >> 1) & 1);
    return k == 8 ? bit : (R[R_FLAGS] & ~(1u << k)) | (bit << k);
}
__device__ __forceinline__ void set_flag_reg(uint8_t* R, uint32_t k, uint32_t v, uint32_t flags) {
    R[R_ENAM0 + k] = (uint8_t)v;
    R[k == 8 ? R_FLAGS2 : R_FLAGS] = (uint8_t)flags;
}


// Apply one queued TIA write of `v` to register `reg` made at cycle t: the
// row-log entries of what it changes for the renderer, then the registers.
__device__ __forceinline__ void tia_apply(Cpu& c, const Wave& W, uint32_t reg, uint32_t v, uint32_t t) {
    uint8_t* R = W.tia + c.tia_off;
    const bool lg = c.log != nullptr;
    if (W.track && reg == 0x2C) {               // CXCLR: the latches restart at clock 3(t+1)
        const int32_t ln = (int32_t)((t + 1) / 76), h = 3 * ((int32_t)(t + 1) - 76 * ln);
        const int32_t row = ln - c.fl - kFirstRow;
        c.cx = 0;
        if (row < 0) {
            c.cx_row = 0;
            c.cx_x = 0;
        } else if (row >= kRows) {
            c.cx_row = kRows;
            c.cx_x = 0;
        } else if (row > c.cx_row || (row == c.cx_row && h - 68 > c.cx_x)) {
            c.cx_row = row;
            c.cx_x = h >= 68 ? h - 68 : 0;
        }
        return;
    }
    switch (reg) {
    case 0x00:
        if ((v & 2) && !(c.vsync & 2)) c.ev |= EV_VSYNC;
        c.vsync = v;
        return;
    case 0x02: c.ev |= EV_WSYNC; return;
    case 0x20: c.hmp0 = v; return;
    case 0x21: c.hmp1 = v; return;
    case 0x22: case 0x23: case 0x24: R[R_HMM0 + reg - 0x22] = (uint8_t)v; return;
    case 0x2B: c.hmp0 = 0; c.hmp1 = 0; R[R_HMM0] = R[R_HMM1] = R[R_HMBL] = 0; return;
    case 0x1B:                                  // GRP0; GRP1 to its delayed copy
        if (lg) log_event(c, W, t, R_GRP0, v, 0);
        R[R_GRP1_OLD] = R[R_GRP1];
        R[R_GRP0] = (uint8_t)v;
        return;
    case 0x1C:                                  // GRP1; GRP0 and ENABL to their delayed copies
        if (lg) log_event(c, W, t, R_GRP1, v, 0);
        R[R_GRP0_OLD] = R[R_GRP0];
        R[R_GRP1] = (uint8_t)v;
        R[R_ENABL_OLD] = R[R_ENABL];
        R[R_FLAGS] = (uint8_t)((R[R_FLAGS] & ~8u) | ((R[R_FLAGS] & 4u) << 1));
        return;
    case 0x1D: case 0x1E: case 0x1F: case 0x25: case 0x26: case 0x27: {
        // (every entry is logged before the registers change: logging first
        // takes the snapshots of the rows before the write)
        const uint32_t k = reg <= 0x1F ? reg - 0x1D : reg - 0x25 + 4;
        const uint32_t fl = flags_after(R, k, v);
        if (lg) log_event(c, W, t, R_FLAGS, fl, 0);
        set_flag_reg(R, k, v, fl);
        return;
    }
    case 0x28: case 0x29: {                     // RESMP: the release puts the missile at the player's centre
        const uint32_t i = reg - 0x28;
        const uint32_t was = (R[R_RESMP0 + i] >> 1) & 1;
        const uint32_t fl = flags_after(R, 7 + i, v);
        const bool release = !(v & 2) && was;
        const uint32_t mode = R[R_NUSIZ0 + i] & 7;
        const uint32_t pos = (R[R_P0X + i] + (mode == 5 ? 6u : mode == 7 ? 10u : 3u)) % 160;
        if (lg) log_event(c, W, t, R_RESMP + i, fl, release ? pos : R[R_M0X + i]);
        if (release) R[R_M0X + i] = (uint8_t)pos;
        set_flag_reg(R, 7 + i, v, fl);
        return;
    }
    case 0x2A: {                                // HMOVE: every object by the pulses its blank takes, now
        const uint32_t ln = (t + 1) / 76, h = 3 * (t + 1 - 76 * ln);
        const uint32_t p0 = hm_move(R[R_P0X], hmove_left(h, c.hmp0 >> 4));
        const uint32_t p1 = hm_move(R[R_P1X], hmove_left(h, c.hmp1 >> 4));
        const uint32_t m0 = hm_move(R[R_M0X], hmove_left(h, R[R_HMM0] >> 4));
        const uint32_t m1 = hm_move(R[R_M1X], hmove_left(h, R[R_HMM1] >> 4));
        const uint32_t bl = hm_move(R[R_BLX], hmove_left(h, R[R_HMBL] >> 4));
        if (lg)   // one entry: the renderer applies the five motion nibbles itself
            log_event(c, W, t, R_HMOVE | ((R[R_HMBL] >> 4) & 15), ((c.hmp0 >> 4) & 15) | (c.hmp1 & 0xF0),
                      ((R[R_HMM0] >> 4) & 15) | (R[R_HMM1] & 0xF0));
        R[R_P0X] = (uint8_t)p0; R[R_P1X] = (uint8_t)p1;
        R[R_M0X] = (uint8_t)m0; R[R_M1X] = (uint8_t)m1; R[R_BLX] = (uint8_t)bl;
        if (h < 68) {                           // written in the horizontal blank: pixels 0-7 of the line blank
            c.hmb_line = (int32_t)ln;
            const int32_t row = (int32_t)ln - c.fl - kFirstRow;
            if (row >= 0 && row < kRows) R[R_HMB] = (uint8_t)(row + 1);
        }
        return;
    }
    default: break;
    }
    uint32_t code, v0 = v;
    if (reg >= 0x06 && reg <= 0x0F) code = reg - 0x06;
    else if (reg == 0x01) code = R_VBLANK;
    else if (reg == 0x04 || reg == 0x05) code = R_NUSIZ0 + (reg - 0x04);
    else if (reg == 0x10 || reg == 0x11) {
        code = R_P0X + (reg - 0x10);
        v0 = reset_pos(t, 5);
    } else if (reg >= 0x12 && reg <= 0x14) {
        code = R_M0X + (reg - 0x12);
        v0 = reset_pos(t, 4);
    } else {
        return;   // audio and the rest: no emulated effect
    }
    if (lg) log_event(c, W, t, code, v0, 0);
    R[code] = (uint8_t)v0;
}

__device__ __forceinline__ void apply_queue(Cpu& c, const Wave& W, uint32_t t) {
    if (c.tqm) {
        if (c.tqm & 1) tia_apply(c, W, c.tqr0, c.tqv0, t);
        if (c.tqm & 2) tia_apply(c, W, c.tqr1, c.tqv1, t);
        if (c.tqm & 4) tia_apply(c, W, c.tqr2, c.tqv2, t);
    }
}

__device__ __forceinline__ uint32_t rfl(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ int32_t rfl(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }

// ------------------------------------------------------- wave-uniform path
//
// The full dispatch of a group of lanes at one place (run_cold): bank, pc, cycle,
// frame line and open row are scalars (Fast), the predecoded word gives opcode
// and operands, addressing and timing run on the scalar unit, and only the data
// (A, X, Y, P, SP, RAM, TIA registers, log position and stores) is per lane.
// Branches whose outcome differs end the run with the lanes parted; penalties or
// stack targets that differ leave the instruction to the per-lane path, as do
// those not covered here (indirect modes, JMP (ind), RTI, BRK, indexed accesses
// outside RAM and cartridge).
struct Fast {
    uint32_t pc, bank, cyc, orow;
    int32_t fl;
    uint32_t logon;
};

__device__ __forceinline__ bool all_lanes(bool p) { return __builtin_amdgcn_ballot_w64(!p) == 0; }

// Stores that the full dispatch leaves to the per-lane path: VSYNC (it may end
// the frame), the motion registers, HMOVE, HMCLR, RESMP, CXCLR and timer writes.
// (The hot loop takes the motion registers, HMCLR and a VSYNC that ends no frame
// itself.)
__device__ __forceinline__ bool tia_exit_reg(uint32_t reg) {
    return reg == 0x00 || (reg >= 0x20 && reg <= 0x24) || reg == 0x28 || reg == 0x29 || reg == 0x2A || reg == 0x2B ||
           reg == 0x2C;
}
__device__ __forceinline__ uint32_t fast_store_ok(uint32_t a) {
    if (a & 0x1000) return 1;                             // cartridge: bank hotspots only
    if (!(a & 0x80)) return tia_exit_reg(a & 0x3F) ? 0u : 1u;   // TIA
    if (!(a & 0x200)) return 1;                           // RAM
    return (a & 0x14) != 0x14 ? 1u : 0u;                  // RIOT: everything but the timer
}

// Store classes of a static address (cart_store_class): the full dispatch's
// cases, and what k_predecode picks a store's hot-loop slot by.
constexpr uint32_t SC_RAM = 0, SC_WSYNC = 1, SC_IGNORE = 2, SC_EXIT = 3, SC_CART = 4, SC_TIA = 0x20;
// SC_TIA | code: a register stored as is; SC_TIAS | code: a position from
// the cycle or a flags byte; SC_TIAG | code: GRP0 / GRP1 (the delayed copies)
constexpr uint32_t SC_TIAS = 0x40, SC_TIAG = 0x60;
// classes that depend on the cartridge: an absolute access to the Superchip RAM
// window, and a 3F slice-select store to an ignored TIA register
constexpr uint32_t SC_XRAM = 5, SC_3F = 6;
// TIA store codes past the snapshot registers: ENAM0, ENAM1, ENABL, VDELP0,
// VDELP1, VDELBL (SC_TIAS | kScFlag0 + i), written as their full byte and a
// new flags byte
constexpr uint32_t kScFlag0 = 26;

// Class of a store to a (13 bits): RAM, WSYNC, a TIA register the scalar path
// writes (SC_TIA, SC_TIAS or SC_TIAG | its code), a write that changes nothing emulated, a
// cartridge access, or one the scalar path leaves to the per-lane path
// (fast_store_ok).
__device__ __forceinline__ uint32_t store_class(uint32_t a) {
    if (a & 0x1000) return SC_CART;
    if (!(a & 0x80)) {
        const uint32_t reg = a & 0x3F;
        if (reg == 0x02) return SC_WSYNC;
        if (tia_exit_reg(reg)) return SC_EXIT;
        if (reg >= 0x06 && reg <= 0x0F) return SC_TIA | (reg - 0x06);
        if (reg == 0x01) return SC_TIA | R_VBLANK;
        if (reg == 0x04 || reg == 0x05) return SC_TIA | (R_NUSIZ0 + reg - 0x04);
        if (reg == 0x1B) return SC_TIAG | R_GRP0;
        if (reg == 0x1C) return SC_TIAG | R_GRP1;
        if (reg == 0x10 || reg == 0x11) return SC_TIAS | (R_P0X + reg - 0x10);
        if (reg >= 0x12 && reg <= 0x14) return SC_TIAS | (R_M0X + reg - 0x12);
        if (reg >= 0x1D && reg <= 0x1F) return SC_TIAS | (kScFlag0 + reg - 0x1D);
        if (reg >= 0x25 && reg <= 0x27) return SC_TIAS | (kScFlag0 + 3 + reg - 0x25);
        return SC_IGNORE;   // audio and the rest
    }
    if (!(a & 0x200)) return SC_RAM;
    return (a & 0x14) == 0x14 ? SC_EXIT : SC_IGNORE;
}

// The class on the tile's cartridge: on 3F cartridges a store to $00-$3F also
// selects a slice (SC_3F when the TIA register it reaches is not emulated,
// else left to the per-lane path); with a Superchip its RAM window is SC_XRAM.
__device__ __forceinline__ uint32_t cart_store_class(uint32_t kind, uint32_t sc, uint32_t a) {
    const uint32_t k = store_class(a);
    if (kind == CART_3F && a <= 0x3F) return k == SC_IGNORE ? SC_3F : SC_EXIT;
    return sc && (a & 0x1000) && !(a & 0xF00) ? SC_XRAM : k;
}
__device__ __forceinline__ uint32_t cart_store_class(const Wave& W, uint32_t a) {
    return cart_store_class(cm_kind(W), cm_sc(W), a);
}

// Predecoded word: store class (7 bits) | slot << 7 | b1 << 16 | b2 << 24.  The
// slot is the hot loop's handler (hotloop.h); a HOT_REAL word carries the
// opcode in bits 0-6 and 15 instead of a class.
//
// The two-step reads' operation (HW_*), and the modes whose slots they have.
constexpr uint32_t hot_work(int mn) {
    switch (mn) {
    case LDA: return HW_LDA; case LDX: return HW_LDX; case LDY: return HW_LDY; case AND: return HW_AND;
    case ORA: return HW_ORA; case EOR: return HW_EOR; case CMP: return HW_CMP; case CPX: return HW_CPX;
    case CPY: return HW_CPY; case BIT: return HW_BIT; case ADC: return HW_ADC; case SBC: return HW_SBC;
    case ASL: return HW_ASL; case ROL: return HW_ROL; case LSR: return HW_LSR; case ROR: return HW_ROR;
    case DEC: return HW_DEC; case INC: return HW_INC;
    }
    return HW_NONE;
}
constexpr uint32_t kTwoStepFirst = HOT_Z_CONST, kTwoStepEnd = HOT_SEG_Y + 1;
constexpr int two_step_mode(uint32_t slot) {
    switch (slot) {
    case HOT_Z_CONST: case HOT_Z_INPT4: return ZP;
    case HOT_ZX: case HOT_ZX_RMW: return ZPX;
    case HOT_ZY: return ZPY;
    case HOT_AX_ROM: case HOT_AX_RAM: case HOT_SEG_X: return ABX;
    case HOT_AY_ROM: case HOT_AY_RAM: case HOT_SEG_Y: return ABY;
    case HOT_IY_ROM: return IZY;
    default: return ABS;
    }
}
// The opcode a slot runs, whole words for the scalar unit: op[slot], two[32
// (slot - kTwoStepFirst) + operation] for the two-step reads, st[register] for
// stores of any register (the class's bits 5-6: A, X, Y).
struct HotOps {
    uint32_t op[kHotSlots], two[32 * (kTwoStepEnd - kTwoStepFirst)], st_zp[4], st_abs[4];
    constexpr HotOps() : op(), two(), st_zp(), st_abs() {
        for (uint32_t i = 0; i < kHotSlots; ++i) op[i] = kHotSlotOp[i];
        for (uint32_t o = 0; o < 256; ++o) {
            const OpInfo I = decode((int)o);
            const uint32_t w = hot_work(I.mn);
            for (uint32_t s = kTwoStepFirst; w != HW_NONE && s < kTwoStepEnd; ++s)
                if (two_step_mode(s) == I.md) two[32 * (s - kTwoStepFirst) + w] = o;
        }
        st_zp[0] = 0x85; st_zp[1] = 0x86; st_zp[2] = 0x84;
        st_abs[0] = 0x8D; st_abs[1] = 0x8E; st_abs[2] = 0x8C;
    }
};
__constant__ HotOps kHotOps = HotOps();
struct HotWorks {                                // an opcode's operation
    uint8_t w[256];
    constexpr HotWorks() : w() {
        for (int i = 0; i < 256; ++i) w[i] = (uint8_t)hot_work(decode(i).mn);
    }
};
__constant__ HotWorks kHotWorkOf = HotWorks();
struct HotSlots {                                // an opcode's slot (hot_slot)
    uint8_t s[256];
    constexpr HotSlots() : s() {
        for (uint32_t i = 0; i < 256; ++i) s[i] = (uint8_t)hot_slot(i);
    }
};
__constant__ HotSlots kHotSlot = HotSlots();
__device__ __forceinline__ uint32_t pre_slot(uint32_t q) { return (q >> 7) & 0xFF; }
__device__ __forceinline__ uint32_t pre_op(uint32_t q) {
    const uint32_t slot = pre_slot(q);
    if (slot == HOT_REAL) return (q & 0x7F) | ((q >> 8) & 0x80);
    if (slot - kTwoStepFirst < kTwoStepEnd - kTwoStepFirst) return kHotOps.two[32 * (slot - kTwoStepFirst) + (q & 31)];
    if (slot == HOT_RESP || slot == HOT_RESM || slot == HOT_HMCLR) return kHotOps.st_zp[(q >> 5) & 3];
    if (slot == HOT_HS_ST) return kHotOps.st_abs[(q >> 5) & 3];
    return kHotOps.op[slot];
}

// Write of per-lane value v to TIA register class `sc` (SC_TIA/S/G | code) at
// scalar cycle t, with its row-log entry.  The scalar path takes the colour,
// playfield, control, reflection, VBLANK and NUSIZ registers, the object
// resets, the players' graphics and the enable and vertical-delay bits
// (logged as the new flags byte); motion, HMOVE, RESMP and CXCLR go to the
// per-lane path.  A GRP0 / GRP1 entry also stands for the copy to the delayed
// registers (the other player's graphics; with GRP1, ENABL), which the
// renderer repeats from its own state.  Returns 0, before changing a register,
// when a lane's row is full (the per-lane path then records the error).
__device__ __forceinline__ uint32_t fast_tia_code(Cpu& c, const Wave& W, Fast& F, uint32_t sc, uint32_t v,
                                                  uint32_t t) {
    const uint32_t ln = (t + 1) / 76;
    const uint32_t h = 3 * (t + 1 - 76 * ln);
    uint8_t* R = W.tia + c.tia_off;
    uint32_t code = sc & 0x1F;
    uint32_t v0 = v, full = 0;
    if (sc >= SC_TIAS && sc < SC_TIAG) {
        if (code == R_P0X || code == R_P1X) {
            v0 = h < 68 ? 3u : (h - 68 + 5) % 160;
        } else if (code >= R_M0X && code <= R_BLX) {
            v0 = h < 68 ? 2u : (h - 68 + 4) % 160;
        } else if (code >= kScFlag0) {       // ENAM0/1, ENABL (D1), VDELP0/1, VDELBL (D0)
            const uint32_t i = code - kScFlag0;
            const uint32_t k = i < 3 ? i : i + 1;
            const uint32_t bit = i < 3 ? (v >> 1) & 1 : v & 1;
            v0 = (R[R_FLAGS] & ~(1u << k)) | (bit << k);
            full = R_ENAM0 + k;
            code = R_FLAGS;
        }
    }
    if (F.logon) {
        // rows before the one the write lands in (its own row too when the
        // write lands in the visible part) get their snapshots first
        const int32_t row = (int32_t)ln - F.fl - kFirstRow;
        const int32_t vis = h >= 68 ? 1 : 0;
        int32_t target = row - 1 + vis;
        target = target > kRows - 1 ? kRows - 1 : target;
        if ((int32_t)F.orow <= target) {
            if (F.orow > 0) c.log[(F.orow - 1) * kSnapBytes + 15] = (uint8_t)c.open_cnt;
            c.open_base += c.open_cnt;   // the new rows' entries start after the open row's
            c.open_cnt = 0;
            const uint32_t* src = reinterpret_cast<const uint32_t*>(R);
            const uint4 snap0 = make_uint4(src[0], src[1], src[2], src[3] & 0x00FFFFFFu);
            const uint4 snap1 = make_uint4(src[4], src[5], src[6], (src[7] & 0xFFFF0000u) | c.open_base);
            do {    // F.orow holds the open row + 1 (0 = none)
                uint4* d = reinterpret_cast<uint4*>(c.log + F.orow * kSnapBytes);
                d[0] = snap0;
                d[1] = snap1;
                F.orow++;
            } while ((int32_t)F.orow <= target);
        }
        if (vis) {
            if ((uint32_t)row < (uint32_t)kRows) {
                // the row is the open one here; past the guard the per-lane path records the error
                if (!all_lanes(c.open_cnt < kCountMask && c.open_base + c.open_cnt < (uint32_t)kFrameEntries)) return 0;
                *reinterpret_cast<uint32_t*>(c.log + kSnapArea + 4 * (c.open_base + c.open_cnt)) =
                    (h - 68) | (code << 8) | (v0 << 16);
                c.open_cnt++;
            }
        }
    }
    if (sc >= SC_TIAG) {
        if (code == R_GRP0) {
            R[R_GRP1_OLD] = R[R_GRP1];
        } else {
            R[R_GRP0_OLD] = R[R_GRP0];
            R[R_ENABL_OLD] = R[R_ENABL];
            R[R_FLAGS] = (uint8_t)((R[R_FLAGS] & ~8u) | ((R[R_FLAGS] & 4u) << 1));
        }
    } else if (full) {
        R[full] = (uint8_t)v;
    }
    R[code] = (uint8_t)v0;
    return 1;
}

// TIA write of per-lane `v` to scalar register `reg` at scalar cycle t (a
// register fast_store_ok accepts).  Sets `wsync`.  Returns 0 when the
// per-lane path must take the write (a full row log).
__device__ __forceinline__ uint32_t fast_tia(Cpu& c, const Wave& W, Fast& F, uint32_t reg, uint32_t v, uint32_t t,
                                             uint32_t& wsync) {
    const uint32_t sc = store_class(reg);
    if (sc == SC_WSYNC) {
        wsync = 1;
        return 1;
    }
    if (sc < SC_TIA) return 1;
    return fast_tia_code(c, W, F, sc, v, t);
}

// Read of scalar address a (13 bits) at scalar cycle t.
__device__ __forceinline__ uint32_t fast_rd(Cpu& c, const Wave& W, Fast& F, uint32_t a, uint32_t t) {
    if (a & 0x1000) {
        F.bank = hotspot(W, F.bank, a);
        return W.rom[rom_off(W, F.bank, a)];
    }
    if (!(a & 0x80)) {
        const uint32_t r = a & 0x0F;
        return r == 0x0C ? c.inpt4 : (r == 0x0D ? 0x80u : 0u);
    }
    if (!(a & 0x200)) return W.ram[c.ram_off + (a & 0x7F)];
    return riot_read(c, W, a, t);
}

// Write of per-lane v to scalar address a (fast_store_ok) at scalar cycle t.
// Returns false when the per-lane path must take the instruction.
__device__ __forceinline__ uint32_t fast_wr(Cpu& c, const Wave& W, Fast& F, uint32_t a, uint32_t v, uint32_t t,
                                            uint32_t& wsync) {
    if (a & 0x1000) {
        F.bank = hotspot(W, F.bank, a);
        return 1;
    }
    if (!(a & 0x80)) return fast_tia(c, W, F, a & 0x3F, v & 0xFF, t, wsync);
    if (!(a & 0x200)) W.ram[c.ram_off + (a & 0x7F)] = (uint8_t)v;
    return 1;   // other RIOT writes (ports) change nothing emulated
}

// Decimal mode of the lanes in exec for ADC/SBC: 0 all binary, 1 all
// decimal, 2 mixed (the per-lane path then takes the instruction).  Keeping
// the choice uniform keeps the scalar loop free of per-lane branches.
__device__ __forceinline__ uint32_t dec_mode(const Cpu& c) {
    const uint64_t d = __builtin_amdgcn_ballot_w64((c.p & FD) != 0);
    if (d == 0) return 0;
    return d == __builtin_amdgcn_ballot_w64(true) ? 1u : 2u;
}

__device__ __forceinline__ void adc_bin(Cpu& c, uint32_t v) {
    const uint32_t bin = c.a + v + (c.p & FC);
    const uint32_t ovf = (c.a ^ bin) & (v ^ bin) & 0x80;
    c.p = (c.p & ~(FC | FV)) | (bin > 0xFF ? FC : 0) | (ovf ? FV : 0);
    c.a = bin & 0xFF;
    c.p = nz(c.p, c.a);
}

// the decimal ADC and SBC of the per-lane path, for lanes known to be in
// decimal mode (their arithmetic compiles to selects)
__device__ __forceinline__ void adc_dec(Cpu& c, uint32_t v) {
    const uint32_t cin = c.p & FC;
    const uint32_t bin = c.a + v + cin;
    int32_t lo = (int32_t)((c.a & 0x0F) + (v & 0x0F) + cin);
    lo = lo > 9 ? ((lo + 6) & 0x0F) + 0x10 : lo;
    int32_t sum = (int32_t)(c.a & 0xF0) + (int32_t)(v & 0xF0) + lo;
    const int32_t ss = sext8(c.a & 0xF0) + sext8(v & 0xF0) + lo;
    sum = sum >= 0xA0 ? sum + 0x60 : sum;
    c.p = (c.p & ~(FC | FV | FN | FZ)) | (sum >= 0x100 ? FC : 0) | ((ss < -128 || ss > 127) ? FV : 0) |
          (ss & 0x80 ? FN : 0) | ((bin & 0xFF) == 0 ? FZ : 0);
    c.a = (uint32_t)sum & 0xFF;
}

__device__ __forceinline__ void sbc_any(Cpu& c, uint32_t v, uint32_t dec) {
    const uint32_t cin = c.p & FC;
    const uint32_t inv = (~v) & 0xFF;
    const uint32_t bin = c.a + inv + cin;
    const uint32_t ovf = (c.a ^ bin) & (inv ^ bin) & 0x80;
    uint32_t res = bin & 0xFF;
    if (dec) {
        int32_t lo = (int32_t)(c.a & 0x0F) - (int32_t)(v & 0x0F) + (int32_t)cin - 1;
        lo = lo < 0 ? ((lo - 6) & 0x0F) - 0x10 : lo;
        int32_t d = (int32_t)(c.a & 0xF0) - (int32_t)(v & 0xF0) + lo;
        d = d < 0 ? d - 0x60 : d;
        res = (uint32_t)d & 0xFF;
    }
    c.p = (c.p & ~(FC | FV)) | (bin > 0xFF ? FC : 0) | (ovf ? FV : 0);
    c.p = nz(c.p, bin & 0xFF);
    c.a = res;
}

// Per-lane ALU part of the read-class operations (operand v); `dm` is the
// uniform decimal mode (dec_mode) for ADC and SBC.
__device__ __forceinline__ void fast_alu(Cpu& c, uint32_t mn, uint32_t v, uint32_t dm = 0) {
    switch (mn) {
    case LDA: c.a = v; c.p = nz(c.p, v); break;
    case LDX: c.x = v; c.p = nz(c.p, v); break;
    case LDY: c.y = v; c.p = nz(c.p, v); break;
    case ADC: if (dm) adc_dec(c, v); else adc_bin(c, v); break;
    case SBC: sbc_any(c, v, dm); break;
    case AND: c.a &= v; c.p = nz(c.p, c.a); break;
    case ORA: c.a |= v; c.p = nz(c.p, c.a); break;
    case EOR: c.a ^= v; c.p = nz(c.p, c.a); break;
    case CMP: do_cmp(c, c.a, v); break;
    case CPX: do_cmp(c, c.x, v); break;
    case CPY: do_cmp(c, c.y, v); break;
    default: c.p = (c.p & ~(FN | FV | FZ)) | (v & (FN | FV)) | ((c.a & v) == 0 ? FZ : 0); break;   // BIT
    }
}

__device__ __forceinline__ uint32_t fast_rmw(Cpu& c, uint32_t mn, uint32_t x) {
    const uint32_t ci = c.p & FC;
    uint32_t r, co = ci;
    if (mn == ASL) { r = (x << 1) & 0xFF; co = x >> 7; }
    else if (mn == LSR) { r = x >> 1; co = x & 1; }
    else if (mn == ROL) { r = ((x << 1) | ci) & 0xFF; co = x >> 7; }
    else if (mn == ROR) { r = (x >> 1) | (ci << 7); co = x & 1; }
    else if (mn == INC) { r = (x + 1) & 0xFF; }
    else { r = (x - 1) & 0xFF; }
    c.p = nz((c.p & ~FC) | co, r);
    return r;
}

// Outcome of one instruction on the wave-uniform path.
enum : uint32_t {
    FS_NEXT = 0,     // executed; F holds the next pc and cycle
    FS_EXIT = 1,     // not executed: the per-lane path takes this instruction
    FS_LANE = 2      // executed; lanes parted, c.pc / c.cyc hold each lane's
};

constexpr bool read_mn(int mn) {
    return mn == LDA || mn == LDX || mn == LDY || mn == ADC || mn == SBC || mn == AND || mn == ORA || mn == EOR ||
           mn == CMP || mn == CPX || mn == CPY || mn == BIT;
}
constexpr bool store_mn(int mn) { return mn == STA || mn == STX || mn == STY; }
constexpr bool rmw_mn(int mn) { return mn == ASL || mn == LSR || mn == ROL || mn == ROR || mn == INC || mn == DEC; }

template <int MN>
__device__ __forceinline__ uint32_t store_value(const Cpu& c) {
    return MN == STA ? c.a : (MN == STX ? c.x : c.y);
}

// End of an instruction that may have written a TIA register: next pc and
// cycle (a WSYNC write stalls to the next line start).
__device__ __forceinline__ uint32_t fast_finish(Fast& F, uint32_t next, uint32_t t, uint32_t wsync) {
    F.pc = next;
    F.cyc = wsync ? 76 * (t / 76 + 1) : t + 1;
    return FS_NEXT;
}

// One instruction with opcode OP (a compile-time constant, so addressing
// mode, operation and base cycles are folded) for every lane in exec;
// TRACK: collision latches tracked.
template <int OP, bool TRACK>
__device__ __forceinline__ uint32_t fop(Cpu& c, const Wave& W, Fast& F, uint32_t b1, uint32_t b2) {
    constexpr OpInfo I = decode(OP);
    constexpr int MD = I.md, MN = I.mn;
    constexpr uint32_t N = (uint32_t)I.cyc;
    const uint32_t next = (F.pc + (uint32_t)op_len(MD)) & 0xFFFF;
    if constexpr (MN == ILL || MN == BRK || MN == RTI || MD == IZX || MD == IZY || MD == IND || MN >= SLO ||
                  (MN == NOP && MD != IMP)) {
        return FS_EXIT;   // left to the per-lane path (undocumented opcodes included)
    } else if constexpr (MD == IMM) {
        uint32_t dm = 0;
        if constexpr (MN == ADC || MN == SBC) {
            dm = dec_mode(c);
            if (dm == 2) return FS_EXIT;
        }
        fast_alu(c, MN, b1, dm);
        F.pc = next;
        F.cyc += N;
        return FS_NEXT;
    } else if constexpr (MD == ACC) {
        c.a = fast_rmw(c, MN, c.a);
        F.pc = next;
        F.cyc += N;
        return FS_NEXT;
    } else if constexpr (MD == IMP) {
        if constexpr (MN == PHA || MN == PHP) {
            if (!all_lanes(c.sp >= 0x80)) return FS_EXIT;
            W.ram[c.ram_off + (c.sp & 0x7F)] = (uint8_t)(MN == PHA ? c.a : (c.p | FB | FU));
            c.sp = (c.sp - 1) & 0xFF;
        } else if constexpr (MN == PLA || MN == PLP) {
            if (!all_lanes(c.sp >= 0x7F && c.sp <= 0xFE)) return FS_EXIT;
            c.sp = (c.sp + 1) & 0xFF;
            const uint32_t v = W.ram[c.ram_off + (c.sp & 0x7F)];
            if constexpr (MN == PLA) {
                c.a = v;
                c.p = nz(c.p, v);
            } else {
                c.p = (v & ~FB) | FU;
            }
        } else if constexpr (MN == RTS) {
            if (!all_lanes(c.sp >= 0x7F && c.sp <= 0xFD)) return FS_EXIT;
            const uint32_t lo = W.ram[c.ram_off + ((c.sp + 1) & 0x7F)];
            const uint32_t hi = W.ram[c.ram_off + ((c.sp + 2) & 0x7F)];
            c.sp = (c.sp + 2) & 0xFF;
            const uint32_t tgt = ((lo | (hi << 8)) + 1) & 0xFFFF;
            const uint32_t t0 = rfl(tgt);
            if (!all_lanes(tgt == t0)) {
                c.pc = tgt;
                c.cyc = F.cyc + N;
                return FS_LANE;
            }
            F.pc = t0;
            F.cyc += N;
            return FS_NEXT;
        } else if constexpr (MN == INX) { c.x = (c.x + 1) & 0xFF; c.p = nz(c.p, c.x); }
        else if constexpr (MN == INY) { c.y = (c.y + 1) & 0xFF; c.p = nz(c.p, c.y); }
        else if constexpr (MN == DEX) { c.x = (c.x - 1) & 0xFF; c.p = nz(c.p, c.x); }
        else if constexpr (MN == DEY) { c.y = (c.y - 1) & 0xFF; c.p = nz(c.p, c.y); }
        else if constexpr (MN == TAX) { c.x = c.a; c.p = nz(c.p, c.x); }
        else if constexpr (MN == TAY) { c.y = c.a; c.p = nz(c.p, c.y); }
        else if constexpr (MN == TXA) { c.a = c.x; c.p = nz(c.p, c.a); }
        else if constexpr (MN == TYA) { c.a = c.y; c.p = nz(c.p, c.a); }
        else if constexpr (MN == TSX) { c.x = c.sp; c.p = nz(c.p, c.x); }
        else if constexpr (MN == TXS) { c.sp = c.x; }
        else if constexpr (MN == CLC) { c.p &= ~FC; }
        else if constexpr (MN == SEC) { c.p |= FC; }
        else if constexpr (MN == CLI) { c.p &= ~FI; }
        else if constexpr (MN == SEI) { c.p |= FI; }
        else if constexpr (MN == CLV) { c.p &= ~FV; }
        else if constexpr (MN == CLD) { c.p &= ~FD; }
        else if constexpr (MN == SED) { c.p |= FD; }
        F.pc = next;
        F.cyc += N;
        return FS_NEXT;
    } else if constexpr (MD == ZP || MD == ABS) {
        const uint32_t ea = MD == ZP ? b1 : (b1 | (b2 << 8));
        const uint32_t a = ea & 0x1FFF;
        const uint32_t t = F.cyc + N - 1;
        if constexpr (MN == JMP) {
            F.pc = ea;
            F.cyc += N;
            return FS_NEXT;
        } else if constexpr (MN == JSR) {
            if (!all_lanes(c.sp >= 0x81)) return FS_EXIT;
            const uint32_t ret = (next - 1) & 0xFFFF;
            W.ram[c.ram_off + (c.sp & 0x7F)] = (uint8_t)(ret >> 8);
            W.ram[c.ram_off + ((c.sp - 1) & 0x7F)] = (uint8_t)(ret & 0xFF);
            c.sp = (c.sp - 2) & 0xFF;
            F.pc = ea;
            F.cyc += N;
            return FS_NEXT;
        } else if constexpr (read_mn(MN)) {
            uint32_t dm = 0;
            if constexpr (MN == ADC || MN == SBC) {
                dm = dec_mode(c);
                if (dm == 2) return FS_EXIT;
            }
            uint32_t v;
            if (TRACK && !(a & 0x1080) && (a & 0xF) < 8) return FS_EXIT;   // a latch read: the per-lane path scans the log
            if (MD == ABS && (a & 0x1000) && sc_window(W, a))   // Superchip RAM: read port, or the write port (0)
                v = (a & 0x80) ? (uint32_t)c.xram[a & 0x7F] : 0u;
            else
                v = fast_rd(c, W, F, a, t);
            fast_alu(c, MN, v, dm);
            F.pc = next;
            F.cyc += N;
            return FS_NEXT;
        } else if constexpr (store_mn(MN)) {
            const uint32_t aux = cart_store_class(W, a);
            const uint32_t v = store_value<MN>(c);
            if (aux == SC_RAM) {
                W.ram[c.ram_off + (a & 0x7F)] = (uint8_t)v;
            } else if (aux >= SC_TIA) {
                if (!fast_tia_code(c, W, F, aux, v & 0xFF, t)) return FS_EXIT;
            } else if (aux == SC_WSYNC) {
                return fast_finish(F, next, t, 1);
            } else if (aux == SC_EXIT) {
                return FS_EXIT;
            } else if (aux == SC_CART) {
                F.bank = hotspot(W, F.bank, a);
            } else if (aux == SC_XRAM) {
                if (!(a & 0x80)) c.xram[a & 0x7F] = (uint8_t)v;   // writes to the read port do nothing
            } else if (aux == SC_3F) {
                // the slice number must agree across the lanes to stay uniform
                const uint32_t sl = v & cm_tf_mask(W), s0 = rfl(sl);
                if (!all_lanes(sl == s0)) return FS_EXIT;
                F.bank = s0;
            }
            F.pc = next;
            F.cyc += N;
            return FS_NEXT;
        } else {
            static_assert(rmw_mn(MN), "read-modify-write");
            // a TIA register reads back as an input port or 0: RMW on one is
            // left to the per-lane path, as are the stores fast_store_ok refuses
            if (!(a & 0x1000) && !(a & 0x80)) return FS_EXIT;
            if (!fast_store_ok(a)) return FS_EXIT;
            if constexpr (MD == ABS) {
                if ((a & 0x1000) && sc_window(W, a)) return FS_EXIT;   // RMW on the Superchip RAM window
            }
            const uint32_t v = fast_rd(c, W, F, a, t);
            const uint32_t r = fast_rmw(c, MN, v);
            uint32_t wsync = 0;
            fast_wr(c, W, F, a, r, t, wsync);
            return fast_finish(F, next, t, wsync);
        }
    } else if constexpr (MD == ZPX || MD == ZPY || MD == ABX || MD == ABY) {
        const uint32_t idx = (MD == ZPX || MD == ABX) ? c.x : c.y;
        uint32_t ea;
        bool cross = false;
        if constexpr (MD == ZPX || MD == ZPY) {
            ea = (b1 + idx) & 0xFF;
        } else {
            const uint32_t base = b1 | (b2 << 8);
            ea = (base + idx) & 0xFFFF;
            cross = ((base ^ ea) & 0xFF00) != 0;
        }
        const uint32_t a = ea & 0x1FFF;
        const bool in_ram = (a & 0x1280) == 0x0080;
        if constexpr (read_mn(MN)) {
            // cartridge addresses that are plain ROM: no hotspot, no Superchip RAM
            const bool in_cart = (a & 0x1000) && hotspot(W, F.bank, a) == F.bank && !sc_window(W, a);
            if (!all_lanes(in_ram || in_cart)) return FS_EXIT;
        } else {
            if (!all_lanes(in_ram)) return FS_EXIT;
        }
        uint32_t n = N;
        if constexpr (I.pen) {
            const uint32_t cr = rfl(cross ? 1u : 0u);
            if (!all_lanes(cross == (cr != 0))) return FS_EXIT;
            n += cr;
        }
        if constexpr (read_mn(MN)) {
            uint32_t dm = 0;
            if constexpr (MN == ADC || MN == SBC) {
                dm = dec_mode(c);
                if (dm == 2) return FS_EXIT;
            }
            // one LDS read from RAM or cartridge, whichever each lane's address is in
            const uint8_t* src = in_ram ? W.ram + c.ram_off + (a & 0x7F) : W.rom + rom_off(W, F.bank, a);
            fast_alu(c, MN, *src, dm);
        } else if constexpr (store_mn(MN)) {
            W.ram[c.ram_off + (a & 0x7F)] = (uint8_t)store_value<MN>(c);
        } else {
            static_assert(rmw_mn(MN), "read-modify-write");
            uint8_t* m = &W.ram[c.ram_off + (a & 0x7F)];
            *m = (uint8_t)fast_rmw(c, MN, *m);
        }
        F.pc = next;
        F.cyc += n;
        return FS_NEXT;
    } else {
        static_assert(MD == REL, "branch");
        bool taken;
        if constexpr (MN == BPL) taken = !(c.p & FN);
        else if constexpr (MN == BMI) taken = (c.p & FN) != 0;
        else if constexpr (MN == BVC) taken = !(c.p & FV);
        else if constexpr (MN == BVS) taken = (c.p & FV) != 0;
        else if constexpr (MN == BCC) taken = !(c.p & FC);
        else if constexpr (MN == BCS) taken = (c.p & FC) != 0;
        else if constexpr (MN == BNE) taken = !(c.p & FZ);
        else taken = (c.p & FZ) != 0;
        const uint32_t tgt = (next + (uint32_t)sext8(b1)) & 0xFFFF;
        const uint32_t extra = 1 + (((tgt ^ next) & 0xFF00) ? 1 : 0);
        const uint64_t tk = __builtin_amdgcn_ballot_w64(taken);
        if (tk == 0) {
            F.pc = next;
            F.cyc += N;
            return FS_NEXT;
        }
        if (tk == __builtin_amdgcn_ballot_w64(true)) {
            F.pc = tgt;
            F.cyc += N + extra;
            return FS_NEXT;
        }
        c.pc = taken ? tgt : next;            // the lanes part here
        c.cyc = F.cyc + N + (taken ? extra : 0);
        return FS_LANE;
    }
}

#define VCS_FAST_CASE(o) \
    case (o): st = fop<(o), TRACK>(c, W, F, b1, b2); break;
#define VCS_FAST_4(o) VCS_FAST_CASE(o) VCS_FAST_CASE((o) + 1) VCS_FAST_CASE((o) + 2) VCS_FAST_CASE((o) + 3)
#define VCS_FAST_16(o) VCS_FAST_4(o) VCS_FAST_4((o) + 4) VCS_FAST_4((o) + 8) VCS_FAST_4((o) + 12)
#define VCS_FAST_64(o) VCS_FAST_16(o) VCS_FAST_16((o) + 16) VCS_FAST_16((o) + 32) VCS_FAST_16((o) + 48)

// Runs instructions of the lanes in exec (one group of the hot loop, at a place
// inside the cartridge window) through the full dispatch: the one that the loop
// left, and those after it up to one that the loop runs (the way there and back
// costs about three instructions here), a place the per-lane path must take, a
// branch that parts the lanes, or, when others wait (`partial`), the next line.
// Returns how many it ran; 0: the per-lane path must execute the first.
template <bool TRACK>
__device__ __forceinline__ uint32_t run_cold(Cpu& c, const Wave& W, uint32_t partial) {
    Fast F;
    F.pc = rfl(c.pc);
    F.bank = rfl(c.bank);
    F.cyc = rfl(c.cyc);
    F.fl = rfl(c.fl);
    F.orow = (uint32_t)(rfl(c.open_row) + 1);
    F.logon = rfl(c.log != nullptr ? 1u : 0u);
    const uint32_t cap = rfl(c.cap), stop = partial ? min(cap, 76 * (F.cyc / 76 + 1)) : cap;
    uint32_t st, n = 0;
    uint32_t q = rfl(W.pre[(F.bank << 12) | (F.pc & 0xFFF)]);
    for (;;) {
        const uint32_t op = pre_op(q), b1 = (q >> 16) & 0xFF, b2 = q >> 24;
        st = FS_EXIT;
        switch (op) {
            VCS_FAST_64(0x00)
            VCS_FAST_64(0x40)
            VCS_FAST_64(0x80)
            VCS_FAST_64(0xC0)
        }
        if (st == FS_EXIT) break;
        ++n;
        if (st == FS_LANE || F.cyc >= stop || (F.pc & 0x1FFF) - 0x1000u > 0xFFCu) break;
        q = rfl(W.pre[(F.bank << 12) | (F.pc & 0xFFF)]);
        if (pre_slot(q) != HOT_REAL) break;
    }
    if (n == 0) return 0;
    if (st != FS_LANE) {                      // pc and cycle are still common to all lanes
        c.pc = F.pc;
        c.cyc = F.cyc;
    }
    c.icount += n;
    c.ucount += n;
    c.bank = F.bank;
    c.open_row = (int32_t)F.orow - 1;
    return n;
}
#undef VCS_FAST_64
#undef VCS_FAST_16
#undef VCS_FAST_4
#undef VCS_FAST_CASE

__device__ __forceinline__ uint32_t bcd_value(uint32_t b) { return 10 * (b >> 4) + (b & 15); }

// Next tile of a persistent launch (lane 0 takes it, the wave shares it).
__device__ __forceinline__ uint32_t take_tile(uint32_t* queue) {
    uint32_t t = 0;
    if (threadIdx.x == 0) t = atomicAdd(queue, 1u);
    return __builtin_amdgcn_readfirstlane(t);
}

// Orders LDS accesses between the lanes of the emulating wave (its helpers, if
// any, wait at the block's barrier meanwhile).
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Waves of a block that tracks collisions, at most: one emulates, the others
// share its scans.
constexpr int kScanWaves = 8;

// LL = envs a tile may hold (64 or 32): RAM and TIA registers get LL + 1
// slots in LDS (lanes at LL and above, always idle, share the last one), so
// narrow tiles take less LDS and more waves fit on a compute unit.
// RC = bytes of cartridge staged in LDS (8 KB), or 0: the cartridge is read
// from its HBM slot through the caches (launches with a ROM larger than 8 KB,
// which would otherwise need 32 KB of LDS per wave and cut the waves per CU
// by three).
// TRACK: collision latches tracked (TRACK_NONE has no scan code and keeps its
// registers; in TRACK_HELPERS the scan's registers are not the emulating wave's,
// so nothing spills).  NOOPS: the reset no-op
// frames of restarted envs (envs with no frames to run leave at once, the
// step counter stays); a separate instantiation, so the step's kernel keeps
// its code.  Registers for three waves per SIMD where the LDS holds as many (no
// latches; 170 were 2 too many), else for two.
template <int LL, int RC, int TRACK, bool NOOPS>
__global__ void __launch_bounds__(TRACK ? kLanes * kScanWaves : kLanes, TRACK ? 2 : 3)
    k_interp(InterpArgs A, const uint32_t* __restrict__ pre_all) {
    __shared__ uint32_t s_rom[RC ? RC / 4 + 4 : 1];
    __shared__ uint32_t s_ram[(LL + 1) * kRamStride / 4];
    __shared__ uint32_t s_tia[(LL + 1) * kTiaStride / 4];
    __shared__ CxJob s_jobs[TRACK ? kLanes : 1];
    __shared__ uint32_t s_njobs;              // jobs to scan, or 0: the block is done
    if constexpr (TRACK) {
        if (threadIdx.x >= (uint32_t)kLanes) {     // a helper wave: scans until the emulating wave is done
            for (;;) {
                __syncthreads();
                const uint32_t m = __builtin_amdgcn_readfirstlane(s_njobs);
                if (m == 0) return;
                constexpr uint32_t first = TRACK == TRACK_HELPERS ? kLanes : 0;
                cx_scan_rows(s_jobs, m, threadIdx.x - first, blockDim.x - first);
                __syncthreads();
            }
        }
    }

    const uint32_t n_tiles = *A.n_tiles;
    uint32_t tile_id = A.queue ? take_tile(A.queue) : blockIdx.x;
    while (tile_id < n_tiles) {
        const Tile& T = A.tiles[tile_id];
        const int lane = threadIdx.x;
        const int rom_id = T.rom;

        Wave W;
        if constexpr (RC > 0) {   // stage the cartridge in LDS
            const uint4* rsrc = reinterpret_cast<const uint4*>(A.roms + (size_t)rom_id * kRomSlot);
            for (int i = lane; i < RC / 16; i += kLanes) reinterpret_cast<uint4*>(s_rom)[i] = rsrc[i];
            if (lane < 4) s_rom[RC / 4 + lane] = 0;
            W.rom = reinterpret_cast<const uint8_t*>(s_rom);
        } else {
            W.rom = A.roms + (size_t)rom_id * kRomSlot;
        }
        W.ram = reinterpret_cast<uint8_t*>(s_ram);
        W.tia = reinterpret_cast<uint8_t*>(s_tia);
        W.ram_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t*)s_ram;
        W.tia_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t*)s_tia;
        W.cm = A.cmap[rom_id];
        W.pre = (PreWords)(pre_all + A.pre_off[rom_id]);
        W.track = TRACK ? 1u : 0u;

        const int env = lane < T.count ? T.env[lane] : -1;
        const int out = lane < T.count ? T.out[lane] : 0;
        bool active = env >= 0;

        Cpu c;
        c.ram_off = (lane < LL ? lane : LL) * kRamStride;
        c.tia_off = (lane < LL ? lane : LL) * kTiaStride;
        c.ptr_memo = -1;
        DevEnv* E = active ? &A.envs[env] : nullptr;
        uint64_t base_line = 0;
        uint32_t prev_action = 0, act = 0, step_idx = 0, score0 = 0, nfr = A.nframes;
        uint64_t sticky_prefix = 0;
        if (active) {
            const uint4* src = reinterpret_cast<const uint4*>(E->ram);
            for (int i = 0; i < 8; ++i) {
                const uint4 q = src[i];
                uint32_t* d = s_ram + (c.ram_off >> 2) + 4 * i;
                d[0] = q.x; d[1] = q.y; d[2] = q.z; d[3] = q.w;
            }
            const uint4 qt = reinterpret_cast<const uint4*>(E->tia)[0];
            const uint4* q2 = reinterpret_cast<const uint4*>(E->tia2);
            uint32_t* dt = s_tia + (c.tia_off >> 2);
            dt[0] = qt.x; dt[1] = qt.y; dt[2] = qt.z; dt[3] = qt.w;
            for (int i = 0; i < 2; ++i) {
                const uint4 q = q2[i];
                dt[4 + 4 * i] = q.x; dt[5 + 4 * i] = q.y; dt[6 + 4 * i] = q.z; dt[7 + 4 * i] = q.w;
            }
            dt[12] = 0;
            c.a = E->a; c.x = E->x; c.y = E->y; c.sp = E->sp; c.p = E->p;
            c.bank = E->bank | ((uint32_t)E->bank_hi << 8);
            c.xram = E->xram;
            c.vsync = E->vsync; c.hmp0 = E->hmp0; c.hmp1 = E->hmp1;
            c.tv = E->tv; c.tshift = E->tshift; c.tbase = E->tbase;
            c.pc = E->pc;
            const uint64_t cyc = E->cycle;
            base_line = cyc / 76;
            c.cyc = (uint32_t)(cyc - base_line * 76);
            c.fl = (int32_t)((int64_t)E->frame_line0 - (int64_t)base_line);
            c.hmb_line = E->hmb_now ? 0 : -1;     // the line of `cycle` is the base line
            c.cx = E->cx;
            c.cx_need = -1;
            prev_action = E->prev_action;
            step_idx = E->step_idx;
            c.err = E->err;
            act = A.actions ? A.actions[out] : 0;
            if (A.nframes_per_out) nfr = A.nframes_per_out[out];
            sticky_prefix = rng_prefix(A.seed, (uint64_t)env, kStickyPurpose);
        }
        wave_sync();
        score0 = active ? W.ram[c.ram_off + 0x50] : 0;
        c.base = base_line * 76;
        c.icount = 0;
        c.ucount = 0;
        c.slots = 0;
        c.slot = 0;
        c.log = nullptr;
        c.open_row = -1;
        c.open_cnt = 0;
        c.open_base = 0;
        c.tqm = 0;
        c.ev = 0;
        uint32_t k = 0, done = 0;
        uint32_t f = 0;
        uint32_t passes = 0;       // the wave's instruction passes (one per group instruction or opcode pass)
        uint32_t rounds = 0;       // its scheduling rounds (group formed, then scalar run or per-lane passes)

        auto begin_frame = [&]() {
            uint32_t eff = act;
            if (A.sticky_thr) {
                const uint64_t ctr = (uint64_t)step_idx * A.frameskip + f;
                if ((uint32_t)(rng_draw(sticky_prefix, ctr) >> 32) < A.sticky_thr) eff = prev_action;
            }
            prev_action = eff;
            c.swcha = (0xF0u & ~joy_pressed(eff)) | 0x0Fu;
            c.inpt4 = fire_pressed(eff) ? 0x00u : 0x80u;
            c.cap = 76u * (uint32_t)(320 + c.fl);
            const int32_t slot = A.render_all ? (int32_t)f : (int32_t)f - ((int32_t)nfr - 2);
            c.log = (A.log_enabled && slot >= 0 && slot < (int32_t)A.n_slots)
                        ? A.logs + ((size_t)out * A.n_slots + slot) * kFrameLogBytes
                        : nullptr;
            c.slot = (uint32_t)slot;
            c.log_scratch = 0;
            if (TRACK && !c.log) {                 // tracked collisions read every frame's log
                c.log = A.cx_logs + (size_t)out * kFrameLogBytes;
                c.log_scratch = 1;
            }
            c.open_row = -1;
            c.open_cnt = 0;
            c.open_base = 0;
            c.cx_row = 0;
            c.cx_x = 0;
            W.tia[c.tia_off + R_HMB] = 0;          // an earlier frame's blanked row is not this frame's
        };

        if constexpr (NOOPS) {
            if (nfr == 0) active = false;        // not restarted: nothing to run
        }
        if (active) {
            if (act >= 18) {
                c.err |= ERR_BAD_ACTION;
                done = 1;
                active = false;
            } else if (nfr == 0) {
                active = false;
            } else {
                begin_frame();
            }
        }

        const uint64_t pre_addr = (uint64_t)W.pre, rom_addr = (uint64_t)(A.roms + (size_t)rom_id * kRomSlot);
        const uint64_t table = (uint64_t)rfl((uint32_t)pre_addr) | ((uint64_t)rfl((uint32_t)(pre_addr >> 32)) << 32);
        const uint64_t rom_hbm = (uint64_t)rfl((uint32_t)rom_addr) | ((uint64_t)rfl((uint32_t)(rom_addr >> 32)) << 32);
        const uint32_t sc_end = cm_sc(W) ? 0x100u : 0u, hs_n = (W.cm.a >> 4) & 15;
        HotRom hot_rom{RC > 0 ? (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t*)s_rom : ~0u, sc_end,
                       (hs_n ? W.cm.a >> 8 : 0x1000u) - sc_end};
        if (cm_kind(W) == CART_E0) hot_rom.span = 0;
        if (cm_kind(W) == CART_3F) {
            hot_rom.first = W.cm.b & 0xFFFF;
            hot_rom.span = 1;
        }
        // ---------------------------------------------------------- main loop
        while (__any(active)) {
            uint32_t op = 0, b1 = 0, b2 = 0;
            bool want = false, ended = false;
            uint32_t end_t = 0;
            // The hot loop runs every group of lanes as far as it can, to the
            // first one at an instruction it does not run (`in`).
            const bool hot = active && (c.pc & 0x1000) && (c.pc & 0xFFF) <= 0xFFC && c.cyc < c.cap;
            const uint32_t line = c.cyc / 76;
            HotLane H;
            H.po = hot ? ((c.bank << 12) | (c.pc & 0xFFF)) << 2 : kHotNone;
            H.acc = (kAccBias + (c.cyc - 76 * line)) << kAccShift;
            H.lines = 320u + (uint32_t)c.fl - line;
            H.orow = (uint32_t)(c.open_row + 1);
            H.obase = c.open_base + kSnapArea / 4;
            H.lp = (uint64_t)c.log + 4 * (H.obase + c.open_cnt);
            H.key = ((c.pc >> 12) << 28) | (c.log ? kHotLogged : 0u) | ((uint32_t)c.fl & (kHotLogged - 1));
            uint32_t nzv = ((c.p & FN) << 1) | (((c.p >> 1) & 1) ^ 1), cf = c.p & FC, vf = c.p << 1;
            uint32_t ic = 0, hot_passes = 0, hot_rounds = 0;
            // (a timer that ran out long ago is kept in 32 bits: only the low byte of its age shows)
            const int64_t age = (int64_t)c.base - c.tbase;
            const HotTimer timer{age < (1 << 30) ? (uint32_t)age : (1u << 30) + ((uint32_t)age & 0xFF), c.tv, c.tshift};
            const uint64_t group =
                hot_wave(__builtin_amdgcn_ballot_w64(active), table, rom_hbm, H, c.a, c.x, c.y, c.p, nzv, cf, vf, c.hmp0, c.hmp1, c.vsync, c.inpt4,
                         c.swcha, ic,
                         hot_passes, hot_rounds, W.ram_lds + c.ram_off, W.tia_lds + c.tia_off, (uint64_t)c.log,
                         (uint64_t)c.xram, c.sp, timer, hot_rom);
            passes += hot_passes;
            rounds += hot_rounds;
            if (active) {
                c.p = (c.p & ~(FN | FV | FZ | FC)) | cf | ((vf >> 1) & FV) | ((nzv & 0xFF) == 0 ? FZ : 0u) |
                      ((nzv & 0x180) ? FN : 0u);
                c.icount += ic;
                c.ucount += ic;
            }
            if (hot) {
                c.pc = ((H.key >> 28) << 12) | ((H.po >> 2) & 0xFFF);
                c.bank = H.po >> 14;
                c.cyc = 76 * (320u + (uint32_t)c.fl - H.lines) + (H.acc >> kAccShift) - kAccBias;
                c.open_row = (int32_t)H.orow - 1;
                c.open_cnt = ((uint32_t)(H.lp - (uint64_t)c.log) >> 2) - H.obase;
                c.open_base = H.obase - kSnapArea / 4;
            }
            const bool in = group ? __builtin_amdgcn_inverse_ballot_w64(group) : active;
            uint32_t cold = 0;
            const uint32_t partial = __builtin_amdgcn_ballot_w64(active) != group ? 1u : 0u;
            if (group != 0 && in && hot && c.cyc < c.cap) cold = run_cold<TRACK != TRACK_NONE>(c, W, partial);
            if (__any(cold != 0)) {
                // Nothing else happens this round (no per-lane pass, no frame
                // change): the next one starts at once.
                passes += (uint32_t)__builtin_amdgcn_readlane((int)cold, (int)__builtin_ctzll(group));
                continue;
            }
            const bool go = in;
            const bool away = !((c.pc & 0x1000) && (c.pc & 0xFFF) <= 0xFFD);   // not fetched from one bank
            if constexpr (TRACK) {
                // bytes fetched from the TIA read registers show the latches
                // through the fetch cycle's pixels, 3t+2
                const bool scan = go && away && c.cyc < c.cap;
                if (__any(scan)) cx_catch_up<TRACK>(c, W, s_jobs, &s_njobs, scan, 3 * (int32_t)c.cyc + 2);
            }
            if (go) {
                if (c.cyc >= c.cap) {
                    c.err |= ERR_FRAME_CAP;
                    ended = true;
                    end_t = c.cyc - 1;
                } else {
                    const uint32_t pc = c.pc;
                    const uint32_t off = pc & 0xFFF;
                    if (!away) {
                        uint32_t v;
                        if (cm_kind(W) == CART_LINEAR) {   // the 4 KB bank is contiguous in LDS
                            const uint32_t boff = (c.bank << 12) | off;
                            const uint32_t* rw = reinterpret_cast<const uint32_t*>(W.rom);
                            const uint32_t w0 = rw[boff >> 2], w1 = rw[(boff >> 2) + 1];
                            v = __builtin_amdgcn_alignbyte(w1, w0, boff & 3);
                        } else {                          // segments: the predecoded word
                            const uint32_t q = W.pre[(c.bank << 12) | off];
                            v = pre_op(q) | ((q >> 8) & 0xFFFF00u);
                        }
                        op = v & 0xFF;
                        b1 = (v >> 8) & 0xFF;
                        b2 = (v >> 16) & 0xFF;
                    } else {
                        op = peek(c, W, pc, c.cyc);
                        b1 = peek(c, W, pc + 1, c.cyc);
                        b2 = peek(c, W, pc + 2, c.cyc);
                    }
                    want = true;
                    c.ev = 0;
                    c.tqm = 0;
                }
            }
            // one pass per distinct opcode among the lanes that fetched one.
            // The instruction is counted, and `ran_lane` set, where it
            // completes: counting after the passes under the fetch mask
            // counted more instructions than ran in waves whose lanes took
            // the undocumented RRA / ISC at different places.
            bool todo = want;
            uint32_t ran_lane = 0;
            while (__any(todo)) {
                ++passes;
                if constexpr (TRACK) {
                    const bool again = todo && c.cx_need >= 0;   // an instruction that read the latches runs again
                    if (__any(again)) {
                        cx_catch_up<TRACK>(c, W, s_jobs, &s_njobs, again, c.cx_need);
                        if (again) c.cx_need = -1;
                    }
                }
                if (todo) {
                    const uint32_t sop = __builtin_amdgcn_readfirstlane(op);
                    // an opaque scalar copy: inside the branch below the compiler
                    // would otherwise switch on the per-lane `op` (equal there)
                    uint32_t sw = sop;
                    asm volatile("" : "+s"(sw));
                    uint32_t d = kDecode.w[sw];
                    asm volatile("" : "+s"(d));
                    if (op == sop) {
                        const uint32_t sa = c.a, sx = c.x, sy = c.y, ssp = c.sp, sp_ = c.p, spc = c.pc,
                                       scy = c.cyc, sbk = c.bank;
                        exec_generic(d, c, W, b1, b2);
                        if (TRACK && c.cx_need >= 0) {   // undo; the latches are scanned before it runs again
                            c.a = sa; c.x = sx; c.y = sy; c.sp = ssp; c.p = sp_; c.pc = spc; c.cyc = scy;
                            c.bank = sbk;
                            c.tqm = 0;
                            c.ev = 0;
                        } else {
                            todo = false;
                            ran_lane = 1;
                            if (!(c.err & ERR_ILLEGAL)) c.icount++;
                            if constexpr (TRACK) c.ptr_memo = -1;
                        }
                    }
                }
            }
            if (ran_lane) {
                if (c.err & ERR_ILLEGAL) {
                    ended = true;
                    end_t = c.cyc - 1;
                } else {
                    const uint32_t t = c.ac;
                    apply_queue(c, W, t);
                    if (c.ev & EV_WSYNC) c.cyc = 76 * (t / 76 + 1);
                    if (c.ev & EV_VSYNC) {
                        ended = true;
                        end_t = t;
                    }
                }
            }
            // Every iteration moves some lane on (the earliest lane always
            // runs); if none moved, stop the wave's frames with an error
            // instead of spinning.
            if (!__any(ran_lane != 0 || ended) && active) {
                c.err |= ERR_FRAME_CAP;
                ended = true;
                end_t = c.cyc;
            }
            if constexpr (TRACK) {
                if (__any(ended)) {                // the latches take the frame's remaining rows
                    uint8_t* lg = c.log;
                    const bool close = ended && c.log;
                    if (close) {
                        log_close(c, W, end_t);
                        c.log = lg;
                    }
                    cx_scan<TRACK>(c, s_jobs, &s_njobs, close, kRows, 0);
                    if (close) c.log = nullptr;
                }
            }
            if (ended) {
                if constexpr (!TRACK) {
                    if (c.log) log_close(c, W, end_t);
                }
                c.fl = (int32_t)(end_t / 76);
                ++k;
                ++f;
                const bool term = A.early_stop && W.ram[c.ram_off + 0x51] != 0;
                if (c.err || term) {
                    done = 1;
                    active = false;
                } else if (f >= nfr) {
                    active = false;
                } else {
                    begin_frame();
                }
            }
        }

        // ---------------------------------------------------------- write back
        if (env >= 0) {
            const uint32_t* sr = s_ram + (c.ram_off >> 2);
            uint4* dst = reinterpret_cast<uint4*>(E->ram);
            for (int i = 0; i < 8; ++i) dst[i] = make_uint4(sr[4 * i], sr[4 * i + 1], sr[4 * i + 2], sr[4 * i + 3]);
            const uint32_t* st = s_tia + (c.tia_off >> 2);
            reinterpret_cast<uint4*>(E->tia)[0] = make_uint4(st[0], st[1], st[2], st[3]);
            reinterpret_cast<uint4*>(E->tia2)[0] = make_uint4(st[4], st[5], st[6], st[7]);
            reinterpret_cast<uint4*>(E->tia2)[1] = make_uint4(st[8], st[9], st[10], st[11]);
            E->hmb_now = c.hmb_line >= 0 && (uint32_t)c.hmb_line == c.cyc / 76 ? 1 : 0;
            E->cx = (uint16_t)c.cx;
            E->a = c.a; E->x = c.x; E->y = c.y; E->sp = c.sp; E->p = c.p;
            E->bank = (uint8_t)c.bank;
            E->bank_hi = (uint8_t)(c.bank >> 8);
            E->vsync = c.vsync; E->hmp0 = c.hmp0; E->hmp1 = c.hmp1;
            E->tv = c.tv; E->tshift = c.tshift; E->tbase = c.tbase;
            E->pc = c.pc;
            E->cycle = c.base + c.cyc;
            E->frame_line0 = (uint64_t)((int64_t)base_line + c.fl);
            E->instr += c.icount;
            E->prev_action = prev_action;
            E->err = c.err;
            E->step_idx = step_idx + (NOOPS ? 0u : 1u);
            StepInfo si;
            si.k = (uint8_t)k;
            si.done = (uint8_t)done;
            si.err = (uint8_t)c.err;
            si.slots = (uint8_t)c.slots;
            A.info[out] = si;
            if (A.done) A.done[out] = (uint8_t)done;
            if (A.reward) {
                const uint32_t s1 = W.ram[c.ram_off + 0x50];
                A.reward[out] = (int32_t)bcd_value(s1) - (int32_t)bcd_value(score0);
            }
            if (c.err) {
                atomicOr(&A.err_word[0], c.err);
                atomicMin(&A.err_word[1], (uint32_t)env);
            }
            if (A.instr_total) {
                atomicAdd(&A.instr_total[0], (unsigned long long)c.icount);
                atomicAdd(&A.instr_total[1], (unsigned long long)c.ucount);
            }
        }
        if (A.instr_total && lane == 0) {
            atomicAdd(&A.instr_total[2], (unsigned long long)passes);
            atomicAdd(&A.instr_total[3], (unsigned long long)rounds);
        }
        if (!A.queue) break;
        wave_sync();   // every lane is done with the LDS of this tile
        tile_id = take_tile(A.queue);
    }
    if constexpr (TRACK) {                    // the helpers leave
        s_njobs = 0;
        __syncthreads();
    }
}

// Predecoded ROM: for every virtual bank and offset, the word (pre_op) of the
// instruction that starts there, each byte read through the bank's mapping, so
// instructions that cross an E0 or 3F segment boundary decode exactly.  An
// instruction gets a hot-loop slot when the loop has a handler for what it does
// at that address (HOT_REAL otherwise) and leaves the pc inside $000-$FFC of the
// bank: it does not end past $FFC, and a branch's, jump's or call's target is
// inside.  What the address does not settle -- an index that leads elsewhere, a
// stack outside RAM -- the handler finds out and leaves.  track: collision
// latches are tracked, so a read of one needs the scan.  Entries past offset
// $FFD are never used.
__global__ void k_predecode(const uint8_t* rom, RomInfo R, uint32_t* pre, uint32_t track) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= R.n_vbanks * 4096u) return;
    const uint32_t bank = i >> 12, off = i & 0xFFF;
    const uint32_t op = rom[cart_rom_off(R, bank, 0x1000 | off)];
    const uint32_t b1 = off + 1 < 4096 ? rom[cart_rom_off(R, bank, 0x1000 | (off + 1))] : 0;
    const uint32_t b2 = off + 2 < 4096 ? rom[cart_rom_off(R, bank, 0x1000 | (off + 2))] : 0;
    const uint32_t d = kDecode.w[op];
    const uint32_t md = d & 15, len = (d >> DW_LEN) & 3, work = kHotWorkOf.w[op];
    const bool st_abs = op == 0x8C || op == 0x8D || op == 0x8E;
    uint32_t slot = HOT_REAL, cls = 0;
    if (off + len <= 0xFFC) {                          // (the hot loop loads four words from there)
        const bool st = op == 0x84 || op == 0x85 || op == 0x86;
        if (st) {
            cls = cart_store_class(R.kind, R.sc, b1);
            const uint32_t k = op == 0x85 ? 0 : op == 0x86 ? HOT_STX_TIA : HOT_STY_TIA;   // then + 1 GRP0, + 2 GRP1
            if (cls == SC_RAM) slot = kHotSlot.s[op];
            else if (cls == SC_WSYNC) slot = HOT_WSYNC;
            else if (cls == SC_IGNORE) slot = HOT_ST_NOP;
            else if (cls >= SC_TIA && cls < SC_TIAS) slot = k ? k : hot_tia_slot(cls & 0x1F);
            else if (cls >= (SC_TIAS | kScFlag0) && cls < SC_TIAG) {
                const uint32_t f = (cls & 0x1F) - kScFlag0;
                slot = op == 0x85 ? HOT_FLAG + 2 * f : (op == 0x86 ? HOT_FLAG_X : HOT_FLAG_Y) + f;
            } else if (cls >= SC_TIAS && cls < SC_TIAG) {      // an object reset
                slot = (cls & 0x1F) <= R_P1X ? HOT_RESP : HOT_RESM;
                cls = (cls & 0x1F) | ((op == 0x85 ? 0u : op == 0x86 ? 1u : 2u) << 5);
            } else if (cls == SC_3F) {
                slot = HOT_3F + (op == 0x85 ? 0 : op == 0x86 ? 1 : 2);
                cls = R.tf_mask;
            }
            else if (cls == SC_EXIT && !(R.kind == CART_3F && b1 <= 0x3F)) {   // VSYNC, motion registers
                const uint32_t reg = b1 & 0x3F, r = op == 0x85 ? 0u : op == 0x86 ? 1u : 2u;
                if (reg == 0 && r == 0) slot = HOT_VSYNC;
                else if (reg == 0x20 || reg == 0x21) slot = HOT_HMP + 2 * r + (reg & 1);
                else if (reg >= 0x22 && reg <= 0x24 && r == 0) slot = HOT_HMM + reg - 0x22;
                else if (reg == 0x2B) {
                    slot = HOT_HMCLR;
                    cls = r << 5;
                }
            }
            else if (cls == (SC_TIAG | R_GRP0)) slot = k ? k + 1 : HOT_STA_GRP0;
            else if (cls == (SC_TIAG | R_GRP1)) slot = k ? k + 2 : HOT_STA_GRP1;
        } else if ((op & 0x1F) == 0x10) {              // conditional branch
            const uint32_t next = off + 2, t = next + (uint32_t)(int32_t)(int8_t)b1;
            const uint32_t k = op >> 5;
            const uint32_t cross = HOT_BPL_X + k;
            if (t <= 0xFFC) slot = ((t ^ next) & 0xF00) ? cross : kHotSlot.s[op];
        } else if (op == 0x4C || op == 0x20) {         // JMP, JSR: the target's window
            const uint32_t t = (b1 | (b2 << 8)) & 0x1FFF;
            if (t - 0x1000u <= 0xFFCu) slot = op == 0x4C ? kHotSlot.s[op] : HOT_JSR;
        } else if (md == ABS && st_abs) {
            const uint32_t a = (b1 | (b2 << 8)) & 0x1FFF, r = op == 0x8D ? 0u : op == 0x8E ? 1u : 2u;
            cls = cart_store_class(R.kind, R.sc, a);
            if (cls == SC_RAM) slot = HOT_STA_A + r;
            else if (cls >= SC_TIA && cls < SC_TIAS) slot = HOT_A_TIA + 3 * r;
            else if (cls == (SC_TIAG | R_GRP0)) slot = HOT_A_TIA + 3 * r + 1;
            else if (cls == (SC_TIAG | R_GRP1)) slot = HOT_A_TIA + 3 * r + 2;
            else if (cls == SC_XRAM) {
                if (!(a & 0x80) && op == 0x8D) slot = HOT_XW;
            } else if ((a & 0x1000) && R.kind == CART_LINEAR) {
                const uint32_t to = cart_hotspot(R.kind, R.hs_first, R.hs_n, 8, a);
                if (to < 8) {
                    slot = HOT_HS_ST;
                    cls = to | (r << 5);
                }
            }
        } else if (md == ABS && work > HW_SBC && work <= HW_INC) {
            cls = work;
            if (((b1 | (b2 << 8)) & 0x1280) == 0x0080) slot = HOT_A_RMW;
        } else if (md == ABS && work <= HW_SBC) {
            const uint32_t a = (b1 | (b2 << 8)) & 0x1FFF;
            cls = work;
            if ((a & 0x1000) && R.sc && !(a & 0xF00)) {    // Superchip RAM: reads of the read port
                if (a & 0x80)
                    slot = op == 0xAD ? HOT_XR_LDA : op == 0x6D ? HOT_XR_ADC : op == 0x2D ? HOT_XR_AND
                         : op == 0x4D ? HOT_XR_EOR : op == 0x0D ? HOT_XR_ORA : HOT_REAL;
            } else if (a & 0x1000) {
                if (R.kind == CART_LINEAR) {
                    const uint32_t to = cart_hotspot(R.kind, R.hs_first, R.hs_n, 8, a);
                    if (to >= 8) slot = op == 0xAD ? HOT_ABS : HOT_A_ROM;
                    else if (op == 0xAD) {
                        slot = HOT_HS;
                        cls = to;
                    }
                } else if (R.kind == CART_E0 && op == 0xAD && (a & 0xFFF) - 0xFE0u < 24u) {
                    slot = HOT_E0;
                } else if (cart_hotspot(R.kind, R.hs_first, R.hs_n, bank, a) == bank &&
                           !(R.kind == CART_E0 && (a & 0xFFF) >= 0xFE0)) {
                    slot = HOT_SEG;
                }
            } else if (!(a & 0x80)) {                      // TIA
                if ((a & 0xF) != 0xC && ((a & 0xF) >= 8 || !track)) {
                    slot = HOT_A_CONST;
                    cls |= (a & 0xF) == 0xD ? 1u << 5 : 0u;
                }
            } else if (!(a & 0x200)) {
                slot = HOT_A_RAM;
            } else if (!(a & 4)) {                         // the ports
                if ((a & 3) == 0) slot = op == 0xAD ? HOT_SWCHA_LDA : op == 0x4D ? HOT_SWCHA_EOR : HOT_A_SWCHA;
                else slot = HOT_A_CONST;
                if ((a & 3) == 2) cls |= 2u << 5;
            } else if (!(a & 1)) {
                slot = HOT_A_INTIM;
            }
        } else if (md == ZP && work <= HW_SBC && b1 < 0x80) {  // a TIA read
            cls = work;
            if ((b1 & 0xF) == 0xC) {
                slot = op == 0xA5 ? HOT_INPT4 : HOT_Z_INPT4;
            } else if ((b1 & 0xF) >= 8 || !track) {
                slot = HOT_Z_CONST;
                cls |= (b1 & 0xF) == 0xD ? 1u << 5 : 0u;
            }
        } else if (md == ZPX || md == ZPY) {
            cls = work;
            if (work <= HW_SBC) slot = md == ZPX ? HOT_ZX : HOT_ZY;
            else if (work <= HW_INC && md == ZPX) slot = HOT_ZX_RMW;
            else slot = op == 0x95 ? HOT_STA_ZX : op == 0x94 ? HOT_STY_ZX : op == 0x96 ? HOT_STX_ZY : HOT_REAL;
        } else if (md == ABX || md == ABY) {
            const uint32_t base = (b1 | (b2 << 8)) & 0x1FFF;
            cls = work;
            if (base >= 0x80 && base <= 0xFF) {            // RAM, as far as the index leaves it there
                if (work <= HW_SBC) slot = md == ABX ? HOT_AX_RAM : HOT_AY_RAM;
                else slot = op == 0x9D ? HOT_STA_AX : op == 0x99 ? HOT_STA_AY : HOT_REAL;
            } else if ((base & 0x1000) && work <= HW_SBC) {
                if (R.kind == CART_LINEAR) slot = md == ABX ? HOT_AX_ROM : HOT_AY_ROM;
                else slot = md == ABX ? HOT_SEG_X : HOT_SEG_Y;
            }
        } else if (md == IZY && R.kind == CART_LINEAR && work <= HW_SBC && b1 >= 0x80 && b1 < 0xFF) {
            slot = HOT_IY_ROM;
            cls = work;
        } else if (op == 0x08 || op == 0x28) {
            slot = op == 0x08 ? HOT_PHP : HOT_PLP;
        } else if (md == IMP || md == ACC || md == IMM || (md == ZP && b1 >= 0x80)) {
            slot = kHotSlot.s[op];
        }
    }
    const uint32_t low = slot == HOT_REAL ? (op & 0x7F) | ((op & 0x80) << 8) : cls;
    pre[i] = low | (slot << 7) | (b1 << 16) | (b2 << 24);
}

void launch_predecode(const uint8_t* rom, const RomInfo& info, uint32_t* pre, uint32_t track, hipStream_t s) {
    const uint32_t n = info.n_vbanks * 4096u;
    hipLaunchKernelGGL(k_predecode, dim3((n + 255) / 256), dim3(256), 0, s, rom, info, pre, track);
}

// Waves per block of a launch that tracks collisions: as many as the chip can
// hold at once for that many tiles.
static int scan_waves(uint32_t tiles) {
    return tiles <= 256 ? 8 : (tiles <= 512 ? 4 : (tiles <= 1024 ? 2 : 1));
}

template <int TRACK, bool NOOPS>
static void launch_interp_t(const InterpArgs& a, uint32_t grid, uint32_t tile_envs, uint32_t rom_lds, hipStream_t s) {
    const dim3 block(TRACK ? kLanes * scan_waves(grid) : kLanes);
    if (rom_lds == 0) {
        if (tile_envs <= 32)
            hipLaunchKernelGGL((k_interp<32, 0, TRACK, NOOPS>), dim3(grid), block, 0, s, a, a.pre);
        else
            hipLaunchKernelGGL((k_interp<64, 0, TRACK, NOOPS>), dim3(grid), block, 0, s, a, a.pre);
    } else if (tile_envs <= 32) {
        hipLaunchKernelGGL((k_interp<32, 8192, TRACK, NOOPS>), dim3(grid), block, 0, s, a, a.pre);
    } else {
        hipLaunchKernelGGL((k_interp<64, 8192, TRACK, NOOPS>), dim3(grid), block, 0, s, a, a.pre);
    }
}

template <int TRACK>
static void launch_interp_n(const InterpArgs& a, uint32_t grid, uint32_t tile_envs, uint32_t rom_lds, hipStream_t s) {
    if (a.count_step) launch_interp_t<TRACK, false>(a, grid, tile_envs, rom_lds, s);
    else launch_interp_t<TRACK, true>(a, grid, tile_envs, rom_lds, s);
}

// With 8 waves the helpers alone scan: the emulating wave is one of eight, and
// without the scan's call it spills nothing.  With fewer, its share is worth
// more.  Steps of 4,096 / 16,384 / 24,576 / 49,152 envs with objects (8, 8, 4, 2
// waves), ms, helpers alone against every wave: 2.07 / 2.09, 3.71 / 3.76, 5.19 /
// 5.10, 9.93 / 9.32.
void launch_interp(const InterpArgs& a, uint32_t grid, uint32_t tile_envs, uint32_t rom_lds, hipStream_t s) {
    if (!a.track) launch_interp_n<TRACK_NONE>(a, grid, tile_envs, rom_lds, s);
    else if (scan_waves(grid) == kScanWaves) launch_interp_n<TRACK_HELPERS>(a, grid, tile_envs, rom_lds, s);
    else launch_interp_n<TRACK_ALL>(a, grid, tile_envs, rom_lds, s);
}

}  // namespace vcs
