"""Small cartridges made of what games use besides zero-page loads and stores:
timer waits, tables read by index or through pointers, routines and the stack,
indexed RAM, port reads, object resets, decimal scores.  Each frame waits on
INTIM through the vertical blank and the overscan, and draws 180 lines of
`body` (X: the line), so all envs of one cartridge stay in lockstep unless
`body` looks at the joystick.
"""
import random

from helpers import cart

HEAD = """
reset:
    ldx #$FF
    txs
    cld
    lda #0
    sta VBLANK
frame:
    lda #2
    sta VSYNC
    sta WSYNC
    sta WSYNC
    lda #0
    sta VSYNC
    inc $80
"""
# tables at $1E00; the routine that calls go to; a pointer to the tables at $F0
TAIL = """
    .org $1C00
sub:
    inc $8A
    lda $8A
    sta COLUBK
    rts
sub2:
    pha
    txa
    pha
    lda tab,x
    sta GRP1
    pla
    tax
    pla
    rts
    .org $1E00
tab:
"""
TAIL += "".join(f"    .byte {(i * 37 + 11) & 0xFF}\n" for i in range(448))


def waiting(body, vblank="", overscan="", before=""):
    """A frame that waits for its blanks on the timer and draws `body` on 180 lines."""
    return HEAD + f"""
    lda #<tab
    sta $F0
    lda #>tab
    sta $F1
    lda #40
    sta TIM64T
{vblank}
w1:
    lda INTIM
    bne w1
{before}
    ldx #180
ln:
{body}
    sta WSYNC
    dex
    beq lo
    jmp ln
lo:
    lda #28
    sta TIM64T
{overscan}
w2:
    lda INTIM
    bne w2
    jmp frame
""" + TAIL


def plain(body, n=230):
    """A frame without the timer: n lines of `body`, each ended by WSYNC."""
    return HEAD + f"""
    lda #<tab
    sta $F0
    lda #>tab
    sta $F1
    ldx #{n}
ln:
{body}
    sta WSYNC
    dex
    beq lo
    jmp ln
lo:
    jmp frame
""" + TAIL


def filler(n):
    """n instructions that the hot loop has always run."""
    ops = ["lda $80", "eor $81", "sta $82", "and #$3C", "iny", "sta $83", "lda $82", "clc", "adc $83", "sta $84"]
    return "".join(f"    {ops[i % len(ops)]}\n" for i in range(n))


SRC = {
    # the blanks only: two instructions in turn
    "timer": waiting(filler(6)),
    # sprites and playfield out of tables
    "tables": plain("    lda tab,x\n    sta GRP0\n    ldy tab+20,x\n    lda tab+32,y\n    sta GRP1\n"
                    "    lda tab+180,x\n    sta PF1\n    ldy $80\n    lda tab,y\n    sta COLUBK\n"),
    "pointers": plain("    ldy #3\n    lda ($F0),y\n    sta GRP0\n    iny\n    lda ($F0),y\n    sta GRP1\n"
                      "    lda $80\n    sta COLUBK\n"),
    # a routine per line, and one that saves registers
    "calls": plain("    jsr sub\n    jsr sub2\n    lda $8A\n    sta COLUPF\n"),
    "stack": plain("    lda $80\n    pha\n    txa\n    pha\n    tsx\n    stx $88\n    pla\n    tax\n    pla\n"
                   "    sta COLUBK\n    php\n    pla\n    sta $89\n"),
    "ram": plain("    stx $90\n    txa\n    and #$1F\n    tay\n    ldx $90\n    lda $80,x\n    txa\n    lsr\n    tax\n"
                 "    lda $A0\n    sta $94\n    ldx #5\n    lda $90,x\n    sta $98,x\n    inc $98,x\n    lda $98,x\n"
                 "    ldy $9A,x\n    sty COLUBK\n    ldx $90\n"),
    "resets": plain("    lda $80\n    sta RESP0\n    sta COLUBK\n    sta RESM0\n    sta RESBL\n    sta $8B\n"
                    "    sta RESP1\n"),
    "motion": plain("    lda $80\n    sta HMP0\n    sta HMM0\n    stx HMP1\n    sta HMBL\n    sty COLUBK\n    sta HMM1\n    cpx #90\n"
                    "    bcs mo\n    stx HMCLR\n    sta HMM1\nmo:\n"),
    "decimal": plain("    sed\n    clc\n    lda $8C\n    adc #$19\n    sta $8C\n    lda $8D\n    adc $8C\n    sta $8D\n"
                     "    sec\n    sbc #$07\n    sta COLUBK\n    cld\n"),
    "ports": plain("    lda SWCHB\n    and #$08\n    sta $8E\n    bit INPT4\n    bpl po\n    inc $8F\npo:\n"
                   "    lda $8F\n    cmp tab\n    ldy tab+3\n    sty COLUBK\n    bit SWCHA\n    lda $08\n    sta $86\n"),
    # one call among many plain instructions
    "rare": plain(filler(11) + "    jsr nothing\n", 230).replace("sub:\n", "nothing:\n    rts\nsub:\n"),
    # instructions no handler is meant for, among plain ones and back to back
    "seldom": plain("    lda $80\n    asl.w $0082\n    sta $83\n    lda $84\n    cpx.w tab\n    sta $85\n    ora tab,x\n"
                    "    eor tab+7,x\n    asl $87,x\n    cmp $82\n"),
    # absolute stores to TIA registers, and other forms of what the loop runs
    "absolute": plain("    lda.w $0080\n    sta.w COLUBK\n    ldy.w $0081\n    sty.w GRP0\n    stx.w GRP1\n    php\n    asl.w $0082\n"
                      "    plp\n    rol.w $0082\n    stx.w COLUPF\n    sta.w $0084\n    sty.w PF1\n"),
    # next to nothing but instructions without a handler
    "cold": plain("    inc COLUBK\n    asl $87,x\n    asl.w $0207\n    nop.w $1000\n    stx.w AUDV0\n    inc tab,x\n"
                  "    sta.w AUDF0\n    sty.w AUDF1\n    sta tab\n"),
    # a bit of everything, as a game's frame has it
    "game": waiting("    lda tab,x\n    sta GRP0\n    cpx $80\n    bcc nb\n    lda #2\n    sta ENABL\nnb:\n"
                    "    lda ($F0),y\n    sta PF2\n    lda tab+64,x\n    sta COLUPF\n",
                    vblank="    jsr sub\n    jsr sub2\n    lda SWCHA\n    and #$10\n    bne v1\n    inc $91\nv1:\n    lda $91\n"
                           "    and #7\n    tax\n    lda tab,x\n    sta $92\n    sed\n    clc\n    lda $93\n    adc #1\n    sta $93\n"
                           "    cld\n    lda #$20\n    sta HMP0\n    sta HMM0\n    sta HMBL\n    sta WSYNC\n    sta HMOVE\n    sta WSYNC\n    sty HMCLR\n    sta HMM1\n    sta RESP0\n"
                           "    lda $94,x\n    sta $96,x\n    ldy #9\n",
                    overscan="    lda INPT4\n    bmi o1\n    jsr sub\no1:\n    lda CXP0FB\n    sta $98\n    sta CXCLR\n    dec $99\n"),
}


def rom(name):
    return cart(SRC[name])[0]


# ---- random frames of the same instructions, branching on the joystick
_TIA = ["COLUBK", "COLUPF", "COLUP0", "GRP0", "GRP1", "PF0", "PF1", "PF2", "ENAM0", "ENAM1", "ENABL", "NUSIZ0", "CTRLPF",
        "REFP0", "VDELP0", "VDELBL", "HMP0", "HMP1", "HMM0", "HMM1", "HMBL", "RESP0", "RESP1", "RESM0", "RESBL", "HMCLR",
        "AUDV0"]
_ALU = ["lda", "and", "ora", "eor", "cmp", "adc", "sbc"]
_READ = _ALU + ["ldx", "ldy", "cpx", "cpy", "bit"]
_RMW = ["inc", "dec", "asl", "lsr", "rol", "ror"]


def _random_body(r, k):
    def ram():
        return f"${r.randint(0x80, 0xBF):02X}"

    def store():
        return r.choice(["sta", "stx", "sty"])

    out = []
    for i in range(r.randint(6, 16)):
        out += r.choice([
            lambda: [f"{r.choice(_READ)} {ram()}"],
            lambda: [f"{r.choice(_READ)}.w $00{r.randint(0x80, 0xBF):02X}"],
            lambda: [f"{r.choice(_READ)} tab+{r.randint(0, 200)}"],
            lambda: [f"{r.choice(_ALU + ['ldy'])} tab+{r.randint(0, 190)},x"],
            lambda: [f"{r.choice(_ALU + ['ldx'])} tab+{r.randint(0, 190)},y"],
            lambda: [f"{r.choice(_ALU)} ($F0),y"],
            lambda: [f"ldx #{r.randint(0, 40)}", f"{r.choice(_ALU + _RMW + ['ldy', 'sta', 'sty'])} ${r.randint(0x80, 0xA0):02X},x"],
            lambda: [f"ldy #{r.randint(0, 40)}", f"{r.choice(_ALU + ['sta'])}.w $00{r.randint(0x80, 0xA0):02X},y"],
            lambda: [f"{store()}{r.choice(['', '', '.w'])} {r.choice(_TIA)}"],
            lambda: [f"{store()}{r.choice(['', '.w'])} $0090"],
            lambda: [r.choice(["jsr sub", "jsr sub2"])],
            lambda: [r.choice(["pha", "php"]), r.choice(["inx", "iny", "clc"]), r.choice(["pla", "plp"])],
            lambda: [r.choice(["sed", "cld", "sec", "clc", "clv", "tsx", "tya", "txa", "tax", "tay", "asl", "ror"])],
            lambda: [f"{r.choice(['adc', 'sbc'])} #{r.randint(0, 255)}"],
            lambda: [f"{r.choice(_ALU + ['bit'])} {r.choice(['SWCHA', 'SWCHB', 'INTIM', 'INPT4', 'TIMINT', '$0D', '$03'])}"],
            lambda: [f"{r.choice(_RMW)}{r.choice(['', '.w'])} $00{r.randint(0x80, 0xBF):02X}"],
            lambda: [f"lda {r.choice(['INPT4', 'SWCHA'])}", r.choice(["asl", "lsr", "nop"]),
                     f"{r.choice(['bpl', 'bmi', 'bcc', 'bcs'])} q{k}_{i}", f"inc {ram()}", r.choice(["nop", "jsr sub"]),
                     f"sta {r.choice(_TIA)}", f"q{k}_{i}:"],
            lambda: [r.choice(["sta HMOVE", "sta TIM8T", "sta WSYNC", f"lda ({ram()}),y", "dey", "nop"])],
        ])()
    return "".join((l if l.endswith(":") else "    " + l) + "\n" for l in out)


def random_rom(seed):
    """Loops of such bodies, some of them a line each, and lines to the frame's end."""
    r = random.Random(seed)
    src = HEAD + ("    lda #<tab\n    sta $F0\n    lda #>tab\n    sta $F1\n    ldx #$E8\n    txs\n    cld\n"
                  "    lda #44\n    sta TIM64T\n")
    for k in range(r.randint(2, 4)):
        src += f"    lda #{r.randint(10, 40)}\n    sta $C{k}\nL{k}:\n" + _random_body(r, k)
        src += ("    sta WSYNC\n" if r.random() < 0.75 else "") + f"    dec $C{k}\n    beq E{k}\n    jmp L{k}\nE{k}:\n"
    return cart(src + "    jmp frame\n" + TAIL)[0]
