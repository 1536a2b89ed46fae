"""The interpreter's hot loop at its edges, against the oracle: frames, rewards
and states of small cartridges whose envs run in lockstep, part by their
joysticks and meet again."""
import numpy as np
import pytest

from helpers import cart
from parity import make_pair, step_both
from test_gpu_tia import compare_all

pytestmark = pytest.mark.gpu

HEAD = """
reset:
    ldx #$FF
    txs
    cld
    lda #0
    sta VBLANK
"""
FRAME = """
frame:
    lda #2
    sta VSYNC
    lda #0
    sta VSYNC
    inc $80
"""


def lines(body, n=100, label="ln"):
    """n lines of `body`, each ended by WSYNC."""
    return f"    ldx #{n}\n{label}:\n{body}\n    sta WSYNC\n    dex\n    bne {label}\n"


def dense(n):
    regs = ["COLUBK", "COLUPF", "PF1", "GRP0", "GRP1", "ENAM0", "PF2", "COLUP0", "ENABL"]
    return HEAD + FRAME + lines("    lda $80\n    eor $81\n" + "".join(f"    sta {regs[i % 9]}\n" for i in range(n)), 90) + \
        "    inc $81\n    jmp frame\n"


def wsync_at(k):
    """WSYNC and a colour write around the end of a line: k cycles of filler."""
    fill = "    nop\n" * (k // 2) if k % 2 == 0 else "    lda $80\n" + "    nop\n" * ((k - 3) // 2)
    return HEAD + FRAME + lines(fill + "    sty COLUBK\n    stx COLUBK\n    iny", 60) + "    jmp frame\n"


def overflow():
    """Lines that run over without WSYNC, a loop across many lines, colours on the way."""
    return HEAD + FRAME + """
    ldy #200
ov:
    sty COLUBK
    lda $80
    adc #3
    sta $80
    stx PF0
    inx
    stx GRP1
    dey
    bne ov
    jmp frame
"""


def paging():
    """Branches and indexed reads across a page, both taken and not."""
    return HEAD + FRAME + """
    ldx #40
pg:
    ldy #0
    lda $80
    lsr
    bcs odd
    jmp even
odd:
    jmp near
    .org $10F8
even:
    iny
    cpy #5
    bne over
    jmp out
near:
    iny
    nop
over:
    lda $10F0,y
    sta COLUBK
    lda $10FD,x
    sta COLUPF
    cpy #5
    bne even
out:
    sta WSYNC
    dex
    beq done
    jmp pg
done:
    jmp frame
"""


def decimal():
    return HEAD + FRAME + """
    ldx #60
dc:
    sed
    clc
    lda $82
    adc $80
    sta $82
    sta COLUBK
    sec
    lda $83
    sbc $82
    sta $83
    cld
    sta PF1
    php
    pla
    sta PF2
    bvs dv
    inc $84
dv:
    asl $82
    ror $83
    rol $84
    lsr $85
    bit $82
    bmi dm
    dec $85
dm:
    sta WSYNC
    dex
    bne dc
    jmp frame
"""


def parting():
    """Paths of different lengths by joystick and button, calls, and a meeting at WSYNC or without one."""
    return HEAD + FRAME + """
    ldx #70
pt:
    lda INPT4
    bmi nofire
    jsr sub
    sta COLUBK
nofire:
    lda SWCHA
    asl
    bcs noright
    inc $86
    inc $86
    lda $86
    sta COLUPF
noright:
    asl
    bcs noleft
    ldy #3
pl:
    dey
    bne pl
    sty PF0
noleft:
    asl
    bcs nodown
    sta RESP0
    sta HMP0
nodown:
    cpx #20
    bcc nosync
    sta WSYNC
nosync:
    lda $86
    sta GRP0
    dex
    bne pt
    sta HMOVE
    jmp frame
sub:
    lda #1
    sta VDELP0
    inc $87
    lda $87
    sta GRP1
    rts
"""


CASES = [(f"dense{n}", dense(n)) for n in (7, 8, 9, 16, 18)] + \
        [(f"wsync{k}", wsync_at(k)) for k in (40, 54, 55, 56, 57, 58, 59, 60, 61, 62)] + \
        [("overflow", overflow()), ("paging", paging()), ("decimal", decimal()), ("parting", parting())]


@pytest.mark.parametrize("name,src", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("n,mode", [(70, 0), (3, 1)])
def test_hot_loop(name, src, n, mode):
    print(f"case: hot loop {name}, {n} envs, render mode {mode}", flush=True)
    rom = cart(src)[0]
    o, g = make_pair([(rom, 0)], np.zeros(n, np.uint16), seed=4, frameskip=4, render_mode=mode)
    rng = np.random.default_rng(n)
    for s in range(5):
        step_both(o, g, rng.integers(0, 18, n), want_frames=True, tag=f"{name} step {s}")
        compare_all(o, g, n, f"{name} step {s}")
    assert g.poll_errors() == o.poll_errors()
    g.close()
    o.close()
