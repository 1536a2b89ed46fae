"""Cartridges made of what games use (gamecarts.py) against the oracle, and how
often the interpreter has to leave its hot loop on them: an instruction that
the loop left one at a time cost as much as a dozen that it ran."""
import numpy as np
import pytest

import gamecarts
from paper_1907_08467_amd.inputs.romgen import RomSpec, generate
from parity import make_pair, step_both
from test_gpu_tia import compare_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", list(gamecarts.SRC))
@pytest.mark.parametrize("n,mode,collisions,big", [(70, 0, False, False), (5, 1, False, True), (3, 1, True, False)])
def test_against_the_oracle(name, n, mode, collisions, big):
    """`big`: another env of a 32 KB cartridge, so that cartridges are read from HBM."""
    print(f"case: game cartridge {name}, {n} envs, render mode {mode}, collisions {collisions}, big {big}", flush=True)
    roms, env_rom = [(gamecarts.rom(name), 0)], np.zeros(n, np.uint16)
    if big:
        f4 = generate(RomSpec(6003, "f4", True))
        roms.append((f4.data, f4.scheme))
        env_rom[-1] = 1
    o, g = make_pair(roms, env_rom, seed=8, frameskip=3, render_mode=mode, collisions=collisions)
    rng = np.random.default_rng(n)
    for s in range(5):
        step_both(o, g, rng.integers(0, 18, n), want_frames=True, tag=f"{name} step {s}")
        compare_all(o, g, n, f"{name} step {s}")
    assert g.poll_errors() == o.poll_errors()
    g.close()
    o.close()


@pytest.mark.parametrize("seed", range(1, 17))
def test_random_frames(seed):
    """The same instructions in random order; envs part on their joysticks and meet again."""
    n, collisions = (70, 5, 64, 33)[seed % 4], seed % 3 == 0
    print(f"case: random game cartridge {seed}, {n} envs, collisions {collisions}", flush=True)
    o, g = make_pair([(gamecarts.random_rom(seed), 0)], np.zeros(n, np.uint16), seed=seed, frameskip=3,
                     render_mode=seed % 2, collisions=collisions)
    rng = np.random.default_rng(seed)
    for s in range(5):
        step_both(o, g, rng.integers(0, 18, n), want_frames=True, tag=f"{seed} step {s}")
    compare_all(o, g, n, f"random {seed}")
    assert g.poll_errors() == o.poll_errors()
    g.close()
    o.close()


@pytest.mark.parametrize("name", ["timer", "tables", "pointers", "calls", "resets", "motion", "decimal", "rare", "stack",
                                  "absolute"])
def test_the_hot_loop_is_not_left(name):
    """Envs of these run in lockstep: what is left to the other paths is a few
    instructions of each frame, whatever its lines are made of."""
    print(f"case: game cartridge {name}, rounds", flush=True)
    n, frames = 64, 4
    o, g = make_pair([(gamecarts.rom(name), 0)], np.zeros(n, np.uint16), seed=8, frameskip=frames, render_mode=1)
    for s in range(3):
        step_both(o, g, np.zeros(n, np.uint8), tag=f"{name} step {s}")
    instr, uniform, passes, rounds = g.last_step_counts()
    assert passes > 180 * frames and uniform > 0.99 * instr
    assert rounds <= 16 * frames, f"{rounds} rounds for {passes} passes"
    g.close()
    o.close()
