"""Collision scans shared by the waves of a block: a launch of more tiles has
fewer waves per block (8 up to 256 tiles, 4 up to 512, 2 up to 1,024, then 1),
and whatever their number, and with blocks that take tile after tile, a step's
outputs and states are the same byte for byte."""
import numpy as np
import pytest
import torch

from paper_1907_08467_amd.env import VcsEnv
from paper_1907_08467_amd.inputs.palette import GRAY
from test_gpu_tia import decode, objects_roms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,width,workers", [
    (4112, 16, 0),       # 4 waves (257 tiles) and, 64 wide, 8
    (8208, 16, 0),       # 2 and 8
    (16400, 16, 0),      # 1 and 4
    (1000, 16, 3),       # 3 blocks of 8 waves over all tiles
    (33, 32, 0),
    (1, 64, 0),
])
def test_scan_waves_agree(n, width, workers):
    print(f"case: collision scans, {n} envs in tiles of {width}, workers {workers}", flush=True)
    roms = objects_roms()
    env_rom = (np.arange(n) % len(roms)).astype(np.uint16)
    cfg = dict(seed=77, frameskip=4, render_mode=1, collisions=True)
    a, b = VcsEnv(roms, env_rom, GRAY, **cfg), VcsEnv(roms, env_rom, GRAY, **cfg)
    b.set_launch(width, workers, 256)
    rng = np.random.default_rng(n)
    for s in range(6):
        acts = torch.from_numpy(rng.integers(0, 18, n).astype(np.uint8)).cuda()
        ra, rb = a.step(acts), b.step(acts)
        torch.cuda.synchronize()
        for x, y in zip(ra[:3], rb[:3]):
            assert torch.equal(x, y), f"step {s}"
        for e in {0, n // 3, n // 2, n - 1}:
            sa, sb = a.get_state(int(e)), b.get_state(int(e))
            assert np.array_equal(sa, sb), f"step {s} env {e}"
    # the players met (the cartridges count it in RAM and clear the latches)
    hits = [int(decode(a.get_state(e))["ram"][0x56]) for e in range(min(n, 64))]
    assert sum(hits) > 0 or n == 1
    assert a.poll_errors() == b.poll_errors()
    a.close()
    b.close()
