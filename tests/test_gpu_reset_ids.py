"""A reset of listed envs validates the ids itself, before an env is touched:
negative, too large and repeated ones are refused."""
import numpy as np
import pytest
import torch

from paper_1907_08467_amd.inputs.romgen import RomSpec, generate
from parity import compare_states, make_pair, step_both

pytestmark = pytest.mark.gpu


def test_bad_and_repeated_ids():
    n = 12
    print(f"case: reset of listed ids, some refused, {n} envs", flush=True)
    rom = generate(RomSpec(1000))
    o, g = make_pair([(rom.data, rom.scheme)], np.zeros(n, np.uint16), seed=21)
    rng = np.random.default_rng(2)
    for s in range(3):
        step_both(o, g, rng.integers(0, 18, n), tag=f"step {s}")
    assert g.poll_errors()[1] == 0
    ids = [5, -1, 7, 5, n, 9, 2**31 - 1, -2**31]
    refused = {1, 4, 6, 7}
    for again in range(2):                     # the same ids again: another call's claim
        obs = g.reset(torch.tensor(ids, dtype=torch.int32, device="cuda")).cpu().numpy()
        want = o.reset(np.array([5, 7, 9], np.int32))
        assert all(not obs[i].any() for i in refused)
        assert np.array_equal(obs[2], want[1]) and np.array_equal(obs[5], want[2])
        served = [i for i in (0, 3) if np.array_equal(obs[i], want[0])]
        assert len(served) == 1 and want[0].any() and not obs[3 - served[0]].any()
        compare_states(o, g, range(n), f"reset {again}")      # (each episode advanced once, the others not at all)
        first, bits = g.poll_errors()
        assert bits == 8 and first == 5        # the refused repeat is the smallest valid id named
    step_both(o, g, rng.integers(0, 18, n), want_frames=True, tag="after")
    compare_states(o, g, range(n), "after")
    g.close()
    o.close()
