"""Frame stack pushes from and into buffers that are not 16-byte aligned (moved
in 4-byte words) equal the aligned ones (16-byte words) and the oracle, at the
depths where the loads go in one, two or many groups."""
import numpy as np
import pytest
import torch

from oracle.stack import FrameStack as OracleStack
from paper_1907_08467_amd.env import FrameStack
from test_gpu_policy import env_for

pytestmark = pytest.mark.gpu


def shifted(n_bytes, by):
    return torch.zeros(n_bytes + 16, dtype=torch.uint8, device="cuda")[by:by + n_bytes]


@pytest.mark.parametrize("depth", [1, 2, 4, 5, 7, 16])
@pytest.mark.parametrize("bits", [8, 4])
def test_stack_alignment(depth, bits):
    print(f"case: stack alignment, depth {depth} bits {bits}", flush=True)
    n = 9
    g = env_for(n)
    oracle, a = OracleStack(n, depth=depth, bits=bits), FrameStack(g, depth, bits)
    others = [(FrameStack(g, depth, bits), ob, ot) for ob, ot in ((4, 0), (0, 4), (8, 12))]
    rng = np.random.default_rng(depth * 10 + bits)
    for s in range(depth + 3):
        obs = rng.integers(0, 256, (n, 84, 84)).astype(np.uint8)
        done = (rng.random(n) < 0.2).astype(np.uint8)
        d, dn = torch.from_numpy(obs).cuda(), torch.from_numpy(done).cuda()
        want = oracle.push(obs, done)
        assert np.array_equal(a.push(d, dn).cpu().numpy(), want), f"push {s}"
        for fs, ob, ot in others:
            src = shifted(d.numel(), ob).view(n, 84, 84)
            src.copy_(d)
            out = shifted(n * depth * 7056, ot).view(n, depth, 84, 84)
            fs.push(src, dn, out=out)
            assert np.array_equal(out.cpu().numpy(), want), f"push {s}, buffers at {ob} and {ot}"
    for fs, _, _ in others:
        fs.close()
    a.close()
