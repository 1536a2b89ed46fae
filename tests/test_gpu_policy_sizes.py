"""The policy's blockings, at the batch sizes where the choice between them
changes: every env's logits and action are bit for bit those of the same env in
a small batch (the order of each sum does not depend on the blocking), and the
action is the first maximal logit, with infinities and NaN as in a scan."""
import numpy as np
import pytest
import torch

from paper_1907_08467_amd.env import Policy
from paper_1907_08467_amd.inputs.policy_weights import policy_weights
from test_gpu_policy import check_outputs, env_for, make_policy
from oracle.policy import forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [15, 16, 17, 252, 253, 417, 418, 1280, 1281])
def test_policy_blockings_agree(n):
    print(f"case: policy blockings, {n} envs", flush=True)
    g = env_for(n)
    layers = policy_weights(11)
    P = make_policy(g, layers)
    stack = np.random.default_rng(n).integers(0, 256, (n, 4, 84, 84)).astype(np.uint8)
    d = torch.from_numpy(stack).cuda()
    act, lg = P.act(d, want_logits=True)
    act, lg = act.cpu().numpy(), lg.cpu().numpy()
    for i in range(0, n, 13):
        a, l = P.act(d[i:i + 13].contiguous(), want_logits=True)
        assert np.array_equal(l.cpu().numpy().view(np.uint32), lg[i:i + 13].view(np.uint32)), f"envs from {i}"
        assert np.array_equal(a.cpu().numpy(), act[i:i + 13])
    check_outputs(lg[:17].astype(np.float64), act[:17], forward(stack[:17], layers))
    check_outputs(lg[-17:].astype(np.float64), act[-17:], forward(stack[-17:], layers))
    P.close()


def scan(l):
    best = 0
    for a in range(1, 18):
        if l[a] > l[best]:
            best = a
    return best


@pytest.mark.parametrize("row", [
    [0.0] * 18,
    [float(a == 17) for a in range(18)],
    [1.0 if a in (5, 16) else 0.0 for a in range(18)],
    [float("-inf")] * 18,
    [float("-inf") if a != 9 else -1.0 for a in range(18)],
    [float("nan")] + [2.0] * 17,
    [1.0, float("nan")] + [5.0 if a == 13 else 0.0 for a in range(2, 18)],
    [float("nan") if a in (4, 8, 12, 16) else float(a % 7) for a in range(18)],
    [float("inf") if a in (3, 17) else 0.0 for a in range(18)],
])
def test_policy_first_maximal_logit(row):
    print("case: policy actions from logits", row, flush=True)
    g = env_for(17)
    layers = policy_weights(3)
    w = [l[0] for l in layers]
    b = [l[2] for l in layers]
    w[4] = np.zeros_like(w[4])                   # the logits are the head's biases
    b[4] = np.array(row + [100.0], b[4].dtype)
    P = Policy(g, w, b)
    act, lg = P.act(torch.zeros(17, 4, 84, 84, dtype=torch.uint8, device="cuda"), want_logits=True)
    assert np.array_equal(lg.cpu().numpy()[:, :18], np.tile(np.array(row, np.float32), (17, 1)), equal_nan=True)
    assert act.cpu().numpy().tolist() == [scan(row)] * 17
    P.close()
