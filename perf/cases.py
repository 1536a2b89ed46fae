"""The work a user has the framework do, as cases that can be timed and compared.

Every case goes through the public torch-facing entry points: `VcsEnv.step`
(whole populations, listed env ids, captured graphs), `VcsEnv.reset`,
`FrameStack.push`, `Policy.act`, and the loop of the last two with the step
(actions from the network).  Sizes are those of the workload configurations
(`inputs/workloads.py`) and the benchmark; cartridges come from the seeded
generator, as everywhere in this repository.

Consoles run on: each pass steps the states the pass before left, with the
next of a set of action vectors, as a program that plays does.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_1907_08467_amd import binding as B
from paper_1907_08467_amd.env import FrameStack, Policy, VcsEnv
from paper_1907_08467_amd.inputs.palette import GRAY
from paper_1907_08467_amd.inputs.romgen import RomSpec, generate
from paper_1907_08467_amd.inputs.workloads import zipf_counts

DEV = "cuda:0"
OBS = 84 * 84
FRAME = 210 * 160
STATE = 384
ACTION_SETS = 16                       # action vectors a state cycles through
SCHEMES = "4k,f8,f6,f4,f8sc,f6sc,f4sc,e0,3f"
# the policy network's layers: (outputs, reduction length), then its convolutions (channels, kernel, stride)
LAYERS = [(32, 256), (64, 512), (64, 576), (512, 3136), (19, 512)]
CONVS = [(4, 8, 4), (32, 4, 2), (64, 3, 1)]
LOGITS = 19                            # 18 action logits and the value; the rest of a logits row is unspecified
POLICY_FLOPS = 18705408                # per env


def _step(name, n, **kw):
    """A step of n envs; `resident` > n: of n listed ids among that many."""
    c = dict(name=name, path="step", n=n, resident=n, kinds="4k", roms=1, divergent=False, objects=False, zipf=0.0,
             frameskip=4, sticky=0.0, frames=False, last2=False, steps=1, rom_seed=2000)
    c.update(kw)
    return c


def listed():
    return [
        # a handful of consoles: an evaluation or a debugging session; one launch of few waves, latency only
        _step("step_8", 8, frames=True, rom_seed=1000),
        # the plain batched step of an actor-critic learner's population, every frame kept
        _step("step_4096_frames", 4096, frames=True),
        # several games, envs that part on random branches, sticky actions, every frame kept
        _step("divergent_16384_frames", 16384, kinds="4k,f8", roms=8, divergent=True, sticky=0.25, frames=True,
              rom_seed=3000),
        # the largest fixed batch on one GPU: 16 games in uneven populations, captured steps, observations only
        _step("graph_65536x4", 65536, kinds="4k,f8", roms=16, divergent=True, zipf=1.2, last2=True, steps=4,
              rom_seed=4000),
        # every cartridge scheme in one batch: the cartridges are read from HBM
        _step("schemes_36864", 36864, kinds=SCHEMES, roms=9, divergent=True, sticky=0.25, last2=True, rom_seed=6000),
        # missiles, ball, object motion and collision latches, every frame kept
        _step("objects_4096_frames", 4096, objects=True, frames=True, rom_seed=7000),
        # one merged batch of a server: listed ids out of a large resident population
        _step("served_6529", 6529, resident=131072, kinds="4k,f8", roms=16, divergent=True, zipf=1.2, last2=True,
              rom_seed=4000),
        # restarting some envs from the reset cache
        dict(name="reset_1000", path="reset", n=1000, resident=4096, kinds="4k", roms=1, divergent=False,
             objects=False, zipf=0.0, frameskip=4, sticky=0.0, last2=True, rom_seed=2000),
        # the learner's input: the last four observations of a large population
        dict(name="stack_16384", path="stack", n=16384, resident=16384, depth=4, bits=8),
        # the policy network: a learner's batch, and a few envs
        dict(name="policy_4096", path="policy", n=4096),
        dict(name="policy_33", path="policy", n=33),
        # inference only: the network picks the actions, the envs step, the stack takes the observations
        dict(name="loop_4096", path="loop", n=4096, kinds="4k", roms=1, divergent=False, objects=False, zipf=0.0,
             frameskip=4, sticky=0.0, last2=True, rom_seed=2000, depth=4, bits=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    path = rng.choice(["step", "step", "step", "step", "graph", "served", "reset", "stack", "policy", "loop"])
    if path == "stack":
        n = _log(rng, 1, 16384)
        return dict(path="stack", n=n, resident=n + rng.choice([0, 0, 7, 1000]), depth=rng.randint(1, 6),
                    bits=rng.choice([8, 4]))
    if path == "policy":
        return dict(path="policy", n=_log(rng, 1, 6000))
    kinds = rng.choice(["4k", "f8", "4k,f8", "4k,f8", SCHEMES, rng.choice(SCHEMES.split(","))])
    roms = rng.randint(1, 12) if "," in kinds else rng.choice([1, 1, 2, 3])
    objects = kinds == "4k" and rng.random() < 0.4
    c = dict(kinds=kinds, roms=roms, divergent=rng.random() < 0.6, objects=objects,
             zipf=rng.choice([0.0, 0.0, 1.2]), frameskip=rng.choice([2, 3, 4, 4, 4, 5]),
             sticky=rng.choice([0.0, 0.25]), last2=rng.random() < 0.6, rom_seed=100 * rng.randint(20, 90))
    if path == "loop":
        return dict(c, path="loop", n=_log(rng, 4, 4096), depth=4, bits=rng.choice([8, 4]))
    if path == "reset":
        n = _log(rng, 1, 4096)
        return dict(c, path="reset", n=n, resident=n + rng.randint(0, 4096))
    if path == "served":
        n = _log(rng, 64, 8192)
        return dict(c, path="step", n=n, resident=n + _log(rng, 100, 60000), frames=False, steps=1, last2=True)
    steps = rng.randint(2, 4) if path == "graph" else 1
    n = _log(rng, 1, 2048 if objects else 12288)
    return dict(c, path="step", n=n, resident=n, frames=rng.random() < 0.4 and n <= 8192, steps=steps)


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _env(case, seed):
    kinds = case["kinds"].split(",")
    k = case["roms"]
    roms = [generate(RomSpec(case["rom_seed"] + r, kinds[r % len(kinds)], case["divergent"], objects=case["objects"]))
            for r in range(k)]
    n = case.get("resident", case["n"])
    if case["zipf"]:
        counts = zipf_counts(n, k, case["zipf"])
    else:
        counts = [n // k + (r < n % k) for r in range(k)]
    lab = np.repeat(np.arange(k, dtype=np.uint16), counts)
    if k > 1:
        lab = np.random.Generator(np.random.PCG64(seed)).permutation(lab)
    return VcsEnv([(r.data, r.scheme) for r in roms], lab, GRAY, frameskip=case["frameskip"],
                  sticky_threshold=int(case["sticky"] * 2**32), seed=seed,
                  render_mode=B.VCS_RENDER_LAST2 if case["last2"] else B.VCS_RENDER_ALL, max_batch=case["n"],
                  pipelines=2 if case.get("steps", 1) > 1 else 1, collisions=case["objects"])


def _images(g, n):
    """Observations as the emulator makes them: a few flat bands of gray,
    blocks of playfield over them and small bright objects, as u8 [n][84][84]."""
    band = torch.randint(0, 256, (n, 12, 1), generator=g, device=DEV)
    field = torch.randint(0, 256, (n, 12, 21), generator=g, device=DEV)
    on = torch.rand((n, 12, 21), generator=g, device=DEV) < 0.4
    img = torch.where(on, field, band).to(torch.uint8)
    img = img.repeat_interleave(7, 1).repeat_interleave(4, 2)
    spot = torch.rand((n, 84, 84), generator=g, device=DEV) < 0.01
    return torch.where(spot, torch.full_like(img, 236), img).contiguous()


def _weights(g):
    """He-uniform bf16 weights and small biases: [(bit patterns, values)] and the biases."""
    ws, bs = [], []
    for n, k in LAYERS:
        lim = math.sqrt(6.0 / k)
        w = ((torch.rand((n, k), generator=g, device=DEV) * 2 - 1) * lim).to(torch.bfloat16)
        ws.append(w)
        bs.append((torch.rand(n, generator=g, device=DEV) - 0.5) * 0.1)
    return ws, bs


def _policy(env, ws, bs):
    return Policy(env, [w.view(torch.int16).cpu().numpy().view(np.uint16) for w in ws], [b.cpu().numpy() for b in bs])


def _small_env(n):
    """The context a frame stack or a policy belongs to, where no env is stepped."""
    rom = generate(RomSpec(1000))
    return VcsEnv([(rom.data, rom.scheme)], np.zeros(n, np.uint16), GRAY, reset_cache_k=1, startup_frames=2,
                  noop_max=0, render_mode=B.VCS_RENDER_LAST2)


def _policy_inputs(n, seed):
    g = _gen(seed)
    ws, bs = _weights(g)
    return _images(g, 4 * n).reshape(n, 4, 84, 84), ws, bs


def prepare(case, seed):
    n, path = case["n"], case["path"]
    if path == "policy":
        stack, ws, bs = _policy_inputs(n, seed)
        env = _small_env(n)
        return dict(case=case, env=env, policy=_policy(env, ws, bs), stack=stack)
    g = _gen(seed)
    if path == "stack":
        env = _small_env(case["resident"])
        ids = None
        if case["resident"] > n:
            ids = torch.randperm(case["resident"], generator=g, device=DEV)[:n].to(torch.int32)
        fs = FrameStack(env, depth=case["depth"], bits=case["bits"])
        obs = [_images(g, n) for _ in range(3)]
        done = [(torch.rand(n, generator=g, device=DEV) < 0.01).to(torch.uint8) for _ in range(3)]
        return dict(case=case, env=env, fs=fs, obs=obs, done=done, ids=ids, k=0,
                    out=torch.empty((n, case["depth"], 84, 84), dtype=torch.uint8, device=DEV))
    env = _env(case, seed)
    st = dict(case=case, env=env, k=0)
    if path == "reset":
        st["ids"] = torch.randperm(env.num_envs, generator=g, device=DEV)[:n].to(torch.int32)
        st["obs"] = torch.empty((n, 84, 84), dtype=torch.uint8, device=DEV)
        return st
    if path == "loop":
        ws, bs = _weights(g)
        st["policy"] = _policy(env, ws, bs)
        st["fs"] = FrameStack(env, depth=4, bits=case["bits"])
        st["done"] = torch.ones(n, dtype=torch.uint8, device=DEV)
        st["reward"] = torch.empty(n, dtype=torch.int32, device=DEV)
        st["obs"] = env.reset()
        st["stack"] = st["fs"].push(st["obs"], st["done"])
        st["actions"] = torch.empty(n, dtype=torch.uint8, device=DEV)
        st["logits"] = torch.empty((n, 32), dtype=torch.float32, device=DEV)
        return st
    st["actions"] = torch.randint(0, 18, (ACTION_SETS, case["steps"], n), generator=g, device=DEV, dtype=torch.uint8)
    if case["steps"] > 1:
        st["graph"] = env.capture(steps=case["steps"], want_frames=case["frames"])
        return st
    st["ids"] = None
    if case["resident"] > n:
        st["ids"] = torch.randperm(case["resident"], generator=g, device=DEV)[:n].to(torch.int32)
    st["out"] = (torch.empty((n, 84, 84), dtype=torch.uint8, device=DEV),
                 torch.empty(n, dtype=torch.int32, device=DEV), torch.empty(n, dtype=torch.uint8, device=DEV),
                 torch.empty((n, env.n_slots, 210, 160), dtype=torch.uint8, device=DEV) if case["frames"] else None)
    return st


def run(st):
    case, path = st["case"], st["case"]["path"]
    if path == "policy":
        actions, logits = st["policy"].act(st["stack"], want_logits=True)
        return dict(actions=actions, logits=logits[:, :LOGITS])
    if path == "reset":
        return dict(obs=st["env"].reset(st["ids"], obs=st["obs"]))
    k = st["k"]
    st["k"] = k + 1
    if path == "stack":
        return dict(stack=st["fs"].push(st["obs"][k % 3], st["done"][k % 3], env_ids=st["ids"], out=st["out"]))
    if path == "loop":
        st["policy"].act(st["stack"], logits=st["logits"], actions=st["actions"])
        st["env"].step(st["actions"], out=(st["obs"], st["reward"], st["done"], None))
        st["fs"].push(st["obs"], st["done"], out=st["stack"])
        return dict(logits=st["logits"][:, :LOGITS], actions=st["actions"], reward=st["reward"], done=st["done"],
                    stack=st["stack"])
    acts = st["actions"][k % ACTION_SETS]
    if "graph" in st:
        obs, reward, done, frames = st["graph"].launch(acts)
    else:
        obs, reward, done, frames = st["env"].step(acts[0], st["ids"], out=st["out"])
    return dict(obs=obs, reward=reward, done=done, frames=frames)


def _step_work(case, steps=1):
    n, fs = case["n"], case["frameskip"]
    slots = (2 if case["last2"] else fs) if case.get("frames") else 0
    # per env-step: state in and out, action, the observation, reward and done, the frames kept
    b = 2 * STATE + 1 + OBS + 4 + 1 + slots * FRAME + (4 if case.get("resident", n) > n else 0)
    # one operation per emulated 6507 instruction: about 3,300 a frame, 4,000 in the cartridges with random branches
    ops = fs * (4000 if case["divergent"] else 3300)
    return dict(bytes=steps * n * b, flops=steps * n * ops)


def work(case):
    n, path = case["n"], case["path"]
    if path == "policy":
        return dict(bytes=n * (4 * OBS + 32 * 4 + 1) + 2 * sum(a * b for a, b in LAYERS), flops=n * POLICY_FLOPS)
    if path == "reset":
        return dict(bytes=n * (2 * STATE + 2 * OBS + 4), flops=0)
    if path == "stack":
        slot = OBS * case["bits"] // 8
        d = case["depth"]      # the observation in, one slot written, the other slots read, the stack out
        return dict(bytes=n * (OBS + slot + (d - 1) * slot + d * OBS + 2), flops=0)
    if path == "loop":
        w = _step_work(case)
        slot = OBS * case["bits"] // 8
        return dict(bytes=w["bytes"] + n * (4 * OBS + 128 + 1 + OBS + slot + 3 * slot + 4 * OBS) +
                    2 * sum(a * b for a, b in LAYERS), flops=w["flops"] + n * POLICY_FLOPS)
    return _step_work(case, case["steps"])


def exact(case, seed):
    """The network's outputs in 64 bits; everything else is whole numbers."""
    if case["path"] != "policy":
        return None
    stack, ws, bs = _policy_inputs(case["n"], seed)
    ws = [w.double() for w in ws]
    bs = [b.double() for b in bs]
    # reduction orders: the first layer (channel, ky, kx), the others (ky, kx, channel)
    taps = [ws[0].reshape(32, 4, 8, 8).permute(0, 2, 3, 1).reshape(32, 256), ws[1], ws[2]]
    outs = []
    for lo in range(0, case["n"], 256):
        x = stack[lo:lo + 256].double().permute(0, 2, 3, 1) / 255.0
        for (_, k, s), w, b in zip(CONVS, taps, bs):
            p = x.unfold(1, k, s).unfold(2, k, s)                  # [n][oh][ow][channel][ky][kx]
            m, oh, ow = p.shape[:3]
            p = p.permute(0, 1, 2, 4, 5, 3).reshape(m * oh * ow, -1)
            x = torch.relu(p @ w.t().contiguous() + b).reshape(m, oh, ow, -1)
        h = torch.relu(x.reshape(x.shape[0], -1) @ ws[3].t().contiguous() + bs[3])
        outs.append(h @ ws[4].t().contiguous() + bs[4])
    return dict(actions=None, logits=torch.cat(outs))
