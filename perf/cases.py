"""What users of this library have it do, as cases that can be timed and compared.

Seven kinds of call, each through the public binding:

  step      one pcgrl_step per pass, called eagerly, as a policy in the loop does
  graph     a HIP graph of consecutive pcgrl_step launches, replayed once per pass
  rollout   one pcgrl_rollout of `steps` steps per pass, a slot per step
  reset     pcgrl_reset with the first observations
  levels    levels made elsewhere are installed, scored and read back
            (pcgrl_set_state, pcgrl_metrics, pcgrl_get_state)
  unpack    one slot of bit-packed observations is widened for the network
  diameter  the exact diameter of every level

Environments are in mid-episode when they are handed over (a stretch of random edits lies behind
them), actions are those of a random agent and already on the GPU, observation buffers belong to
the caller.  A case is a dict of plain values; `listed()` gives the ones that are watched, `draw()`
others of the same ranges.
"""
import math

import torch

from paper_2408_12525_amd import binding, workloads as wl

PROBLEMS = {"binary": wl.BINARY, "maze": wl.MAZE, "dungeon": wl.DUNGEON}
PROBS = {"binary": [.5, .5], "maze": [.45, .45, .05, .05],
         "dungeon": [.40, .40, .04, .04, .04, .04, .04]}
DTYPES = {"uint8": torch.uint8, "float16": torch.float16, "bfloat16": torch.bfloat16,
          "float32": torch.float32}
WARM_STEPS = 200            # random edits before the environments are handed over
ACTION_BYTES = 32 << 20     # the pre-generated actions stay below this
MAX_BYTES = 500 << 20       # a drawn case's observations, all steps of a pass together
MAX_RING = 2 << 30          # a drawn case's observation buffers


def _case(kind, problem, batch, h, w, **more):
    """The fields of a case with their usual values: a fixed shape, the 31-cell window, border
    padding, dense one-hot observations, random positions, 1000 steps an episode."""
    c = dict(kind=kind, problem=problem, batch=batch, h=h, w=w, min_h=h, min_w=w, obs_w=31, wall_pad=False,
             scan=False, frozen=0, max_changes=0, lines=False, packed=False, slots=1, steps=1, dtype="uint8")
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: 64 levels, one buffer that a policy reads before the next step; what
        # counts is the host's path and the launch
        _case("step", "binary", 64, 16, 16, wall_pad=True, name="step_binary16_b64"),
        # the usual training batch, every observation kept by the learner
        _case("step", "maze", 4096, 16, 16, lines=True, slots=64, name="step_maze16_b4096"),
        # random shapes with pinpoints and a small window
        _case("step", "binary", 16384, 32, 32, min_h=8, min_w=8, obs_w=15, frozen=3, lines=True, slots=32,
              name="step_binary32_ow15_b16384"),
        # seven tile types; a change limit, so that some levels restart in every step
        _case("step", "dungeon", 16384, 32, 32, obs_w=15, max_changes=205, name="step_dungeon32_b16384"),
        # the largest batch
        _case("step", "binary", 262144, 16, 16, wall_pad=True, lines=True, slots=4, name="step_binary16_b262144"),
        # large maps, the steps captured once and replayed
        _case("graph", "maze", 8192, 64, 64, lines=True, slots=16, steps=16, name="graph_maze64_b8192"),
        # a small batch taken through many steps in one launch
        _case("rollout", "binary", 64, 16, 16, wall_pad=True, slots=256, steps=256, name="rollout_binary16_b64"),
        # large maps in one launch, every observation kept
        _case("rollout", "maze", 8192, 64, 64, lines=True, slots=32, steps=32, name="rollout_maze64_b8192"),
        # a learner reads a packed slot for its first convolution
        _case("unpack", "maze", 8192, 64, 64, packed=True, dtype="bfloat16", name="unpack_maze64_bf16_b8192"),
        # a fresh batch of episodes
        _case("reset", "maze", 8192, 64, 64, lines=True, name="reset_maze64_b8192"),
        # a ragged buffer and batch: levels of a designer or of another generator are scored
        _case("levels", "dungeon", 5001, 27, 45, min_h=9, min_w=9, obs_w=15, name="levels_dungeon27x45_b5001"),
        # how far the two-sweep estimate is off
        _case("diameter", "binary", 1024, 64, 64, name="diameter_binary64_b1024"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["step", "graph", "rollout", "reset", "levels", "unpack", "diameter"],
                       [34, 10, 24, 9, 8, 9, 6])[0]
    problem = "binary" if kind == "diameter" else rng.choice(["binary", "maze", "dungeon"])
    h = rng.choice([16, 32, 64, rng.randint(8, 64)])
    w = h if rng.random() < .6 else rng.randint(8, 64)
    c = _case(kind, problem, 1, h, w)
    if rng.random() < .3:
        c.update(min_h=rng.randint(3, h), min_w=rng.randint(3, w))
    c.update(obs_w=rng.choice([31, 15, rng.randint(3, 63)]), wall_pad=rng.random() < .3, scan=rng.random() < .2,
             frozen=rng.choice([0, 0, rng.randint(1, 8)]),
             max_changes=rng.choice([0, 0, 0, rng.randint(30, 300)]), lines=rng.random() < .5,
             packed=kind == "unpack" or (kind in ("step", "graph", "rollout") and rng.random() < .2))
    one = observation_bytes(c)
    if kind == "diameter":
        c["batch"] = _log_int(rng, 16, min(16384, 1024 * 64 ** 4 // max(h, w) ** 4))
    elif kind == "unpack":
        c["dtype"] = rng.choice(sorted(DTYPES))
        c["batch"] = _log_int(rng, 64, min(65536, MAX_BYTES // (one * 8 * DTYPES[c["dtype"]].itemsize)))
    elif kind == "levels":
        c["batch"] = _log_int(rng, 64, min(65536, 8192 * 64 * 64 // (h * w)))
    else:
        c["steps"] = 1 if kind in ("step", "reset") else rng.choice([8, 16, 32, _log_int(rng, 4, 256)])
        # (the from-scratch work of a reset and the floods of a step grow with the map, so the
        # largest batches are those of small maps)
        most = min(262144 * 256 // max(h, w) ** 2, MAX_BYTES // (one * c["steps"]))
        c["batch"] = _log_int(rng, 64, max(65, most))
        if kind == "step":
            c["slots"] = rng.choice([1, max(1, min(rng.choice([16, 32, 64]), MAX_RING // (one * c["batch"])))])
        elif kind != "reset":
            c["slots"] = c["steps"]
    if rng.random() < .5 and c["batch"] > 256:
        c["batch"] |= 1             # a batch that no wavefront divides
    return c


def config(case):
    """The library's configuration of a case."""
    return wl.make_config(
        PROBLEMS[case["problem"]], case["batch"], case["h"], case["obs_w"], max_w=case["w"],
        min_size=case["min_h"], min_w=case["min_w"],
        pad_mode=wl.PAD_WALL if case["wall_pad"] else wl.PAD_BORDER,
        pos_mode=wl.POS_SCAN if case["scan"] else wl.POS_RANDOM, n_frozen=case["frozen"], max_steps=1000,
        max_changes=case["max_changes"], probs=PROBS[case["problem"]], obs_format=1 if case["packed"] else 0,
        obs_pitch=-1 if case["lines"] else 0)


def observation_bytes(case):
    """Bytes of one level's observation."""
    return wl.obs_bytes(config(case))


def _levels(case, gen):
    """Levels in the plain layout: tiles, frozen cells, shapes and positions."""
    dev, B, H, W = "cuda", case["batch"], case["h"], case["w"]
    p = torch.tensor(PROBS[case["problem"]], device=dev)
    u = torch.rand((B, H, W), generator=gen, device=dev)
    tiles = torch.searchsorted(p.cumsum(0)[:-1].contiguous(), u).to(torch.int8)
    frozen = (torch.rand((B, H, W), generator=gen, device=dev) < case["frozen"] / (H * W)).to(torch.uint8)
    span = lambda lo, hi: torch.randint(lo, hi + 1, (B,), generator=gen, device=dev)  # noqa: E731
    hw = torch.stack([span(case["min_h"], H), span(case["min_w"], W)], 1).to(torch.int16)
    pos = torch.zeros_like(hw)
    return tiles, frozen, hw, pos


def prepare(case, seed):
    kind, dev = case["kind"], torch.device("cuda", 0)
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    cfg = config(case)
    B, K = case["batch"], wl.NUM_TILES[cfg["problem"]]
    env = binding.Pcgrl(cfg, 0)
    env.pcgrl_reset(seed)
    s = {"kind": kind, "env": env, "t": 0, "seed": seed}
    if kind == "levels":
        s["levels"] = _levels(case, gen)
        return s
    if kind == "reset":
        s["obs"] = env.new_obs()
        return s

    def acts(n):
        return torch.randint(0, K, (n, B), dtype=torch.int32, generator=gen, device=dev)

    env.pcgrl_rollout(acts(WARM_STEPS))
    if kind == "diameter":
        s["out"] = torch.empty(B, dtype=torch.int32, device=dev)
        return s
    if kind == "unpack":
        s["packed"] = env.pcgrl_observe()
        s["out"] = torch.empty(env.onehot_shape, dtype=DTYPES[case["dtype"]], device=dev)
        return s
    slots, steps = case["slots"], case["steps"]
    ring = torch.empty((slots,) + tuple(env.obs_shape), dtype=torch.uint8, device=dev)
    if kind == "step":
        n = max(8, min(64, ACTION_BYTES // (4 * B)))
        s["actions"] = acts(n).unbind(0)
        s["obs"] = ring.unbind(0)
        s["reward"] = torch.empty((slots, B), dtype=torch.float32, device=dev).unbind(0)
        s["done"] = torch.empty((slots, B), dtype=torch.uint8, device=dev).unbind(0)
        return s
    s["actions"] = acts(steps)
    s["obs"] = ring
    s["reward"] = torch.empty((steps, B), dtype=torch.float32, device=dev)
    s["done"] = torch.empty((steps, B), dtype=torch.uint8, device=dev)
    if kind == "graph":
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            for t in range(steps):
                env.pcgrl_step(s["actions"][t], ring[t], s["reward"][t], s["done"][t])
    return s


def run(s):
    kind, env = s["kind"], s["env"]
    if kind == "step":
        t = s["t"]
        s["t"] = t + 1
        i = t % len(s["obs"])
        obs, reward, done = s["obs"][i], s["reward"][i], s["done"][i]
        env.pcgrl_step(s["actions"][t % len(s["actions"])], obs, reward, done)
        return obs, reward, done
    if kind == "graph":
        s["graph"].replay()
        return s["obs"], s["reward"], s["done"]
    if kind == "rollout":
        env.pcgrl_rollout(s["actions"], s["obs"], s["reward"], s["done"])
        return s["obs"], s["reward"], s["done"]
    if kind == "reset":
        s["seed"] += 1
        env.pcgrl_reset(s["seed"], s["obs"])
        return s["obs"], env.pcgrl_metrics()
    if kind == "levels":
        env.pcgrl_set_state(*s["levels"])
        return env.pcgrl_metrics(), env.pcgrl_get_state()
    if kind == "unpack":
        return env.pcgrl_unpack_obs(s["packed"], s["out"], s["out"].dtype)
    return env.pcgrl_exact_diameter(s["out"])


def work(case):
    """Bytes of one pass: a level is its tile code as bit-planes, a 32-byte record and its rows of
    metrics and targets; what a call reads of that is counted once, and so is what it writes.  The
    path has no floating-point work to speak of."""
    cfg = config(case)
    M, B, cells = wl.num_metrics(cfg["problem"]), case["batch"], case["h"] * case["w"]
    planes = {"binary": 1, "maze": 2, "dungeon": 3}[case["problem"]]
    level = -(-planes * cells // 8)
    obs = wl.obs_bytes(cfg)
    kind, steps = case["kind"], case["steps"]
    if kind in ("step", "graph"):
        one = level + 32 + 8 * M + 4 + obs + 4 + 1 + 32 + 4 * M
        return {"bytes": B * steps * one, "flops": 0}
    if kind == "rollout":
        return {"bytes": B * (2 * (level + 32) + 12 * M + steps * (4 + obs + 4 + 1)), "flops": 0}
    if kind == "reset":
        return {"bytes": B * (level + 32 + 8 * M + obs + 4 * M), "flops": 0}
    if kind == "levels":
        return {"bytes": B * (2 * cells + 8 + 4 * M + 2 * cells + 8 + 12), "flops": 0}
    if kind == "unpack":
        onehot = wl.obs_bytes(dict(cfg, obs_format=0))
        return {"bytes": B * (obs + onehot * DTYPES[case["dtype"]].itemsize), "flops": 0}
    return {"bytes": B * (level + 4), "flops": 0}


def tolerance(case):
    """Whole numbers everywhere, and rewards that are one sum of float32 products in a fixed order."""
    return "exact"
