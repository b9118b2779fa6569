"""The library's rules for steps and rollouts of one or two wavefronts a level group (csrc/pcgrl_split.h)."""
import host_rule
from paper_2408_12525_amd import workloads as wl

STORES = {"cached": 0, "stream": 1, "through": 2}
SOURCE = """
#include "pcgrl_split.h"
extern "C" void rule(const int64_t* v, int64_t* out) {
  const pcgrl::SplitCase c = {(int)v[0], (int)v[1], v[2], v[3], v[4], v[5] != 0};
  out[0] = v[6] != 0 ? pcgrl::split_rollout(c, pcgrl::ring_of((int)v[7], v[8])) : pcgrl::split_step(c, (int)v[7]);
}
"""


def _case(cfg):
    rows = next(s for s in (16, 32, 64) if max(cfg["max_h"], cfg["max_w"]) <= s)
    stride = host_rule.obs_stride(cfg)
    return [rows, cfg["problem"], cfg["batch"], wl.obs_bytes(cfg), stride * cfg["batch"], stride % 128 == 0]


def step(cfg, store):
    """Whether a step that stores its observations this way takes two wavefronts."""
    return bool(host_rule.call(SOURCE, _case(cfg) + [0, STORES[store], 0], 1)[0])


def rollout(cfg, slots, store):
    """Whether a rollout into that many slots, stored this way, takes two wavefronts."""
    return bool(host_rule.call(SOURCE, _case(cfg) + [1, STORES[store], slots * host_rule.obs_stride(cfg) * cfg["batch"]], 1)[0])
