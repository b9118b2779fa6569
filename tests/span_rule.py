"""The library's rule for rollouts that are cut up along their steps (csrc/pcgrl_spans.h), compiled for the host."""
import host_rule
from paper_2408_12525_amd import workloads as wl

FIELDS = ("rows", "problem", "observed", "batch", "steps", "cells", "max_w", "obs_bytes", "window_bits", "step_bytes", "episode")
SOURCE = """
#include "pcgrl_spans.h"
extern "C" void rule(const int64_t* v, int64_t* out) {
  const pcgrl::SpanCase c = {(int)v[0], (int)v[1], v[2] != 0, v[3], v[4], v[5], v[6], v[7], v[8], v[9], v[10]};
  const pcgrl::SpanShape s = pcgrl::span_shape(c);
  out[0] = s.spans; out[1] = s.steps; out[2] = pcgrl::span_room((int)v[0], (int)v[1], v[3]);
}
"""


def shape_and_room(**case):
    """(spans, steps of a span, levels that a context keeps room for); every field of a case has to be given."""
    assert set(case) == set(FIELDS)
    return host_rule.call(SOURCE, [case[k] for k in FIELDS], 3)


def shape(**case):
    return shape_and_room(**case)[:2]


def case_of(cfg, steps, observed):
    """What pcgrl_rollout works out for a configuration that leaves the shape of the launches open."""
    rows = next(s for s in (16, 32, 64) if max(cfg["max_h"], cfg["max_w"]) <= s)
    ends = [cfg["max_steps"]] + [cfg["max_changes"]] * (cfg["max_changes"] > 0)
    mean = (cfg["min_h"] + cfg["max_h"]) * (cfg["min_w"] + cfg["max_w"]) // 4
    return dict(rows=rows, problem=cfg["problem"], observed=observed, batch=cfg["batch"], steps=steps, cells=(mean + cfg["max_h"] * cfg["max_w"]) // 2,
                max_w=cfg["max_w"], obs_bytes=wl.obs_bytes(cfg), window_bits=wl.obs_bytes(dict(cfg, obs_format=0)),
                step_bytes=host_rule.obs_stride(cfg) * cfg["batch"] if observed else 0, episode=min(ends) if cfg["autoreset"] else 0)


def spans(cfg, steps, slots):
    """Into how many spans a rollout with this many slots (0: without observations) is cut."""
    opened = all(cfg.get(k, 0) == 0 for k in ("split_step", "rollout_turns", "levels_per_wave", "split_obs_levels"))
    return shape(**case_of(cfg, steps, slots > 0))[0] if opened and slots in (0, steps) else 1
