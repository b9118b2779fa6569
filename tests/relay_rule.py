"""The library's rule for rollouts as a relay (csrc/pcgrl_relay.h), compiled for the host, and what a
configuration hands to it."""
import json
import os
import re

import host_rule
from paper_2408_12525_amd import binding, build, workloads as wl

COMPUTE_UNITS = 256
FIELDS = ("rows", "binary", "per_simd", "compute_units", "workgroups", "observers", "obs_bytes", "step_bytes", "lds_tables",
          "lds_observer", "steps", "slots")
SOURCE = """
#include "pcgrl_relay.h"
extern "C" void rule(const int64_t* v, int64_t* out) {
  pcgrl::RelayCase c;
  c.rows = (int)v[0]; c.binary = v[1] != 0; c.per_simd = (int)v[2]; c.compute_units = (int)v[3]; c.workgroups = v[4];
  c.observers = (int)v[5]; c.obs_bytes = v[6]; c.step_bytes = v[7]; c.lds_tables = v[8]; c.lds_observer = v[9];
  c.steps = v[10]; c.slots = v[11];
  const pcgrl::RelayShape s = pcgrl::relay_shape(c);
  out[0] = s.searchers; out[1] = s.turns;
}
"""


def shape(**case):
    """(searchers, turns) of one case; every field of it has to be given."""
    assert set(case) == set(FIELDS)
    return host_rule.call(SOURCE, [case[k] for k in FIELDS], 2)


def resources(kernel):
    """What the build noted of the instances of a kernel, by their template arguments."""
    binding.load()
    rep = json.load(open(build.SCAN_REPORT)) if os.path.exists(build.SCAN_REPORT) else {}
    if "resources" not in rep:                     # a library from before the note: build again
        build.build(force=True)
        rep = json.load(open(build.SCAN_REPORT))
    out = {}
    for name, res in rep["resources"].items():
        m = re.match(r"_ZN5pcgrl\d+%sI((?:L[ib]\d+E)+)E" % kernel, name)
        if m:
            out[tuple(int(v) for v in re.findall(r"L[ib](\d+)E", m.group(1)))] = res
    return out


def wavefronts_per_simd(vgprs):
    """That a SIMD's 512 vector registers, handed out in eights, hold of a kernel (at most eight)."""
    return min(8, 512 // (-(-vgprs // 8) * 8))


def case_of(cfg, steps, slots):
    """What pcgrl_create and pcgrl_rollout work out for a configuration of which a metrics wavefront and
    observation wavefronts share the rollouts."""
    rows = next(s for s in (16, 32, 64) if max(cfg["max_h"], cfg["max_w"]) <= s)
    B, most = cfg["batch"], 64 // rows

    def fit(want, limit):
        n = 1
        while n * 2 <= want and n * 2 <= limit:
            n *= 2
        return n

    obs, stride = wl.obs_bytes(cfg), host_rule.obs_stride(cfg)
    levels = most
    while levels > 1 and -(-B // levels) < 1024:
        levels //= 2
    per_observer = levels // 2 if rows == 16 and obs >= 4096 and levels >= 2 else levels
    if cfg.get("levels_per_wave", 0) > 0:
        levels = per_observer = fit(cfg["levels_per_wave"], most)
    if cfg.get("split_obs_levels", 0) > 0:
        per_observer = fit(cfg["split_obs_levels"], levels)
    bits = stride * (8 if cfg.get("obs_format", 0) else 1)
    res = resources("rollout_relay_kernel")[rows, cfg["problem"]]
    return dict(rows=rows, binary=int(cfg["problem"] == wl.BINARY), per_simd=wavefronts_per_simd(res["vgprs"]), compute_units=COMPUTE_UNITS,
                workgroups=-(-B // levels), observers=levels // per_observer, obs_bytes=obs, step_bytes=stride * B, lds_tables=res["lds"],
                lds_observer=(((120 + per_observer * (bits + 8) + 31) // 32 + 6) * 4 + 15) // 16 * 16, steps=steps, slots=slots)


def relays(cfg, steps, slots):
    """Whether such a rollout runs as a relay, whose pieces have no room for an episode that ends twice in one."""
    ends = [cfg["max_steps"]] + [cfg["max_changes"]] * (cfg["max_changes"] > 0)
    return (not cfg["autoreset"] or min(ends) >= 8) and shape(**case_of(cfg, steps, slots))[0] > 0
