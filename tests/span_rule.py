"""The library's rule for rollouts that are cut up along their steps (csrc/pcgrl_spans.h), compiled for the host."""
import ctypes as C
import functools
import os
import subprocess
import tempfile

import relay_rule
from paper_2408_12525_amd import workloads as wl

FIELDS = ("rows", "binary", "observed", "batch", "steps", "step_bytes")
SOURCE = """
#include "pcgrl_spans.h"
extern "C" void shape(const int64_t* v, int64_t* out) {
  const pcgrl::SpanCase c = {(int)v[0], v[1] != 0, v[2] != 0, v[3], v[4], v[5]};
  const pcgrl::SpanShape s = pcgrl::span_shape(c);
  out[0] = s.spans; out[1] = s.steps; out[2] = pcgrl::span_room((int)v[0], v[1] != 0, v[3]);
}
"""


@functools.lru_cache(None)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        with open(os.path.join(d, "spans.cpp"), "w") as f:
            f.write(SOURCE)
        so = os.path.join(d, "spans.so")
        subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC", "-I", relay_rule.CSRC, f.name, "-o", so], check=True)
        return C.CDLL(so)


def shape_and_room(**case):
    """(spans, steps of a span, levels that a context keeps room for); every field of a case has to be given."""
    assert set(case) == set(FIELDS)
    v, out = (C.c_int64 * len(FIELDS))(*[int(case[k]) for k in FIELDS]), (C.c_int64 * 3)()
    _lib().shape(v, out)
    return tuple(out)


def shape(**case):
    return shape_and_room(**case)[:2]


def case_of(cfg, steps, observed):
    """What pcgrl_rollout works out for a configuration that leaves the shape of the launches open."""
    rows = next(s for s in (16, 32, 64) if max(cfg["max_h"], cfg["max_w"]) <= s)
    return dict(rows=rows, binary=cfg["problem"] == wl.BINARY, observed=observed, batch=cfg["batch"], steps=steps,
                step_bytes=wl.obs_bytes(cfg) * cfg["batch"] if observed else 0)
