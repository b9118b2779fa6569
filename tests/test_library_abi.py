"""Host-only checks of the C ABI: the built library exports what include/pcgrl.h declares, and
its defaults agree with the workload tables.  No GPU call is made."""
import ctypes as C
import os
import re

import pytest

from paper_2408_12525_amd import binding, build, workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_functions():
    src = open(os.path.join(ROOT, "include", "pcgrl.h")).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b(pcgrl_[a-z_]+)\s*\(", src)))


def test_library_exports_every_declared_entry_point():
    binding.load()                      # compiles the library first if it was never built
    lib = C.CDLL(build.LIB)
    names = header_functions()
    assert {"pcgrl_create", "pcgrl_reset", "pcgrl_step", "pcgrl_metrics"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n
    assert sorted(binding.EXPORTS) == names


@pytest.mark.parametrize("problem", [wl.BINARY, wl.MAZE, wl.DUNGEON])
def test_default_config_matches_workload_table(problem):
    c = binding.pcgrl_config_default(problem)
    w, lo, hi = wl.default_reward_table(problem)
    M = wl.num_metrics(problem)
    assert list(c.weights)[:M] == w and list(c.target_lo)[:M] == lo and list(c.target_hi)[:M] == hi
    K = wl.NUM_TILES[problem]
    cdf = list(c.init_cdf)
    assert cdf[K - 1] == 2**32 - 1 and all(cdf[i] <= cdf[i + 1] for i in range(K - 1))


def test_host_side_argument_errors_need_no_gpu():
    L = binding.load()
    assert L.pcgrl_create(None, None, 0) == -1
    assert L.pcgrl_config_default(7, C.byref(binding.PcgrlConfig())) == -2
    assert L.pcgrl_destroy(None) == 0
    assert L.pcgrl_strerror(-2).decode().startswith("configuration")
    h = C.c_void_p()
    bad = binding.make_config(wl.workload("maze16", batch=4, obs_w=99))
    assert L.pcgrl_create(C.byref(h), C.byref(bad), 0) == -2 and not h


SHIFT_ASM = """
_Z3fooPi:
	v_and_b32_e32 v{amt}, 31, v41
	v_lshlrev_b64 v[60:61], v{amt}, v[42:43]
	v_lshrrev_b64 v[4:5], s7, v[42:43]
	s_endpgm
	.amdhsa_kernel _Z3fooPi
		.amdhsa_next_free_vgpr {n}
	.end_amdhsa_kernel
"""


def test_build_scan_finds_a_shift_amount_in_the_highest_allocated_register():
    """The check the build runs on the compiler's device assembly (64-bit vector shifts whose
    amount sits in the last register of the kernel's allocation, which comes in blocks of eight):
    found where it is, not found one register lower, with a larger allocation, or with the amount
    in a scalar register."""
    n, found = build.scan_shift_amounts(SHIFT_ASM.format(amt=63, n=64))
    assert n == 1 and len(found) == 1 and found[0][0] == "_Z3fooPi" and found[0][1] == 64
    assert build.scan_shift_amounts(SHIFT_ASM.format(amt=63, n=58))[1] != []      # 58 registers are handed out as 64
    assert build.scan_shift_amounts(SHIFT_ASM.format(amt=62, n=64))[1] == []
    assert build.scan_shift_amounts(SHIFT_ASM.format(amt=63, n=65))[1] == []
    assert build.scan_shift_amounts(SHIFT_ASM.format(amt=71, n=65))[1] != []


def test_built_library_passed_the_scan():
    """build() refuses to hand out a library with such a shift; the report it leaves says how many
    kernels it looked at."""
    import json
    binding.load()
    if not os.path.exists(build.SCAN_REPORT):      # a library from before the check: build again
        build.build(force=True)
    rep = json.load(open(build.SCAN_REPORT))
    assert rep["findings"] == [] and rep["kernels"] >= 80


def test_compiled_call_path_leaves_doubtful_arguments_to_the_python_checks():
    """Arguments that are not device tensors of the right type and shape, missing ones and a closed
    environment are answered with LOOK, before any library call (no GPU is touched)."""
    import torch
    py = binding._load_py()
    env = py.Env(1, 0, 4, 16, 16, (3, 2, 31, 31), (3, 2, 31, 31))   # (the handle is never followed)
    act, obs = torch.zeros(3, dtype=torch.int32), torch.zeros((3, 2, 31, 31), dtype=torch.uint8)
    calls = lambda e: [e.step(act, None, None, None), e.step(None, obs, None, None), e.step(act), e.rollout(act, None, None, None),
                       e.rollout(act[None], obs, None, None), e.reset("1", None), e.reset(1, obs), e.metrics(act),
                       e.observe(obs), e.unpack_obs(obs, obs), e.exact_diameter(act), e.set_state(act, None, act, act)]
    assert set(calls(env)) == {py.LOOK}
    env.close()
    assert set(calls(env) + [env.get_state(), env.reset(1, None)]) == {py.LOOK}


WRAPPED = """
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
from paper_2408_12525_amd import binding
py = binding._load_py()
env = py.Env(1, 0, 4, 16, 16, (3, 2, 31, 31), (3, 2, 31, 31))   # (the handle is never followed)
shapes = dict(env=((3,), torch.int32), two=((5, 3), torch.int32), obs=((3, 2, 31, 31), torch.uint8), met=((3, 4), torch.int32),
              grid=((3, 16, 16), torch.int8), pair=((3, 2), torch.int16))
asked = []
def inside(env_, two, obs, met, grid, pair):
    try:
        env_.data_ptr()
        raise SystemExit("the wrapped tensor has storage after all")
    except RuntimeError:
        pass
    asked.extend([env.step(env_, None, None, None), env.rollout(two, None, None, None), env.reset(1, obs), env.metrics(met),
                  env.exact_diameter(env_), env.observe(obs), env.unpack_obs(obs, obs), env.set_state(grid, None, pair, pair)])
    return env_
with FakeTensorMode():
    torch.vmap(inside)(*[torch.empty((2,) + s, dtype=d, device="cuda:0") for s, d in shapes.values()])
assert asked == [py.LOOK] * 8, asked
print("asked")
"""


def test_compiled_call_path_outlives_tensors_without_storage():
    """A tensor of the right device, type and shape whose accessors throw inside torch (a batched
    tensor of torch.vmap without storage) is answered with LOOK by every entry point that takes
    tensors: the exception ends neither the call nor the process.  In a process of its own, which is
    what an escaping exception would end."""
    import subprocess
    import sys
    res = subprocess.run([sys.executable, "-c", WRAPPED], cwd=ROOT, capture_output=True, text=True)
    assert res.returncode == 0 and res.stdout.split() == ["asked"], res.stderr[-2000:]
