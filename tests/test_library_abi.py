"""Host-only checks of the C ABI: the built library exports what include/pcgrl.h declares, and
its defaults agree with the workload tables.  No GPU call is made."""
import ctypes as C
import os
import random
import re

import pytest

import host_rule
import relay_rule
import span_rule
import split_rule
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


PLANES = {0: 1, 1: 2, 2: 3}   # bit-planes of binary, maze and dungeon levels


def test_single_steps_load_their_state_and_nothing_else():
    """A step asks memory for the level, its record, action, metrics, ranges and weights: beside the
    planes twelve loads at most, and three for the observation wavefront, which loads the planes
    again.  More of them are configuration read as if it differed from lane to lane, in the middle of a
    chain and behind the wavefront's own stores (as the draws of a restart once were).  Nor does a step
    use scratch memory."""
    steps = relay_rule.resources("step_kernel")
    assert len(steps) == 54
    for (S, problem, split, pin, wide), res in steps.items():
        assert res["loads"] <= (1 + split) * PLANES[problem] + 12 + 3 * split, (S, problem, split, pin, wide, res)
        assert res["scratch"] == 0, (S, problem, split, pin, wide, res)


# wavefronts that a SIMD's 512 vector registers hold of a rollout with observation wavefronts; a lost one
# showed as 11 % on 32-row binary levels
ROLLOUT_WAVEFRONTS = {(16, 0): 6, (16, 1): 5, (16, 2): 4, (32, 0): 6, (32, 1): 5, (32, 2): 4, (64, 0): 8, (64, 1): 7, (64, 2): 6}


def test_rollouts_of_large_batches_keep_their_wavefronts():
    rollouts = relay_rule.resources("rollout_kernel")
    assert {(S, p) for S, p, mode in rollouts if mode == 3} == set(ROLLOUT_WAVEFRONTS)
    for (S, problem, mode), res in rollouts.items():
        assert res["scratch"] == 0, (S, problem, mode, res)
        if mode == 3:
            assert relay_rule.wavefronts_per_simd(res["vgprs"]) >= ROLLOUT_WAVEFRONTS[S, problem], (S, problem, res)


# us a step of 32-step rollouts with 31-cell windows, one level a workgroup: no relay, then 4 searchers and 4
# observers that take turns, 4 and 2, 2 and 2, 2 and 1
RELAY_TIMES = {
    (16, wl.BINARY): {64: (1.39, .87, .91, 1.05, 1.24), 512: (1.82, 1.15, 1.13, 1.29, 1.44), 768: (1.95, 1.66, 1.29, 1.45, 1.54),
                      1024: (1.97, 2.20, 1.81, 1.96, 1.64), 1280: (2.14, 2.47, 2.05, 2.21, 2.49), 1536: (2.22, 2.92, 2.39, 2.61, 2.75)},
    (32, wl.BINARY): {64: (1.38, .96, .99, .99, 1.15), 512: (2.02, 1.34, 1.30, 1.45, 1.55), 768: (1.99, 1.71, 1.47, 1.56, 1.65),
                      1024: (2.14, 2.27, 1.91, 1.98, 1.80), 1280: (2.32, 2.48, 2.05, 2.19, 2.26), 1536: (2.29, 2.89, 2.31, 2.44, 2.59)},
    (64, wl.BINARY): {64: (1.11, .82, .88, .90, 1.04), 512: (1.41, 1.17, 1.18, 1.15, 1.27), 768: (1.50, 1.70, 1.36, 1.29, 1.39),
                      1024: (1.65, 2.26, 1.81, 1.79, 1.58), 1280: (1.70, 2.49, 2.08, 2.04, 2.16), 1536: (1.88, 3.00, 2.35, 2.40, 2.43)},
    (16, wl.MAZE): {64: (1.02, .67, .85, .85, 1.28), 512: (1.19, 1.25, 1.03, 1.01, 1.40), 768: (1.35, 1.79, 1.70, 1.75, 1.48),
                    1024: (1.37, 2.31, 1.85, 1.93, 2.58), 1280: (1.72, 2.85, 2.48, 2.52, 2.85)},
    (32, wl.MAZE): {64: (1.12, .66, .79, .79, 1.15), 512: (1.30, .90, .98, .97, 1.25), 768: (1.46, 1.31, 1.11, 1.10, 1.34),
                    1024: (1.49, 1.94, 1.59, 1.58, 1.43), 1280: (1.60, 2.07, 1.80, 1.93, 2.32)},
    (64, wl.MAZE): {64: (1.23, .78, .89, .92, 1.22), 512: (1.45, 1.07, 1.13, 1.15, 1.37), 768: (1.64, 1.57, 1.31, 1.31, 1.49),
                    1024: (1.67, 2.27, 1.82, 1.83, 1.59), 1280: (1.79, 2.43, 2.10, 2.20, 2.50)},
    (16, wl.DUNGEON): {64: (1.28, .80, 1.05, 1.04, 1.63), 512: (1.46, 1.46, 1.25, 1.21, 1.75), 768: (1.66, 2.09, 2.06, 2.08, 1.82),
                       1024: (1.68, 2.71, 2.27, 2.35, 3.25), 1280: (2.50, 3.40, 3.09, 3.10, 3.58)},
    (32, wl.DUNGEON): {64: (1.39, .76, .97, .95, 1.44), 512: (1.56, 1.39, 1.18, 1.13, 1.54), 768: (1.75, 1.98, 1.88, 1.86, 1.65),
                       1024: (1.81, 2.57, 2.12, 2.17, 2.81), 1280: (2.44, 3.19, 2.83, 2.82, 3.21)},
    (64, wl.DUNGEON): {64: (1.52, .91, 1.07, 1.10, 1.53), 512: (1.75, 1.23, 1.36, 1.35, 1.66), 768: (2.00, 1.80, 1.57, 1.55, 1.81),
                       1024: (2.06, 2.65, 2.17, 2.17, 1.96), 1280: (2.58, 2.88, 2.55, 2.71, 3.16)}}
RELAY_SHAPES = [(0, 0), (4, 4), (4, 2), (2, 2), (2, 1)]


@pytest.mark.parametrize("rows,problem", sorted(RELAY_TIMES))
def test_the_relay_takes_the_shape_that_was_fastest(rows, problem):
    """For the kernels as they are built now; within 7 %, which is what the shapes of a size class that the rule
    takes as one lie apart."""
    for batch, times in RELAY_TIMES[rows, problem].items():
        got = relay_rule.shape(**relay_rule.case_of(wl.make_config(problem, batch, rows, 31, obs_pitch=-1), 32, 32))
        assert times[RELAY_SHAPES.index(got)] <= 1.07 * min(times), (batch, got, times)


def test_the_relay_is_left_where_it_does_not_pay():
    """Rollouts of a step or two, observations that the stores are the time of, slots that leave a step to
    one observer, and workgroups that would not fit their compute unit together."""
    case = dict(rows=32, binary=0, per_simd=6, compute_units=256, workgroups=64, observers=1, obs_bytes=4805, step_bytes=64 * 4805,
                lds_tables=4000, lds_observer=700, steps=32, slots=32)
    shape = lambda **more: relay_rule.shape(**dict(case, **more))  # noqa: E731
    assert shape() == (4, 4) and shape(workgroups=512) == (4, 4) and shape(workgroups=513) == (4, 2) and shape(workgroups=769) == (2, 1)
    assert [shape(steps=n, slots=n) for n in (1, 2, 3)] == [(0, 0), (0, 0), (4, 4)]
    assert [shape(binary=1, steps=n, slots=n) for n in (1, 2)] == [(0, 0), (4, 4)]
    assert shape(rows=16, per_simd=5, workgroups=512, steps=8, slots=8) == (0, 0) and shape(rows=16, per_simd=5, workgroups=512) == (2, 2)
    assert shape(step_bytes=11 << 20) == (4, 4) and shape(step_bytes=(11 << 20) + 1) == (0, 0)
    assert [shape(slots=n) for n in (1, 2, 3, 4, 6, 7, 8, 31)] == [(4, n) for n in (1, 2, 1, 4, 2, 1, 4, 1)]
    assert shape(rows=64, binary=1, obs_bytes=11907, slots=1) == (0, 0) and shape(rows=64, binary=1, obs_bytes=11907) == (4, 4)
    assert [shape(observers=n) for n in (2, 4)] == [(4, 2), (4, 1)] and shape(observers=2, slots=1) == (4, 1)
    assert shape(lds_observer=16 * 1024) == (0, 0) and shape(lds_observer=15 * 1024) == (4, 4)
    assert shape(workgroups=768, lds_observer=25 * 1024) == (0, 0) and shape(workgroups=768, lds_observer=24 * 1024) == (4, 2)


def test_compiled_call_path_leaves_doubtful_arguments_to_the_python_checks():
    """Tensors that are not on the device, arguments that are missing or no tensors, and a closed
    environment are answered with LOOK, before any library call (no GPU is touched; device tensors of
    a wrong type or shape are tested on the GPU)."""
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


def test_compiled_call_path_belongs_to_one_torch_and_one_interpreter(monkeypatch, tmp_path):
    """The compiled part of the binding is looked for under a name that changes with torch and with
    the interpreter, is built where that one is missing, and a file that cannot be loaded is
    reported as the binding reports everything else."""
    import shutil
    import sysconfig
    import torch
    here = binding._load_py().__file__
    monkeypatch.setattr(build, "LIB_DIR", str(tmp_path))
    built = []
    monkeypatch.setattr(build, "build_py", lambda: built.append(shutil.copy(here, build.py_lib())))
    monkeypatch.setattr(binding, "_py", None)
    binding._load_py()
    assert len(built) == 1
    monkeypatch.setattr(binding, "_py", None)
    binding._load_py()
    assert len(built) == 1                          # (there now)
    monkeypatch.setattr(torch, "__version__", "0.0.1")
    monkeypatch.setattr(binding, "_py", None)
    binding._load_py()
    assert len(built) == 2 and "0.0.1" in built[1]
    monkeypatch.setattr(sysconfig, "get_config_var", lambda name: "other-" + name)
    monkeypatch.setattr(binding, "_py", None)
    binding._load_py()
    assert len(built) == 3 and "other-SOABI" in built[2]
    monkeypatch.setattr(torch, "__version__", "0.0.2")
    open(build.py_lib(), "wb").write(b"no module")
    monkeypatch.setattr(binding, "_py", None)
    with pytest.raises(binding.PcgrlError, match="cannot be loaded"):
        binding._load_py()


INDEX = """
#include "pcgrl_index.h"
extern "C" void grid(uint32_t batch, uint32_t cells, int with_cells, uint32_t* out) {
  const pcgrl::GetGrid g = pcgrl::get_grid(batch, cells, with_cells != 0);
  out[0] = g.x; out[1] = g.y;
}
extern "C" void piece(uint32_t bx, uint32_t by, int thread, uint32_t batch, int cells, int max_w, int64_t* out) {
  const pcgrl::GetPiece p = pcgrl::get_piece(bx, by, thread, batch, cells, max_w);
  out[0] = (int64_t)p.at; out[1] = p.n; out[2] = p.env; out[3] = p.y; out[4] = p.x;
  out[5] = (int64_t)pcgrl::get_level(bx, by, thread);
}
// how often `divided` is wrong for this divisor, and by how much its product of reciprocals falls short at the most
extern "C" void wrong(uint32_t by, int64_t* out) {
  const uint32_t r = pcgrl::get_sizes(1, (int)by, (int)by).per_level, most = 0xffffffffu, last = most / by;
  out[0] = out[1] = 0;
  for (int i = 0; i < 64; ++i) {
    const uint32_t k = i < 24 ? (uint32_t)i : i < 48 ? last - (uint32_t)(i - 24) : (uint32_t)((uint64_t)last * (uint64_t)(i - 47) / 17);
    const uint32_t at[] = {k * by, k * by - 1, k * by + 1, most - (uint32_t)i};
    for (uint32_t n : at) {
      uint32_t rest = 0;
      const uint32_t q = pcgrl::divided(n, by, r, rest);
      const int64_t less = (int64_t)(n / by) - (int64_t)(((uint64_t)n * r) >> 32);
      out[0] += q != n / by || rest != n % by;
      out[1] = less > out[1] ? less : out[1];
    }
  }
}
"""


@pytest.fixture(scope="module")
def index(tmp_path_factory):
    import subprocess
    d = tmp_path_factory.mktemp("index")
    (d / "index.cpp").write_text(INDEX)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2408_12525_amd", "csrc"),
                    str(d / "index.cpp"), "-o", str(d / "index.so")], check=True)
    lib = C.CDLL(str(d / "index.so"))
    u32, p64 = C.c_uint32, C.POINTER(C.c_int64 * 6)
    lib.grid.argtypes, lib.grid.restype = [u32, u32, C.c_int, C.POINTER(u32 * 2)], None
    lib.piece.argtypes, lib.piece.restype = [u32, u32, C.c_int, u32, C.c_int, C.c_int, p64], None
    lib.wrong.argtypes, lib.wrong.restype = [u32, C.POINTER(C.c_int64 * 2)], None
    return lib


def test_divisions_by_reciprocals_need_one_correction(index):
    out, most = (C.c_int64 * 2)(), 0
    for by in range(1, 4097):                      # cells of a level, and of a row
        index.wrong(by, C.byref(out))
        assert out[0] == 0, by
        most = max(most, out[1])
    assert most == 1


@pytest.mark.parametrize("batch,h,w", [(1, 1, 1), (300, 1, 1), (5, 3, 7), (1, 64, 64), (37, 27, 45), (2051, 2, 64), (8388608, 64, 64), (8388609, 64, 64),
                                       (8388613, 63, 61), (1 << 24, 64, 64), ((1 << 24) - 1, 64, 63), (1 << 24, 16, 16), (1 << 24, 1, 1)])
def test_get_state_indices_at_every_batch(index, batch, h, w):
    """What the threads of the plain-layout kernel address, from one cell to the largest batch there
    can be: a launch below 2^32 threads either way, workgroups numbered without a gap, every piece
    inside the arrays and where it belongs, and every level's scalars written by the one thread of
    that number (from 2^31 threads on the numbers are no 32-bit integers any more)."""
    cells, total = h * w, batch * h * w
    g, out = (C.c_uint32 * 2)(), (C.c_int64 * 6)()
    for with_cells in (1, 0):
        index.grid(batch, cells, with_cells, C.byref(g))
        gx, gy = g
        want = -(-max(-(-total // 16) if with_cells else 0, batch) // 256)
        assert gx * 256 < 1 << 31 and 1 <= gy < 1 << 16 and gx * gy >= want > gx * (gy - 1)
        for b in sorted({b for b in (0, 1, want // 3, batch // 256, 1 << 22, (1 << 23) - 1, 1 << 23, want - 1, gx * gy - 1) if b < gx * gy}):
            for t in range(256):
                index.piece(b % gx, b // gx, t, batch, cells, w, C.byref(out))
                at, n, env, y, x, level = out
                assert level == b * 256 + t and at == 16 * level and n == max(0, min(16, total - at))
                if n:
                    assert (env, y, x) == (at // cells, at % cells // w, at % cells % w) and env < batch


def test_spans_cover_a_rollout_and_fit_their_room():
    rng = random.Random(7)
    cut = 0
    for _ in range(20000):
        batch, steps = int(2 ** rng.uniform(0, 24)), int(2 ** rng.uniform(0, 20))
        case = dict(rows=rng.choice([16, 32, 64]), problem=rng.choice([wl.BINARY, wl.MAZE, wl.DUNGEON]), observed=rng.random() < .5, batch=batch, steps=steps,
                    cells=rng.choice([9, 300, 1024, 4096]), max_w=rng.choice([3, 16, 40, 64]), obs_bytes=rng.choice([75, 4864, 19845]), window_bits=rng.choice([75, 8000, 19845]), episode=rng.choice([0, 30, 150, 1000]))
        case["step_bytes"] = case["obs_bytes"] * batch if case["observed"] else 0
        spans, each, room = span_rule.shape_and_room(**case)
        assert spans == 1 and each == steps or spans > 1 and (spans - 1) * each < steps <= spans * each, case
        assert spans == 1 or spans * batch <= room <= min(256 * batch, 8192 if case["rows"] == 64 else 16384), case
        cut += spans > 1
    assert cut > 2000
    # where cutting up begins to pay, and where the stores are what a rollout waits for
    shape = lambda **more: span_rule.shape(**dict(dict(rows=16, problem=wl.BINARY, observed=1, batch=64, steps=256, cells=256, max_w=16, obs_bytes=1922, window_bits=1922, step_bytes=64 * 1922, episode=1000), **more))  # noqa: E731
    assert shape() == (64, 4) and shape(steps=11) == (1, 11) and shape(steps=12) == (12, 1)
    assert shape(step_bytes=9 << 20) == (64, 4) and shape(step_bytes=(9 << 20) + 1) == (1, 256)
    assert shape(rows=64) == (32, 8) and shape(rows=64, steps=19) == (1, 19) and shape(rows=32, batch=1536, problem=wl.MAZE) == (2, 128)
    assert shape(batch=4096) == (1, 256) and shape(batch=4096, observed=0, step_bytes=0) == (4, 64) and shape(batch=4097, observed=0, step_bytes=0) == (1, 256)


@pytest.mark.parametrize("problem,rows,ow,batch,whole,cut,more", [
    # (rollouts of so many steps: one that is faster in one piece, one that is faster cut up)
    (wl.DUNGEON, 64, 9, 64, 20, 30, {}), (wl.DUNGEON, 64, 31, 256, 42, 50, {}), (wl.MAZE, 64, 9, 64, 20, 30, {}), (wl.MAZE, 64, 9, 256, 34, 51, {}),
    (wl.BINARY, 64, 9, 64, 16, 20, {}), (wl.DUNGEON, 64, 31, 768, 256, None, {}), (wl.DUNGEON, 64, 31, 640, 50, 72, {}), (wl.DUNGEON, 16, 34, 917, 10, 16, {}), (wl.DUNGEON, 64, 63, 231, 24, 32, dict(h=64, max_w=56)),
    (wl.MAZE, 32, 9, 256, 16, 24, {}), (wl.DUNGEON, 32, 9, 256, 20, 24, {}), (wl.BINARY, 32, 31, 64, 12, 16, {}),
    (wl.DUNGEON, 16, 9, 256, 12, 18, {}), (wl.MAZE, 16, 9, 3072, 12, 18, {}), (wl.BINARY, 16, 9, 2048, 12, 18, {}), (wl.BINARY, 16, 9, 1536, 10, 12, {}),
    # smaller levels
    (wl.DUNGEON, 64, 31, 165, 24, 36, dict(h=8, max_w=54)), (wl.DUNGEON, 64, 49, 261, 24, 32, dict(h=32, max_w=48)), (wl.DUNGEON, 32, 9, 256, 14, 18, dict(max_w=17)),
    (wl.DUNGEON, 64, 9, 64, 18, 20, dict(max_w=8, max_changes=40)), (wl.DUNGEON, 64, 9, 64, 18, 25, dict(min_size=8, min_w=8)),
    # stores that spill from the cache
    (wl.MAZE, 16, 63, 256, 96, 36, {}), (wl.MAZE, 16, 63, 320, 10, 96, {}), (wl.MAZE, 16, 63, 448, 18, None, {}), (wl.DUNGEON, 16, 63, 256, 42, 21, {}),
    # levels that start again on the way
    (wl.DUNGEON, 64, 9, 64, 36, 45, dict(max_changes=150)), (wl.DUNGEON, 64, 9, 768, 640, None, dict(max_changes=40)), (wl.DUNGEON, 64, 31, 397, 60, 246, dict(h=30, max_w=48, max_changes=63, obs_format=1)), (wl.MAZE, 64, 9, 512, 73, 159, dict(max_steps=30)), (wl.BINARY, 64, 9, 1024, 120, None, dict(max_steps=30)),
    (wl.DUNGEON, 64, 9, 64, 20, 30, dict(max_steps=30, autoreset=0)), (wl.DUNGEON, 32, 9, 256, 29, 43, dict(max_changes=150)), (wl.DUNGEON, 16, 9, 64, 13, 18, dict(max_changes=150)), (wl.DUNGEON, 64, 15, 634, 72, 116, dict(max_changes=74)),
    (wl.DUNGEON, 32, 38, 345, 14, 32, dict(max_changes=195))])
def test_rollouts_are_cut_into_spans_where_that_is_ahead(problem, rows, ow, batch, whole, cut, more):
    more = dict(more)
    cfg = wl.make_config(problem, batch, more.pop("h", rows), ow, obs_pitch=-1, **more)
    for steps, spans in ((whole, 0), (cut, 1)):
        assert steps is None or (span_rule.shape(**span_rule.case_of(cfg, steps, True))[0] > 1) == spans


@pytest.mark.parametrize("problem,ow,pitch,batch,one,many", [
    # (one: a single buffer, written through; many: a buffer for each step, so many that they do not fit the caches)
    (wl.DUNGEON, 18, -1, 32768, 0, 0), (wl.DUNGEON, 19, -1, 32768, 0, 0), (wl.DUNGEON, 19, 0, 32768, 0, 1), (wl.DUNGEON, 20, -1, 28000, 0, 1), (wl.DUNGEON, 21, -1, 32768, 1, 1),
    (wl.DUNGEON, 21, -1, 40000, 1, 0), (wl.DUNGEON, 23, -1, 32768, 1, 0), (wl.DUNGEON, 25, 0, 32768, 1, 1), (wl.MAZE, 23, -1, 40000, 0, 1),
    (wl.MAZE, 25, -1, 40000, 1, 1), (wl.MAZE, 25, -1, 50000, 1, 0), (wl.MAZE, 29, 0, 40000, 1, 1), (wl.MAZE, 29, -1, 40000, 1, 0), (wl.MAZE, 31, -1, 32768, 1, 1), (wl.BINARY, 31, -1, 50000, 1, 1),
    (wl.BINARY, 35, -1, 40000, 1, 0), (wl.DUNGEON, 23, 0, 50000, 0, 0), (wl.MAZE, 21, 0, 32768, 0, 0)])
def test_steps_of_large_batches_take_two_wavefronts_where_that_is_ahead(problem, ow, pitch, batch, one, many):
    cfg = wl.make_config(problem, batch, 32, ow, obs_pitch=pitch)
    large = host_rule.obs_stride(cfg) * batch >= 128 << 20 and wl.obs_bytes(cfg) >= 3072
    assert split_rule.step(cfg, "through") == one and split_rule.step(cfg, "cached" if large else "stream") == many


@pytest.mark.parametrize("problem,rows,ow,pitch,batch,slots,store,two", [
    # a ring that the cache holds, one that it does not, and one that is not stored through it
    (wl.MAZE, 64, 20, 0, 14000, 8, "cached", 1), (wl.MAZE, 64, 20, 0, 16000, 8, "cached", 0), (wl.MAZE, 64, 20, 0, 12000, 16, "cached", 0), (wl.MAZE, 64, 20, 0, 24000, 48, "stream", 1),
    (wl.BINARY, 64, 25, -1, 20000, 8, "cached", 0), (wl.BINARY, 64, 9, -1, 24001, 48, "cached", 1), (wl.BINARY, 64, 9, -1, 32768, 48, "cached", 0),
    (wl.DUNGEON, 64, 9, 0, 32768, 8, "cached", 1), (wl.DUNGEON, 64, 14, 0, 10887, 16, "cached", 1), (wl.DUNGEON, 64, 15, 0, 20000, 8, "cached", 0), (wl.DUNGEON, 64, 9, 0, 50000, 8, "cached", 0), (wl.MAZE, 64, 9, 0, 50000, 8, "cached", 0),
    (wl.DUNGEON, 32, 25, 0, 4097, 8, "cached", 1), (wl.DUNGEON, 32, 25, 0, 4097, 16, "cached", 1),
    (wl.DUNGEON, 32, 25, 0, 4097, 48, "cached", 0), (wl.DUNGEON, 32, 23, -1, 4097, 48, "cached", 1), (wl.DUNGEON, 32, 23, -1, 4608, 48, "cached", 0), (wl.DUNGEON, 32, 21, -1, 5120, 48, "cached", 1), (wl.MAZE, 32, 25, -1, 5120, 48, "cached", 1), (wl.MAZE, 32, 15, 0, 120000, 8, "stream", 1),
    (wl.MAZE, 32, 15, 0, 200000, 8, "stream", 0), (wl.MAZE, 32, 45, 0, 10240, 48, "cached", 0), (wl.DUNGEON, 32, 35, 0, 10240, 8, "cached", 0)])
def test_rollouts_of_large_batches_take_two_wavefronts_where_that_is_ahead(problem, rows, ow, pitch, batch, slots, store, two):
    assert split_rule.rollout(wl.make_config(problem, batch, rows, ow, obs_pitch=pitch), slots, store) == two
