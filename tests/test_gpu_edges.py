"""GPU kernels vs the oracle at the sizes where their splits can go wrong (needs an MI355X)."""
import numpy as np
import pytest
import torch

import oracle
import relay_rule
import span_rule
from parity import assert_same, check_obs, compare_state
from paper_2408_12525_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


def _plain_levels(problem, B, h, w, seed, p_wall=None):
    """Random levels in the plain layout, some codes of them no tile of the problem, ragged shapes,
    positions inside and outside."""
    rng = np.random.default_rng(seed)
    K = wl.NUM_TILES[problem]
    if p_wall is None:
        tiles = rng.integers(-2, K + 3, size=(B, h, w)).astype(np.int8)
    else:
        tiles = (rng.random((B, h, w)) < p_wall).astype(np.int8)
    frozen = ((rng.random((B, h, w)) < 0.2) * rng.integers(1, 256, size=(B, h, w))).astype(np.uint8)
    hw = np.stack([rng.integers(1, h + 1, B), rng.integers(1, w + 1, B)], 1).astype(np.int16)
    hw[0] = (h, w)
    pos = rng.integers(-1, 70, size=(B, 2)).astype(np.int16)
    return tiles, frozen, hw, pos


@pytest.mark.parametrize("problem,B,h,w,per_wave", [
    (wl.BINARY, 1, 1, 1, 0), (wl.MAZE, 37, 16, 16, 0), (wl.DUNGEON, 2051, 11, 3, 0), (wl.BINARY, 65, 3, 32, 0), (wl.MAZE, 4099, 31, 17, 0),
    (wl.DUNGEON, 19, 27, 45, 0), (wl.BINARY, 9, 64, 64, 0), (wl.DUNGEON, 5, 2, 64, 0), (wl.MAZE, 7, 63, 5, 0),
    # several levels a wavefront, the last one partly filled, rows that start at odd bits of the run
    (wl.DUNGEON, 37, 11, 3, 2), (wl.DUNGEON, 37, 11, 3, 4), (wl.BINARY, 419, 13, 7, 2), (wl.BINARY, 419, 13, 7, 4), (wl.MAZE, 38, 16, 16, 4),
    (wl.MAZE, 3, 16, 16, 4), (wl.BINARY, 2, 1, 1, 4), (wl.MAZE, 37, 31, 17, 2), (wl.DUNGEON, 5, 32, 32, 2)])
@pytest.mark.parametrize("with_frozen", [True, False])
def test_plain_levels_in_and_out(problem, B, h, w, per_wave, with_frozen):
    """pcgrl_set_state and pcgrl_get_state where rows, levels and the 16-byte pieces they are read
    and written in end at different places, with one and several levels in a wavefront."""
    cfg = wl.make_config(problem, B, h, 5, max_w=w, min_size=1, min_w=1, autoreset=0, levels_per_wave=per_wave)
    gpu, cpu = binding.Pcgrl(cfg, 0), oracle.Oracle(cfg)
    gpu.pcgrl_reset(3)
    cpu.reset(3)
    tiles, frozen, hw, pos = _plain_levels(problem, B, h, w, B + h)
    frozen = frozen if with_frozen else None
    # arrays that do not start on a 16-byte boundary, with guard bytes behind them
    def shifted(a, by):
        buf = torch.full((a.size + 64,), 0x55, dtype=torch.uint8, device=DEV)
        buf[by:by + a.size] = torch.from_numpy(a.reshape(-1).view(np.uint8)).to(DEV)
        return buf[by:by + a.size].view(torch.int8 if a.dtype == np.int8 else torch.uint8).view(a.shape)
    gpu.pcgrl_set_state(shifted(tiles, 7), None if frozen is None else shifted(frozen, 13),
                        torch.from_numpy(hw).to(DEV), torch.from_numpy(pos).to(DEV))
    # (what the library makes of it: unknown codes count as tile 0, positions are clamped)
    known = np.where((tiles < 0) | (tiles >= wl.NUM_TILES[problem]), 0, tiles).astype(np.int8)
    cpu.set_state(known, frozen, hw, np.clip(pos, 0, hw - 1).astype(np.int16))
    compare_state(gpu, cpu, "after set_state")
    assert_same("metrics", gpu.pcgrl_metrics(), cpu.metrics(), "after set_state")
    assert_same("obs", gpu.pcgrl_observe(), cpu.observe(), "after set_state")
    n = B * h * w
    for by in (0, 5):
        t, f = (torch.full((n + 32,), 0x77, dtype=torch.uint8, device=DEV) for _ in range(2))
        rc = gpu.L.pcgrl_get_state(gpu.h, t.data_ptr() + by, f.data_ptr() + by, None, None, None, gpu._st())
        assert rc == 0
        st = cpu.get_state()
        assert_same("tiles", t[by:by + n].view(torch.int8).view(B, h, w), st["tiles"], f"offset {by}")
        assert_same("frozen", f[by:by + n].view(B, h, w), st["frozen"], f"offset {by}")
        for buf in (t, f):
            assert bool((buf[by + n:] == 0x77).all()) and bool((buf[:by] == 0x77).all())
    acts = wl.random_actions(cfg, 4, 12)
    for t in range(12):
        gpu.pcgrl_step(torch.from_numpy(acts[t]).to(DEV))
        cpu.step(acts[t], want_obs=False)
    assert_same("metrics", gpu.pcgrl_metrics(), cpu.metrics(), "after edits")
    gpu.close()


def _loop(h, w):
    """A serpentine closed to one loop by a way back along the first column."""
    n = (h + 1) // 4 * 2
    t = np.ones((h, w), np.int8)
    for i in range(n):
        t[2 * i, 2:] = 0
        if i < n - 1:
            t[2 * i + 1, w - 1 if i % 2 == 0 else 2] = 0
    t[0, :2] = t[2 * n - 2, :2] = 0
    t[:2 * n - 1, 0] = 0
    return t


@pytest.mark.parametrize("h,w,per_wave", [
    (16, 16, 0), (13, 7, 0), (32, 32, 0), (5, 32, 0), (64, 64, 0), (64, 33, 0),
    (16, 16, 2), (16, 16, 4), (13, 7, 2), (13, 7, 4), (32, 32, 2), (5, 32, 2)])
def test_exact_diameter_prunes_no_longest_path(h, w, per_wave):
    """The exact diameter on maps of every density (one huge component to none), rooms, corridors,
    rings and loops, for one and several parts per level, each level in a wavefront of its own (or
    in all of its lane groups) and together with different ones, the last wavefront partly filled."""
    rng = np.random.default_rng(h * 100 + w)
    maps = [(rng.random((h, w)) < d).astype(np.int8) for d in (0, .05, .2, .3, .35, .4, .42, .45, .5, .5, .6, .8, 1)]
    y, x = np.mgrid[:h, :w]
    maps += [((y % 2 == 1) & (x != np.where(y % 4 == 1, w - 1, 0))).astype(np.int8),         # a serpentine
             (np.minimum(np.minimum(y, h - 1 - y), np.minimum(x, w - 1 - x)) % 2).astype(np.int8),  # nested rings
             ((y % 4 == 0) & (x % 7 != 3)).astype(np.int8),                                  # rooms with doors
             ((x % 2 == 1) & (y > 0)).astype(np.int8),                                       # a comb
             ((y + x) % 2).astype(np.int8)]                                                  # single cells
    # loops beside levels of nothing, a few cells and another loop
    maps += [_loop(h, w), np.ones((h, w), np.int8), np.ascontiguousarray(_loop(h, w)[::-1]), (rng.random((h, w)) < .9).astype(np.int8),
             ((y % 4 != 0) & (x % 4 != 0)).astype(np.int8)]                                  # corridors all round blocks
    maps += [(rng.random((h, w)) < .5).astype(np.int8) for _ in range(396)]
    tiles = np.stack(maps)
    B = len(tiles)
    hw = np.full((B, 2), (h, w), np.int16)
    cfg = wl.make_config(wl.BINARY, B, h, 5, max_w=w, min_size=1, min_w=1, autoreset=0, levels_per_wave=per_wave)
    gpu, cpu = binding.Pcgrl(cfg, 0), oracle.Oracle(cfg)
    gpu.pcgrl_reset(1)
    cpu.reset(1)
    gpu.pcgrl_set_state(torch.from_numpy(tiles).to(DEV), None, torch.from_numpy(hw).to(DEV), torch.zeros_like(torch.from_numpy(hw)).to(DEV))
    cpu.set_state(tiles, None, hw, np.zeros_like(hw))
    want = cpu.exact_diameters()
    assert_same("exact diameters", gpu.pcgrl_exact_diameter(), want, (h, w))
    for parts_log2 in (0, 1, 4):
        got = gpu.pcgrl_exact_diameter_static(torch.empty(B, dtype=torch.int32, device=DEV), parts_log2)
        assert_same("exact diameters", got, want, (h, w, parts_log2))
    gpu.close()


def test_exact_diameter_shares_out_a_loop():
    """The cells of one long loop are all equally far from their farthest one, so that half of them
    are swept, each on its own: with 16 wavefronts at that, a level takes less than a quarter of the
    time of one."""
    n = 64
    tiles = _loop(n, n)[None]
    hw = torch.full((1, 2), n, dtype=torch.int16, device=DEV)
    gpu = binding.Pcgrl(wl.make_config(wl.BINARY, 1, n, 5, min_size=1, autoreset=0), 0)
    gpu.pcgrl_reset(1)
    gpu.pcgrl_set_state(torch.from_numpy(tiles).to(DEV), None, hw, torch.zeros_like(hw))
    out = torch.empty(1, dtype=torch.int32, device=DEV)
    took = {}
    for parts_log2 in (4, 0, 4, 0):
        begin, end = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        begin.record()
        gpu.pcgrl_exact_diameter_static(out, parts_log2)
        end.record()
        torch.cuda.synchronize()
        assert int(out[0]) == 1040  # half of the loop's 2080 cells
        took[parts_log2] = begin.elapsed_time(end)
    assert took[4] < took[0] / 4, took
    gpu.close()


@pytest.mark.parametrize("parts_log2", [0, 1, 2, 3, 4])
def test_exact_diameter_components_in_both_words_of_a_row(parts_log2):
    """64-column levels of hooks and zigzags whose first cell lies in the upper half of its row and
    the others in the lower half (two words of the set that the wavefronts of a workgroup take
    components from), some of them small enough to be dropped unswept once a longer one is known."""
    rng = np.random.default_rng(parts_log2)
    B, n = 300, 64
    tiles = np.ones((B, n, n), np.int8)
    for b in range(B):
        y = 0
        while y < n - 1:
            rows = int(rng.integers(2, min(6, n - y + 1)))
            for k in range(rows):
                lo, hi = ((32, 33 + rng.integers(0, 20)) if k == 0 else (33 - rng.integers(1, 30), 33))
                tiles[b, y + k, int(lo):int(hi)] = 0
            tiles[b, y:y + rows, 32] = 0
            y += rows + 1
    hw = np.full((B, 2), n, np.int16)
    cfg = wl.make_config(wl.BINARY, B, n, 5, min_size=1, autoreset=0)
    gpu, cpu = binding.Pcgrl(cfg, 0), oracle.Oracle(cfg)
    gpu.pcgrl_reset(1)
    cpu.reset(1)
    gpu.pcgrl_set_state(torch.from_numpy(tiles).to(DEV), None, torch.from_numpy(hw).to(DEV), torch.zeros((B, 2), dtype=torch.int16, device=DEV))
    cpu.set_state(tiles, None, hw, np.zeros_like(hw))
    want = cpu.exact_diameters()
    for _ in range(5):
        got = gpu.pcgrl_exact_diameter_static(torch.empty(B, dtype=torch.int32, device=DEV), parts_log2)
        assert_same("exact diameters", got, want, parts_log2)
    gpu.close()


@pytest.mark.parametrize("problem,h,w,per_wave", [
    (wl.BINARY, 16, 16, 0), (wl.MAZE, 16, 16, 1), (wl.DUNGEON, 5, 3, 4), (wl.BINARY, 3, 3, 2), (wl.BINARY, 1, 7, 4), (wl.MAZE, 9, 2, 0),
    (wl.BINARY, 32, 32, 2), (wl.DUNGEON, 32, 9, 1), (wl.MAZE, 17, 31, 2), (wl.BINARY, 64, 64, 0), (wl.DUNGEON, 2, 64, 0), (wl.MAZE, 64, 33, 0),
    (wl.BINARY, 64, 1, 0)])
def test_every_ring_around_the_edited_cell(problem, h, w, per_wave):
    """The region update after one edit, for all 256 patterns of walls around the cell, in the middle
    of a map, on each side and in each corner of it (where the ring is partly outside), in random
    surroundings from open to dense; the cell walled up and opened."""
    rng = np.random.default_rng(10 * h + w)
    ys, xs = sorted({0, h // 2, h - 1}), sorted({0, w // 2, w - 1})
    places = [(y, x) for y in ys for x in xs]
    ring = [(-1, -1), (-1, 0), (-1, 1), (0, 1), (1, 1), (1, 0), (1, -1), (0, -1)]
    levels, pos, acts = [], [], []
    for y, x in places:
        for pattern in range(256):
            t = (rng.random((h, w)) < rng.choice([.2, .4, .5])).astype(np.int8)
            for b, (dy, dx) in enumerate(ring):
                if 0 <= y + dy < h and 0 <= x + dx < w:
                    t[y + dy, x + dx] = pattern >> b & 1
            t[y, x] = pattern & 1 ^ (y + x) & 1
            levels.append(t)
            pos.append((y, x))
            acts.append(1 - t[y, x])
    B = len(levels)
    cfg = wl.make_config(problem, B, h, 5, max_w=w, min_size=1, min_w=1, autoreset=0, levels_per_wave=per_wave)
    gpu, cpu = binding.Pcgrl(cfg, 0), oracle.Oracle(cfg)
    gpu.pcgrl_reset(3)
    cpu.reset(3)
    tiles, hw = np.stack(levels), np.tile(np.array([h, w], np.int16), (B, 1))
    pos, acts = np.array(pos, np.int16), np.array(acts, np.int32)
    gpu.pcgrl_set_state(torch.from_numpy(tiles).to(DEV), None, torch.from_numpy(hw).to(DEV), torch.from_numpy(pos).to(DEV))
    cpu.set_state(tiles, None, hw, pos)
    assert_same("metrics", gpu.pcgrl_metrics(), cpu.metrics(), "before the edit")
    gpu.pcgrl_step(torch.from_numpy(acts).to(DEV))
    cpu.step(acts, want_obs=False)
    assert_same("metrics", gpu.pcgrl_metrics(), cpu.metrics(), "after the edit")
    gpu.close()


def _spiral(n):
    """A corridor that winds inwards and the wall beside it, each one cell wide."""
    t = np.ones((n, n), np.int8)
    y, x, dy, dx = 0, 0, 0, 1
    t[0, 0] = 0
    while True:
        for _ in range(2):  # straight on, or round the corner once
            a, b, c, d = y + dy, x + dx, y + 2 * dy, x + 2 * dx
            if 0 <= a < n and 0 <= b < n and t[a, b] == 1 and not (0 <= c < n and 0 <= d < n and t[c, d] == 0):
                break
            dy, dx = dx, -dy
        else:
            return t
        y, x = y + dy, x + dx
        t[y, x] = 0


@pytest.mark.parametrize("n", [16, 31, 64])
def test_regions_of_winding_walls(n):
    """The from-scratch region count where a flood through the walls takes longer than it is allowed
    to (next to levels where it does not, some in the same wavefront), and edits along such walls."""
    spiral = _spiral(n)
    cut = spiral.copy()
    cut[n // 2] = 1
    wall_only = 1 - spiral
    comb = np.ones((n, n), np.int8)
    comb[1::2, 1:] = 0
    few = np.zeros((n, n), np.int8)
    few[n // 3, n // 4:n // 2] = 1
    levels = [spiral, few, cut, wall_only, comb, spiral.T.copy(), np.ones_like(few), np.zeros_like(few), spiral[::-1, ::-1].copy()]
    tiles = np.stack(levels * 3)
    B = len(tiles)
    hw, pos = np.full((B, 2), n, np.int16), np.random.default_rng(n).integers(0, n, (B, 2)).astype(np.int16)
    for mode in (wl.REGIONS_INCREMENTAL, wl.REGIONS_RECOUNT):
        cfg = wl.make_config(wl.BINARY, B, n, 5, autoreset=0, pos_mode=wl.POS_RANDOM, levels_per_wave=4, regions_mode=mode)
        gpu, cpu = binding.Pcgrl(cfg, 0), oracle.Oracle(cfg)
        gpu.pcgrl_reset(3)
        cpu.reset(3)
        gpu.pcgrl_set_state(torch.from_numpy(tiles).to(DEV), None, torch.from_numpy(hw).to(DEV), torch.from_numpy(pos).to(DEV))
        cpu.set_state(tiles, None, hw, pos)
        assert_same("metrics", gpu.pcgrl_metrics(), cpu.metrics(), "set_state")
        acts = wl.random_actions(cfg, 5, 40)
        for t in range(40):
            gpu.pcgrl_step(torch.from_numpy(acts[t]).to(DEV))
            cpu.step(acts[t], want_obs=False)
            assert_same("metrics", gpu.pcgrl_metrics(), cpu.metrics(), f"step {t}")
        gpu.close()


@pytest.mark.parametrize("problem", [wl.BINARY, wl.MAZE, wl.DUNGEON])
@pytest.mark.parametrize("B,h,w", [(5, 1, 1), (37, 16, 15), (9, 3, 31), (33, 32, 32), (7, 5, 33), (6, 64, 63), (5, 64, 64)])
def test_drawn_levels(problem, B, h, w):
    """First levels of pcgrl_reset where the 32 columns that are drawn together end at different
    places, with tiles that never or always come up (equal, lowest and highest thresholds)."""
    K = wl.NUM_TILES[problem]
    rng = np.random.default_rng(B + w)
    odds = [[1 / K] * K, [1.] + [0.] * (K - 1), [0.] * (K - 1) + [1.]]
    some = rng.random(K) * (rng.random(K) < .6)
    some[rng.integers(K)] += .1
    odds.append(list(some / some.sum()))
    for probs in odds:
        cfg = wl.make_config(problem, B, h, 5, max_w=w, min_size=1, min_w=1, probs=probs)
        gpu, cpu = binding.Pcgrl(cfg, 0), oracle.Oracle(cfg)
        gpu.pcgrl_reset(11)
        cpu.reset(11)
        compare_state(gpu, cpu, f"after reset, {probs}")
        assert_same("metrics", gpu.pcgrl_metrics(), cpu.metrics(), f"after reset, {probs}")
        gpu.close()


@pytest.mark.parametrize("problem,size,obs_w,frozen", [
    (wl.BINARY, 16, 1, 0), (wl.BINARY, 16, 6, 0), (wl.BINARY, 16, 13, 0), (wl.DUNGEON, 16, 8, 0), (wl.MAZE, 16, 5, 0), (wl.DUNGEON, 16, 4, 0), (wl.DUNGEON, 16, 63, 3)])
@pytest.mark.parametrize("dtype", [torch.uint8, torch.bfloat16, torch.float32])
def test_unpack_row_lengths(problem, size, obs_w, frozen, dtype):
    """pcgrl_unpack_obs on packed rows of less than 16 bytes, of about 16, and of the most there can
    be, at an odd address, into an array that starts off a 16-byte boundary; guards stay as they are."""
    B = 11
    cfg = wl.make_config(problem, B, size, obs_w, obs_format=1, n_frozen=frozen, obs_frozen_channel=1 if frozen else 0)
    gpu, cpu = binding.Pcgrl(cfg, 0), oracle.Oracle(cfg)
    obs = gpu.new_obs()
    gpu.pcgrl_reset(5, obs)
    want = torch.from_numpy(cpu.reset(5)).to(dtype)
    for by in (0, 1, 7):
        src = torch.full((obs.numel() + 32,), 0xff, dtype=torch.uint8, device=DEV)
        src[by:by + obs.numel()] = obs.reshape(-1)
        buf = torch.full((want.numel() + 32,), 7, dtype=dtype, device=DEV)
        out = buf[by:by + want.numel()].view(want.shape)
        gpu.pcgrl_unpack_obs(src[by:by + obs.numel()].view(obs.shape), out=out)
        assert torch.equal(out.cpu(), want), by
        assert bool((buf[:by] == 7).all()) and bool((buf[by + want.numel():] == 7).all()), by
    gpu.close()


def _spoilt(t, wrong):
    """A tensor like t with one property that is not t's."""
    if wrong == "type":
        return torch.zeros(t.shape, dtype=torch.int64, device=DEV)
    if wrong == "size":
        return torch.zeros(t.shape[:-1] + (t.shape[-1] + 1,), dtype=t.dtype, device=DEV)
    if wrong == "first size":
        return torch.zeros((t.shape[0] + 1,) + t.shape[1:], dtype=t.dtype, device=DEV)
    if wrong == "stride":
        return torch.zeros(t.shape[:-1] + (2 * t.shape[-1],), dtype=t.dtype, device=DEV)[..., ::2]
    if wrong == "one more dimension":
        return torch.zeros((1,) + t.shape, dtype=t.dtype, device=DEV)
    if wrong == "one dimension less":
        return torch.zeros(t.shape[1:], dtype=t.dtype, device=DEV)
    return torch.zeros(t.shape, dtype=t.dtype)  # "device"


@pytest.mark.parametrize("wrong", ["type", "size", "first size", "stride", "one more dimension", "one dimension less", "device"])
@pytest.mark.parametrize("packed", [False, True])
def test_every_argument_of_every_call_is_checked(wrong, packed):
    """Device tensors with one property wrong, one at a time, in every place of every call that goes
    through the compiled path: answered with LOOK there and with PcgrlError by the binding; what
    is right is taken."""
    B, T = 5, 4
    cfg = wl.make_config(wl.MAZE, B, 9, 6, max_w=11, min_size=1, min_w=1, obs_format=int(packed))
    gpu = binding.Pcgrl(cfg, 0)
    z = lambda shape, dtype: torch.zeros(tuple(shape), dtype=dtype, device=DEV)
    i8, u8, i16, i32, f32 = torch.int8, torch.uint8, torch.int16, torch.int32, torch.float32
    obs, grid, pair = tuple(gpu.obs_shape), (B, 9, 11), (B, 2)
    calls = dict(
        step=[z((B,), i32), z(obs, u8), z((B,), f32), z((B,), u8)],
        rollout=[z((T, B), i32), z((T,) + obs, u8), z((T, B), f32), z((T, B), u8)],
        reset=[7, z(obs, u8)], metrics=[z((B, gpu.M), i32)], exact_diameter=[z((B,), i32)], observe=[z(obs, u8)],
        set_state=[z(grid, i8), z(grid, u8), torch.full(pair, 3, dtype=i16, device=DEV), z(pair, i16)])
    if packed:
        calls["unpack_obs"] = [z(obs, u8), z(gpu.onehot_shape, f32)]
    gpu.pcgrl_reset(1)
    for name, args in calls.items():
        fast, method = getattr(gpu._env, name), getattr(gpu, "pcgrl_" + name)
        # (those of one argument take it alone, like every other caller of them)
        assert fast(*args) == 0, name
        method(*args)
        for i, t in enumerate(args):
            if not isinstance(t, torch.Tensor):
                continue
            if wrong == "first size" and name == "rollout" and i == 0:
                continue  # (another number of steps; then the others are wrong)
            bad = args[:i] + [_spoilt(t, wrong)] + args[i + 1:]
            rc = fast(*bad)
            # (more slots than steps is for the library to refuse)
            assert rc == (-2 if wrong == "first size" and name == "rollout" and i == 1 else binding._LOOK), (name, i)
            with pytest.raises(binding.PcgrlError):
                method(*bad)
    torch.cuda.synchronize()
    gpu.close()


def _rollouts_against_steps(cfg, T, S, observed=True):
    """Three rollouts of T steps into S slots, two single steps after each, against the oracle's steps."""
    B = cfg["batch"]
    gpu, cpu = binding.Pcgrl(cfg, 0), oracle.Oracle(cfg)
    gpu.pcgrl_reset(5)
    cpu.reset(5)
    for turn in range(3):
        acts = wl.random_actions(cfg, 30 + turn, T + 2, bad_fraction=0.05)
        obs = torch.zeros((S,) + tuple(gpu.obs_shape), dtype=torch.uint8, device=DEV)
        rew, done = torch.empty((T, B), dtype=torch.float32, device=DEV), torch.empty((T, B), dtype=torch.uint8, device=DEV)
        gpu.pcgrl_rollout(torch.from_numpy(acts[:T].copy()).to(DEV), obs if observed else None, rew, done)
        for t in range(T):
            o, r, d = cpu.step(acts[t])
            assert np.array_equal(rew[t].cpu().numpy(), r) and np.array_equal(done[t].cpu().numpy(), d), f"turn {turn} step {t}"
            if observed and t >= T - S:
                check_obs(gpu, obs[t % S], o, f"turn {turn} step {t}")
        assert_same("metrics", gpu.pcgrl_metrics(), cpu.metrics(), f"turn {turn}")
        assert_same("targets", gpu.pcgrl_get_targets(), cpu.get_targets(), f"turn {turn}")
        compare_state(gpu, cpu, f"turn {turn}")
        for t in range(T, T + 2):
            gpu.pcgrl_step(torch.from_numpy(acts[t]).to(DEV))
            cpu.step(acts[t], want_obs=False)
        assert_same("metrics", gpu.pcgrl_metrics(), cpu.metrics(), f"turn {turn}, single steps")
    gpu.close()


@pytest.mark.parametrize("problem,h,w,T,relay,more", [
    (wl.BINARY, 16, 16, 1, 0, {}), (wl.BINARY, 16, 16, 7, 1, dict(max_steps=8)), (wl.MAZE, 16, 16, 8, 1, dict(max_steps=8)),
    (wl.DUNGEON, 11, 16, 9, 1, dict(max_steps=9, n_frozen=2)), (wl.BINARY, 32, 20, 17, 1, dict(max_steps=11, min_size=5, min_w=5)),
    (wl.MAZE, 32, 32, 16, 1, dict(max_changes=8, obs_format=1)), (wl.DUNGEON, 32, 32, 33, 1, dict(max_steps=8, max_changes=8, pos_mode=wl.POS_SCAN)),
    (wl.BINARY, 64, 64, 24, 1, dict(max_steps=13, n_frozen=3, min_size=20)), (wl.MAZE, 64, 40, 15, 1, dict(autoreset=0, max_steps=4)),
    (wl.DUNGEON, 64, 64, 25, 1, dict(max_steps=10, regions_mode=wl.REGIONS_RECOUNT)),
    # episodes that would end twice within a piece of a relay: turns without one
    (wl.BINARY, 16, 16, 20, 0, dict(max_steps=3)), (wl.MAZE, 32, 32, 20, 0, dict(max_changes=2))])
@pytest.mark.parametrize("slots", ["all", "two"])
def test_rollouts_in_pieces(problem, h, w, T, relay, more, slots):
    """Rollouts of a small batch around the sizes of the pieces that their wavefronts hand on to each
    other, episodes that end in every one of them, three in a row and single steps in between: what
    they leave behind is what the next one starts from.  (Two wavefronts are asked for, so that none is cut into spans.)"""
    B, n_slots = 21, T if slots == "all" else min(2, T)
    cfg = wl.make_config(problem, B, h, 9, **dict(dict(max_w=w, max_steps=50, pos_mode=wl.POS_RANDOM, split_step=2), **more))
    assert relay_rule.relays(cfg, T, n_slots) == bool(relay) and span_rule.spans(cfg, T, n_slots) == 1
    _rollouts_against_steps(cfg, T, n_slots)


@pytest.mark.parametrize("problem,B,h,T,slots,shape,more", [
    # several levels to a workgroup, of which some restart while the others go on
    (wl.BINARY, 21, 16, 25, 25, (4, 4), dict(levels_per_wave=4)), (wl.MAZE, 37, 16, 20, 20, (4, 4), dict(levels_per_wave=2, n_frozen=2)),
    (wl.DUNGEON, 38, 16, 33, 33, (4, 4), dict(levels_per_wave=4)), (wl.BINARY, 21, 32, 24, 24, (4, 4), dict(levels_per_wave=2, min_size=7)),
    (wl.DUNGEON, 9, 32, 19, 19, (4, 4), dict(levels_per_wave=2)), (wl.MAZE, 15, 32, 17, 6, (4, 2), dict(levels_per_wave=2)),
    # several observers to a step; some of the last workgroup have no level at all
    (wl.BINARY, 21, 16, 25, 25, (4, 2), dict(levels_per_wave=4, split_obs_levels=2)), (wl.DUNGEON, 21, 16, 18, 18, (4, 1), dict(levels_per_wave=4, split_obs_levels=1)),
    (wl.MAZE, 37, 16, 27, 3, (4, 1), dict(levels_per_wave=2, split_obs_levels=1)), (wl.BINARY, 7, 32, 22, 2, (4, 2), dict(levels_per_wave=2, split_obs_levels=1)),
    # one slot, an odd ring, a ring of two
    (wl.MAZE, 21, 16, 20, 1, (4, 1), {}), (wl.DUNGEON, 21, 64, 17, 3, (4, 1), {}), (wl.BINARY, 33, 64, 20, 2, (4, 2), {}),
    # the shapes of larger batches
    (wl.MAZE, 300, 16, 18, 18, (4, 2), {}), (wl.DUNGEON, 300, 16, 17, 17, (2, 2), dict(obs_w=31, n_frozen=1)), (wl.DUNGEON, 511, 32, 12, 12, (2, 2), dict(obs_w=21)),
    (wl.BINARY, 513, 16, 19, 19, (4, 2), {}), (wl.MAZE, 700, 64, 10, 10, (4, 2), {}), (wl.BINARY, 769, 16, 25, 25, (2, 1), {}),
    (wl.MAZE, 800, 32, 18, 18, (2, 1), {}), (wl.DUNGEON, 770, 64, 10, 5, (2, 1), {}), (wl.BINARY, 2047, 32, 18, 18, (2, 1), {}),
    (wl.BINARY, 1100, 16, 17, 17, (4, 2), {}), (wl.BINARY, 1030, 32, 9, 9, (4, 2), {}),
    # ... with several observers, and without a relay
    (wl.MAZE, 601, 16, 11, 11, (4, 2), dict(levels_per_wave=2, split_obs_levels=1)), (wl.BINARY, 1100, 16, 17, 3, (0, 0), {}),
    (wl.MAZE, 37, 32, 2, 2, (0, 0), {}), (wl.DUNGEON, 300, 16, 8, 8, (0, 0), {}), (wl.BINARY, 21, 16, 1, 1, (0, 0), {})])
def test_every_shape_of_a_relay(problem, B, h, T, slots, shape, more):
    """Rollouts in every shape that the rule for them gives out, in levels whose episodes end at different
    steps (a change limit)."""
    more = dict(dict(max_steps=60, max_changes=9, obs_w=9, pos_mode=wl.POS_RANDOM, split_step=2), **more)
    cfg = wl.make_config(problem, B, h, more.pop("obs_w"), **more)
    assert relay_rule.shape(**relay_rule.case_of(cfg, T, slots)) == shape
    _rollouts_against_steps(cfg, T, slots)


@pytest.mark.parametrize("problem,B,h,w,T,observed,shape,more", [
    # one step a span, the last span of a rollout, several levels to a wavefront and some without one
    (wl.BINARY, 21, 16, 16, 12, True, (12, 1), {}), (wl.MAZE, 130, 16, 11, 70, True, (35, 2), dict(max_changes=5)),
    (wl.DUNGEON, 9, 32, 20, 131, True, (131, 1), dict(max_steps=40, n_frozen=2)), (wl.BINARY, 300, 30, 32, 33, True, (11, 3), dict(max_changes=3)),
    (wl.MAZE, 601, 32, 32, 25, False, (13, 2), dict(max_steps=7)), (wl.DUNGEON, 100, 64, 64, 60, True, (20, 3), dict(max_steps=13, min_size=30)),
    (wl.BINARY, 33, 64, 50, 67, True, (34, 2), dict(max_changes=9, obs_format=1)), (wl.MAZE, 530, 16, 16, 40, True, (14, 3), dict(obs_pitch=-1)),
    # several episodes within 64 steps, one that ends with every step, and none that ends
    (wl.DUNGEON, 21, 16, 16, 90, True, (90, 1), dict(max_steps=7, ctrl={1: (3, 9), 2: (2, 6)})),
    (wl.MAZE, 65, 16, 16, 64, True, (32, 2), dict(max_steps=1)), (wl.BINARY, 70, 16, 16, 129, False, (43, 3), dict(autoreset=0, max_steps=20)),
    # many steps of 64 on the same cell; round a small map and round again; pinpoints that show
    (wl.DUNGEON, 17, 2, 3, 140, True, (140, 1), {}), (wl.MAZE, 200, 3, 3, 80, True, (40, 2), dict(pos_mode=wl.POS_SCAN, max_changes=30)),
    (wl.BINARY, 90, 1, 1, 65, True, (33, 2), dict(max_changes=20)),
    (wl.DUNGEON, 150, 9, 33, 49, True, (13, 4), dict(pos_mode=wl.POS_SCAN, n_frozen=8, min_size=3, min_w=5, obs_frozen_channel=1, regions_mode=wl.REGIONS_RECOUNT))])
def test_rollouts_cut_into_spans(problem, B, h, w, T, observed, shape, more):
    """Rollouts that are cut up along their steps: the state that a wavefront runs ahead to at the start of
    every span (64 steps at a time, edits of the same cell among them, episodes that end) and what the spans
    leave behind, against the same steps of the oracle."""
    cfg = wl.make_config(problem, B, h, 9, **dict(dict(max_w=w, max_steps=500, pos_mode=wl.POS_RANDOM), **more))
    assert span_rule.shape(**span_rule.case_of(cfg, T, observed)) == shape
    _rollouts_against_steps(cfg, T, T, observed)


@pytest.mark.parametrize("problem,B,h,w,T,more", [
    (wl.MAZE, 70, 16, 13, (24, 41, 17), {}), (wl.DUNGEON, 40, 30, 32, (30, 19, 64), dict(ctrl={1: (3, 9)}, max_changes=11)),
    (wl.BINARY, 20, 64, 50, (40, 30, 70), dict(max_steps=29, obs_frozen_channel=1))])
def test_rollouts_cut_into_spans_from_a_state_of_the_callers(problem, B, h, w, T, more):
    """Levels of mixed shapes with pinpoints, in a context configured without any, and targets of the caller's: what runs ahead,
    the spans and the end of a rollout take both from there.  Rollouts of several lengths, one of them without
    observations, share the room for the starts; then one is captured and replayed."""
    cfg = wl.make_config(problem, B, h, 9, **dict(dict(max_w=w, max_steps=500, pos_mode=wl.POS_RANDOM), **more))
    gpu, cpu = binding.Pcgrl(cfg, 0), oracle.Oracle(cfg)
    rng = np.random.default_rng(B)
    gpu.pcgrl_reset(6)
    cpu.reset(6)
    M, K = gpu.pcgrl_metrics().shape[1], gpu.K
    tiles = rng.integers(0, K, (B, h, w)).astype(np.int8)
    frozen = (rng.random((B, h, w)) < 0.3).astype(np.uint8)
    hw = np.stack([rng.integers(2, h + 1, B), rng.integers(2, w + 1, B)], 1).astype(np.int16)
    pos = np.stack([rng.integers(0, hw[:, 0]), rng.integers(0, hw[:, 1])], 1).astype(np.int16)
    lo = rng.integers(0, 20, (B, M))
    targets = np.stack([lo, lo + rng.integers(0, 30, (B, M))], 2).astype(np.int32)
    gpu.pcgrl_set_state(*(torch.from_numpy(a).to(DEV) for a in (tiles, frozen, hw, pos)))
    cpu.set_state(tiles, frozen, hw, pos)
    gpu.pcgrl_set_targets(torch.from_numpy(targets).to(DEV))
    cpu.set_targets(targets)

    def check(acts, obs, rew, done, turn):
        for t in range(len(acts)):
            o, r, d = cpu.step(acts[t])
            assert np.array_equal(rew[t].cpu().numpy(), r) and np.array_equal(done[t].cpu().numpy(), d), f"{turn} step {t}"
            if obs is not None:
                check_obs(gpu, obs[t], o, f"{turn} step {t}")
        assert_same("metrics", gpu.pcgrl_metrics(), cpu.metrics(), turn)
        assert_same("targets", gpu.pcgrl_get_targets(), cpu.get_targets(), turn)
        compare_state(gpu, cpu, turn)

    buffers = lambda n: (torch.zeros((n,) + tuple(gpu.obs_shape), dtype=torch.uint8, device=DEV), torch.empty((n, B), dtype=torch.float32, device=DEV),  # noqa: E731
                         torch.empty((n, B), dtype=torch.uint8, device=DEV))
    for turn, n in enumerate(T):
        assert span_rule.spans(cfg, n, 0 if turn == 1 else n) > 1
        acts = wl.random_actions(cfg, 40 + turn, n, bad_fraction=0.05)
        obs, rew, done = buffers(n)
        gpu.pcgrl_rollout(torch.from_numpy(acts).to(DEV), None if turn == 1 else obs, rew, done)
        check(acts, None if turn == 1 else obs, rew, done, f"rollout {turn}")
    acts = wl.random_actions(cfg, 50, T[0])
    on_gpu, (obs, rew, done) = torch.from_numpy(acts).to(DEV), buffers(T[0])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        gpu.pcgrl_rollout(on_gpu, obs, rew, done)
    for replay in range(3):
        graph.replay()
        torch.cuda.synchronize()
        check(acts, obs, rew, done, f"replay {replay}")
        (obs.float().sum() + 1).item()                             # unrelated eager work between replays
    gpu.close()


@pytest.mark.parametrize("n,corridor", [(64, 40), (32, 25)])
def test_exact_diameter_of_snakes_beside_a_corridor(n, corridor):
    """A corridor and a snake in a square of side 16, of a few cells less or more than the corridor has: squares with
    no more cells than the longest path so far are dropped unswept, wherever they lie against the grid."""
    snake = [(2 * r + k, c) for r in range(8) for k, c in
             [(0, c) for c in (range(14) if r % 2 == 0 else range(13, -1, -1))] + [(1, 13 if r % 2 == 0 else 0)]]
    maps, want = [], []
    for oy in range(2, n - 15, 5):
        for ox in range(0, n - 13, 3):
            for cells in range(corridor - 1, corridor + 4):
                t = np.ones((n, n), np.int8)
                t[0, :corridor] = 0
                for y, x in snake[:cells]:
                    t[oy + y, ox + x] = 0
                maps.append(t)
                want.append(max(corridor, cells) - 1)  # (both are paths: one edge less than cells)
    B = len(maps)
    hw = torch.full((B, 2), n, dtype=torch.int16, device=DEV)
    gpu = binding.Pcgrl(wl.make_config(wl.BINARY, B, n, 5, min_size=1, autoreset=0), 0)
    gpu.pcgrl_reset(1)
    for tiles in (np.stack(maps), np.stack(maps)[:, ::-1].copy(), np.stack(maps)[:, :, ::-1].copy()):
        gpu.pcgrl_set_state(torch.from_numpy(tiles).to(DEV), None, hw, torch.zeros_like(hw))
        for parts_log2 in (-1, 0, 3):
            got = gpu.pcgrl_exact_diameter_static(torch.empty(B, dtype=torch.int32, device=DEV), parts_log2)
            assert_same("exact diameters", got, np.array(want, np.int32), parts_log2)
    gpu.close()
