"""pcgrl_exact_diameter_static, whose caller chooses how many wavefronts share a level, against
pcgrl_exact_diameter, through the C ABI: same results for every choice, on calls in a row of
different sizes (needs an MI355X)."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
from paper_2408_12525_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu


def _diameters(gpu, static, parts_log2=-1):
    dev = torch.device("cuda", 0)
    out = torch.full((gpu.B,), -7, dtype=torch.int32, device=dev)
    st = C.c_void_p(torch.cuda.current_stream(dev).cuda_stream)
    if static:
        rc = gpu.L.pcgrl_exact_diameter_static(gpu.h, C.c_void_p(out.data_ptr()), parts_log2, st)
    else:
        rc = gpu.L.pcgrl_exact_diameter(gpu.h, C.c_void_p(out.data_ptr()), st)
    assert rc == 0, rc
    torch.cuda.synchronize()
    return out.cpu().numpy()


def test_static_scratch_variant_equals_the_allocating_entry_point():
    dev = torch.device("cuda", 0)
    # 700 levels with the wavefronts the other entry point takes, 45 larger ones with 32 wavefronts
    # each asked for (16 are used), 3 with 64, and 9000 with one: each workgroup leaves its sets of
    # cells in LDS for the next one, which has to start from its own
    cases = [("binary16", 700, -1), ("dungeon32", 45, 5), ("maze64", 3, 6), ("binary16", 9000, 0)]
    envs = []
    for name, batch, lg in cases:
        cfg = wl.workload(name, batch=batch, max_steps=10**6, autoreset=0)
        gpu, cpu = binding.Pcgrl(cfg, 0), oracle.Oracle(cfg)
        gpu.pcgrl_reset(11)
        cpu.reset(11, want_obs=False)
        acts = wl.random_actions(cfg, 12, 30)
        for a in acts:
            gpu.pcgrl_step(torch.from_numpy(a).to(dev))
            cpu.step(a, want_obs=False)
        envs.append((gpu, cpu, lg, name))
    # the static calls back to back, nothing in between
    got = [_diameters(gpu, True, lg) for gpu, _, lg, _ in envs]
    for (gpu, cpu, lg, name), g in zip(envs, got):
        want = _diameters(gpu, False)
        assert np.array_equal(g, want), name
        assert np.array_equal(g, cpu.exact_diameters()), name
    # again in reverse order (large after small), and with every split the buffer size allows
    for gpu, cpu, lg, name in reversed(envs):
        side = 16 if max(gpu.Hm, gpu.Wm) <= 16 else 32 if max(gpu.Hm, gpu.Wm) <= 32 else 64
        for p in range(0, side.bit_length()):
            if (gpu.B << p) > (1 << 18) and p > 0:
                break
            assert np.array_equal(_diameters(gpu, True, p), cpu.exact_diameters()), (name, p)
    for gpu, *_ in envs:
        gpu.close()


def test_static_scratch_variant_rejects_what_does_not_fit():
    dev = torch.device("cuda", 0)
    cfg = wl.workload("binary16", batch=40000, max_steps=10**6, autoreset=0)
    gpu = binding.Pcgrl(cfg, 0)
    out = torch.empty((gpu.B,), dtype=torch.int32, device=dev)
    st = C.c_void_p(torch.cuda.current_stream(dev).cuda_stream)
    call = lambda lg: gpu.L.pcgrl_exact_diameter_static(gpu.h, C.c_void_p(out.data_ptr()), lg, st)
    assert call(3) == -6                       # 40 000 levels x 8 parts = 320 000 > 262 144
    assert call(2) == 0                        # 160 000 are accepted
    assert call(5) == -2 and call(-2) == -2    # more parts than rows / no such code
    assert gpu.L.pcgrl_exact_diameter_static(None, C.c_void_p(out.data_ptr()), 0, st) == -1
    assert b"static scratch" in gpu.L.pcgrl_strerror(-6) and b"262 144" in gpu.L.pcgrl_strerror(-6)
    torch.cuda.synchronize()
    gpu.close()
