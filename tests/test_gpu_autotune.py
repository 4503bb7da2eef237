"""mmx_autotune: with the profiler on, every launch it counts is timed and the
context stays usable; the Heun path it chooses is the faster one."""
import time

import numpy as np
import pytest

from workloads import random_unit

from _mmx_case import Case, dev, host, open_ctx

pytestmark = pytest.mark.gpu

TERMS = ("exchange", "anisotropy", "zeeman", "demag")


@pytest.mark.parametrize("n,R", [((32, 32, 1), 4), ((64, 48, 1), 2), ((16, 12, 3), 2)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_autotune_with_the_profiler_on(n, R):
    import paper_2608_15253_amd as mmx
    print(f"[case] autotune profiled {n} R={R}", flush=True)
    case = Case(n, (4e-9, 4e-9, 4e-9), R=R, Ku=3e5, B=(0.0, 0.0, 0.05), terms=TERMS)
    m0 = random_unit(n, seed=4, replicas=R).astype(np.float32)
    out = []
    for profiled in (False, True):
        ctx = open_ctx(case, mmx.MMX_F32)
        try:
            mmx.mmx_profile_enable(ctx, profiled)
            for _ in range(3):
                mmx.mmx_autotune(ctx)
            table = mmx.mmx_profile_get(ctx)
            md = dev(m0, mmx.MMX_F32)
            mmx.mmx_heun(ctx, md, 1e-14, 3, 0)
            mmx.mmx_sync(ctx)
            mmx.mmx_profile_enable(ctx, False)
            # the tiles do not change results, the Heun path may (round-off)
            mmx.mmx_set_path(ctx, mmx.MMX_PATH_STAGED)
            mmx.mmx_heun(ctx, md, 1e-14, 3, 3)
            out.append(host(md))
        finally:
            mmx.mmx_destroy(ctx)
        if profiled:
            assert sum(c for _, c in table.values()) > 0
            for name, (ms, count) in table.items():
                # a launch takes 1 us at least, and these grids far below 1 ms
                assert count == 0 or 1e-3 <= ms / count <= 1.0, (name, ms, count)
        else:
            assert all(c == 0 for _, c in table.values())
    assert np.abs(out[0] - out[1]).max() <= 1e-5


@pytest.mark.parametrize("n,R", [((16, 16, 1), 256), ((32, 32, 1), 256)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_autotune_keeps_the_faster_heun_path(n, R):
    """Runs of 64 steps on the chosen path take no longer than on the faster
    of the two by more than 7 % (the least of 12 timings repeats within 2 %)."""
    import torch
    import paper_2608_15253_amd as mmx
    print(f"[case] autotune heun path {n} R={R}", flush=True)
    case = Case(n, (4e-9, 4e-9, 4e-9), R=R, alpha=0.02, Ku=5e5, B=(0.0, 0.0, -0.1), T=300.0,
                seeds=list(range(1, R + 1)), terms=TERMS + ("thermal",))
    ctx = open_ctx(case, mmx.MMX_F32)
    try:
        md = dev(random_unit(n, seed=4, replicas=R), mmx.MMX_F32)
        mmx.mmx_autotune(ctx)
        t = {}
        for path in (mmx.MMX_PATH_AUTO, mmx.MMX_PATH_STAGED, mmx.MMX_PATH_FUSED):
            mmx.mmx_set_path(ctx, path)
            mmx.mmx_heun(ctx, md, 1e-14, 64, 0)
            runs = []
            for _ in range(12):
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                mmx.mmx_heun(ctx, md, 1e-14, 64, 0)
                torch.cuda.synchronize()
                runs.append(time.perf_counter() - t0)
            t[path] = min(runs)
    finally:
        mmx.mmx_destroy(ctx)
    print({k: f"{v / 64 * 1e6:.1f} us" for k, v in t.items()}, flush=True)
    assert t[mmx.MMX_PATH_AUTO] <= 1.07 * min(t[mmx.MMX_PATH_STAGED], t[mmx.MMX_PATH_FUSED])
