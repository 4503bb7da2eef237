"""Heun and rotation runs whose replicas are split into parts (working sets
beyond the memory-side cache): every
replica bit for bit as in a context of few replicas, which is one part, with
switching times and through retire/refill; several groups, one of them split.
"""
import numpy as np
import pytest

from workloads import replica_seeds, uniform

from _mmx_case import Case, dev, host, open_ctx

pytestmark = pytest.mark.gpu


def _case(n, R, base=3):
    return Case(n, (4e-9, 4e-9, 4e-9), R=R, Ms=8e5, A=1.3e-11, alpha=0.02, Ku=5e5,
                B=(0.0, 0.0, -0.15), T=300.0, seeds=list(replica_seeds(base, R)),
                terms=("exchange", "anisotropy", "zeeman", "demag", "thermal"))


def _sub(case, rs):
    return Case(**{**case.__dict__, "R": len(rs), "seeds": [case.seeds[r] for r in rs]})


def _start(case):
    m = uniform(case.n, (0.02, 0.01, 1.0), replicas=case.R)
    # replicas differ, and some start past their switching
    m[::3, 2] *= -1.0
    return m.astype(np.float32).astype(np.float64)


# 64 x 64: 198 KB of spectrum and states per replica in FP32 (247 KB with the
# rotation), so 1, 2 and 3 parts
@pytest.mark.parametrize("R", [1024, 1400, 2300])
@pytest.mark.parametrize("rot", [False, True], ids=["heun", "rotation"])
def test_parts_equal_single_contexts(R, rot):
    import paper_2608_15253_amd as mmx
    print(f"[case] run parts R={R} rot={rot}", flush=True)
    case = _case((64, 64, 1), R)
    m0 = _start(case)
    call = mmx.mmx_depondt if rot else mmx.mmx_heun
    few = sorted({0, 1, R // 3, R // 2 - 1, R // 2, R // 2 + 1, 2 * R // 3, R - 1})

    def run(c, start):
        ctx = open_ctx(c, mmx.MMX_F32)
        try:
            md, ts = dev(start, mmx.MMX_F32), dev(-np.ones(c.R), mmx.MMX_F64)
            call(ctx, md, 1e-14, 5, 2, ts)
            call(ctx, md, 1e-14, 3, 7, ts)   # the captured runs again
            return host(md), host(ts)
        finally:
            mmx.mmx_destroy(ctx)

    got, ts = run(case, m0)
    ref, tr = run(_sub(case, few), m0[few])
    assert np.array_equal(got[few], ref)
    assert np.array_equal(ts[few], tr)
    assert np.all((ts[::3] > 0)) and np.all(np.delete(ts, np.s_[::3]) < 0)


def test_parts_with_refill():
    import paper_2608_15253_amd as mmx
    R, cap = 1200, 4
    case = _case((64, 64, 1), R)
    m0 = _start(case)
    few = [0, 3, 599, 600, 601, 1199]

    def run(c, start):
        ctx = open_ctx(c, mmx.MMX_F32)
        try:
            import torch
            md, mi = dev(start, mmx.MMX_F32), dev(start, mmx.MMX_F32)
            times = torch.zeros(c.R * cap, dtype=torch.float64, device="cuda:0")
            counts = torch.zeros(c.R, dtype=torch.int32, device="cuda:0")
            mmx.mmx_depondt_refill(ctx, md, mi, 1e-14, 5, times, cap, counts)
            return host(md), host(times).reshape(c.R, cap), host(counts)
        finally:
            mmx.mmx_destroy(ctx)

    got, ref = run(case, m0), run(_sub(case, few), m0[few])
    for a, b in zip(got, ref):
        assert np.array_equal(a[few], b)
    assert got[2].max() >= 1


def test_parts_of_several_groups():
    import paper_2608_15253_amd as mmx
    groups = [_case((32, 32, 1), 24, 5), _case((64, 64, 1), 1400, 6), _case((16, 12, 1), 9, 7)]
    m0 = [_start(c) for c in groups]

    def run(cs, starts):
        ctx = open_ctx(cs[0], mmx.MMX_F32, groups=cs)
        try:
            md = dev(np.concatenate([s.ravel() for s in starts]), mmx.MMX_F32)
            ts = dev(-np.ones(sum(c.R for c in cs)), mmx.MMX_F64)
            mmx.mmx_heun(ctx, md, 1e-14, 7, 0, ts)
            return host(md), host(ts)
        finally:
            mmx.mmx_destroy(ctx)

    got, ts = run(groups, m0)
    at = rt = 0
    for c, s in zip(groups, m0):
        ref, tr = run([c], [s])
        assert np.array_equal(got[at:at + s.size], ref)
        assert np.array_equal(ts[rt:rt + c.R], tr)
        at, rt = at + s.size, rt + c.R
