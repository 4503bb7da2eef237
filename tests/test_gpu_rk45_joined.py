"""RK45 whose attempts are joined by one pass (captured chunks) against the
separate controller, commit and combine passes (the profiler's plain launches,
and a run with an energy trace): bit for bit, over chunk ends and rejected
attempts, for several groups, per-cell materials, lengths known at compile and
at run time, resumed runs and replayed steps."""
import numpy as np
import pytest

from workloads import random_unit

from _mmx_case import Case, dev, host, open_ctx

pytestmark = pytest.mark.gpu

TERMS = ("exchange", "anisotropy", "zeeman", "demag")
CELL = (4e-9, 4e-9, 4e-9)
GROUPS = {
    "film-32": [Case((32, 20, 1), CELL, R=2, Ku=3e5, B=(0.01, 0.0, 0.05), terms=TERMS)],
    "film-45": [Case((45, 18, 1), CELL, R=1, Ku=3e5, terms=TERMS)],
    "groups": [Case((16, 12, 1), CELL, R=3, terms=TERMS),
               Case((64, 6, 1), CELL, R=1, Ku=3e5, B=(0.0, 0.05, 0.0), terms=TERMS),
               Case((10, 9, 4), CELL, R=2, terms=TERMS)],
}


def _run(groups, prec, mode):
    import torch
    import paper_2608_15253_amd as mmx
    m0 = np.concatenate([random_unit(c.n, seed=5 + g, replicas=c.R).ravel()
                         for g, c in enumerate(groups)])
    rng = np.random.default_rng(2)
    R = sum(c.R for c in groups)
    ctx = open_ctx(groups[0], prec, groups=groups)
    out = []
    try:
        Ms = rng.uniform(4e5, 8e5, groups[0].n[::-1])
        mmx.mmx_set_material_cells(ctx, 0, Ms=dev(Ms, prec))
        mmx.mmx_profile_enable(ctx, mode == "profiled")
        kw = {}
        if mode == "traced":
            trace = torch.zeros(4000 * R, dtype=torch.float64, device="cuda:0")
            kw = dict(energy_trace=trace, trace_cap=4000)

        def note(m, s):
            out.append(host(m))
            out.append(np.array([s.t, s.dt, s.err, s.accepted, s.rejected]))
            out.append(np.array(mmx.mmx_rk45_dts(ctx)))

        m = dev(m0, prec)
        note(m, mmx.mmx_rk45(ctx, m, 0.0, 5e-12, 1e-5, 1e-13, **kw))
        note(m, mmx.mmx_rk45_resume(ctx, m, 7e-12, 1e-5, **kw))
        # tighter, from a step that has to be rejected first
        note(m, mmx.mmx_rk45(ctx, m, 0.0, 1e-12, 1e-7, 1e-12, **kw))
        m = dev(m0, prec)
        dts = [1e-14 * (1 + i % 3) for i in range(21)]
        note(m, mmx.mmx_rk45(ctx, m, 0.0, float(sum(dts)), 1e-5, dt_replay=dts, **kw))
    finally:
        mmx.mmx_destroy(ctx)
    return out


@pytest.mark.parametrize("prec", [2, 1], ids=["f64", "f32"])
@pytest.mark.parametrize("name", list(GROUPS))
def test_joined_attempts(name, prec):
    print(f"[case] rk45 joined {name} prec={prec}", flush=True)
    runs = {mode: _run(GROUPS[name], prec, mode) for mode in ("joined", "profiled", "traced")}
    stats = [runs["joined"][i] for i in (1, 4, 7, 10)]
    print([s.tolist() for s in stats], flush=True)
    assert stats[0][3] > 16 and stats[2][4] >= 1 and stats[3][3] == 21
    for mode in ("profiled", "traced"):
        for a, b in zip(runs["joined"], runs[mode]):
            assert np.array_equal(a, b), mode
