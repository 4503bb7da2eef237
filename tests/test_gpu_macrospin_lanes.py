"""Single-cell ensembles with several lanes per replica: the lane counts (16, 8,
4, 1) that the ensemble size selects, run lengths that are no multiple of
them, and ensembles that do not fill the last wave, against the staged path
(one workgroup per replica, whose noise and steps are pinned to the oracle
elsewhere) and against the oracle.

Bars: the two paths contract multiply-adds differently: FP64 1e-12, FP32 1e-5
over 23 steps (the state bars of the integrator tests).
"""
import numpy as np
import pytest

from oracle import integrators as oit
from oracle import rotation as orot
from workloads import random_unit, replica_seeds

from _mmx_case import Case, dev, host, open_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [2, 1], ids=["f64", "f32"])
@pytest.mark.parametrize("rot", [False, True], ids=["heun", "rotation"])
@pytest.mark.parametrize("R", [1, 37, 8200, 16400, 33000])
def test_lanes(R, rot, prec):
    import paper_2608_15253_amd as mmx
    print(f"[case] macrospin lanes R={R} rot={rot} prec={prec}", flush=True)
    steps, dt, step0 = 23, 5e-14, 5
    case = Case((1, 1, 1), (10e-9, 10e-9, 10e-9), R=R, Ms=1.1e6, A=0.0, alpha=0.05, Ku=5e5,
                B=(0.02, 0.0, -0.1), T=300.0, seeds=list(replica_seeds(19, R)),
                terms=("anisotropy", "zeeman", "thermal"))
    m0 = random_unit(case.n, seed=4, replicas=R)
    if prec == 1:
        m0 = m0.astype(np.float32).astype(np.float64)
    bar = {2: 1e-12, 1: 1e-5}[prec]
    got = {}
    for path in (mmx.MMX_PATH_AUTO, mmx.MMX_PATH_STAGED):
        ctx = open_ctx(case, prec)
        try:
            mmx.mmx_set_path(ctx, path)
            md = dev(m0, prec)
            (mmx.mmx_depondt if rot else mmx.mmx_heun)(ctx, md, dt, steps, step0)
            got[path] = host(md)
        finally:
            mmx.mmx_destroy(ctx)
    assert np.abs(got[mmx.MMX_PATH_AUTO] - got[mmx.MMX_PATH_STAGED]).max() <= bar
    few = [0, R // 2, R - 1]
    run = orot.depondt_run if rot else oit.heun_run
    ref = run(m0[few], case.grid, case.material(), dt, steps,
              seed=np.array(case.seeds, dtype=np.uint64)[few], step0=step0)
    assert np.abs(got[mmx.MMX_PATH_AUTO][few] - ref).max() <= bar
