"""The longest lines that a workgroup's LDS takes (rows of 1000 and 500 points,
whose integrator epilogues also hold the split factors, columns of 500 and 250
cells): field, RK4, RK45 in dt replay and Heun against the oracle.

Bars: fields FP64 1e-11 / FP32 4e-6 of max |H|; states FP64 1e-12 / FP32 1e-5.
"""
import numpy as np
import pytest

from oracle import fields as ofl
from oracle import integrators as oit
from workloads import random_unit

from _mmx_case import Case, dev, host, open_ctx

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,prec", [((1000, 2, 1), 1), ((500, 2, 1), 2), ((4, 500, 1), 1),
                                    ((4, 250, 1), 2)],
                         ids=["1000x2-f32", "500x2-f64", "4x500-f32", "4x250-f64"])
def test_longest_lines(n, prec):
    import paper_2608_15253_amd as mmx
    print(f"[case] long lines {n} prec={prec}", flush=True)
    case = Case(n, (4e-9, 4e-9, 4e-9), alpha=0.1, Ku=3e5, B=(0.01, 0.0, 0.05),
                terms=("exchange", "anisotropy", "zeeman", "demag"))
    m0 = random_unit(n, seed=2, replicas=1)
    if prec == 1:
        m0 = m0.astype(np.float32).astype(np.float64)
    barf, barm = {2: 1e-11, 1: 4e-6}[prec], {2: 1e-12, 1: 1e-5}[prec]
    mat = case.material()
    dts = [1e-14, 2e-14]
    ctx = open_ctx(case, prec)
    try:
        H = dev(np.zeros_like(m0), prec)
        mmx.mmx_field(ctx, dev(m0, prec), H)
        got = [host(H)[0]]
        for call in (lambda m: mmx.mmx_rk4(ctx, m, 1e-14, 2),
                     lambda m: mmx.mmx_rk45(ctx, m, 0.0, sum(dts), 1e-6, dt_replay=dts),
                     lambda m: mmx.mmx_heun(ctx, m, 1e-14, 2, 0)):
            m = dev(m0, prec)
            call(m)
            got.append(host(m)[0])
    finally:
        mmx.mmx_destroy(ctx)
    ref = ofl.effective_field(m0[0], case.grid, mat)
    assert np.abs(got[0] - ref).max() <= barf * np.abs(ref).max()
    for g, r in zip(got[1:], (oit.rk4_run(m0[0], case.grid, mat, 1e-14, 2),
                              oit.rk45_run(m0[0], case.grid, mat, 0.0, sum(dts), 1e-6,
                                           dt_replay=dts).m,
                              oit.heun_run(m0[0], case.grid, mat, 1e-14, 2))):
        assert np.abs(g - r).max() <= barm
