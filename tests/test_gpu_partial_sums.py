"""Energies, switching times and trial ends from the workgroups' partial sums:
tiles that give one partial per replica, a few, and more than a wave sums at
once.  Energies against the oracle; switching and trials the same for every
tile, with replicas that start on either side of m_z = 0.

Bars: energies FP64 1e-12 / FP32 2e-6 of the largest term.
"""
import numpy as np
import pytest

from oracle import observables as oob
from workloads import random_unit

from _mmx_case import Case, dev, host, open_ctx

pytestmark = pytest.mark.gpu

TERMS = ("exchange", "anisotropy", "zeeman", "demag")
TOLE = {2: 1e-12, 1: 2e-6}


@pytest.mark.parametrize("prec", [2, 1], ids=["f64", "f32"])
@pytest.mark.parametrize("n,R", [((12, 8, 1), 70), ((12, 40, 1), 3), ((6, 30, 18), 2)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_energies_of_every_tile(n, R, prec):
    import paper_2608_15253_amd as mmx
    print(f"[case] partial sums energies {n} R={R} prec={prec}", flush=True)
    case = Case(n, (3e-9, 3e-9, 3e-9), R=R, Ku=3e5, B=(0.01, 0.0, 0.05), terms=TERMS)
    m0 = random_unit(n, seed=3, replicas=R)
    if prec == 1:
        m0 = m0.astype(np.float32).astype(np.float64)
    ctx = open_ctx(case, prec)
    try:
        md, got = dev(m0, prec), {}
        t0 = mmx.mmx_get_tiles(ctx, 0)
        for L in (1, 2, n[1]):   # 8 to 540 partial sums, and one per layer
            mmx.mmx_set_tiles(ctx, 0, (L, t0[1], t0[2]))
            E = dev(np.zeros((R, 6)), 2)
            mmx.mmx_energy(ctx, md, E)
            got[L] = host(E)
    finally:
        mmx.mmx_destroy(ctx)
    for r in sorted({0, R // 2, R - 1}):
        e = oob.energies(m0[r], case.grid, case.material())
        ref = np.array([e[k] for k in ("exchange", "dmi", "demag", "anisotropy", "zeeman",
                                       "total")])
        for L, E in got.items():
            assert np.abs(E[r] - ref).max() <= TOLE[prec] * np.abs(ref[:5]).max(), (r, L)


@pytest.mark.parametrize("n,R", [((12, 8, 1), 70), ((6, 30, 18), 5)],
                         ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_switching_and_trials_of_every_tile(n, R):
    import torch
    import paper_2608_15253_amd as mmx
    print(f"[case] partial sums switching {n} R={R}", flush=True)
    case = Case(n, (3e-9, 3e-9, 3e-9), R=R, alpha=0.3, Ku=3e5, T=300.0,
                seeds=list(range(1, R + 1)), B=(0.0, 0.0, -0.1), terms=TERMS + ("thermal",))
    m0 = random_unit(n, seed=3, replicas=R) * 0.2
    m0[:, 2] += np.where(np.arange(R) % 3 == 0, -1.0, 1.0)[:, None, None, None]
    m0 /= np.linalg.norm(m0, axis=1, keepdims=True)
    ctx = open_ctx(case, mmx.MMX_F64)
    try:
        mi, out = dev(m0, 2), []
        t0 = mmx.mmx_get_tiles(ctx, 0)
        for L in (1, n[1]):
            mmx.mmx_set_tiles(ctx, 0, (L, t0[1], t0[2]))
            ts = dev(-np.ones(R), 2)
            mmx.mmx_heun(ctx, mi.clone(), 1e-14, 3, 0, ts)
            times = torch.zeros(R * 4, dtype=torch.float64, device="cuda:0")
            counts = torch.zeros(R, dtype=torch.int32, device="cuda:0")
            m = mi.clone()
            mmx.mmx_depondt_refill(ctx, m, mi, 1e-14, 3, times, 4, counts)
            out.append((host(ts), host(times), host(counts), host(m)))
    finally:
        mmx.mmx_destroy(ctx)
    ts, times, counts, _ = out[0]
    assert np.array_equal(ts > 0, np.arange(R) % 3 == 0) and np.all(ts[::3] == 1e-14)
    # a replica that starts with m_z < 0 ends a trial after every step
    assert np.array_equal(counts, np.where(np.arange(R) % 3 == 0, 3, 0))
    for a, b in zip(*out):
        assert np.array_equal(a, b)
