"""Sequences of mmx_rk4 calls: two groups (one with per-cell materials) with
setters, other step sizes and other arrays between the calls, against the
oracle; no call waits for the device; launches into a caller's capture.

Bars: states FP64 1e-12 / FP32 1e-5 max |dm| (the parity bar of the precision
forms).
"""
import dataclasses

import numpy as np
import pytest

from oracle import integrators as oit
from workloads import random_unit

from _mmx_case import Case, dev, host, open_ctx

pytestmark = pytest.mark.gpu

BAR = {2: 1e-12, 1: 1e-5}
TERMS = ("exchange", "anisotropy", "zeeman", "demag")
FILM = Case((32, 12, 1), (3e-9, 2.5e-9, 2e-9), R=2, Ms=6e5, Ku=3e5, B=(0.01, 0.0, 0.05),
            alpha=0.1, terms=TERMS)
BLOCK = Case((15, 10, 4), (3e-9, 3e-9, 3e-9), R=1, Ms=8e5, alpha=0.05, B=(0.0, 0.02, 0.0),
             terms=TERMS)


def _round(a, prec):
    return a.astype(np.float32).astype(np.float64) if prec == 1 else a


@pytest.mark.parametrize("prec", [2, 1], ids=["f64", "f32"])
def test_calls_between_setters_arrays_and_step_sizes(prec):
    import paper_2608_15253_amd as mmx
    print(f"[case] rk4 calls prec={prec}", flush=True)
    rng = np.random.default_rng(5)
    cells = {"Ms": _round(rng.uniform(4e5, 8e5, FILM.n[::-1]), prec),
             "alpha": _round(rng.uniform(0.02, 0.3, FILM.n[::-1]), prec)}
    mats = [dataclasses.replace(FILM.material(), Ms_cells=cells["Ms"],
                                alpha_cells=cells["alpha"]), BLOCK.material()]
    start = {a: [_round(random_unit(c.n, seed=s + g, replicas=c.R), prec)
                 for g, c in enumerate((FILM, BLOCK))] for a, s in (("A", 3), ("B", 11))}
    ref = {a: [m.copy() for m in v] for a, v in start.items()}
    ctx = open_ctx(FILM, prec, groups=[FILM, BLOCK])
    try:
        mmx.mmx_set_material_cells(ctx, 0, **{k: dev(v, prec) for k, v in cells.items()})
        md = {a: dev(np.concatenate([m.ravel() for m in v]), prec) for a, v in start.items()}

        def step(a, dt, n):
            mmx.mmx_rk4(ctx, md[a], dt, n)
            for g, c in enumerate((FILM, BLOCK)):
                for r in range(c.R):
                    ref[a][g][r] = oit.rk4_run(ref[a][g][r], c.grid, mats[g], dt, n)

        def field(g, B):
            mmx.mmx_set_field(ctx, g, B)
            mats[g] = dataclasses.replace(mats[g], B=B)

        def precession(on):
            mmx.mmx_set_precession(ctx, on)
            mats[:] = [dataclasses.replace(m, precess=on) for m in mats]

        step("A", 1e-14, 1)
        step("A", 1e-14, 3)
        field(1, (0.0, 0.0, -0.1))
        step("A", 1e-14, 2)
        step("A", 2e-14, 1)
        step("B", 2e-14, 3)
        step("A", 2e-14, 1)
        precession(False)
        step("B", 1e-14, 2)
        precession(True)
        field(0, (0.0, 0.1, 0.0))
        step("B", 1e-14, 1)
        got = {a: host(v) for a, v in md.items()}
    finally:
        mmx.mmx_destroy(ctx)
    for a, v in ref.items():
        want = np.concatenate([m.ravel() for m in v])
        assert np.abs(got[a] - want).max() <= BAR[prec], a


def test_calls_do_not_wait_for_the_device():
    """Work queued ahead on the bound stream is still running when calls with
    two arrays and a setter between them have returned."""
    import torch
    import paper_2608_15253_amd as mmx
    ctx = open_ctx(FILM, mmx.MMX_F32)
    try:
        A, B = (dev(random_unit(FILM.n, seed=s, replicas=FILM.R), 1) for s in (1, 2))
        for m in (A, B):
            mmx.mmx_rk4(ctx, m, 1e-14, 3)
        x = torch.randn(8192, 8192, device="cuda:0")
        y = torch.empty_like(x)
        torch.mm(x, x, out=y)
        torch.cuda.synchronize()
        for _ in range(40):  # 1.1 TFLOP each: some 7 ms
            torch.mm(x, x, out=y)
        queued = torch.cuda.Event()
        queued.record()
        for m in (A, B, A):
            mmx.mmx_rk4(ctx, m, 1e-14, 3)
            mmx.mmx_set_field(ctx, 0, (0.0, 0.0, 0.02))
        ahead = not queued.query()
        torch.cuda.synchronize()
    finally:
        mmx.mmx_destroy(ctx)
    assert ahead


@pytest.mark.parametrize("prec", [2, 1], ids=["f64", "f32"])
def test_calls_in_a_captured_stream(prec):
    import torch
    import paper_2608_15253_amd as mmx
    m0 = _round(random_unit(FILM.n, seed=9, replicas=FILM.R), prec)
    ctx = open_ctx(FILM, prec)
    try:
        m = dev(m0, prec)
        want = []
        for _ in range(3):
            mmx.mmx_rk4(ctx, m, 1e-14, 2)
            want.append(host(m).copy())
        m = dev(m0, prec)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            mmx.mmx_set_stream(ctx, torch.cuda.current_stream().cuda_stream)
            mmx.mmx_rk4(ctx, m, 1e-14, 2)
        mmx.mmx_set_stream(ctx, torch.cuda.current_stream().cuda_stream)
        other = dev(m0, prec)
        for k in range(3):
            g.replay()
            torch.cuda.synchronize()
            assert np.array_equal(host(m), want[k]), k
            mmx.mmx_rk4(ctx, other, 2e-14, 1)  # eager work on the same context between replays
    finally:
        mmx.mmx_destroy(ctx)
