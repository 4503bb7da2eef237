"""GPU parity of the LDS line transforms at the lengths where their plans and
their fixed-length variants change: fixed rows of 32 to 256 and columns of 64
to 512 points (padded lines), lengths on either side of them, the odd radices
and the composite ones (6, 9, 10), pruned and full, tiles with a remainder.
Fields against the oracle, and one RK45 and RK4 run each (the row kernels' RK
epilogues), FP64 and FP32.

Bars as in the field tests: FP64 1e-11 and FP32 4e-6 of max |H| (round-off of
transforms of a few hundred terms); states FP64 1e-12, FP32 1e-5.
"""
import numpy as np
import pytest

from oracle import fields as ofl
from oracle import integrators as oit
from workloads import random_unit

from _mmx_case import Case, dev, host, open_ctx

pytestmark = pytest.mark.gpu

# (nx, ny, nz, periodic x and y): the transforms are nx (or nx / 2 if periodic)
# along x, 2 ny (or ny) along y and 2 nz along z
GRIDS = [
    (32, 32, 1, 0), (64, 6, 1, 0), (128, 5, 1, 0), (256, 3, 1, 0), (64, 64, 1, 1),
    (16, 16, 1, 0), (512, 4, 1, 1), (5, 128, 1, 0), (3, 256, 1, 0), (6, 128, 1, 1),
    (18, 27, 1, 0), (27, 25, 1, 0), (30, 45, 1, 0), (54, 50, 1, 0), (100, 9, 1, 0),
    (20, 81, 1, 1), (90, 75, 1, 0), (8, 6, 9, 0), (12, 10, 15, 0),
]


def _case(g, R=1):
    nx, ny, nz, per = g
    return Case((nx, ny, nz), (3e-9, 2.5e-9, 2e-9), pbc=(per, per, 0), images=(per, per, 0), R=R,
                Ms=5.8e5, A=1.5e-11, alpha=0.2, Ku=3e5, D=2e-3, B=(0.01, 0.0, 0.05))


@pytest.mark.parametrize("prec", [2, 1], ids=["f64", "f32"])
@pytest.mark.parametrize("g", GRIDS, ids=lambda g: "x".join(map(str, g[:3])) + "p" * g[3])
def test_field_of_every_plan(g, prec):
    import paper_2608_15253_amd as mmx
    case = _case(g, R=2)
    print(f"[case] line fft {g} prec={prec}", flush=True)
    m0 = random_unit(case.n, seed=5, replicas=2)
    if prec == 1:
        m0 = m0.astype(np.float32).astype(np.float64)
    ref = np.stack([ofl.effective_field(m0[r], case.grid, case.material()) for r in range(2)])
    bar = {2: 1e-11, 1: 4e-6}[prec] * np.abs(ref).max()
    ctx = open_ctx(case, prec)
    try:
        H = dev(np.zeros_like(m0), prec)
        md = dev(m0, prec)
        tiles = mmx.mmx_get_tiles(ctx, 0)
        # the default tiles, one row and column, and a number that leaves a remainder
        few = tuple(min(3, n) for n in (g[1], tiles[1] + 1, tiles[2] + 1))
        for t in (tiles, (1, 1, 1), few):
            try:
                mmx.mmx_set_tiles(ctx, 0, t)
            except mmx.MMXError:
                continue  # beyond the columns or the LDS of this grid
            mmx.mmx_field(ctx, md, H)
            assert np.abs(host(H) - ref).max() <= bar, t
    finally:
        mmx.mmx_destroy(ctx)


@pytest.mark.parametrize("prec", [2, 1], ids=["f64", "f32"])
@pytest.mark.parametrize("g", [(32, 12, 1, 0), (64, 10, 1, 0), (128, 6, 1, 0), (256, 4, 1, 0),
                               (48, 20, 1, 0), (45, 9, 1, 0), (32, 6, 4, 0)],
                         ids=lambda g: "x".join(map(str, g[:3])))
def test_rk_epilogues(g, prec):
    import paper_2608_15253_amd as mmx
    case = _case(g)
    print(f"[case] line fft rk {g} prec={prec}", flush=True)
    rng = np.random.default_rng(3)
    m0 = np.zeros((1, 3) + (g[2], g[1], g[0]))
    m0[:, 2] = 1.0
    m0 += 0.3 * rng.standard_normal(m0.shape)
    m0 /= np.linalg.norm(m0, axis=1, keepdims=True)
    if prec == 1:
        m0 = m0.astype(np.float32).astype(np.float64)
    bar = {2: 1e-12, 1: 1e-5}[prec]
    dts = [1e-14, 2e-14, 3e-14, 2e-14]
    ctx = open_ctx(case, prec)
    try:
        md = dev(m0, prec)
        mmx.mmx_rk45(ctx, md, 0.0, float(sum(dts)), 1e-6, dt_replay=dts)
        ref = oit.rk45_run(m0[0], case.grid, case.material(), 0.0, float(sum(dts)), 1e-6,
                           dt_replay=dts)
        assert np.abs(host(md)[0] - ref.m).max() <= bar
        md = dev(m0, prec)
        mmx.mmx_rk4(ctx, md, 2e-14, 5)
        assert np.abs(host(md)[0] - oit.rk4_run(m0[0], case.grid, case.material(), 2e-14,
                                                5)).max() <= bar
    finally:
        mmx.mmx_destroy(ctx)
