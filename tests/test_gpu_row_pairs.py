"""Register row and column kernels at the edges of their work split: column
counts below, at and beyond a wave's, zero halves left out or not, odd replica
counts; rows that pair their spectrum columns (every split, open and periodic,
row counts that leave a wave partly empty), against the oracle.

Bars as for the other FP32 kernels: fields 4e-6 of max |H|, states 1e-5; a
replica of a batch equals the same replica alone bit for bit.
"""
import numpy as np
import pytest

from oracle import fields as ofl
from oracle import integrators as oit
from workloads import random_unit, replica_seeds, uniform

from _mmx_case import Case, dev, host, open_ctx

pytestmark = pytest.mark.gpu


def _case(n, R, per=0, T=0.0, base=13):
    return Case(n, (3e-9, 2.5e-9, 2e-9), pbc=(per, per, 0), images=(per, per, 0), R=R, Ms=8e5,
                A=1.3e-11, alpha=0.1, Ku=2e5, B=(0.01, 0.0, 0.03), T=T,
                seeds=list(replica_seeds(base, R)) if T else [],
                terms=("exchange", "anisotropy", "zeeman", "demag") + (("thermal",) if T else ()))


# padded columns of 64, 128 and 256 points, nx + 1 (nx / 2 + 1 periodic) of them
@pytest.mark.parametrize("R", [1, 3, 7])
@pytest.mark.parametrize("g", [(1, 32, 0), (2, 32, 0), (5, 32, 0), (8, 64, 0), (3, 128, 0),
                               (16, 32, 0), (30, 64, 1), (4, 128, 1)],
                         ids=lambda g: f"{g[0]}x{g[1]}" + "p" * g[2])
def test_columns_of_every_count(g, R):
    import paper_2608_15253_amd as mmx
    print(f"[case] columns {g} R={R}", flush=True)
    case = _case((g[0], g[1], 1), R, g[2])
    m0 = random_unit(case.n, seed=9, replicas=R).astype(np.float32).astype(np.float64)

    def field(c, m):
        ctx = open_ctx(c, mmx.MMX_F32)
        try:
            H = dev(np.zeros_like(m), mmx.MMX_F32)
            mmx.mmx_field(ctx, dev(m, mmx.MMX_F32), H)
            return host(H)
        finally:
            mmx.mmx_destroy(ctx)

    got = field(case, m0)
    for r in range(R):
        ref = ofl.effective_field(m0[r], case.grid, case.material())
        assert np.abs(got[r] - ref).max() <= 4e-6 * np.abs(ref).max()
    alone = field(_case((g[0], g[1], 1), 1, g[2]), m0[R - 1:])
    assert np.array_equal(got[R - 1:], alone)


# half lengths 16 to 256: nx open, nx / 2 periodic
@pytest.mark.parametrize("per", [0, 1], ids=["open", "periodic"])
@pytest.mark.parametrize("hx", [16, 32, 64, 96, 128, 256])
def test_rows_of_every_split(hx, per):
    import paper_2608_15253_amd as mmx
    case = _case((hx * (1 + per), 5, 1), 2, per, T=300.0)
    print(f"[case] rows hx={hx} periodic={per}", flush=True)
    m0 = uniform(case.n, (0.2, 0.1, 1.0), replicas=2)
    m0 += 0.2 * random_unit(case.n, seed=4, replicas=2)
    m0 /= np.linalg.norm(m0, axis=1, keepdims=True)
    m0 = m0.astype(np.float32).astype(np.float64)
    ctx = open_ctx(case, mmx.MMX_F32)
    try:
        md = dev(m0, mmx.MMX_F32)
        mmx.mmx_heun(ctx, md, 2e-14, 4, 3)
        got = host(md)
    finally:
        mmx.mmx_destroy(ctx)
    ref = oit.heun_run(m0, case.grid, case.material(), 2e-14, 4, seed=np.array(case.seeds),
                       step0=3)
    assert np.abs(got - ref).max() <= 1e-5
