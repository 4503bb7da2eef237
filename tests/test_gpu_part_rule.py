"""Working sets beyond the sizes at which Heun and rotation runs are split into
parts, for films and blocks of either precision and through retire/refill:
every replica bit for bit as in a context of few replicas, which is one part."""
import numpy as np
import pytest

from _mmx_case import dev, host, open_ctx
from test_gpu_run_parts import _case, _start, _sub

pytestmark = pytest.mark.gpu


def _few(R):
    return sorted({0, 1, R // 3, R // 2 - 1, R // 2, R // 2 + 1, 2 * R // 3, R - 1})


# working set per replica (spectrum and states): 396 KB, 1.19 MB, 2.38 MB; split
# above 320 MB (FP64 films), 380 MB (FP32 blocks), 450 MB (FP64 blocks)
@pytest.mark.parametrize("n,prec,R", [((64, 64, 1), 2, 860), ((64, 64, 4), 1, 340),
                                      ((64, 64, 4), 2, 200)],
                         ids=["film-f64", "block-f32", "block-f64"])
def test_split_groups_equal_single_contexts(n, prec, R):
    import paper_2608_15253_amd as mmx
    print(f"[case] parts {n} prec={prec} R={R}", flush=True)
    case = _case(n, R)
    m0, few = _start(case), _few(R)

    def run(c, start):
        ctx = open_ctx(c, prec)
        try:
            md, ts = dev(start, prec), dev(-np.ones(c.R), mmx.MMX_F64)
            mmx.mmx_heun(ctx, md, 1e-14, 3, 2, ts)
            mmx.mmx_heun(ctx, md, 1e-14, 2, 5, ts)
            return host(md), host(ts)
        finally:
            mmx.mmx_destroy(ctx)

    got, ts = run(case, m0)
    ref, tr = run(_sub(case, few), m0[few])
    assert np.array_equal(got[few], ref)
    assert np.array_equal(ts[few], tr)
    assert np.all((ts[::3] > 0)) and np.all(np.delete(ts, np.s_[::3]) < 0)


def test_split_refill_equals_single_context():
    import torch
    import paper_2608_15253_amd as mmx
    R, cap = 1400, 4   # 346 MB with the rotation's slopes
    case = _case((64, 64, 1), R)
    m0, few = _start(case), _few(R)

    def run(c, start):
        ctx = open_ctx(c, mmx.MMX_F32)
        try:
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
