"""Every parameter's gradient of the matrix-core network by itself (a small one
beside large ones would not show in a norm over all) against the FP32 kernels
of the same library, on channel counts of every padding; the reverse pass is
given other weights than the forward pass.

Bar: relative 2-norm 5e-2 of each, the BF16 operand rounding (2^-9 per product,
through the layers), as for each gradient in the network tests.
"""
import numpy as np
import pytest

from test_gpu_fno_project import _run

pytestmark = pytest.mark.gpu


def _split(flat, shape):
    H, W, C, M, L, Cp = shape
    sizes = [("P", 5 * C), ("p", C)]
    for l in range(L):
        sizes += [(f"R{l}", 4 * M * M * C * C), (f"W{l}", C * C), (f"b{l}", C)]
    sizes += [("Q1", Cp * C), ("q1", Cp), ("Q2", 3 * Cp), ("q2", 3)]
    at, out = 0, {}
    for name, n in sizes:
        out[name] = flat[at:at + n]
        at += n
    assert at == flat.size
    return out


@pytest.mark.parametrize("shape,batch", [
    ((16, 16, 32, 4, 2, 128), 3), ((18, 15, 20, 4, 2, 20), 2), ((16, 20, 40, 5, 2, 48), 2),
    ((17, 19, 70, 3, 1, 100), 2), ((16, 16, 100, 3, 1, 128), 2),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_each_gradient(shape, batch):
    print(f"[case] fno gradients {shape} batch {batch}", flush=True)
    got = _split(_run(shape, batch, True)[1], shape)
    ref = _split(_run(shape, batch, False)[1], shape)
    rel = {k: np.linalg.norm(got[k] - v) / np.linalg.norm(v) for k, v in ref.items()}
    print({k: f"{v:.1e}" for k, v in rel.items()}, flush=True)
    assert max(rel.values()) <= 5e-2, rel
