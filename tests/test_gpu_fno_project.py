"""The fused projection of the network (both maps and the GELU between them in
one pass, recomputed in the reverse pass) and the multi-plane transforms on
channel counts of every padding (one to four reduction steps, projection widths
that are no multiple of the instruction's), odd pixel counts and batches beyond
the workgroups of one launch: forward and every gradient against the FP32
kernels of the same library, which the oracle pins elsewhere.  The reverse pass
is given other weights than the forward pass, whose activations it must keep.

Bars: relative 2-norm 2e-2 forward and 5e-2 per gradient, the BF16 operand
rounding (2^-9 per product, through the layers) as in the network tests.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _run(shape, batch, mfma):
    import torch
    import paper_2608_15253_amd as mmx
    H, W, C, M, L, Cp = shape
    net = mmx.mmx_fno_create(H, W, C, M, M, L, Cp, batch, mfma)
    try:
        mmx.mmx_fno_set_stream(net, torch.cuda.current_stream().cuda_stream)
        n = mmx.mmx_fno_param_count(net)
        p = torch.empty(n, dtype=torch.float32, device="cuda:0")
        mmx.mmx_fno_init(net, p, 3)
        g = torch.Generator().manual_seed(5)
        # biases and modes of ordinary size, so that every term counts
        p += 0.02 * torch.randn(n, generator=g).to("cuda:0")
        m = torch.randn((batch, 3, H, W), generator=g)
        m = (m / m.norm(dim=1, keepdim=True)).to("cuda:0").contiguous()
        t = torch.randn((batch, 3, H, W), generator=g).to("cuda:0").contiguous()
        h, grad = torch.empty_like(m), torch.empty_like(p)
        out = []
        for _ in range(2):   # the second pass on warm buffers equals the first
            mmx.mmx_fno_forward(net, p, m, h, batch)
            # moved weights: the activations stay those of the forward pass
            mmx.mmx_fno_backward(net, 1.25 * p, h, t, grad, want_loss=False)
            torch.cuda.synchronize()
            out.append((h.double().cpu().numpy(), grad.double().cpu().numpy()))
        assert all(np.array_equal(a, b) for a, b in zip(*out))
        return out[0]
    finally:
        mmx.mmx_fno_destroy(net)


@pytest.mark.parametrize("shape,batch", [
    ((16, 16, 32, 4, 2, 128), 3), ((18, 15, 20, 4, 2, 20), 2), ((16, 20, 40, 5, 2, 48), 2),
    ((17, 19, 70, 3, 1, 100), 2), ((16, 16, 100, 3, 1, 128), 2), ((128, 16, 32, 5, 1, 64), 40),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_projection_and_transforms(shape, batch):
    print(f"[case] fno projection {shape} batch {batch}", flush=True)
    h, g = _run(shape, batch, True)
    hr, gr = _run(shape, batch, False)
    assert np.linalg.norm(h - hr) <= 2e-2 * np.linalg.norm(hr)
    assert np.linalg.norm(g - gr) <= 5e-2 * np.linalg.norm(gr)
