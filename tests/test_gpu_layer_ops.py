"""The row-wise kernels of the layer slice at the edges of their chunks, and
the tensors that they leave to the framework's own operations.

Tolerances: one bf16 rounding of the exact result (2^-8 relative, half an ulp
being 2^-9), plus a few fp32 roundings."""

import numpy as np
import pytest
import torch

import workloads as W
from oracle import layer_oracle as LO

pytestmark = pytest.mark.gpu


def _draw(*shape, seed=0, scale=1.0):
    g = torch.Generator().manual_seed(seed)
    return (scale * torch.randn(*shape, generator=g)).to(torch.bfloat16).cuda()


def _close(got, want):
    err = (got.double() - want).abs()
    assert bool((err <= 2.0 ** -8 * want.abs() + 1e-30).all()), float(err.max())


@pytest.mark.parametrize("rows,width", [(1, 8), (3, 2040), (5, 2048), (4, 2056), (7, 4096), (2, 8200),
                                        (3, 16384)])
def test_rms_norm(rows, width):
    from paper_2606_09441_amd._lib import rms_norm
    x, w = _draw(rows, width, scale=3.0), 1 + 0.1 * _draw(width, seed=1)
    want = x.double() * torch.rsqrt(x.double().square().mean(-1, keepdim=True) + 1e-5) * w.double()
    _close(rms_norm(x, w, 1e-5), want)


@pytest.mark.parametrize("shape", [(1, 8), (3, 24), (257, 2048)])
def test_silu_mul(shape):
    from paper_2606_09441_amd._lib import silu_mul
    g, u = _draw(*shape, scale=4.0), _draw(*shape, seed=1)
    g.view(-1)[:3] = torch.tensor([-200.0, 200.0, 0.0])
    want = g.double() / (1 + torch.exp(-g.double())) * u.double()
    _close(silu_mul(g, u), want)


@pytest.mark.parametrize("n,hq,hkv,d,skew", [(1, 1, 1, 16, 0), (5, 3, 1, 64, 0), (9, 4, 2, 128, 0),
                                             (6, 2, 2, 512, 0), (7, 2, 1, 20, 0), (5, 2, 1, 64, 4)])
def test_rope(n, hq, hkv, d, skew):
    """Whole 16-byte chunks, other head sizes, and storage off a 16-byte line."""
    from paper_2606_09441_amd import rope_
    rng = np.random.default_rng(d)
    pos = rng.integers(0, 70000, size=n).astype(np.int32)
    f = W.rope_inv_freq(d)
    xs = []
    for h in (hq, hkv):
        buf = _draw(n * h * d + skew, seed=h)
        xs.append(buf[skew:].view(n, h, d))
    want = [LO.rope(x.float().cpu().numpy(), pos, f) for x in xs]
    rope_(*xs, torch.from_numpy(pos).cuda(), torch.from_numpy(f).cuda())
    for x, r in zip(xs, want):
        err = np.abs(x.float().cpu().numpy() - r)
        # angles up to 70000 rad are fp32 products: off by up to 70000 * 2^-24
        assert (err <= 2.0 ** -8 * np.abs(r) + 70000 * 2.0 ** -24 * 8).all(), err.max()


def test_left_to_the_framework():
    from paper_2606_09441_amd._lib import rms_norm, silu_mul
    x, w = _draw(4, 64), _draw(64, seed=1)
    assert rms_norm(x, w, 1e-5) is not None
    assert rms_norm(x.float(), w, 1e-5) is None
    assert rms_norm(x[:, :60], w[:60], 1e-5) is None           # width, not contiguous
    assert rms_norm(_draw(65)[1:].view(1, 64), w, 1e-5) is None    # off a 16-byte line
    assert rms_norm(x.clone().requires_grad_(), w, 1e-5) is None
    assert rms_norm(x.cpu(), w.cpu(), 1e-5) is None
    with torch.autograd.forward_ad.dual_level():
        assert rms_norm(x, w, 1e-5) is None
    assert silu_mul(x, x.float()) is None
    assert silu_mul(x.t(), x.t()) is None


def test_layer_keeps_float_residuals_and_gradients():
    """An fp32 residual stream and a recorded gradient, through the MLP too."""
    from paper_2606_09441_amd import Plan
    from paper_2606_09441_amd.layer import PrefillLayer
    hq, hkv, d = 4, 2, 128
    wl = W.custom([[130, 60, 33]], tile=64, hq=hq, hkv=hkv, d=d, dtype="bf16", seed=5)
    n, hidden = wl.tokens, hq * d
    w = {k: torch.from_numpy(v).cuda().bfloat16()
         for k, v in W.layer_weights(hidden, hq, hkv, d, 2 * hidden, seed=1).items()}
    layer = PrefillLayer(w, hq, hkv, d, torch.from_numpy(W.rope_inv_freq(d)).cuda())
    pos = torch.from_numpy(W.prompt_positions(wl.seg_offsets, wl.prompt_seg_ptr)).cuda()
    la, ca = torch.from_numpy(wl.la).cuda(), torch.from_numpy(wl.ca).cuda()
    x = torch.from_numpy(W.layer_input(n, hidden, seed=2)).cuda()
    with Plan(wl.seg_offsets, wl.prompt_seg_ptr, hq, hkv, d, 64) as plan:
        a = layer.forward(x, plan, pos, la, ca)
        b = layer.forward(x.bfloat16(), plan, pos, la, ca)
        assert a.dtype == torch.float32 and b.dtype == torch.bfloat16
        assert float((a - b.float()).abs().max()) <= 0.02 * float(a.abs().max())
        xg = x.bfloat16().requires_grad_()
        layer.forward(xg, plan, pos, la, ca).float().sum().backward()
        # beside the residual's own 1 there is the MLP's part
        assert float((xg.grad.float() - 1).abs().max()) > 0.1
        torch.cuda.synchronize()
