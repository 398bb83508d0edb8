"""bf16 calls whose stages share launches: the first rows and the others in one launch or in two (by the number of workgroups), and the
padded copies of d = 16 / 32 beside the row maxima and the re-tiled keys, which read the narrow rows themselves.  The parts do the same
sums whoever launches them, so what they give is compared bit for bit; dK and dV of many heads come from a sweep with two key blocks per
wave (d = 16, 32 and 64), whose sums round in another order."""
import math

import pytest
import torch

import paper_2510_01450_amd as llla

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _inputs(B, H, n, d, seed, count=4):
    g = torch.Generator(device=DEV).manual_seed(seed)
    return [torch.randn((B, H, n, d), generator=g, device=DEV).to(torch.bfloat16) for _ in range(count)]


@pytest.mark.parametrize("d,n", [(16, 129), (32, 130), (64, 193), (64, 128), (128, 257), (128, 320)])
def test_many_heads_as_few(d, n):
    """More heads than the rule takes into one launch, and four of them alone, which it does (at n = 128, d = 64 there are first rows only).
    dK and dV: 1e-4 of a head's norm, see test_gpu_backward_blocks.py."""
    H = 4
    blocks = max(1, (n - min(n, 2 * max(d, 64)) + 63) // 64)
    B = 2048 // (H * blocks) + 2
    Q, K, V, G = _inputs(B, H, n, d, 100 + n)
    scale = 1 / math.sqrt(d)
    O, rho, delta = llla.llla_forward(Q, K, V, 1e-2, scale, path="mfma", return_stats=True)
    dQ, dK, dV, dlam = llla.llla_backward(Q, K, V, G, 1e-2, scale, path="mfma", return_dlambda=True)
    for b in (0, B // 2, B - 1):
        q, k, v, g = [t[b:b + 1].contiguous() for t in (Q, K, V, G)]
        few = (*llla.llla_forward(q, k, v, 1e-2, scale, path="mfma", return_stats=True),)
        grad = llla.llla_backward(q, k, v, g, 1e-2, scale, path="mfma", return_dlambda=True)
        for x, r in zip((O, rho, delta, dQ, dlam), (*few, grad[0], grad[3])):
            assert torch.isfinite(r).all() and torch.equal(x[b:b + 1], r)
        for x, r in zip((dK, dV), grad[1:3]):
            err = (x[b:b + 1].double() - r.double()).flatten(2).norm(dim=2) / r.double().flatten(2).norm(dim=2)
            assert float(err.max()) < 1e-4, err


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("d,n", [(16, 33), (16, 97), (16, 200), (32, 64), (32, 161)])
def test_narrow_rows_end_where_they_end(d, n, causal):
    """Rows of d features inside wider ones whose other elements are not numbers: the features beyond d are zero, not what lies there."""
    packed = _inputs(2, 3, n, d, 200 + n)
    wide = [torch.full((2, n, 3, 64 + 8 * t), float("nan"), dtype=torch.bfloat16, device=DEV) for t in range(4)]
    views = [w[..., 8:8 + d].transpose(1, 2) for w in wide]
    for v, p in zip(views, packed):
        v.copy_(p)
    scale = -0.2
    kw = dict(path="mfma", causal=causal)
    for x, r in zip(llla.llla_forward(*views[:3], 1e-2, scale, return_stats=True, **kw), llla.llla_forward(*packed[:3], 1e-2, scale, return_stats=True, **kw)):
        assert torch.isfinite(r).all() and torch.equal(x, r)
    if causal:
        for x, r in zip(llla.llla_backward(*views, 1e-2, scale, path="mfma", return_dlambda=True),
                        llla.llla_backward(*packed, 1e-2, scale, path="mfma", return_dlambda=True)):
            assert torch.isfinite(r).all() and torch.equal(x, r)
