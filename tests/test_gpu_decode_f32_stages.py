"""fp32 caches at d = 64: rows staged in LDS by DMA, one step of 32 keys ahead.  Lengths that leave the four waves of a workgroup no step, one, two
and several, whole last steps and partial ones; more heads than the GPU holds at once; the flat cut of 129 heads of 4095 and 4096 keys; the even cut
of 256 heads of as many, which from 4096 on get two workgroups each.  Rows 2 d apart, everything beyond the sequence NaN."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_01450_amd as llla
import workloads
from parity import check

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("B,H,L", [(2, 2, 66), (2, 2, 96), (2, 2, 128), (2, 3, 129), (2, 2, 250), (3, 2, 256), (1, 2, 385), (70, 8, 70), (70, 8, 300),
                                   (43, 3, 4095), (43, 3, 4096), (16, 16, 4095), (16, 16, 4096)])
def test_steps_and_cuts(B, H, L):
    d = 64
    w = workloads.C5.with_shape(name="stages", B=B, H=H, n=L, d=d, dtype="f32", index=2800 + L, values="l2", tol=1e-4, scale=d ** -0.5)
    q, Kc, Vc = workloads.make_inputs(w)
    nb = min(B, 2)
    ref = oracle.decode(q[:nb], Kc[:nb], Vc[:nb], w.lam, w.scale)
    buf = torch.full((2, B, H, L + 3, 2 * d), float("nan"), device=DEV)
    buf[0, :, :, :L, :d] = Kc.to(DEV)
    buf[1, :, :, :L, d:] = Vc.to(DEV)
    got = llla.llla_decode(q.to(DEV), buf[0, :, :, :L, :d], buf[1, :, :, :L, d:], w.lam, w.scale)
    assert torch.isfinite(got).all()
    # (the gate: 24-bit operands and fp32 sums leave some 2^-24 sqrt(L) of the moments, times a condition number of about 4, and more below 4 d keys)
    check(got[:nb].cpu().numpy()[:, :, None], ref[:, :, None], np.array([L - 1]), d, 1e-5 if L >= 256 else 1e-4, "L=%d heads %d" % (L, B * H))
    # the same keys as the first L of longer caches
    lens = torch.full((B,), L, dtype=torch.int32, device=DEV)
    again = llla.llla_decode(q.to(DEV), buf[0, ..., :d], buf[1, ..., d:], w.lam, w.scale, seqlens=lens)
    check(again[:nb].cpu().numpy()[:, :, None], ref[:, :, None], np.array([L - 1]), d, 1e-5 if L >= 256 else 1e-4, "lengths, L=%d" % L)


@pytest.mark.parametrize("d", [16, 32])
@pytest.mark.parametrize("L", [40, 700])
def test_values_of_any_size(d, L):
    """The output is linear in V, so values times a power of two give the same bits times it, as long as neither is subnormal: the solve takes the
    value moments' columns in three bf16, whose third term would be lost from 2^-110 on and whose first overflows at 2^127.99."""
    g = torch.Generator(device="cpu").manual_seed(3000 + L + d)
    q, K, V = [torch.randn(s, generator=g).to(DEV) for s in ((2, 3, d), (2, 3, L, d), (2, 3, L, d))]
    base = llla.llla_decode(q, K, V, 1e-2, d ** -0.5)
    assert torch.isfinite(base).all()
    for k in (-110, -100, -60, 60, 110):
        got = llla.llla_decode(q, K, V * 2.0 ** k, 1e-2, d ** -0.5)
        assert torch.equal(got.double(), base.double() * 2.0 ** k), k


@pytest.mark.parametrize("dtype,d", [(torch.float32, 16), (torch.float32, 32), (torch.float32, 64), (torch.bfloat16, 16), (torch.bfloat16, 32)])
@pytest.mark.parametrize("L", [80, 700, 3000])
def test_value_features_of_different_sizes(dtype, d, L):
    """The same with a power of two of its own for every feature of V: no feature of the output hangs on the size of another."""
    g = torch.Generator(device="cpu").manual_seed(3100 + L + d)
    q, K, V = [torch.randn(s, generator=g).to(dtype).to(DEV) for s in ((2, 3, d), (2, 3, L, d), (2, 3, L, d))]
    k = [-110, 110, 0, -60, 60, -100, 0, -85] * (d // 8)
    size = torch.tensor([2.0 ** k[i] for i in torch.randperm(d, generator=g)], dtype=torch.float64).to(DEV)
    base = llla.llla_decode(q, K, V, 1e-2, d ** -0.5)
    got = llla.llla_decode(q, K, (V.double() * size).to(dtype), 1e-2, d ** -0.5)
    assert torch.isfinite(base).all() and torch.equal(got.double(), base.double() * size)


@pytest.mark.parametrize("H", [3, 300])
def test_value_features_that_grow(H):
    """Features of V that are zero, or as good as zero, up to some key and of ordinary size from there on, another one after every wave's first step."""
    d, L = 64, 900
    w = workloads.C5.with_shape(name="grow", B=2, H=H, n=L, d=d, dtype="f32", index=3150 + H, values="l2", tol=1e-4, scale=d ** -0.5)
    q, K, V = workloads.make_inputs(w)
    from_key = torch.arange(d) * 13                            # feature 0 is whole, feature 63 begins at key 819
    before = (torch.arange(L)[:, None] < from_key).to(V.dtype)
    zero, tiny = V * (1 - before), V * (1 - before) + V * before * 2.0 ** -100
    ref = oracle.decode(q[:1, :3], K[:1, :3], zero[:1, :3], w.lam, w.scale)
    for x in (zero, tiny):
        got = llla.llla_decode(q.to(DEV), K.to(DEV), x.to(DEV), w.lam, w.scale)
        # (24-bit operands and fp32 sums, as in test_steps_and_cuts)
        check(got[:1, :3].cpu().numpy()[:, :, None], ref[:, :, None], np.array([L - 1]), d, 1e-5, "H=%d" % H)


@pytest.mark.parametrize("d", [16, 32, 64])
def test_queries_of_any_size(d):
    """Keys and values in pairs of opposite sign have no mean, and queries so small that all weights are one then give an output that is linear in
    them: the same bits times the power of two."""
    g = torch.Generator(device="cpu").manual_seed(3200 + d)
    L = 640
    q, K, V = [torch.randn(s, generator=g) for s in ((2, 3, d), (2, 3, L // 2, d), (2, 3, L // 2, d))]
    K, V = [torch.stack((x, -x), dim=3).reshape(2, 3, L, d).to(DEV) for x in (K, V)]
    q = q.to(DEV)
    base = llla.llla_decode(q * 2.0 ** -60, K, V, 1e-2, d ** -0.5)
    assert torch.isfinite(base).all() and (base != 0).any()
    for k in (-112, -90):
        assert torch.equal(llla.llla_decode(q * 2.0 ** k, K, V, 1e-2, d ** -0.5).double(), base.double() * 2.0 ** (k + 60)), k


@pytest.mark.parametrize("dtype,d,H,e", [(torch.float32, 16, 3, 58), (torch.float32, 32, 3, 54), (torch.float32, 32, 3, 58), (torch.bfloat16, 32, 3, 54),
                                         (torch.float32, 64, 3, 52), (torch.float32, 64, 150, 52)])
@pytest.mark.parametrize("L", [100, 700])
def test_keys_and_ridges_of_any_size(dtype, d, H, e, L):
    """Query and keys times 2^-e, the scale times 2^2e and the ridge times 2^-2e are the same problem: the same bits, as long as the moments that the
    matrix cores sum are not subnormal (fp32 caches at d = 64, whose products are taken of three bf16 terms: from 2^-54 on)."""
    g = torch.Generator(device="cpu").manual_seed(3300 + d + L)
    q, K, V = [torch.randn(s, generator=g).to(dtype).to(DEV) for s in ((2, H, d), (2, H, L, d), (2, H, L, d))]
    base = llla.llla_decode(q, K, V, 1e-2, d ** -0.5)
    s = 2.0 ** -e
    assert torch.isfinite(base).all() and torch.equal(llla.llla_decode(q * s, K * s, V, 1e-2 * s * s, d ** -0.5 / (s * s)), base)


@pytest.mark.parametrize("B,H,L", [(16, 16, 1024), (4, 3, 21760), (5, 12, 4352)])
def test_order_of_shares(B, H, L):
    """Sequences of lengths of their own: up to two units of 256 keys of full caches per slot (the capacities here, to within a unit) the heads' first
    shares start first, beyond it a head's shares together.  The shares are the same, and so are the bits."""
    d = 64
    g = torch.Generator(device="cpu").manual_seed(3400 + L)
    units = 1024 // (B * H)
    assert L == 256 * units
    q, K, V = [torch.randn(s, generator=g).to(DEV) for s in ((B, H, d), (B, H, L + 1, d), (B, H, L + 1, d))]
    lens = torch.randint(1, L + 1, (B,), generator=g, dtype=torch.int32)
    lens[B - 1] = L
    lens = lens.to(DEV)
    got = llla.llla_decode(q, K[:, :, :L], V[:, :, :L], 1e-2, d ** -0.5, seqlens=lens)
    assert torch.isfinite(got).all() and torch.equal(got, llla.llla_decode(q, K, V, 1e-2, d ** -0.5, seqlens=lens))
