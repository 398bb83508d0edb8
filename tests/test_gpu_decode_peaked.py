"""Decode where one key far from the origin holds nearly all the weight: a common offset of all keys and the query, and keys of
ten times the usual size.  The moments carry rounding errors of 2^-24 |k|^2 (2^-11 where the weighted keys are 16-bit floats), which the
solve divides by the ridge, so an output is known to |k|^2 / lambda of those at best; where that is more than one it can be
anything of its size, but it has to be finite.  Bound: 8 times that, against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_01450_amd as llla
from parity import row_errors

pytestmark = pytest.mark.gpu
DEV = "cuda"
LAM = 1e-2


def _inputs(kind, B, H, L, d, dtype, seed):
    g = torch.Generator(device="cpu").manual_seed(seed)
    q, K, V = (torch.randn(s, generator=g) for s in ((B, H, d), (B, H, L, d), (B, H, L, d)))
    if kind == "large":
        q, K = 4 * q, 10 * K
    else:
        q, K = q + kind, K + kind
    return [x.to(torch.float32 if dtype == "f32" else torch.bfloat16) for x in (q, K, V)]


def _check(kind, d, dtype, L, seqlens=None, heads=8):
    B = 3 if seqlens is None else len(seqlens)
    q, K, V = _inputs(kind, B, heads, L, d, dtype, 7 * d + L)
    sl = None if seqlens is None else torch.tensor(seqlens, dtype=torch.int32, device=DEV)
    got = llla.llla_decode(q.to(DEV), K.to(DEV), V.to(DEV), LAM, d ** -0.5, seqlens=sl).cpu().numpy()
    assert np.isfinite(got).all(), "%d of %d heads are not finite" % ((~np.isfinite(got).all(-1)).sum(), B * heads)
    ref = oracle.decode(q, K, V, LAM, d ** -0.5, seqlens=seqlens)
    k2 = (K.float() ** 2).sum(-1).amax().item()
    bound = 8 * k2 / LAM * 2.0 ** (-11 if dtype == "bf16" and d >= 64 and L >= 256 else -24)
    err = row_errors(got, ref)
    print("median %.2e max %.2e bound %.2e" % (np.median(err), err.max(), bound))
    assert err.max() <= bound


# every family of decode kernels, with one workgroup per head and with several; bf16 at d = 64 / 128 on the 16-bit kernels from 256 keys on
@pytest.mark.parametrize("d,dtype,L", [(16, "f32", 1000), (16, "bf16", 1000), (32, "f32", 1000), (32, "bf16", 1000), (32, "f32", 4096),
                                       (64, "f32", 1000), (64, "bf16", 200), (64, "f32", 65), (128, "f32", 1000), (128, "f32", 90),
                                       (128, "bf16", 200), (64, "bf16", 1000), (64, "bf16", 4096), (128, "bf16", 1000)])
@pytest.mark.parametrize("kind", ["large", 3.0, 30.0, 100.0])
def test_finite_and_within_the_conditioning(kind, d, dtype, L):
    _check(kind, d, dtype, L)


@pytest.mark.parametrize("d,dtype", [(32, "bf16"), (64, "f32"), (128, "f32")])
def test_lengths_of_their_own(d, dtype):
    _check(30.0, d, dtype, 2000, seqlens=[65, 500, 1999, 2000, 70, 1000])
