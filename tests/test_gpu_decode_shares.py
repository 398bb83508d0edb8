"""How a batch of sequences of different lengths is cut into the shares of workgroups (fewest keys worth a workgroup: 256, or 128
for fp32 caches at d = 128): one sequence far longer than the others, about as many slots as sequences (two rounds of parts), more
sequences than the search for a share serves (129: even cut), lengths on both sides of a share, and calls with one workgroup per
head.  Sampled sequences against the fp64 oracle; every sequence against a call of its own."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_01450_amd as llla
import workloads
from parity import check

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _lens(kind, B, L):
    g = torch.Generator().manual_seed(B + L)
    if kind == "one_long":
        lens = torch.randint(1, 40, (B,), generator=g)
    elif kind == "edges":
        lens = torch.tensor([(1, 255, 256, 257, 511, 512, 513, L - 1)[i % 8] for i in range(B)])
    else:
        lens = torch.randint(L // 8, L + 1, (B,), generator=g)
    lens[B // 2] = L
    return lens.to(torch.int32)


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "f32"), (128, "f32"), (32, "bf16"), (16, "f32")])
@pytest.mark.parametrize("kind,B,H,L", [("one_long", 3, 2, 5000), ("edges", 9, 3, 1100), ("spread", 20, 16, 1500),
                                         ("spread", 36, 16, 700), ("spread", 129, 2, 600)])
def test_different_lengths(d, dtype, kind, B, H, L):
    tol = 2e-2 if dtype == "bf16" and d >= 64 else 1e-4
    w = workloads.C5.with_shape(name="shares", B=B, H=H, n=L, d=d, dtype=dtype, index=2500 + d, values="l2", tol=tol, scale=d ** -0.5)
    q, Kc, Vc = workloads.make_inputs(w)
    lens = _lens(kind, B, L)
    qd, Kd, Vd = q.to(DEV), Kc.to(DEV), Vc.to(DEV)
    got = llla.llla_decode(qd, Kd, Vd, w.lam, w.scale, seqlens=lens.to(DEV))
    assert torch.equal(got, llla.llla_decode(qd, Kd, Vd, w.lam, w.scale, seqlens=lens.to(DEV)))
    got = got.cpu().numpy()
    for b in sorted({0, 1, B // 2, B - 1}):
        n = int(lens[b])
        ref = oracle.decode(q[b:b + 1, :2], Kc[b:b + 1, :2], Vc[b:b + 1, :2], w.lam, w.scale, seqlens=[n])
        check(got[b:b + 1, :2, None], ref[:, :, None], np.array([n - 1]), d, tol, "b=%d len=%d d=%d" % (b, n, d))
    # each sequence in a call of its own (other shares, other partial sums): rounding apart the same numbers
    for b in range(0, B, max(1, B // 12)):
        alone = llla.llla_decode(qd[b:b + 1], Kd[b:b + 1], Vd[b:b + 1], w.lam, w.scale, seqlens=lens[b:b + 1].to(DEV)).cpu().numpy()
        n = int(lens[b])
        check(got[b:b + 1, :, None], alone[:, :, None], np.array([n - 1]), d, tol, "alone b=%d len=%d d=%d" % (b, n, d))


@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (128, "bf16"), (64, "f32"), (128, "f32"), (32, "bf16")])
def test_full_lengths_that_do_not_divide_the_gpu(d, dtype):
    """600 heads for 512 or 1024 slots: equal shares that end in the middle of a sequence."""
    B, H, L = 75, 8, 1100
    tol = 2e-2 if dtype == "bf16" and d >= 64 else 1e-4
    w = workloads.C5.with_shape(name="uneven", B=B, H=H, n=L, d=d, dtype=dtype, index=2600 + d, values="l2", tol=tol, scale=d ** -0.5)
    q, Kc, Vc = workloads.make_inputs(w)
    qd, Kd, Vd = q.to(DEV), Kc.to(DEV), Vc.to(DEV)
    got = llla.llla_decode(qd, Kd, Vd, w.lam, w.scale).cpu().numpy()
    for b in (0, 1, 37, B - 1):
        ref = oracle.decode(q[b:b + 1, :2], Kc[b:b + 1, :2], Vc[b:b + 1, :2], w.lam, w.scale)
        check(got[b:b + 1, :2, None], ref[:, :, None], np.array([L - 1]), d, tol, "b=%d d=%d" % (b, d))
    for b in range(0, B, 7):
        alone = llla.llla_decode(qd[b:b + 1], Kd[b:b + 1], Vd[b:b + 1], w.lam, w.scale).cpu().numpy()
        check(got[b:b + 1, :, None], alone[:, :, None], np.array([L - 1]), d, tol, "alone b=%d d=%d" % (b, d))
