"""How a batch of sequences of different lengths is cut into the shares of workgroups (fewest keys worth a workgroup: 512 for bf16
caches at d = 64, 256, or 128 for fp32 caches at d = 128): one sequence far longer than the others, about as many slots as sequences
(two rounds of parts), every group of 64 sequences that the search for a share looks at together (256) and more than it serves (257: even
cut), lengths on both sides of a share, and calls with one workgroup per head.  bf16 caches at d = 128 take equal shares only from some
2^21 keys on (test_equal_shares_at_d128); the others here take the even cut there.  Sampled sequences against the fp64 oracle; every
sequence, or one of a few, against a call of its own."""
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


@pytest.mark.parametrize("B", [256, 257])
@pytest.mark.parametrize("d,dtype", [(64, "bf16"), (64, "f32"), (32, "bf16"), (16, "f32")])
def test_many_sequences(d, dtype, B):
    H, L = 2, 600
    tol = 2e-2 if dtype == "bf16" and d >= 64 else 1e-4
    w = workloads.C5.with_shape(name="many", B=B, H=H, n=L, d=d, dtype=dtype, index=2700 + d, values="l2", tol=tol, scale=d ** -0.5)
    q, Kc, Vc = workloads.make_inputs(w)
    lens = _lens("spread", B, L)
    got = llla.llla_decode(q.to(DEV), Kc.to(DEV), Vc.to(DEV), w.lam, w.scale, seqlens=lens.to(DEV)).cpu().numpy()
    for b in (0, 1, 62, 63, 64, 65, 127, 128, 129, 190, 191, 192, 193, 254, 255, B - 1):
        n = int(lens[b])
        ref = oracle.decode(q[b:b + 1], Kc[b:b + 1], Vc[b:b + 1], w.lam, w.scale, seqlens=[n])
        check(got[b:b + 1, :, None], ref[:, :, None], np.array([n - 1]), d, tol, "b=%d len=%d d=%d" % (b, n, d))


@pytest.mark.parametrize("equal", [False, True])
def test_equal_shares_at_d128(equal):
    """40 sequences x 16 heads x up to 4096 keys in 512 workgroups: shares of unequal pieces, with sequences of at most 4 d keys (weights in
    two terms) and longer ones in turn in one workgroup; and 40 equal ones."""
    B, H, L, d, tol = 40, 16, 4096, 128, 2e-2
    # (with the flat cut the scratch holds 512 + 640 records, with the even one 640)
    assert llla.decode_workspace_bytes(B, H, L, d, torch.bfloat16) >= (512 + B * H) * 25920 * 4
    g = torch.Generator(device=DEV).manual_seed(128)
    q, Kc, Vc = (torch.randn(s, generator=g, device=DEV, dtype=torch.bfloat16) for s in ((B, H, d), (B, H, L, d), (B, H, L, d)))
    kinds = (1, 700, 64, 4096, 511, 65, 4095, 512, 33, 513, 2000, 128, 1025, 300, 4096, 5)
    lens = torch.tensor([L if equal else kinds[(3 * b) % len(kinds)] for b in range(B)], dtype=torch.int32)
    sl = None if equal else lens.to(DEV)
    if not equal:
        for b in range(B):                                               # rows beyond a sequence are never read
            Kc[b, :, int(lens[b]):] = float("nan")
            Vc[b, :, int(lens[b]):] = float("nan")
    got = llla.llla_decode(q, Kc, Vc, 1e-2, d ** -0.5, seqlens=sl)
    assert torch.equal(got, llla.llla_decode(q, Kc, Vc, 1e-2, d ** -0.5, seqlens=sl))
    got = got.cpu().numpy()
    for b in range(0, B, 3 if equal else 1):
        n = int(lens[b])
        heads = slice(b % 8, b % 8 + 9, 8)
        k, v = Kc[b:b + 1, heads, :n].contiguous(), Vc[b:b + 1, heads, :n].contiguous()
        ref = oracle.decode(q[b:b + 1, heads].cpu(), k.cpu(), v.cpu(), 1e-2, d ** -0.5)
        check(got[b:b + 1, heads, None], ref[:, :, None], np.array([n - 1]), d, tol, "b=%d len=%d" % (b, n))
