"""Backward of bf16 inputs at d = 64 with many workgroups: the key sweep with two key blocks per wave and the r sweep with two
query blocks, against the oracle for one head of the call, and for some forty of all its parts against the same heads in a call of
eight heads, which runs with one block per wave (and which test_gpu_backward.py holds to the oracle).  Lengths on both sides of the 32-row steps, the 64- and 128-row blocks and the first
128 rows; operands strided differently from each other.

Tolerance: the two forms differ in the order of the fp32 sums behind dK only, at most n terms of three kinds per element: n 2^-24 of the
largest partial sum, which cancellation makes some ten times the result: 1e-4 of a head's norm is far above it and far below what a wrong
row, key or fragment does (1e-2 and more)."""
import math

import numpy as np
import pytest
import torch

import paper_2510_01450_amd as llla
from oracle import backward as oracle_backward
from parity import check_grad

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,heads", [(129, 1536), (160, 1536), (257, 768), (300, 768), (384, 768), (513, 384)])
def test_two_blocks_per_wave(n, heads):
    d, H = 64, 8
    g = torch.Generator(device=DEV).manual_seed(n)
    B = heads // H
    def make(order):
        if order == "seq":                                    # [B, n, H, d] in memory
            return torch.randn((B, n, H, d), generator=g, device=DEV).to(torch.bfloat16).transpose(1, 2)
        return torch.randn((B, H, n, d), generator=g, device=DEV).to(torch.bfloat16)
    Q, K, V, G = make("head"), make("seq"), make("head"), make("seq")
    scale = -1 / math.sqrt(d) if n == 300 else 1 / math.sqrt(d)
    got = llla.llla_backward(Q, K, V, G, 1e-2, scale, return_dlambda=True)
    assert all(torch.isfinite(x).all() for x in got)
    for b in (0, B // 3, B // 2, 2 * B // 3, B - 1):
        sl = [t[b:b + 1].contiguous() for t in (Q, K, V, G)]
        ref = llla.llla_backward(*sl, 1e-2, scale, return_dlambda=True)
        for name, x, r in zip(("dQ", "dK", "dV", "dlambda"), got, ref):
            x = x[b:b + 1].double()
            err = (x - r.double()).flatten(2).norm(dim=2) / r.double().flatten(2).norm(dim=2)
            assert float(err.max()) < 1e-4, (name, n, err)
    b, h = B - 2, 5
    head = [t[b, h].cpu().double() for t in (Q, K, V, G)]
    ref = oracle_backward.backward_head(*head, 1e-2, scale)
    floor = [float(head[3].norm() * head[2].norm(dim=-1).pow(2).mean().sqrt())] * 3 + [0.0]
    for name, x, r, fl in zip(("dQ", "dK", "dV", "dlambda"), got, ref, floor):
        print(name, check_grad(x[b, h][None, None].cpu().numpy(), np.asarray(r)[None, None], d, 2e-2, "%s n=%d" % (name, n), floor=fl))


@pytest.mark.parametrize("d,dq_bound,dlam_bound", [(16, 2.5e-4, 1.5e-3), (32, 2.5e-4, 1.5e-3), (64, 2.5e-4, 1.5e-3), (128, 4e-4, 2.5e-3)])
def test_first_rows_have_fp32_accuracy(d, dq_bound, dlam_bound):
    """The first 2 d rows, whose coefficients cancel, take row sweeps with three-term operands.  Bounds on the error of four heads together, some
    twice what the moments leave, whose scaled operand has 22 bits and whose systems have condition numbers of some 10^3 here (seen,
    d = 16 to 128: dQ 5.7e-5 to 2.1e-4, dlambda 2.4e-4 to 1.3e-3; with two-term operands 3.7e-4 to 1.4e-3 and 2.1e-3 to 9.2e-3)."""
    n = 2 * d
    g = torch.Generator(device="cpu").manual_seed(9900 + d)
    Q, K, V, G = [torch.randn((1, 4, n, d), generator=g).bfloat16() for _ in range(4)]
    got = llla.llla_backward(*[t.to(DEV) for t in (Q, K, V, G)], 1e-2, d ** -0.5, path="mfma", return_dlambda=True)
    ref = oracle_backward.backward(Q, K, V, G, 1e-2, d ** -0.5)
    dq, dlam = [np.linalg.norm(got[t].cpu().double().numpy() - ref[t]) / np.linalg.norm(ref[t]) for t in (0, 3)]
    print("dQ %.2e dlambda %.2e" % (dq, dlam))
    assert dq < dq_bound and dlam < dlam_bound


@pytest.mark.parametrize("pitch", [2 ** 24 - 8, 2 ** 24, 2 ** 24 + 64])
def test_rows_far_apart(pitch):
    """Rows 2^24 elements apart: from there on the sweeps of the forward and the backward form an address per row instead of 32-bit offsets from
    a common base.  The same bits as from packed tensors (161 rows: both kinds of blocks, first rows and later ones)."""
    d, H, n = 64, 2, 161
    g = torch.Generator(device="cpu").manual_seed(161)
    packed = [torch.randn((1, H, n, d), generator=g).bfloat16().to(DEV) for _ in range(4)]
    store = torch.empty(n * pitch, dtype=torch.bfloat16, device=DEV)         # 5.4 GB: all four tensors side by side in each row
    far = [store.as_strided((1, H, n, d), (n * pitch, d, pitch, 1), 2 * H * d * t) for t in range(4)]
    for x, y in zip(far, packed):
        x.copy_(y)
    for a, b in zip(llla.llla_forward(*far[:3], 1e-2, 0.125, return_stats=True), llla.llla_forward(*packed[:3], 1e-2, 0.125, return_stats=True)):
        assert torch.isfinite(b).all() and torch.equal(a, b)
    for a, b in zip(llla.llla_backward(*far, 1e-2, 0.125, return_dlambda=True), llla.llla_backward(*packed, 1e-2, 0.125, return_dlambda=True)):
        assert torch.isfinite(b).all() and torch.equal(a, b)
