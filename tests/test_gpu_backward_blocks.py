"""Backward of bf16 inputs at d = 64 with many workgroups: the key sweep with two key blocks per wave and the r sweep with two
query blocks, against the same heads in a call of four heads, which runs with one block per wave (and which
test_gpu_backward.py holds to the oracle).  Lengths on both sides of the 32-row steps, the 64- and 128-row blocks and the first
128 rows; operands strided differently from each other.

Tolerance: the two forms differ in the order of the fp32 sums behind dK only, at most n terms of three kinds per element: n 2^-24 of the
largest partial sum, which cancellation makes some ten times the result: 1e-4 of a head's norm is far above it and far below what a wrong
row, key or fragment does (1e-2 and more)."""
import math

import pytest
import torch

import paper_2510_01450_amd as llla

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
    for b in (0, B - 1):
        sl = [t[b:b + 1, 2:6].contiguous() for t in (Q, K, V, G)]
        ref = llla.llla_backward(*sl, 1e-2, scale, return_dlambda=True)
        for name, x, r in zip(("dQ", "dK", "dV", "dlambda"), got, ref):
            x = x[b:b + 1, 2:6].double()
            err = (x - r.double()).flatten(2).norm(dim=2) / r.double().flatten(2).norm(dim=2)
            assert torch.isfinite(x).all() and float(err.max()) < 1e-4, (name, n, err)
