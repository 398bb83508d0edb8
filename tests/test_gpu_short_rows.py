"""Forward of few short fp32 sequences at d = 16 / 32 (one wave per row): lengths around the key-space rows, the 64 keys of a lane
pass, the chunks of 32 keys and the longest length served, causal and not, a ridge per row, statistics, strided operands, both output
types, and calls on both sides of the rule.  Gate and oracle as in the other parity tests."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2510_01450_amd as llla
import workloads
from parity import check

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _inputs(B, H, n, d, seed):
    g = torch.Generator(device="cpu").manual_seed(seed)
    Q, K, V = [torch.randn((B, n, H, d), generator=g).transpose(1, 2) for _ in range(3)]       # [B, n, H, d] in memory
    lam = 1e-2 * torch.exp(0.5 * torch.randn((B, H, n), generator=g))
    return Q, K, V, lam


@pytest.mark.parametrize("d", [16, 32])
@pytest.mark.parametrize("n", [17, 31, 33, 63, 64, 65, 95, 128, 129, 191, 193, 255, 256, 257])
def test_lengths(n, d):
    Q, K, V, lam = _inputs(1, 3, n, d, 8000 + n + d)
    scale = 1 / math.sqrt(d)
    O, rho, delta = llla.llla_forward(Q.to(DEV), K.to(DEV), V.to(DEV), lam.to(DEV), scale, return_stats=True)
    ref, r, dl = oracle.forward_ex(Q.contiguous(), K.contiguous(), V.contiguous(), lam, scale)
    check(O.cpu().numpy(), ref, np.arange(n), d, 1e-4, "n=%d d=%d" % (n, d))
    check(rho.cpu().numpy(), r, np.arange(n), d, 1e-4, "rho n=%d d=%d" % (n, d))
    check(delta.cpu().numpy()[..., None], dl[..., None], np.arange(n), d, 1e-4, "delta n=%d d=%d" % (n, d))
    half = llla.llla_forward(Q.to(DEV), K.to(DEV), V.to(DEV), lam.to(DEV), scale, out_dtype=torch.bfloat16)
    assert torch.equal(half, O.to(torch.bfloat16))


@pytest.mark.parametrize("d,n", [(16, 20), (16, 200), (32, 40), (32, 256)])
def test_not_causal(d, n):
    Q, K, V, _ = _inputs(2, 2, n, d, 8300 + n)
    O = llla.llla_forward(Q.to(DEV), K.to(DEV), V.to(DEV), 1e-2, -0.2, causal=False).cpu().numpy()
    ref = oracle.forward(Q.contiguous(), K.contiguous(), V.contiguous(), 1e-2, -0.2, causal=False)
    check(O, ref, np.full(n, n - 1), d, 1e-4, "not causal n=%d d=%d" % (n, d))


@pytest.mark.parametrize("d,B,H,n,taken", [(16, 4, 8, 128, True), (16, 2, 8, 256, True), (32, 2, 4, 70, True), (32, 2, 4, 256, True),
                                           (16, 4, 8, 129, False), (16, 3, 11, 60, False), (32, 3, 3, 70, False), (16, 1, 2, 257, False)])
def test_both_sides_of_the_rule_agree(d, B, H, n, taken):
    """The call as it is dispatched, on both sides of the rule and at its extremes, against the oracle; what the rule refuses runs on the vector
    kernels and gives their bits, what it takes does not."""
    Q, K, V, lam = _inputs(B, H, n, d, 8600 + n)
    args = [t.to(DEV) for t in (Q, K, V, lam)]
    a = llla.llla_forward(*args, 0.25)
    ref = oracle.forward_ex(Q.contiguous(), K.contiguous(), V.contiguous(), lam, 0.25)[0]
    check(a.cpu().numpy(), ref, np.arange(n), d, 1e-4, "d=%d %d x %d x %d" % (d, B, H, n))
    assert torch.equal(a, llla.llla_forward(*args, 0.25, path="valu")) == (not taken)


@pytest.mark.parametrize("d,bound", [(16, 6.2), (32, 9.0)])
def test_errors_of_the_moments(d, bound):
    """rho of the rows 2 d .. 255, whose systems are well conditioned, so that its error is that of the moments.  Bound on the relative error of all
    these rows together, in 2^-24: each of four sums of 16 chunks rounds 64 times, one sum of 64 chunks 256 times, which doubles the
    error of the moments and, with the errors of weights and solve, which both have, makes 1.6 times here (d = 16 / 32: 4.6 / 7.1 with four
    sums, 7.1 / 11.4 with one, 7.5 to 8.5 / 11.5 to 12.4 on the vector kernels)."""
    n, H = 256, 8
    g = torch.Generator(device="cpu").manual_seed(8900 + d)
    Q, K, V = [torch.randn((1, H, n, d), generator=g) for _ in range(3)]
    lam = 1e-2 * torch.exp(0.5 * torch.randn((1, H, n), generator=g))
    rho = llla.llla_forward(Q.to(DEV), K.to(DEV), V.to(DEV), lam.to(DEV), d ** -0.5, return_stats=True)[1].cpu().double().numpy()[:, :, 2 * d:]
    ref = oracle.forward_ex(Q, K, V, lam, d ** -0.5)[1][:, :, 2 * d:]
    err = np.linalg.norm(rho - ref) / np.linalg.norm(ref) * 2 ** 24
    print("error %.2f x 2^-24" % err)
    assert err < bound
