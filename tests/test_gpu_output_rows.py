"""Output sweep of the bf16 forward: lengths around its blocks of 32 keys, its workgroups of 64 rows and the first 2 d rows (three-term
operands), causal and not, strided operands, both output types, every head dimension.  Gate and oracle as in the other parity tests."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2510_01450_amd as llla
from parity import check

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _inputs(B, H, n, d, seed):
    g = torch.Generator(device="cpu").manual_seed(seed)
    return [torch.randn((B, n, H, d), generator=g).bfloat16().transpose(1, 2) for _ in range(3)]      # [B, n, H, d] in memory


@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("n", [1, 31, 32, 33, 64, 65, 127, 128, 129, 160, 161, 193, 256, 257, 289, 321])
def test_lengths(n, d):
    Q, K, V = _inputs(1, 2, n, d, 9000 + n + d)
    scale = 1 / math.sqrt(d)
    O = llla.llla_forward(Q.to(DEV), K.to(DEV), V.to(DEV), 1e-2, scale, path="mfma")
    ref = oracle.forward(Q.contiguous(), K.contiguous(), V.contiguous(), 1e-2, scale)
    check(O.cpu().numpy(), ref, np.arange(n), d, 2e-2, "n=%d d=%d" % (n, d))
    half = llla.llla_forward(Q.to(DEV), K.to(DEV), V.to(DEV), 1e-2, scale, out_dtype=torch.bfloat16, path="mfma")
    assert torch.equal(half, O.to(torch.bfloat16))


@pytest.mark.parametrize("d,n", [(16, 130), (32, 100), (64, 33), (64, 129), (64, 161), (128, 256), (128, 300)])
def test_not_causal(d, n):
    Q, K, V = _inputs(2, 2, n, d, 9300 + n)
    O = llla.llla_forward(Q.to(DEV), K.to(DEV), V.to(DEV), 1e-2, -0.1, causal=False, path="mfma").cpu().numpy()
    ref = oracle.forward(Q.contiguous(), K.contiguous(), V.contiguous(), 1e-2, -0.1, causal=False)
    check(O, ref, np.full(n, n - 1), d, 2e-2, "not causal n=%d d=%d" % (n, d))


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_a_value_behind_a_first_row_does_not_reach_it(d, bad):
    """The first 2 d rows are strictly causal in the values too: an entry of value j that is not finite leaves the rows before j as they
    were (to the rounding of another order of the sums, 1e-5 of a row), every other column of the rows from j on too, and reaches its own
    column of those."""
    n = 2 * d + 37
    Q, K, V = [t.to(DEV) for t in _inputs(1, 2, n, d, 9500 + d)]
    scale = 1 / math.sqrt(d)
    clean = llla.llla_forward(Q, K, V, 1e-2, scale, path="mfma")[0, 1].double()
    for j in sorted({1, 5, 17, 31, d, 2 * d - 20, 2 * d - 1}):
        Vb = V.clone()
        Vb[0, 1, j, d - 3] = bad
        got = llla.llla_forward(Q, K, Vb, 1e-2, scale, path="mfma")[0, 1].double()
        other = [c for c in range(d) if c != d - 3]
        for x, r in ((got[:j], clean[:j]), (got[j:2 * d, other], clean[j:2 * d, other])):
            assert torch.isfinite(x).all() and float(((x - r).norm(dim=-1) / r.norm(dim=-1)).max()) < 1e-5, (j, bad)
        assert not torch.isfinite(got[j:2 * d, d - 3]).any(), (j, bad)


@pytest.mark.parametrize("values", ["normal", "regression"])
@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_first_rows_are_summed_in_fp32_accuracy(d, values):
    """The output sweep alone: O of the first 2 d rows against the sum over keys in 64 bits from the call's own rho and delta.  A coefficient
    w (y0 + k . y1) cancels to a few digits in these rows, so errors are measured against the sum T_i of the sizes of its terms.  Bounds
    4 x 2^-24 T_i for every row and 0.5 x 2^-24 T_i for the median one: a term has the errors of the logit and the exponential, an ulp or
    two of its own, and of rho and delta, rounded to fp32 here, at random signs (seen: largest 1.1 to 2.2, median 0.12 to 0.24); two-term
    operands, 2^-17 of a term at worst, were seen at 5 to 20 and 0.9 to 6.2."""
    n, scale = 2 * d, 1 / math.sqrt(d)
    Q, K, V = _inputs(1, 2, n, d, 9700 + d)
    if values == "regression":
        V = (K.float() @ (torch.randn((d, d), generator=torch.Generator().manual_seed(d)) / math.sqrt(d)) + 0.1 * V.float()).bfloat16()
    O, rho, delta = [t.cpu().double() for t in llla.llla_forward(Q.to(DEV), K.to(DEV), V.to(DEV), 1e-2, scale, path="mfma", return_stats=True)]
    q, k, v = Q.double(), K.double(), V.double()
    y1, y0 = -rho / delta[..., None], (1 + (q * rho).sum(-1)) / delta
    lg = (scale * q @ k.transpose(-1, -2)).masked_fill(torch.ones(n, n).triu(1).bool(), -math.inf)
    w = torch.exp(lg - lg.max(-1, keepdim=True).values)
    ref = (w * (y0[..., None] + y1 @ k.transpose(-1, -2))) @ v
    terms = (w * (y0[..., None].abs() + y1.abs() @ k.abs().transpose(-1, -2))) @ v.abs()
    err = (O - ref).norm(dim=-1) / terms.norm(dim=-1) * 2 ** 24
    print("largest error %.3f, median %.3f x 2^-24 of the terms" % (float(err.max()), float(err.median())))
    assert float(err.max()) < 4.0 and float(err.median()) < 0.5
