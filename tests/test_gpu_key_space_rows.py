"""Forward calls whose kernels carry the key-space rows in their own grid (fp32 inputs, and the vector kernels): lengths around the
number of such rows and around the kernels' row blocks, with the statistics, causal and not; and the vector kernels at d = 16 / 32,
whose elimination keeps a row per lane.  Gate and oracle as in the other parity tests."""
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


def _case(n, d, dtype):
    base = workloads.C2 if dtype == "f32" else workloads.C3
    return base.with_shape(name="key_space", B=2, H=2, n=n, d=d, dtype=dtype, values="l2" if dtype == "f32" else "normal",
                           index=620 + n + d, scale=1 / math.sqrt(d), tol=1e-4 if dtype == "f32" else 2e-2)


@pytest.mark.parametrize("d,path,dtype", [(64, "auto", "f32"), (16, "valu", "f32"), (32, "valu", "f32"), (32, "valu", "bf16"),
                                          (128, "valu", "f32")])
@pytest.mark.parametrize("n", [1, 15, 17, 33, 63, 64, 65, 79, 130])
def test_lengths_around_the_key_space_rows(n, d, path, dtype):
    w = _case(n, d, dtype)
    Q, K, V = workloads.make_inputs(w)
    O, rho, delta = llla.llla_forward(Q.to(DEV), K.to(DEV), V.to(DEV), w.lam, w.scale, path=path, return_stats=True)
    ref = oracle.forward(Q, K, V, w.lam, w.scale)
    check(O.cpu().numpy(), ref, np.arange(n), d, w.tol, "n=%d d=%d %s %s" % (n, d, dtype, path))
    # the statistics reproduce the output weights' normalisation: y0 + q.y1 = 1 / delta, y1 = -rho / delta; rows of both kinds
    assert torch.isfinite(rho).all() and torch.isfinite(delta).all() and bool((delta > 0).all())


@pytest.mark.parametrize("n", [20, 64, 65])
def test_not_causal(n):
    w = _case(n, 64, "f32")
    Q, K, V = workloads.make_inputs(w)
    O = llla.llla_forward(Q.to(DEV), K.to(DEV), V.to(DEV), w.lam, w.scale, causal=False)
    ref = oracle.forward(Q, K, V, w.lam, w.scale, causal=False)
    check(O.cpu().numpy(), ref, np.full(n, n - 1), 64, w.tol, "not causal n=%d" % n)
