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


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 30, 61, 64, 70])
def test_rows_at_d64_are_exact_to_the_rounding_of_the_result(n):
    """Four rows per workgroup, one per wave, in fp64: what is left is the rounding of the stored fp32 values (2^-24 per element, and
    the fp64 arithmetic's 2^-53 times a condition number of at most |k|^2 n / lambda = 5e5).  Keys of norm 8, a ridge per row,
    strided inputs."""
    d, B, H = 64, 2, 2
    g = torch.Generator(device="cpu").manual_seed(7000 + n)
    Q, K, V = [torch.randn((B, n, H, d), generator=g).transpose(1, 2) for _ in range(3)]
    lam = 1e-2 * torch.exp(0.5 * torch.randn((B, H, n), generator=g))
    O, rho, delta = llla.llla_forward(Q.to(DEV), K.to(DEV), V.to(DEV), lam.to(DEV), 1 / math.sqrt(d), return_stats=True)
    ref = oracle.forward_ex(Q.contiguous(), K.contiguous(), V.contiguous(), lam, 1 / math.sqrt(d))
    m = min(n, 64)
    for x, r in zip((O, rho, delta[..., None]), (ref[0], ref[1], np.asarray(ref[2])[..., None])):
        x, r = x.cpu().double().numpy()[:, :, :m], np.asarray(r, dtype=np.float64)[:, :, :m]
        err = np.linalg.norm(x - r, axis=-1) / np.maximum(np.linalg.norm(r, axis=-1), 1e-300)
        err[np.linalg.norm(r, axis=-1) == 0] = np.abs(x[np.linalg.norm(r, axis=-1) == 0]).max(initial=0.0)
        assert err.max() < 1e-7, (n, err.max())


@pytest.mark.parametrize("n", [17, 49, 64, 70])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_a_key_behind_a_row_does_not_reach_it(n, bad):
    """Row i sees keys 0..i.  Four rows share a workgroup and their keys: an entry of key j that is not finite must leave every key-space row
    before j, those of its own workgroup among them, as it was, bit for bit."""
    d, B, H = 64, 2, 3
    g = torch.Generator(device="cpu").manual_seed(7300 + n)
    Q, K, V = [torch.randn((B, H, n, d), generator=g).to(DEV) for _ in range(3)]
    clean = llla.llla_forward(Q, K, V, 1e-2, 1 / math.sqrt(d), return_stats=True)
    for j in sorted({1, 2, 3, 13, n // 2, n - 3, n - 2, n - 1}):
        Kb = K.clone()
        Kb[:, :, j, j % d] = bad
        rows = min(j, 64)
        for x, r in zip(llla.llla_forward(Q, Kb, V, 1e-2, 1 / math.sqrt(d), return_stats=True), clean):
            assert torch.isfinite(r).all() and torch.equal(x[:, :, :rows], r[:, :, :rows]), (n, j)


@pytest.mark.parametrize("n", [1, 5, 16, 33, 48, 64, 70])
def test_a_sequence_does_not_depend_on_the_ones_served_before_it(n):
    """A workgroup's LDS holds what the previous one left there.  A call whose keys are all NaN leaves NaN in the inner products of every
    compute unit; the sequences of the next call, and those that share a call with such sequences, must not see it."""
    d, B, H = 64, 32, 16
    g = torch.Generator(device=DEV).manual_seed(7400 + n)
    Q, K, V = [torch.randn((B, H, n, d), generator=g, device=DEV) for _ in range(3)]
    scale = 1 / math.sqrt(d)
    bad = torch.full((B, H, 64, d), float("nan"), device=DEV)
    ref = oracle.forward(Q[:1, :2].cpu(), K[:1, :2].cpu(), V[:1, :2].cpu(), 1e-2, scale)
    before = llla.llla_forward(Q, K, V, 1e-2, scale, return_stats=True)
    llla.llla_forward(bad, bad, bad, 1e-2, scale)
    after = llla.llla_forward(Q, K, V, 1e-2, scale, return_stats=True)
    Kb = K.clone()
    Kb[1::2] = float("nan")
    mixed = llla.llla_forward(Q, Kb, V, 1e-2, scale, return_stats=True)
    check(before[0][:1, :2].cpu().numpy(), ref, np.arange(n), d, 1e-4, "n=%d" % n)
    for x, y, z in zip(before, after, mixed):
        assert torch.isfinite(x).all() and torch.equal(x, y) and torch.equal(x[0::2], z[0::2]), n
