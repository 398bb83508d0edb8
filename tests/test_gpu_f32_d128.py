"""fp32 inputs at d = 128 on the matrix cores: the edges of the forward's blocks of 8 queries and 64 keys, of its key-space rows and of the
32-row tiles of the sweeps, with statistics; the reference exponent when it moves; values that a row does not see; and the calls that
stay with the vector kernels.  Gates and oracles as in the other parity tests."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2510_01450_amd as llla
import workloads
from oracle import backward as ob
from parity import check
from test_gpu_backward import _backward, _compare, _floor, _upstream
from test_gpu_backward import _case as _backward_case

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
D = 128


def _case(n, B=1, H=2, values="l2", **kw):
    return workloads.C2.with_shape(name="f32_d128", B=B, H=H, n=n, d=D, dtype="f32", values=values, index=660 + n, scale=1 / math.sqrt(D),
                                   tol=1e-4, **kw)


@pytest.mark.parametrize("n", [65, 71, 72, 73, 95, 96, 97, 127, 128, 129, 200])
def test_edges_of_the_blocks(n):
    w = _case(n)
    Q, K, V = workloads.make_inputs(w)
    lam = 1e-2 * torch.exp(0.5 * torch.randn((1, 2, n), generator=torch.Generator().manual_seed(n)))
    O, rho, delta = llla.llla_forward(Q.to(DEV), K.to(DEV), V.to(DEV), lam.to(DEV), w.scale, return_stats=True)
    ref = oracle.forward_ex(Q, K, V, lam, w.scale)
    check(O.cpu().numpy(), ref[0], np.arange(n), D, w.tol, "n=%d" % n)
    for x, r in ((rho, ref[1]), (delta[..., None], np.asarray(ref[2])[..., None])):      # as the same statistics at d = 64
        x, r = x.cpu().double().numpy(), np.asarray(r, dtype=np.float64)
        assert np.linalg.norm(x - r) <= 1e-3 * np.linalg.norm(r)


@pytest.mark.parametrize("heads,n", [(16, 64), (40, 26), (130, 8), (15, 64)])
def test_calls_of_key_space_rows_alone(heads, n):
    """Eight rows per workgroup from 1024 rows on, one below: exact to the rounding of the result either way (keys of length 1; fp64)."""
    w = _case(n, H=heads)
    Q, K, V = workloads.make_inputs(w)
    O = llla.llla_forward(Q.to(DEV), K.to(DEV), V.to(DEV), w.lam, w.scale).cpu().double().numpy()
    ref = np.asarray(oracle.forward(Q, K, V, w.lam, w.scale), dtype=np.float64)
    assert np.linalg.norm(O - ref) <= 2.0 ** -24 * np.linalg.norm(ref)


@pytest.mark.parametrize("n", [20, 64, 65, 130])
def test_not_causal(n):
    w = _case(n, H=60)
    Q, K, V = workloads.make_inputs(w)
    O = llla.llla_forward(Q.to(DEV), K.to(DEV), V.to(DEV), w.lam, w.scale, causal=False)[:, :2]
    ref = oracle.forward(Q[:, :2], K[:, :2], V[:, :2], w.lam, w.scale, causal=False)
    check(O.cpu().numpy(), ref, np.full(n, n - 1), D, w.tol, "not causal n=%d" % n)


def test_strides_and_bf16_output():
    """Heads interleaved with the rows, rows further apart than they are long: the bits of the contiguous call."""
    w = _case(150, B=2)
    T = [t.to(DEV) for t in workloads.make_inputs(w)]
    want = llla.llla_forward(*T, w.lam, w.scale)
    rows = [t.transpose(1, 2).contiguous().transpose(1, 2) for t in T]
    out = torch.empty((2, 150, 2, D + 8), device=DEV).transpose(1, 2)[..., :D]
    assert torch.equal(llla.llla_forward(*rows, w.lam, w.scale, out=out), want)
    wide = [torch.nn.functional.pad(t, (0, 4), value=float("nan"))[..., :D] for t in T]
    assert torch.equal(llla.llla_forward(*wide, w.lam, w.scale), want)
    assert torch.equal(llla.llla_forward(*T, w.lam, w.scale, out_dtype=torch.bfloat16), want.to(torch.bfloat16))


@pytest.mark.parametrize("factor", [-1.0, 40.0])
def test_reference_exponent(factor):
    """Logits that grow along the row by more than the 64 bits after which the reference exponent moves, and a negative scale.  Logits of
    300 carry a rounding of 2e-5 into the weights, which the cancellation of rows with few keys amplifies beyond the gate in any fp32
    evaluation, so the vector kernels are the measure (errors 0.8 times theirs; their sums round in another order: at most 1.25)."""
    w = _case(300)
    Q, K, V = workloads.make_inputs(w)
    if factor > 1:
        K = K * torch.linspace(0.5, 8.0, w.n)[None, None, :, None]
        Q = Q * factor
    scale = -w.scale if factor < 0 else 1.0
    ref = np.asarray(oracle.forward(Q, K, V, w.lam, scale), dtype=np.float64)
    auto, valu = (np.linalg.norm(llla.llla_forward(Q.to(DEV), K.to(DEV), V.to(DEV), w.lam, scale, path=p).cpu().double().numpy() - ref)
                  for p in ("auto", "valu"))
    assert auto <= 1.25 * valu and auto <= 1e-3 * np.linalg.norm(ref)


@pytest.mark.parametrize("first", [70, 79, 100, 128])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_values_that_a_row_does_not_see(first, bad):
    """Keys and values that are not finite from a row on leave the rows before it as they were."""
    w = _case(140)
    Q, K, V = (t.to(DEV) for t in workloads.make_inputs(w))
    want = llla.llla_forward(Q, K, V, w.lam, w.scale)
    for t in (K, V):
        t[:, :, first:] = bad
    got = llla.llla_forward(Q, K, V, w.lam, w.scale)
    a, b = got[:, :, :first], want[:, :, :first]
    # the sums of the diagonal tiles in another order: sixteen fp32 roundings of terms of the size of the result
    assert bool(torch.isfinite(a).all()) and float((a - b).norm()) <= 16 * 2.0 ** -23 * float(b.norm())
    assert not bool(torch.isfinite(got[:, :, first:]).any())


def test_without_workspace_the_vector_kernels_serve():
    w = _case(150)
    T = [t.to(DEV) for t in workloads.make_inputs(w)]
    want = llla.llla_forward(*T, w.lam, w.scale, path="valu")
    small = torch.empty(256, dtype=torch.uint8, device=DEV)
    assert llla.forward_workspace_bytes(1, 2, 150, D, torch.float32) > 256
    assert torch.equal(llla.llla_forward(*T, w.lam, w.scale, workspace=small), want)
    assert not torch.equal(llla.llla_forward(*T, w.lam, w.scale), want)
    with pytest.raises(llla.LlaError):
        llla.llla_forward(*T, w.lam, w.scale, path="mfma")


@pytest.mark.parametrize("n", [1, 7, 8, 9, 31, 32, 33, 64, 65, 130])
def test_backward_edges(n):
    w = _backward_case(1, 2, n, D, "f32", index=690 + n)
    Q, K, V = workloads.make_inputs(w)
    G = _upstream(w, 80 + n)
    _compare(w, _backward(w, Q, K, V, G, w.lam), ob.backward(Q, K, V, G, w.lam, w.scale), "n=%d" % n, _floor(V, G, w.lam))


def test_moments_and_sweeps_see_the_same_logits():
    """Logits of some eight standard deviations of 1: a weight of the moments kernel and of a sweep that differ by the rounding of two orders of
    summation leave e_ij = w_ij (gamma_ij - b_ij) of that size behind, which y1 multiplies by |q| / ridge.  Geometric mean of the heads' errors of
    dK against the vector kernels', whose sweeps share one order: seen WITH, in two orders WITHOUT."""
    w = _backward_case(1, 16, 70, D, "f32", values="normal", index=699)
    Q, K, V = workloads.make_inputs(w)
    Q = 8 * Q
    G = _upstream(w, 99)
    ref = np.asarray(ob.backward(Q, K, V, G, w.lam, w.scale)[1])
    err = [np.linalg.norm((_backward(w, Q, K, V, G, w.lam, path)[1] - ref).reshape(16, -1), axis=1) for path in ("auto", "valu")]
    ratio = float(np.exp(np.mean(np.log(err[0] / err[1]))))
    print("ratio %.3f" % ratio)
    assert ratio < 1.25, ratio
