"""fp32 backward on the matrix cores: the edges of its 32-row tiles and of the halves they are split into,
against the backward oracle, with the fp32 gate of the other backward tests (parity.check_grad, 1e-3)."""
import numpy as np
import pytest
import torch

import paper_2510_01450_amd as llla
import workloads
from oracle import backward as ob
from parity import check_grad
from test_gpu_backward import DEV, _backward, _case, _compare, _floor, _upstream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 97, 130, 257])
def test_edges_of_the_tiles(n):
    w = _case(1, 3, n, 64, "f32", index=540 + n)
    Q, K, V = workloads.make_inputs(w)
    G = _upstream(w, 40 + n)
    _compare(w, _backward(w, Q, K, V, G, w.lam), ob.backward(Q, K, V, G, w.lam, w.scale), "n=%d" % n, _floor(V, G, w.lam))


@pytest.mark.parametrize("d,n", [(32, n) for n in (63, 64, 65, 95, 96, 97, 130, 257)] + [(16, n) for n in (95, 96, 97, 127, 128, 130, 257)])
def test_small_heads(d, n):
    """d = 16 / 32: sweeps at the head's own dimension, moments on copies padded to 64 features; the sizes on both sides of the rule
    that takes them."""
    w = _case(1, 3, n, d, "f32", index=560 + n)
    Q, K, V = workloads.make_inputs(w)
    G = _upstream(w, 60 + n)
    _compare(w, _backward(w, Q, K, V, G, w.lam), ob.backward(Q, K, V, G, w.lam, w.scale), "d=%d n=%d" % (d, n), _floor(V, G, w.lam))


@pytest.mark.parametrize("d", [16, 32])
def test_small_heads_strides_do_not_matter(d):
    """Heads interleaved with the rows, and rows further apart than they are long: the same bits as contiguous tensors."""
    w = _case(2, 3, 131, d, "f32", index=570 + d)
    T = [t.to(DEV) for t in workloads.make_inputs(w)] + [_upstream(w, 70).to(DEV)]
    want = llla.llla_backward(*T, w.lam, w.scale, return_dlambda=True)
    rows = [t.transpose(1, 2).contiguous().transpose(1, 2) for t in T]
    wide = []
    for t in T:
        x = torch.full((2, 3, 131, d + 12), float("nan"), device=DEV)
        x[..., :d] = t
        wide.append(x[..., :d])
    for S in (rows, wide):
        assert all(torch.equal(a, b) for a, b in zip(llla.llla_backward(*S, w.lam, w.scale, return_dlambda=True), want))


@pytest.mark.parametrize("factor", [-1.0, 40.0])
def test_reference_exponent(factor):
    """Logits of growing size: the running reference exponent moves by more than its slack of 64 bits inside a row
    (factor 40: logits of several hundred), and a negative scale."""
    w = _case(1, 2, 150, 64, "f32", index=900)
    Q, K, V = workloads.make_inputs(w)
    if factor > 1:
        K = K * torch.linspace(0.5, 8.0, w.n)[None, None, :, None]
        Q = Q * factor
    w = w.with_shape(scale=w.scale * (-1.0 if factor < 0 else 1.0))
    G = _upstream(w, 41)
    _compare(w, _backward(w, Q, K, V, G, w.lam), ob.backward(Q, K, V, G, w.lam, w.scale), "factor %g" % factor, _floor(V, G, w.lam))


def test_few_keys_small_ridge_features_over_four_decades():
    """Rows with few keys far apart: the system is regular only through the ridge, and the intercept has to be eliminated
    before the features (eliminated last it cancels to zero).  Bounds: four times the errors of the vector kernels, which eliminate in
    that order too (2.4e-4, 2.0e-5, 2.0e-4, 3.0e-4; here 1.4e-4, 1.9e-5, 1.5e-4, 1.7e-4)."""
    n, d = 64, 64
    g = torch.Generator(device="cpu").manual_seed(64)
    Q, K, V, G = (torch.randn((1, 2, n, d), generator=g) for _ in range(4))
    size = 10.0 ** (torch.rand(d, generator=g) * 4 - 3)
    K, Q = K * size, Q / size.clamp(min=0.1)
    got = llla.llla_backward(Q.to(DEV), K.to(DEV), V.to(DEV), G.to(DEV), 1e-4, 1 / 8.0, return_dlambda=True)
    ref = ob.backward(Q, K, V, G, 1e-4, 1 / 8.0)
    for a, b, bound in zip(got, ref, (1e-3, 8e-5, 8e-4, 1.2e-3)):
        a = a.cpu().double().numpy()
        assert np.isfinite(a).all()
        assert np.linalg.norm(a - b) <= bound * np.linalg.norm(b)


@pytest.mark.parametrize("d,n", [(64, 70), (32, 70), (16, 100)])
def test_workspace_of_the_vector_kernels_is_enough(d, n):
    """A caller that brings only what the vector kernels need gets their result."""
    w = _case(1, 2, n, d, "f32", index=901)
    Q, K, V = (t.to(DEV) for t in workloads.make_inputs(w))
    G = _upstream(w, 42).to(DEV)
    small = (w.B * w.H * w.n * (2 * w.d + 8) * 4 + 255) // 256 * 256
    assert small < llla.backward_workspace_bytes(w.B, w.H, w.n, w.d, torch.float32)
    ws = torch.empty(small, dtype=torch.uint8, device=DEV)
    got = llla.llla_backward(Q, K, V, G, w.lam, w.scale, return_dlambda=True, workspace=ws)
    want = llla.llla_backward(Q, K, V, G, w.lam, w.scale, return_dlambda=True, path="valu")
    assert all(torch.equal(a, b) for a, b in zip(got, want))


@pytest.mark.parametrize("n,offset", [(500, 30.0), (130, 100.0), (64, 100.0)])
def test_common_offset_stays_finite(n, offset):
    """Keys and queries far from the origin: the rounding of moments of the size of |k|^2 exceeds the ridge, pivots of the centred
    matrix come out negative, and what they would be divided into must not overflow.  (Nothing but finiteness can be asked for:
    |k|^2 / ridge * 2^-24 is 0.4 and 4.)"""
    g = torch.Generator(device="cpu").manual_seed(n)
    Q, K, V, G = (torch.randn((1, 4, n, 64), generator=g).to(DEV) for _ in range(4))
    Q, K = Q + offset, K + offset
    for x in (llla.llla_forward(Q, K, V, 1e-2, 1 / 8.0),) + llla.llla_backward(Q, K, V, G, 1e-2, 1 / 8.0, return_dlambda=True):
        assert bool(torch.isfinite(x).all())


@pytest.mark.parametrize("what", ["keys", "values"])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("d,n", [(16, 100), (16, 143), (32, 64), (32, 111), (64, 40), (64, 111), (128, 40), (128, 143)])
def test_a_row_does_not_see_what_is_behind_it(d, n, bad, what):
    """Keys or values that are not finite from a row on leave dQ and dlambda of the rows before it as the sequence without them gives
    them.  (dK and dV of the keys before it are sums over all later rows.)  Rows on both sides of the tiles of 16 and the blocks of 32."""
    w = _case(1, 4, n, d, "f32", index=580 + d + n)
    Q, K, V = workloads.make_inputs(w)
    G = _upstream(w, 90 + n)
    floor = _floor(V, G, w.lam)
    full = ob.backward(Q, K, V, G, w.lam, w.scale)
    for first in (5, 17, n - 33, n - 16, n - 7, n - 1):
        T = {"keys": K.clone(), "values": V.clone()}
        T[what][:, :, first:] = bad
        got = _backward(w, Q, T["keys"], T["values"], G, w.lam)
        for name, t in (("dQ", 0), ("dlambda", 3)):
            ref = np.asarray(full[t])[:, :, :first]
            print(name, check_grad(got[t][:, :, :first], ref, d, w.tol, "%s from %d: %s" % (what, first, name), floor=floor[name]))
            assert not np.isfinite(got[t][:, :, first:]).any()


@pytest.mark.parametrize("d,n", [(16, 120), (32, 90)])
def test_small_heads_with_a_common_offset(d, n):
    """Keys with a common offset of 3 in all features: the centred matrix of a row is a difference of sums some 9 d times its size, and what mu~
    and Sigma~ round differently stays in it.  The geometric mean of the heads' errors against the vector kernels', which sum both from the
    same products: seen 0.75 and 0.68 times; with mu~ from rounded weights above 0.8 (0.91 and 0.89 on other inputs)."""
    w = _case(1, 48, n, d, "f32", values="normal", index=595 + d)
    Q, K, V = workloads.make_inputs(w)
    K = K + 3
    G = _upstream(w, 95 + d)
    ref = np.asarray(ob.backward(Q, K, V, G, w.lam, w.scale)[0])
    err = [np.linalg.norm((_backward(w, Q, K, V, G, w.lam, path)[0] - ref).reshape(48, -1), axis=1) for path in ("auto", "valu")]
    ratio = float(np.exp(np.mean(np.log(err[0] / err[1]))))
    print("ratio %.3f" % ratio)
    assert ratio < 0.8


@pytest.mark.parametrize("d,n,bound", [(16, 120, 0.95), (32, 90, 1.1)])
def test_small_heads_few_keys_and_a_small_ridge(d, n, bound):
    """|k|^2 / ridge = 1.6e5 and 3.2e5: what the solve for u1 loses in rows with fewer keys than features is most of the error of dQ.  Geometric
    mean of the heads' errors against the vector kernels': seen 0.91 and 1.03, with L^-1 formed first 1.23 and 1.13."""
    w = _case(1, 48, n, d, "f32", values="normal", index=596 + d, lam=1e-4)
    Q, K, V = workloads.make_inputs(w)
    G = _upstream(w, 97 + d)
    ref = np.asarray(ob.backward(Q, K, V, G, w.lam, w.scale)[0])
    err = [np.linalg.norm((_backward(w, Q, K, V, G, w.lam, path)[0] - ref).reshape(48, -1), axis=1) for path in ("auto", "valu")]
    ratio = float(np.exp(np.mean(np.log(err[0] / err[1]))))
    print("ratio %.3f" % ratio)
    assert ratio < bound, ratio
