"""Decode on the fp32 matrix-core kernels (path='auto' for fp32 caches, and for bf16 caches that the 16-bit kernels do not
serve): step and tile remainders, splits of a cache over several workgroups, per-sequence lengths, strided and poisoned caches,
a call without scratch, both output types.  All outputs against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_01450_amd as llla
import workloads
from parity import check

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _case(B, H, L, d, dtype, index, values="normal"):
    tol = 1e-4                       # fp32 arithmetic for either input type (bf16 widens exactly)
    w = workloads.C5.with_shape(name="decf32", B=B, H=H, n=L, d=d, dtype=dtype, index=index, values=values, tol=tol,
                                scale=d ** -0.5)
    return w, workloads.make_inputs(w)


# bf16 at d = 64 / 128 comes here below 256 cached rows only
@pytest.mark.parametrize("d,dtype,L,BH", [
    (16, "f32", 65, (2, 3)), (16, "bf16", 4097, (1, 2)), (32, "f32", 33, (3, 1)), (32, "bf16", 3000, (2, 2)),
    (32, "bf16", 256, (40, 16)), (64, "f32", 257, (2, 2)), (64, "f32", 5003, (1, 3)), (64, "f32", 1030, (70, 8)),
    (64, "bf16", 255, (2, 3)), (128, "f32", 129, (2, 2)), (128, "f32", 4100, (1, 2)), (128, "f32", 700, (37, 8)),
    (128, "bf16", 130, (3, 2))])
def test_full_length(d, dtype, L, BH):
    B, H = BH
    w, (q, Kc, Vc) = _case(B, H, L, d, dtype, 2100 + d + L)
    nb = min(B, 3)
    ref = oracle.decode(q[:nb], Kc[:nb], Vc[:nb], w.lam, w.scale)
    qd, Kd, Vd = q.to(DEV), Kc.to(DEV), Vc.to(DEV)
    got = llla.llla_decode(qd, Kd, Vd, w.lam, w.scale)
    print(check(got[:nb].cpu().numpy()[:, :, None], ref[:, :, None], np.array([L - 1]), d, w.tol, "L=%d d=%d" % (L, d)))
    again = llla.llla_decode(qd, Kd, Vd, w.lam, w.scale)
    assert torch.equal(got, again)
    half = llla.llla_decode(qd, Kd, Vd, w.lam, w.scale, out_dtype=torch.bfloat16)
    assert torch.equal(half, got.to(torch.bfloat16))


@pytest.mark.parametrize("d,dtype", [(16, "f32"), (16, "bf16"), (32, "f32"), (32, "bf16"), (64, "f32"), (128, "f32")])
def test_lengths_of_their_own_strided_and_poisoned(d, dtype):
    """Lengths on both sides of the key-space limit, of a step (8 to 32 keys) and of a workgroup's share, in a cache whose rows
    are 2 d apart and whose tail is NaN."""
    k = min(d, 64)
    lens = [1, k, k + 1, k + 7, 2 * d + 9, 4 * d, 4 * d + 1, 1111, 2047, 2048]
    w, (q, Kc, Vc) = _case(len(lens), 2, 2048, d, dtype, 2200 + d)
    ref = oracle.decode(q, Kc, Vc, w.lam, w.scale, seqlens=lens)
    wide = torch.full((len(lens), 2, 2048, 2 * d), float("nan"), dtype=Kc.dtype)
    Kw, Vw = wide.clone(), wide.clone()
    Kw[..., :d] = Kc
    Vw[..., d:] = Vc
    for b, L in enumerate(lens):
        Kw[b, :, L:] = float("nan")
        Vw[b, :, L:] = float("nan")
    sl = torch.tensor(lens, dtype=torch.int32, device=DEV)
    got = llla.llla_decode(q.to(DEV), Kw.to(DEV)[..., :d], Vw.to(DEV)[..., d:], w.lam, w.scale, seqlens=sl).cpu().numpy()
    for b, L in enumerate(lens):
        print(L, check(got[b:b + 1, :, None], ref[b:b + 1, :, None], np.array([L - 1]), d, w.tol, "seqlen %d d=%d" % (L, d)))


@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_without_scratch_and_static(d):
    """The scratch is optional here (one workgroup per head without it), and llla_decode_static runs the same kernels."""
    L = 3001
    w, (q, Kc, Vc) = _case(1, 3, L, d, "f32", 2300 + d, values="l2")
    ref = oracle.decode(q, Kc, Vc, w.lam, w.scale)
    qd, Kd, Vd = q.to(DEV), Kc.to(DEV), Vc.to(DEV)
    assert llla.decode_workspace_bytes(1, 3, L, d, torch.float32) > 0
    bare = llla.llla_decode(qd, Kd, Vd, w.lam, w.scale, workspace=torch.empty(16, dtype=torch.uint8, device=DEV))
    full = llla.llla_decode(qd, Kd, Vd, w.lam, w.scale)
    static = llla.llla_decode_static(qd, Kd, Vd, w.lam, w.scale, torch.empty((1, 3, d), device=DEV))
    assert torch.equal(full, static)
    for got in (bare, full):
        print(check(got.cpu().numpy()[:, :, None], ref[:, :, None], np.array([L - 1]), d, w.tol, "scratch d=%d" % d))


@pytest.mark.parametrize("scale", [40.0, -30.0, 0.0])
@pytest.mark.parametrize("d", [32, 64, 128])
def test_reference_exponent_moves(d, scale):
    """Logits that span far more than 2^8 move the reference exponent during the sweep; with scale 0 all weights are equal."""
    L = 900
    w, (q, Kc, Vc) = _case(2, 2, L, d, "f32", 2400 + d, values="l2")
    ref = oracle.decode(q, Kc, Vc, w.lam, scale)
    got = llla.llla_decode(q.to(DEV), Kc.to(DEV), Vc.to(DEV), w.lam, scale).cpu().numpy()
    print(check(got[:, :, None], ref[:, :, None], np.array([L - 1]), d, w.tol, "scale %g d=%d" % (scale, d)))


@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_records_of_a_head(d):
    """Caches cut into one to a few dozen parts, i.e. every size of the last group of records that the merge takes, and as many
    maxima.  Unit keys and a small scale: the matrix is well conditioned and the output known to some tens of roundings,
    which a record with a slightly wrong factor (the gate of the other tests is 1e-4) does not keep."""
    for L in (130, 300, 520, 780, 1030, 1300, 1600, 2100, 2400, 4200, 4700, 8300, 9100):
        w, (q, Kc, Vc) = _case(1, 2, L, d, "f32", 2500 + d + L, values="l2")
        Kc = Kc * torch.linspace(0.5, 1.5, L)[None, None, :, None]                 # the maximum differs from part to part
        ref = oracle.decode(q, Kc, Vc, w.lam, w.scale)
        got = llla.llla_decode(q.to(DEV), Kc.to(DEV), Vc.to(DEV), w.lam, w.scale).cpu().double().numpy()
        err = np.linalg.norm(got - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
        # (hardly more keys than features leave directions that the ridge alone holds: condition number 4 / 10^-2 instead of some tens)
        assert err.max() <= (64 if L >= 4 * d else 640) * 2.0 ** -24, "L=%d: %.2e" % (L, err.max())


@pytest.mark.parametrize("L,BH", [(65, (2, 2)), (95, (2, 2)), (96, (2, 2)), (97, (2, 2)), (127, (1, 3)), (129, (1, 3)), (160, (3, 2)), (257, (2, 2)),
                                  (511, (1, 2)), (1025, (1, 1)), (959, (33, 8)), (960, (33, 8)), (300, (32, 8)), (300, (33, 8))])
def test_three_term_products_at_d64(L, BH):
    """fp32 caches at d = 64: steps of 32 keys and their remainders, one workgroup per head and several, and both sides of the rule that
    chooses between the three-term products and fp32 MFMA (256 heads; 960 keys).  Unit keys.  Bound: 24-bit operands and fp32 sums leave
    some 2^-24 sqrt(L) of the moments, times the condition number of the system (about 4 from 4 d keys on: a tenth of the usual gate;
    below, the usual gate)."""
    B, H = BH
    w, (q, Kc, Vc) = _case(B, H, L, 64, "f32", 2300 + L, values="l2")
    nb = min(B, 3)
    got = llla.llla_decode(q.to(DEV), Kc.to(DEV), Vc.to(DEV), w.lam, w.scale)[:nb].cpu().numpy()
    ref = oracle.decode(q[:nb], Kc[:nb], Vc[:nb], w.lam, w.scale)
    check(got[:, :, None], ref[:, :, None], np.array([L - 1]), 64, 1e-5 if L >= 256 else 1e-4, "L=%d heads %d" % (L, B * H))


@pytest.mark.parametrize("B,H,L,values", [(16, 16, 4096, "unit"), (16, 16, 4096, "normal"), (2, 16, 32768, "unit"), (2, 16, 32768, "normal")])
def test_errors_do_not_grow_with_the_keys_of_a_wave(B, H, L, values):
    """fp32 caches at d = 64 whose waves walk 1024 keys each.  Bound on the root mean square over heads of the relative error: 8 x 2^-24.
    A step of 32 keys rounds a sum once, independently of the others, so that some 32 roundings of half an ulp stay within a few ulp
    (seen: 4.9 to 5.9 x 2^-24; on fp32 MFMA 7.0 and 8.1 at 32768 keys; with six products chained onto the sum 11.0 to 13.9)."""
    d = 64
    g = torch.Generator(device=DEV).manual_seed(2700 + L)
    q, K, V = [torch.randn(s, generator=g, device=DEV) for s in ((B, H, d), (B, H, L, d), (B, H, L, d))]
    if values == "unit":
        q, K = q / q.norm(dim=-1, keepdim=True), K / K.norm(dim=-1, keepdim=True)
    got = llla.llla_decode(q, K, V, 1e-2, d ** -0.5)[:1].cpu().double().numpy()
    ref = oracle.decode(q[:1].cpu(), K[:1].cpu(), V[:1].cpu(), 1e-2, d ** -0.5)
    err = np.linalg.norm(got - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
    rms = float(np.sqrt(np.mean(err ** 2))) * 2 ** 24
    print("rms error %.2f x 2^-24" % rms)
    assert rms < 8.0


@pytest.mark.parametrize("L", [70, 300, 3000])
def test_values_of_any_size_at_d64(L):
    """fp32 arithmetic has no value range: the output is linear in V, so values times a power of two give the same bits times it, as long as
    neither is subnormal; values that are small at first and ordinary later (factors about 2^-18) among them."""
    g = torch.Generator(device="cpu").manual_seed(2900 + L)
    q, K, V = [torch.randn(s, generator=g).to(DEV) for s in ((2, 4, 64), (2, 4, L, 64), (2, 4, L, 64))]
    base = llla.llla_decode(q, K, V, 1e-2, 0.125)
    assert torch.isfinite(base).all()
    for k in (-110, -104, -80, -20, -19, -18, -17, -16, -15, 60, 118):
        got = llla.llla_decode(q, K, V * 2.0 ** k, 1e-2, 0.125)
        assert torch.equal(got.double(), base.double() * 2.0 ** k), k
