"""Decode of bf16 caches at d = 16 / 32, whose weighted keys are split into three bf16 for the 16-bit matrix cores: remainders of the
32-key step and of a wave's share, sequences in key space beside long ones in one call, and keys beyond the range of a 16-bit
float.  Gate 1e-4 as for the other decode calls in fp32 arithmetic."""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_01450_amd as llla
from parity import check
from test_gpu_decode_f32 import DEV, _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [16, 32])
@pytest.mark.parametrize("L", [65, 95, 96, 97, 127, 129, 161, 1025])
def test_remainders(L, d):
    w, (q, Kc, Vc) = _case(2, 3, L, d, "bf16", 2400 + d + L)
    ref = oracle.decode(q, Kc, Vc, w.lam, w.scale)
    got = llla.llla_decode(q.to(DEV), Kc.to(DEV), Vc.to(DEV), w.lam, w.scale)
    check(got.cpu().numpy()[:, :, None], ref[:, :, None], np.array([L - 1]), d, w.tol, "L=%d d=%d" % (L, d))


@pytest.mark.parametrize("d,dtype", [(16, "bf16"), (32, "bf16"), (32, "f32"), (64, "f32")])
def test_short_and_long_sequences_in_one_call(d, dtype):
    lens = [1, 5, 63, 64, 65, 700, 2000, 64]
    w, (q, Kc, Vc) = _case(len(lens), 2, 2000, d, dtype, 2450 + d)
    ref = oracle.decode(q, Kc, Vc, w.lam, w.scale, seqlens=lens)
    sl = torch.tensor(lens, dtype=torch.int32, device=DEV)
    for out in (torch.float32, torch.bfloat16):
        got = llla.llla_decode(q.to(DEV), Kc.to(DEV), Vc.to(DEV), w.lam, w.scale, seqlens=sl, out_dtype=out).float().cpu().numpy()
        # a bf16 result: half a unit in the last of its 8 bits on top
        for b, L in enumerate(lens):
            check(got[b:b + 1, :, None], ref[b:b + 1, :, None], np.array([L - 1]), d, w.tol if out == torch.float32 else 4e-3 + w.tol, "L=%d" % L)


def test_keys_beyond_the_range_of_f16():
    d, L, size = 32, 500, 2.0 ** 20
    w, (q, Kc, Vc) = _case(1, 4, L, d, "bf16", 2490)
    # the same problem with keys and queries in other units: K s, q s, logits' scale / s^2, ridge s^2
    ref = oracle.decode(q, Kc, Vc, w.lam, w.scale)
    got = llla.llla_decode((q * size).to(DEV), (Kc * size).to(DEV), Vc.to(DEV), w.lam * size ** 2, w.scale / size ** 2)
    check(got.cpu().numpy()[:, :, None], ref[:, :, None], np.array([L - 1]), d, w.tol, "size 2^20")
