"""fp32 forward: the order in which the blocks of query rows and the key-space workgroups of a call start hangs on the number of heads and rows, and
changes no bit: every head of a call comes out as in a call of its own, which is small enough to go head by head with the key-space rows last.  At
d = 64 24 blocks of rows (28 with more than 16 heads) and 256 blocks in all are the lines, at d = 16 / 32 256 and 480 blocks, six heads and 480 workgroups in all; the
numbers of heads are multiples of eight and not, the numbers of rows whole blocks and not.  path: a short call of one head at d = 16 / 32 would take the vector kernel."""
import pytest
import torch

import paper_2510_01450_amd as llla

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("d,B,H,n", [(64, 3, 3, 447), (64, 3, 3, 449), (64, 1, 11, 500), (64, 2, 8, 512), (64, 1, 17, 495), (64, 1, 17, 497),
                                     (64, 3, 8, 560), (64, 1, 4, 1100), (32, 1, 6, 755), (32, 1, 6, 770), (32, 1, 7, 770), (32, 2, 8, 545), (32, 2, 5, 560), (32, 2, 5, 577),
                                     (16, 1, 4, 1100), (16, 1, 14, 600), (16, 2, 8, 560), (16, 5, 5, 600)])
@pytest.mark.parametrize("causal", [True, False])
def test_heads_alone_and_together(d, B, H, n, causal):
    g = torch.Generator(device="cpu").manual_seed(4000 + 17 * n + H)
    Q, K, V = [torch.randn(B, H, n, d, generator=g).to(DEV) for _ in range(3)]
    got = llla.llla_forward(Q, K, V, 1e-2, d ** -0.5, causal=causal, return_stats=True, path="mfma")
    for b in range(B):
        for h in range(H):
            one = llla.llla_forward(*[x[b:b + 1, h:h + 1] for x in (Q, K, V)], 1e-2, d ** -0.5, causal=causal, return_stats=True, path="mfma")
            for x, y in zip(got, one):
                assert torch.isfinite(y).all() and torch.equal(x[b, h], y[0, 0])
