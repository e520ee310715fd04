"""Edges of single kernels and dispatch branches, small, against the oracle or
a plain float64 evaluation of the same definition."""
import numpy as np
import pytest
import torch

from oracle import compress as OC
from paper_2407_00066_amd import compress as GC

from _gpu_helpers import say

pytestmark = pytest.mark.gpu


def _f32(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).to("cuda")


@pytest.mark.parametrize("n,r_l,d_out,d_in", [
    (1, 4, 16, 20),       # one LoRA of four: a quarter of the row tile
    (5, 4, 68, 36),       # a last workgroup of one LoRA
    (7, 8, 132, 1028),    # a k tail of 4 past the 16-wide steps
    (3, 16, 64, 16),      # fewer steps than waves
    (2, 32, 1036, 260),
    (2, 64, 100, 516),
])
def test_lora_norms2(n, r_l, d_out, d_in):
    """fp32 Gram entries: each is a sum of d products, error below d eps times
    the sum of their magnitudes; the square norm adds r_l^2 such terms."""
    say("norms2 n=%d r_l=%d %dx%d" % (n, r_l, d_out, d_in))
    rs = np.random.default_rng(1000 + r_l + n)
    A = rs.standard_normal((n, r_l, d_in)).astype(np.float32)
    B = rs.standard_normal((n, d_out, r_l)).astype(np.float32)
    got = GC.lora_norms2(_f32(A), _f32(B), r=16 if n * r_l >= 16 else n * r_l).cpu().numpy().astype(np.float64) \
        if n * r_l >= 16 else None
    if got is None:                                # r must not exceed n r_l: pad the collection with zero LoRAs
        k = -(-16 // r_l)
        A2, B2 = np.zeros((k, r_l, d_in), np.float32), np.zeros((k, d_out, r_l), np.float32)
        A2[:n], B2[:n] = A, B
        got = GC.lora_norms2(_f32(A2), _f32(B2), r=16).cpu().numpy().astype(np.float64)
        assert (got[n:] == 0).all()
        got = got[:n]
    A, B = A.astype(np.float64), B.astype(np.float64)
    want = np.array([np.linalg.norm(P) ** 2 for P in OC.products(A, B)])
    ga = np.einsum("nlc,nmc->nlm", np.abs(A), np.abs(A))
    gb = np.einsum("nol,nom->nlm", np.abs(B), np.abs(B))
    bound = (d_in + d_out + r_l * r_l) * 2.0 ** -24 * (ga * gb).sum((1, 2))
    assert (np.abs(got - want) <= bound).all()
