"""Tokens whose scores of every row are below fp32's range while all norms are within it: decided by their distances, in launches of
their own and in one, with and without rows that pad the table."""
import numpy as np
import pytest
import torch

from oracle import qvg_oracle as O
from paper_2602_02958_amd import binding as B
from conftest import bf16_bits
import parity_util as P

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("N,I", [(300, 0), (640, 1), (3000, 1)])
@pytest.mark.parametrize("K", [1, 2, 3, 62, 63, 64, 65])
def test_every_score_overflows(N, I, K):
    a = 1.5e18                                       # 128 a^2 = 2.9e38
    g = torch.Generator().manual_seed(N + K)
    x = (a * (0.98 + 0.02 * torch.rand(2, N, 128, generator=g))).to(torch.bfloat16)
    x[:, ::7] *= 1e-3                                # (and some whose scores do not)
    init = (-a * (0.9 + 0.1 * torch.rand(2, K, 1, generator=g)).expand(2, K, 128)).to(torch.bfloat16).contiguous()
    enc = B.encode_chunk(x.to(DEV), init.to(DEV), 64, 1, I)
    torch.cuda.synchronize()
    ref = O.encode_batch(bf16_bits(x), bf16_bits(init), K, 64, 1, I)
    assert np.array_equal(P.to_np_u8(enc.ids), ref["ids"][:, 0])
    assert np.array_equal(P.to_np_u16(enc.centroids[:, 0]), ref["cent"][:, 0])
    assert np.array_equal(P.to_np_u8(enc.codes), ref["codes"])
    assert np.array_equal(P.to_np_u16(enc.scales), ref["scales"])
