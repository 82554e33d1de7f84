"""A token that is not a number (or infinite) belongs to no cluster and leaves all others as they would be without it, in one launch and in launches
of their own."""
import numpy as np
import pytest
import torch

from oracle import qvg_oracle as O
from paper_2602_02958_amd import binding as B
from conftest import bf16_bits
import parity_util as P

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("H,N,K,I", [(24, 780, 64, 3), (6, 2000, 64, 2), (2, 1500, 16, 2), (3, 130, 5, 1), (24, 780, 64, 0)])
def test_nan_tokens(H, N, K, I):
    g = torch.Generator().manual_seed(N + K)
    x = torch.randn(H, N, 128, generator=g).to(torch.bfloat16)
    init = x[:, torch.randperm(N, generator=g)[:K]].contiguous()
    bad = torch.zeros(N, dtype=torch.bool)
    bad[[0, 33, 34, 64, 99, 127]] = True
    y = x.clone()
    y[:, bad] = float("nan")
    y[:, 99] = float("inf")
    enc = B.encode_chunk(y.to(DEV), init.to(DEV), 64, 1, I)
    torch.cuda.synchronize()
    ok = (~bad).numpy()
    units = sorted({0, H - 1})
    ref = O.encode_batch(bf16_bits(x[units][:, ~bad].contiguous()), bf16_bits(init[units]), K, 64, 1, I)
    assert np.array_equal(P.to_np_u16(enc.centroids[units, 0]), ref["cent"][:, 0])
    assert np.array_equal(P.to_np_u8(enc.ids[units])[:, ok], ref["ids"][:, 0])
    assert np.array_equal(P.to_np_u8(enc.codes[units])[:, ok], ref["codes"])
    assert np.array_equal(P.to_np_u16(enc.scales[units])[:, ok], ref["scales"])
