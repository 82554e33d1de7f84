"""The encoder's stages behind the first: in one launch, rows dealt to a unit's workgroups by their members (clusters that hold
most of the tokens next to empty ones, more rows for a workgroup than it makes at a time); tables with several rows of
zeros, of which only the first can be nearest (with rows beside them whose norm is zero in fp32 though they are not).
Stored arrays against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import qvg_oracle as O
from paper_2602_02958_amd import binding as B
from conftest import bf16_bits
import parity_util as P

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _inputs(H, N, K, S, zeros, seed):
    g = torch.Generator().manual_seed(seed)
    x = torch.randn(H, N, 128, generator=g)
    heavy = torch.randn(H, 3, 128, generator=g)                  # three clusters with two thirds of the tokens
    at = torch.randint(0, 3, (H, N), generator=g)
    most = torch.rand(H, N, 1, generator=g) < 0.67
    x = torch.where(most, torch.gather(heavy, 1, at[:, :, None].expand(-1, -1, 128)) + 0.02 * x, x).to(torch.bfloat16)
    n0 = min(K, N)
    init = torch.randn(H, S, K, 128, generator=g).to(torch.bfloat16)
    init[:, 0, :n0] = x[:, :n0]                                  # tokens that are centroids: their residual is zero
    for s in range(1, S):
        init[:, s] = (0.05 * init[:, s].float()).to(torch.bfloat16)
        if zeros:
            rows = torch.randperm(K, generator=g)[:max(2, K // 3)]
            init[:, s, rows] = 0.0
            init[:, s, rows[:2]] = -0.0
            tiny = torch.randperm(K, generator=g)[:max(1, K // 8)]
            init[:, s, tiny, :5] = 2.0 ** -120                   # the norm is below fp32's range, the row is not zero
            init[:, s, tiny, 5:] = 0.0
    return x, init


@pytest.mark.parametrize("zeros", [False, True])
@pytest.mark.parametrize("H,N,K,Bg,S,I", [
    (2, 640, 16, 64, 3, 3),            # as many rows as a few blocks can share
    (2, 257, 7, 64, 2, 2),             # fewer rows than 64
    (3, 1999, 64, 32, 2, 2),
    (2, 1300, 256, 16, 4, 2),          # the paper's four stages; more workgroups than blocks
    (1, 1537, 300, 64, 2, 2),          # 16-bit ids, rows in two halves
    (2, 700, 512, 64, 2, 1),
    (1, 15, 12, 64, 2, 2),             # one workgroup
    (27, 3000, 64, 64, 2, 1),          # a full chip, units of twelve blocks
    (2, 1300, 256, 16, 3, 0),          # launches of their own
    (1, 6300, 64, 64, 2, 1),
])
def test_stages_with_unequal_clusters(H, N, K, Bg, S, I, zeros):
    x, init = _inputs(H, N, K, S, zeros, 1000 + N + K)
    enc = B.encode_chunk(x.to(DEV), init.to(DEV), Bg, 1, I)
    torch.cuda.synchronize()
    units = list(range(H)) if H <= 3 else [0, 8, H - 1]
    ref = O.encode_batch(bf16_bits(x[units]), bf16_bits(init[units]), K, Bg, 1, I, S=S)
    assert np.array_equal(P.to_np_u16(enc.centroids[units, 0]), ref["cent"])
    ids = P.to_np_u8(enc.ids[units]) if K <= 256 else P.to_np_u16(enc.ids[units])
    assert np.array_equal(ids, ref["ids"].transpose(0, 2, 1))
    assert np.array_equal(P.to_np_u8(enc.codes[units]), ref["codes"])
    assert np.array_equal(P.to_np_u16(enc.scales[units]), ref["scales"])


@pytest.mark.parametrize("N,I", [(640, 1), (1300, 2), (640, 0)])
@pytest.mark.parametrize("K,zeros", [(3, [0, 1]), (4, [0, 1, 3]), (4, [0]), (2, [0]), (130, [0, 1, 129])])
def test_scores_beyond_fp32(N, I, K, zeros):
    """Finite tokens and rows whose squared norms are not: a score that overflows decides nothing, also where the only row with
    a finite one is a row of zeros and the rows behind it are the table's padding.  (Half of the tokens are + a, half - a, so
    that the first stage, all rows zero, leaves them as they are.)"""
    a = 2.0 ** 66
    g = torch.Generator().manual_seed(N + K)
    x = torch.full((2, N, 128), a)
    x[:, ::2] *= -1.0
    init = torch.zeros(2, 2, K, 128)
    init[:, 1] = -8.0 * a * (1.0 + torch.rand(2, K, 1, generator=g))     # further than zero from every token
    init[:, 1, zeros] = 0.0
    init[:, 1, min(2, K - 1)] = 0.75 * a
    x, init = x.to(torch.bfloat16), init.to(torch.bfloat16)
    enc = B.encode_chunk(x.to(DEV), init.to(DEV), 64, 1, I)
    torch.cuda.synchronize()
    ref = O.encode_batch(bf16_bits(x), bf16_bits(init), K, 64, 1, I, S=2)
    assert len(set(ref["ids"][0, 1])) == 2
    assert np.array_equal(P.to_np_u8(enc.ids), ref["ids"].transpose(0, 2, 1))
    assert np.array_equal(P.to_np_u16(enc.centroids[:, 0]), ref["cent"])
    assert np.array_equal(P.to_np_u8(enc.codes), ref["codes"])
    assert np.array_equal(P.to_np_u16(enc.scales), ref["scales"])
