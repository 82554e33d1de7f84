"""The update's walk over a unit's blocks of tokens: units of more than 64 blocks (the lists are then put
together 64 blocks at a time), and lists of every short length (rows are read sixteen, eight, four
or two at a time).  Means against the oracle's token-order sums, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import qvg_oracle as O
from paper_2602_02958_amd import binding as B
from conftest import bf16_bits, bits_to_f32
import parity_util as P

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _check(x, ids, prev, K, units):
    xb, pb = x.to(torch.bfloat16), prev.to(torch.bfloat16)
    dt = torch.uint8 if K <= 256 else torch.int16
    c, n = B.kmeans_update(xb.to(DEV), ids.to(DEV, dt), pb.to(DEV))
    torch.cuda.synchronize()
    for h in units:
        want, count = O.update(bits_to_f32(bf16_bits(xb)[h]), ids[h].numpy().astype(np.int32), bf16_bits(pb)[h])
        assert np.array_equal(n[h].cpu().numpy(), count), h
        assert np.array_equal(P.to_np_u16(c[h]), want), h


@pytest.mark.parametrize("H,N,K", [(1, 64 * 256 + 1, 16), (1, 65 * 256, 300), (2, 40000, 64), (1, 140000, 5), (1, 700001, 512),
                                   (9, 33000, 256)])
def test_more_than_64_blocks(H, N, K):
    """One cluster with half of the tokens (all blocks, and one channel whose sum depends on the order), one in
    the last blocks only, one empty, one whose members are 70 blocks apart."""
    g = torch.Generator().manual_seed(N + K)
    x = torch.randn(H, N, 128, generator=g)
    ids = torch.randint(0, K, (H, N), generator=g)
    ids[:, ::2] = 1
    ids[ids == K - 1] = 0
    ids[:, -300:] = K - 1
    ids[ids == 2] = 0
    if K > 3:
        ids[ids == 3] = 0
        ids[:, 5::70 * 256] = 3
    x[0, ::4, 0] *= 1.0e18
    x[0, 2::4, 0] *= 1.0e-9
    _check(x, ids, torch.randn(H, K, 128, generator=g), K, range(min(H, 2)))


@pytest.mark.parametrize("H,K,stride", [(40, 64, 1), (1, 64, 1), (5, 512, 3), (20, 256, 2)])
def test_lists_of_every_short_length(H, K, stride):
    """Cluster j of unit h has (stride j + h) mod 67 members, scattered over the unit."""
    g = torch.Generator().manual_seed(H * K)
    lens = [[(stride * j + h) % 67 for j in range(K)] for h in range(H)]
    N = max(sum(l) for l in lens)
    ids = torch.empty(H, N, dtype=torch.int64)
    for h in range(H):
        flat = torch.cat([torch.full((m,), j) for j, m in enumerate(lens[h])])
        flat = torch.cat([flat, torch.full((N - flat.numel(),), K - 1)])
        ids[h] = flat[torch.randperm(N, generator=g)]
    _check(torch.randn(H, N, 128, generator=g), ids, torch.randn(H, K, 128, generator=g), K, sorted({0, H // 2, H - 1}))


@pytest.mark.parametrize("stride", [136, 10240, 16384, 32768])
def test_tokens_far_apart(stride):
    """Views whose unit spans less and more than 2^31 bytes (65793 tokens: 1.35 and 2.16, 4.3 * 10^9): the rows of
    short and of long lists are found in both, as in a dense copy."""
    N, K = 65793, 1000 // 2
    g = torch.Generator(device=DEV).manual_seed(stride)
    base = torch.empty(1, N, stride, dtype=torch.bfloat16, device=DEV)
    x = base[:, :, 8:136]
    x.copy_(torch.randn(1, N, 128, generator=g, device=DEV))
    ids = torch.randint(0, 400, (1, N), generator=g, device=DEV)
    ids[:, :N // 2] = torch.arange(N // 2, device=DEV) % 300 + 100
    ids[:, -900:] = 400 + torch.arange(900, device=DEV) % 100      # lists of nine
    ids = ids.to(torch.int16)
    prev = torch.randn(1, K, 128, generator=g, device=DEV).to(torch.bfloat16)
    far, dense = B.kmeans_update(x, ids, prev), B.kmeans_update(x.contiguous(), ids, prev)
    torch.cuda.synchronize()
    assert torch.equal(far[1], dense[1]) and torch.equal(far[0].view(torch.int16), dense[0].view(torch.int16))
    want, count = O.update(bits_to_f32(bf16_bits(x[0])), ids[0].cpu().numpy().astype(np.int32), bf16_bits(prev[0]))
    assert np.array_equal(dense[1][0].cpu().numpy(), count)
    assert np.array_equal(P.to_np_u16(dense[0][0]), want)
