"""The assignment's error band and the re-evaluation of tokens inside it: centroids of very different
norms, and tokens with two, a few, many, or only equal candidates.  Ids against the oracle, exactly
(fp64 distances, lowest index among equal ones)."""
import numpy as np
import pytest
import torch

from oracle import qvg_oracle as O
from paper_2602_02958_amd import binding as B
from conftest import bf16_bits, bits_to_f32
import parity_util as P

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("K", [1, 2, 63, 64, 65, 128, 256, 300, 512])
@pytest.mark.parametrize("kind", ["far_centroid", "near_pairs", "few", "many", "equal", "zero", "far_tokens"])
def test_ids_equal_the_oracle(K, kind):
    H, N, d = 2, 333, 128
    g = torch.Generator().manual_seed(1000 * K + len(kind))
    c = torch.randn(H, K, d, generator=g)
    if kind == "far_centroid":               # one centroid a thousand times as long as the others
        c[:, K // 2] *= 1000.0
    elif kind == "near_pairs":               # every centroid once more, one unit of the last place away
        c[:, K // 2:] = c[:, :K - K // 2] * (1.0 + 2.0 ** -8)
    elif kind in ("few", "many"):            # groups of 6 / of 40 centroids inside a token's band
        n = 6 if kind == "few" else 40
        base = torch.randn(H, -(-K // n), d, generator=g)
        c = base.repeat_interleave(n, 1)[:, :K].clone()
        c[:, :, 0] += 2.0 ** -9 * torch.randint(-2, 3, (H, K), generator=g)
    elif kind == "equal":                    # all centroids the same: index 0 must win
        c = c[:, :1].expand(H, K, d).clone()
    elif kind == "zero":
        c = torch.zeros(H, K, d)
    pick = torch.randint(0, K, (H, N), generator=g)
    x = torch.gather(c, 1, pick[:, :, None].expand(-1, -1, d)) + 0.05 * torch.randn(H, N, d, generator=g)
    if kind == "zero":
        x[:, ::2] = 0.0
    if kind == "far_tokens":                 # tokens a hundred times further out than any centroid
        x[:, ::3] *= 100.0
    xb, cb = x.to(torch.bfloat16), c.to(torch.bfloat16)
    got = P.to_np_u8(B.kmeans_assign(xb.to(DEV), cb.to(DEV))) if K <= 256 else \
        P.to_np_u16(B.kmeans_assign(xb.to(DEV), cb.to(DEV)))
    for h in range(H):
        want = O.assign(bits_to_f32(bf16_bits(xb)[h]), bf16_bits(cb)[h])
        assert np.array_equal(got[h].astype(np.int64), want.astype(np.int64)), (h, np.flatnonzero(got[h] != want)[:5])


@pytest.mark.parametrize("K,first", [(128, 0), (128, 64), (256, 64), (256, 192), (512, 128), (512, 448)])
def test_a_block_of_zero_rows_beside_near_ties(K, first):
    """64 zero rows that one wavefront places (the table's largest norm must survive them), the others in
    pairs one unit of the last place apart."""
    H, N, d = 2, 333, 128
    g = torch.Generator().manual_seed(K + first)
    c = torch.randn(H, K, d, generator=g) * torch.exp(torch.randn(H, K, 1, generator=g))
    c[:, 1::2] = c[:, ::2] * (1.0 + 2.0 ** -8)
    c[:, first:first + 64] = 0.0
    pick = torch.randint(0, K, (H, N), generator=g)
    x = torch.gather(c, 1, pick[:, :, None].expand(-1, -1, d))
    x = 1.5 * x + 0.05 * x.abs().mean(-1, keepdim=True) * torch.randn(H, N, d, generator=g)
    x[:, ::7] = 0.0
    xb, cb = x.to(torch.bfloat16), c.to(torch.bfloat16)
    ids = B.kmeans_assign(xb.to(DEV), cb.to(DEV))
    got = P.to_np_u8(ids) if K <= 256 else P.to_np_u16(ids)
    for h in range(H):
        want = O.assign(bits_to_f32(bf16_bits(xb)[h]), bf16_bits(cb)[h])
        assert np.array_equal(got[h].astype(np.int64), want.astype(np.int64)), (h, np.flatnonzero(got[h] != want)[:5])
