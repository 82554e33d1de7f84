"""Decode calls whose slices are one per compute unit (slices of up to eight passes of 256 tokens that end anywhere
in a pass, a chunk that is not full) and the 4-bit single round's own instances: bit-equal to the oracle."""
import numpy as np
import pytest
import torch

from oracle import qvg_oracle as O
from paper_2602_02958_amd import binding as B
import parity_util as P

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _check(H, N, L, K, Bg, T, bits, fmt):
    g = torch.Generator().manual_seed(N + K + T)
    cache = B.alloc_cache(H, N, L, K, Bg, T, 128, DEV, bits=bits, scale_format=fmt)
    cache.centroids.copy_(torch.randn(cache.centroids.shape, generator=g).to(torch.bfloat16))
    cache.ids.copy_(torch.randint(0, K, cache.ids.shape, generator=g).to(cache.ids.dtype))
    if bits == 2:
        f = torch.tensor([0, 1, 3], dtype=torch.uint8)[torch.randint(0, 3, cache.codes.shape + (4,), generator=g)]
        cache.codes.copy_(f[..., 0] | (f[..., 1] << 2) | (f[..., 2] << 4) | (f[..., 3] << 6))
    else:
        f = (torch.randint(-7, 8, cache.codes.shape + (2,), generator=g) & 15).to(torch.uint8)
        cache.codes.copy_(f[..., 0] | (f[..., 1] << 4))
    if fmt == B.SCALE_E4M3:
        cache.scales.copy_(torch.randint(0, 0x60, cache.scales.shape, generator=g, dtype=torch.uint8))
    else:
        cache.scales.copy_(torch.rand(cache.scales.shape, generator=g).to(torch.float16))
    out = B.decode(cache)
    torch.cuda.synchronize()
    out = P.to_np_u16(out)
    ids = cache.ids.cpu().numpy().astype(np.uint16)
    codes, cent = P.to_np_u8(cache.codes), P.to_np_u16(cache.centroids)
    sc = P.to_np_u8(cache.scales).astype(np.uint16) if fmt == B.SCALE_E4M3 else P.to_np_u16(cache.scales)
    for h in range(H):
        for c in range(-(-N // L)):
            sl = slice(c * L, min((c + 1) * L, N))
            want = O.decode_unit(cent[h, c], ids[h, sl], codes[h, sl], sc[h, sl], Bg, bits=bits, scale_fmt=fmt)
            assert np.array_equal(out[h, sl], want), (h, c)


@pytest.mark.parametrize("H,N,L", [
    (1, 65537, 65537),       # 241 slices of 272 tokens, the last with 257
    (1, 524288, 524288),     # eight whole passes each: the longest slices of the rule
    (24, 4680, 4680),        # ten slices of 480, the last 360
    (2, 40001, 4680),        # 14 slices of 336 per chunk, the last chunk 2561 tokens
    (208, 257, 257),         # one slice of 272 per unit, its second pass one token
    (207, 257, 257),         # one unit fewer: too few CUs
    (256, 300, 300),
    (257, 300, 300),         # more units than CUs
])
def test_slices_of_small_calls(H, N, L):
    _check(H, N, L, 16, 64, 2, 2, B.SCALE_F16)


@pytest.mark.parametrize("T,bits,fmt,K,Bg", [(4, 2, B.SCALE_F16, 256, 64), (3, 2, B.SCALE_F16, 100, 32), (5, 2, B.SCALE_F16, 64, 64),
                                             (1, 2, B.SCALE_E4M3, 512, 64), (1, 4, B.SCALE_E4M3, 256, 64), (1, 4, B.SCALE_F16, 300, 16),
                                             (2, 4, B.SCALE_E4M3, 256, 128)])
@pytest.mark.parametrize("H,N,L", [(24, 4680, 4680), (3, 1111, 400)])
def test_formats_in_slices(T, bits, fmt, K, Bg, H, N, L):
    _check(H, N, L, K, Bg, T, bits, fmt)
