"""Decode calls whose last chunk has fewer slices than the others, on both sides of the rules that give each compute unit one
slice, and a last slice of one token: bit-equal to the oracle."""
import pytest

from paper_2602_02958_amd import binding as B
from test_gpu_decode_slices import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,T", [(16, 2), (256, 4)])     # up to 2.5 passes a slice and at least 184 busy units; up to 8, and 152
@pytest.mark.parametrize("H,N,L", [
    (1, 65553, 65553),       # 242 slices of 272 tokens, the last with one
    (1, 524288, 524288),     # 256 of 2048 (K = 256)
    (24, 4688, 4680),        # nine slices of 528 and one of 8 tokens
    (24, 6240, 4680),        # seven of 672, three of a chunk of 1560 (K = 256)
    (24, 9368, 4680),        # four of 1184 to a chunk, 192 busy ones (K = 256)
    (54, 3540, 3472),        # three of 1168 and one of 68 tokens, 165 busy ones (K = 256)
    (50, 3540, 3472),        # 152
    (48, 3500, 3472),        # (five to a chunk)
    (3, 9 * 4000 + 1, 4000), # nine chunks in nine slices of 448 each, and one of one token
    (256, 301, 300),
    (2, 40016, 4680),
])
def test_slices(H, N, L, K, T):
    _check(H, N, L, K, 64, T, 2, B.SCALE_F16)


@pytest.mark.parametrize("T,bits,fmt,K,Bg", [(3, 2, B.SCALE_F16, 100, 32), (1, 2, B.SCALE_E4M3, 512, 64), (1, 4, B.SCALE_E4M3, 256, 64)])
@pytest.mark.parametrize("H,N,L", [(24, 4688, 4680), (3, 1111, 400)])
def test_formats(T, bits, fmt, K, Bg, H, N, L):
    _check(H, N, L, K, Bg, T, bits, fmt)
