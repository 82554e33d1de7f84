"""Decode calls whose last chunk has fewer slices than the others, on both sides of the rule that gives each compute unit one
slice, and a last slice of one token: bit-equal to the oracle."""
import pytest

from paper_2602_02958_amd import binding as B
from test_gpu_decode_slices import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,N,L", [
    (1, 65553, 65553),       # 242 slices of 272 tokens, the last with one
    (24, 4688, 4680),        # nine slices of 528 and one of 8 tokens
    (24, 6240, 4680),        # seven of 672, three of a chunk of 1560
    (24, 9368, 4680),        # too few would be busy: 256 tokens each
    (3, 9 * 4000 + 1, 4000), # nine chunks in nine slices of 448 each, and one of one token
    (256, 301, 300),
    (54, 3540, 3472),
    (2, 40016, 4680),
])
def test_slices(H, N, L):
    _check(H, N, L, 16, 64, 2, 2, B.SCALE_F16)


@pytest.mark.parametrize("T,bits,fmt,K,Bg", [(3, 2, B.SCALE_F16, 100, 32), (1, 2, B.SCALE_E4M3, 512, 64), (1, 4, B.SCALE_E4M3, 256, 64)])
@pytest.mark.parametrize("H,N,L", [(24, 4688, 4680), (3, 1111, 400)])
def test_formats(T, bits, fmt, K, Bg, H, N, L):
    _check(H, N, L, K, Bg, T, bits, fmt)
