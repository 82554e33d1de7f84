"""The one-launch encoder writing the presets' stored forms itself (one round, E4M3 scales: 2-bit levels in groups of 64 and
16, 4-bit levels in groups of 64): scales that saturate, are subnormal, round to zero or are zero, ragged ends, one and four
stages, 16-bit ids.  Stored arrays against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import qvg_oracle as O
from paper_2602_02958_amd import binding as B
from conftest import bf16_bits
import parity_util as P

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("H,N,K,S", [(2, 640, 16, 1), (1, 257, 64, 2), (2, 1537, 256, 4), (1, 700, 300, 1), (1, 17, 5, 1), (27, 2950, 64, 1)])
@pytest.mark.parametrize("bits,Bg", [(2, 64), (2, 16), (4, 64)])
def test_presets(H, N, K, S, bits, Bg):
    g = torch.Generator().manual_seed(7 * N + K + bits + Bg)
    x = torch.randn(H, N, 128, generator=g)
    size = torch.tensor([1.0, 3.0e3, 3.0e-2, 2.0e-3, 4.0e-4, 1.0e-6, 0.0])       # of a group's residuals: E4M3 ends at 448 and 2^-9
    pick = torch.randint(0, len(size), (H, N, 128 // Bg), generator=g)
    x = (x * size[pick].repeat_interleave(Bg, 2)).to(torch.bfloat16)
    init = (0.01 * torch.randn(H, S, K, 128, generator=g)).to(torch.bfloat16)
    init[:, :, : max(1, K // 2)] = 0.0                           # residuals of the sizes above
    if S == 1:
        init = init[:, 0]
    enc = B.alloc_cache(H, N, N, K, Bg, 1, 128, DEV, n_smooth=S, bits=bits, scale_format=B.SCALE_E4M3)
    odd = torch.empty(enc.scales.numel() + 1, dtype=enc.scales.dtype, device=DEV)[1:].view(enc.scales.shape)     # scales at any address
    enc.scales = odd
    enc = B.encode_chunk(x.to(DEV), init.to(DEV), Bg, 1, 1, cache=enc)
    assert enc.scales.data_ptr() == odd.data_ptr() and odd.data_ptr() % 2
    torch.cuda.synchronize()
    units = list(range(H)) if H <= 2 else [0, 8, H - 1]
    ref = O.encode_batch(bf16_bits(x[units]), bf16_bits(init[units]), K, Bg, 1, 1, S=S, bits=bits, scale_fmt=1)
    assert np.array_equal(P.to_np_u16(enc.centroids[units, 0]).ravel(), np.asarray(ref["cent"]).ravel())
    ids = P.to_np_u8(enc.ids[units]) if K <= 256 else P.to_np_u16(enc.ids[units])
    assert np.array_equal(ids.ravel(), np.moveaxis(np.asarray(ref["ids"]), 1, 2).ravel())
    assert np.array_equal(P.to_np_u8(enc.codes[units]).ravel(), np.asarray(ref["codes"]).view(np.uint8).ravel())
    assert np.array_equal(P.to_np_u8(enc.scales[units]).ravel(), np.asarray(ref["scales"]).astype(np.uint8).ravel())
