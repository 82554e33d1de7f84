"""The sizes that qvg_encode_chunk_static accepts do not depend on the layout of the workspace: sizes
whose workspace is larger than QVG_STATIC_SCRATCH_BYTES, accepted by the documented sum, encode as with a
lent workspace; sizes just beyond the sum are refused."""
import numpy as np
import pytest
import torch

from paper_2602_02958_amd import binding as B
from paper_2602_02958_amd import synth
from paper_2602_02958_amd.configs import CONFIGS

pytestmark = pytest.mark.gpu
LIMIT = 16 << 20


def _r256(v):
    return -(-v // 256) * 256


def _rule(H, K, S, iters, N):
    o = _r256(H * (-(-K // 64) * 64) * 8) + _r256(H * 4)
    if iters or S > 1:
        o += 2 * _r256(H * K * 256)
    if iters:
        o += _r256(H * N * 4) + _r256(H * (K + 1) * 4)
    return o + min(S - 1, 2) * _r256(H * N * 256)


@pytest.mark.parametrize("H,K,S,N", [(40, 512, 1, 20000), (3, 512, 2, 20000), (80, 300, 1, 10800)])
def test_static_scratch_accepts_by_the_documented_sum(H, K, S, N):
    assert _rule(H, K, S, 1, N) <= LIMIT
    p = B.make_params(H, K, 64, 1, kmeans_iters=1, n_smooth_stages=S)
    assert B.workspace_bytes(p, B.ENTRY_ENCODE, N) > LIMIT
    x = synth.MixtureStream(CONFIGS["cfg3_dit_small"], H, 0, "cuda").next_chunk(N)
    init = synth.cold_start_centroids(x, K)
    if S > 1:
        init = torch.stack([init] * S, 1)
    a = B.encode_chunk(x, init, 64, 1, 1)
    b = B.encode_chunk(x, init, 64, 1, 1, static_scratch=True)
    torch.cuda.synchronize()
    for t, u in ((a.centroids, b.centroids), (a.ids, b.ids), (a.codes, b.codes), (a.scales, b.scales)):
        assert np.array_equal(t.view(torch.uint8).cpu().numpy(), u.view(torch.uint8).cpu().numpy())


def test_static_scratch_refuses_beyond_the_documented_sum():
    H, K = 3, 512
    N = next(n for n in range(20000, 40000, 16) if _rule(H, K, 2, 1, n) > LIMIT)
    x = torch.zeros(H, N, 128, dtype=torch.bfloat16, device="cuda")
    init = torch.zeros(H, 2, K, 128, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(B.QvgError) as e:
        B.encode_chunk(x, init, 64, 1, 1, static_scratch=True)
    assert e.value.status == -7
