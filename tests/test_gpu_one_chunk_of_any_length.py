"""A chunk length that is not shorter than the cache means one chunk, up to the largest the entry points
take (2^63 - 1): decode and every form of the attention give what the exact length gives."""
import pytest
import torch

from paper_2602_02958_amd import binding as B
from paper_2602_02958_amd import synth
from paper_2602_02958_amd.configs import CONFIGS
from test_gpu_attn_integration import _filled_caches

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("chunk_len", [1001, 1 << 31, (1 << 36) + 1, (1 << 63) - 1])
@pytest.mark.parametrize("n", [63, 1000])
def test_one_chunk_of_any_length(chunk_len, n):
    H = 2
    kc, vc = _filled_caches(H, n, 1, n, 64, 32, 2)
    kl, vl = (B.Encoded(c.centroids, c.ids, c.codes, c.scales, chunk_len) for c in (kc, vc))
    assert torch.equal(B.decode(kl), B.decode(kc))
    none = torch.empty(0, dtype=torch.uint8, device=DEV)                 # lent, too small: one kernel
    big = torch.empty(64 << 20, dtype=torch.uint8, device=DEV)           # holds the cache, but no chunk of 2^31 tokens
    for Nq in (33, 600):
        q = synth.queries(CONFIGS["cfg2_window21"], H, Nq, DEV)
        lens = torch.full((Nq,), min(n, 70), dtype=torch.int32, device=DEV)
        for ql in (None, lens):
            want = B.attn_decode(q, kc, vc, q_kv_len=ql)
            for ws in (None, none, big):
                assert torch.equal(B.attn_decode(q, kl, vl, q_kv_len=ql, workspace=ws), want)
    torch.cuda.synchronize()
