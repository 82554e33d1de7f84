"""The memory that an attention takes for itself, and the workspace it is lent: a call with a prefix
length per query takes no tile workspace (every tile of the cache would be decoded, however short the
prefixes)."""
import pytest
import torch

from paper_2602_02958_amd import binding as B
from paper_2602_02958_amd import synth
from paper_2602_02958_amd.configs import CONFIGS
from test_gpu_attn_integration import _filled_caches

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _taken(fn):
    """(result, bytes at the peak of the call beyond what was allocated before and the result itself)"""
    fn()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    torch.cuda.reset_peak_memory_stats()
    before = torch.cuda.memory_allocated()
    out = fn()
    torch.cuda.synchronize()
    return out, torch.cuda.max_memory_allocated() - before - out.numel() * out.element_size()


def test_a_prefix_length_per_query_takes_no_tile_workspace():
    H, Nq, L, n = 12, 600, 4680, 14040
    kc, vc = _filled_caches(H, L, 3, n, 16, 64, 2)
    q = synth.queries(CONFIGS["cfg2_window21"], H, Nq, DEV)
    lens = torch.full((Nq,), 300, dtype=torch.int32, device=DEV)
    out, taken = _taken(lambda: B.attn_decode(q, kc, vc, q_kv_len=lens))
    tiles = H * -(-L // 64) * 64 * 512                       # one chunk's decoded tiles
    states = 256 * 66 * 512 * 4                              # of at most 256 parts
    assert taken <= states + (1 << 20) < tiles + states
    lent = B.attn_decode(q, kc, vc, q_kv_len=lens, workspace=B.attn_workspace(H, Nq, L, 1, DEV))
    torch.cuda.synchronize()
    assert torch.equal(out, lent)
