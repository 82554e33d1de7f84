"""The memory that an attention takes for itself, and the workspace it is lent: a call with a prefix
length per query takes no tile workspace (every tile of the cache would be decoded, however short the
prefixes), nor does one over a few tiles; the fp32 result uses the lent workspace like the bf16 one."""
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


def test_a_cache_of_a_few_tiles_takes_no_tile_workspace():
    H, Nq, L = 12, 600, 4680
    kc, vc = _filled_caches(H, L, 1, 300, 16, 64, 2)
    q = synth.queries(CONFIGS["cfg2_window21"], H, Nq, DEV)
    out, taken = _taken(lambda: B.attn_decode(q, kc, vc, n_kv=255))
    assert taken <= 1 << 20
    lent = B.attn_decode(q, kc, vc, n_kv=255, workspace=B.attn_workspace(H, Nq, L, 1, DEV))
    torch.cuda.synchronize()
    assert torch.equal(out, lent)


def test_the_fp32_result_uses_the_lent_workspace():
    H, Nq, L, n = 12, 600, 4680, 14040
    kc, vc = _filled_caches(H, L, 3, n, 16, 64, 2)
    q = synth.queries(CONFIGS["cfg2_window21"], H, Nq, DEV)
    out = B.attn_decode(q, kc, vc)
    states = 256 * 66 * 512 * 4
    ws = B.attn_workspace(H, Nq, L, 1, DEV).fill_(0xA5)
    f32, taken = _taken(lambda: B.attn_decode(q, kc, vc, f32_out=True, workspace=ws))
    assert taken <= states + (1 << 20)
    assert (ws != 0xA5).any()
    assert torch.equal(f32.to(torch.bfloat16), out)
    none = torch.empty(0, dtype=torch.uint8, device=DEV)     # lent, too small: the one-kernel form
    f32, taken = _taken(lambda: B.attn_decode(q, kc, vc, f32_out=True, workspace=none))
    assert taken <= states + (1 << 20)
    assert torch.equal(f32.to(torch.bfloat16), out)
