"""Scratch that is lent to an attention call and is not what the call asks for: misaligned."""
import pytest
import torch

from paper_2602_02958_amd import binding as B
from paper_2602_02958_amd import synth
from paper_2602_02958_amd.configs import CONFIGS
from test_gpu_attn_integration import _filled_caches
from test_gpu_attn_parts import _decode_parts

pytestmark = pytest.mark.gpu
DEV = "cuda"
L = 1024


def _filled(H, n):
    return [B.Encoded(c.centroids, c.ids[:, :n].contiguous(), c.codes[:, :n].contiguous(), c.scales[:, :n].contiguous(), c.chunk_len)
            for c in _filled_caches(H, L, -(-n // L), n, 16, 64, 1)]


@pytest.mark.parametrize("H,Nq,n,lengths", [(1, 64, 256, False), (1, 64, 448, False), (8, 64, 400, False), (65, 1, 500, False),
                                            (66, 256, 500, True), (1, 40, 300, True)])
def test_misaligned_scratch_over_a_few_tiles_is_ignored(H, Nq, n, lengths):
    """Such calls ran undivided with any scratch before they were divided, and still do."""
    kd, vd = _filled(H, n)
    q = synth.queries(CONFIGS["cfg2_window21"], H, Nq, DEV)
    lens = torch.arange(1, Nq + 1, dtype=torch.int32, device=DEV) * max(n // Nq, 1) if lengths else None
    scratch = torch.full((110 << 20,), 0x7F, dtype=torch.uint8, device=DEV)
    out = _decode_parts(q, kd, vd, lens, scratch[4:])
    torch.cuda.synchronize()
    assert torch.equal(out, _decode_parts(q, kd, vd, lens, None)) and bool((scratch == 0x7F).all())
