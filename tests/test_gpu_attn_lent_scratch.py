"""Scratch that is lent to an attention call and is not what the call asks for: misaligned, or for a longer cache."""
import pytest
import torch

from oracle import qvg_oracle as O
from paper_2602_02958_amd import binding as B
from paper_2602_02958_amd import synth
from paper_2602_02958_amd.configs import CONFIGS
from conftest import bf16_bits
import parity_util as P
from test_gpu_attn_integration import _filled_caches
from test_gpu_attn_parts import _decode_parts, _scratch_bytes

pytestmark = pytest.mark.gpu
DEV = "cuda"
L = 1024
STATE = 66 * 512 * 4


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


@pytest.mark.parametrize("H,Nq,longest,tiles,parts", [
    (8, 64, 33, 32, 16),      # 17 parts' room, 32 would be best
    (9, 64, 48, 47, 12),      # 12, 24
    (16, 200, 43, 42, 11),    # 11, 14
    (1, 40, 300, 256, 128),   # 150, 256
])
def test_scratch_for_a_longer_cache_divides_a_shorter_one(H, Nq, longest, tiles, parts):
    n = tiles * 64 - 5
    kd, vd = _filled(H, n)
    q = synth.queries(CONFIGS["cfg2_window21"], H, Nq, DEV)
    need = _scratch_bytes(H, Nq, longest * 64, L)
    assert need < _scratch_bytes(H, Nq, n, L)
    scratch = torch.full((need,), 0x7F, dtype=torch.uint8, device=DEV)      # as floats: 3.4e38
    lens = torch.randint(0, n + 1, (Nq,), generator=torch.Generator().manual_seed(tiles), dtype=torch.int32)
    lens[-1] = n
    for ql in (None, lens):
        scratch.fill_(0x7F)
        out = _decode_parts(q, kd, vd, None if ql is None else ql.to(DEV), scratch)
        torch.cuda.synchronize()
        touched = (scratch[:need // (H * STATE) * H * STATE].view(-1, H * STATE) != 0x7F).any(1)
        assert touched[:parts].all() and not touched[parts:].any()
        khat, vhat = B.decode(kd), B.decode(vd)
        for h in (0, H - 1):
            for i in (0, Nq // 2, Nq - 1):
                seen = n if ql is None else int(lens[i])
                if seen == 0:
                    assert not out[h, i].any()
                    continue
                want = O.attention(bf16_bits(q[h, i:i + 1]), P.to_np_u16(khat[h, :seen]), P.to_np_u16(vhat[h, :seen]))
                ok, max_abs, worst = P.attn_tolerance_ok(P.to_np_u16(out[h, i:i + 1]), want)
                assert ok, (h, i, seen, max_abs, worst)
