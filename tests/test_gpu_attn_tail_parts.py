"""More than 256 query blocks: the blocks of the last, partly filled round are divided, the others taken whole.  Sizes at the
rule's edges (two blocks left over and 128, 129 of them, 15 and 16 tiles, a block of one query); equal bits with a tile
workspace (one slab or several), without one and in fp32; the whole blocks have the bits of the undivided call."""
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
L = 520


@pytest.mark.parametrize("H,Nq,n,tail,parts", [
    (43, 1290, 2075, 2, 9),           # 258 blocks, 36 tiles; a last block of ten queries
    (37, 1537, 2080, 3, 9),           # 259, a last block of one
    (32, 3000, 2080, 128, 2),
    (35, 2816, 2080, 0, 1),           # 129 left over: nothing is divided
    (43, 1290, 905, 2, 4),            # 16 tiles
    (43, 1290, 904, 0, 1),            # 15
])
def test_the_last_round_is_divided(H, Nq, n, tail, parts):
    chunks = -(-n // L)
    kc, vc = _filled_caches(H, L, chunks, n, 16, 64, 1)
    blocks, state = -(-Nq // 256), 66 * 512 * 4
    need = _scratch_bytes(H, Nq, n, L)
    assert need == tail * parts * state
    q = synth.queries(CONFIGS["cfg2_window21"], H, Nq, DEV)
    none = torch.empty(0, dtype=torch.uint8, device=DEV)
    out, lse = B.attn_decode(q, kc, vc, want_lse=True, n_kv=n, workspace=none)
    for k in (1, 3, chunks):
        ws = B.attn_workspace(H, Nq, L, k, DEV)
        lent, lse_lent = B.attn_decode(q, kc, vc, want_lse=True, n_kv=n, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(out, lent) and torch.equal(lse, lse_lent), k
    assert torch.equal(B.attn_decode(q, kc, vc, n_kv=n, f32_out=True).to(torch.bfloat16), out)
    kd, vd = (B.Encoded(c.centroids, c.ids[:, :n].contiguous(), c.codes[:, :n].contiguous(), c.scales[:, :n].contiguous(),
                        c.chunk_len) for c in (kc, vc))
    one = _decode_parts(q, kd, vd, None, None)
    scratch = torch.full((max(need, 16),), 0x7F, dtype=torch.uint8, device=DEV)
    assert torch.equal(_decode_parts(q, kd, vd, None, scratch), out)
    torch.cuda.synchronize()
    if tail:
        assert (scratch.view(parts * tail, -1) != 0x7F).any(1).all()
    whole = H * blocks - tail
    for h in range(H):
        rows = min(max(whole - h * blocks, 0) * 256, Nq)
        assert torch.equal(out[h, :rows], one[h, :rows])
    # one output's rounding and the order of the sums apart
    assert (out.float() - one.float()).abs().max() <= 2 ** -8 * one.float().abs().max() + 2e-3
    khat, vhat = B.decode(kc), B.decode(vc)
    for h in (0, H - 1):
        kb, vb = P.to_np_u16(khat[h, :n]), P.to_np_u16(vhat[h, :n])
        for i in (0, Nq - 257, Nq - 1):
            want, lse_w = O.attention(bf16_bits(q[h, i:i + 1]), kb, vb, want_lse=True)
            ok, max_abs, worst = P.attn_tolerance_ok(P.to_np_u16(out[h, i:i + 1]), want)
            assert ok, (h, i, max_abs, worst)
            assert abs(float(lse[h, i]) - lse_w[0]) < 2e-3


@pytest.mark.parametrize("lengths", [False, True])
def test_scratch_that_is_not_aligned_is_ignored(lengths):
    """Calls of more than 128 blocks ran undivided with any scratch before they were divided, and still do."""
    H, Nq, n = (43, 768, 12480) if lengths else (43, 1290, 905)
    kc, vc = _filled_caches(H, L, -(-n // L), n, 16, 64, 1)
    kd, vd = (B.Encoded(c.centroids, c.ids[:, :n].contiguous(), c.codes[:, :n].contiguous(), c.scales[:, :n].contiguous(),
                        c.chunk_len) for c in (kc, vc))
    q = synth.queries(CONFIGS["cfg2_window21"], H, Nq, DEV)
    lens = torch.arange(1, Nq + 1, dtype=torch.int32, device=DEV) * (n // Nq) if lengths else None
    scratch = torch.full((110 << 20,), 0x7F, dtype=torch.uint8, device=DEV)
    out = _decode_parts(q, kd, vd, lens, scratch[4:])
    torch.cuda.synchronize()
    assert torch.equal(out, _decode_parts(q, kd, vd, lens, None)) and bool((scratch == 0x7F).all())
