"""Few query blocks in many parts: the join whose wavefronts share the parts of 32 queries, on both sides of the rules that choose it,
with prefix lengths that end in the first part, between the wavefronts' shares and nowhere."""
import pytest
import torch

from oracle import qvg_oracle as O
from paper_2602_02958_amd import binding as B
from paper_2602_02958_amd import synth
from paper_2602_02958_amd.configs import CONFIGS
from conftest import bf16_bits
import parity_util as P
from test_gpu_attn_integration import _filled_caches
from test_gpu_attn_parts import _scratch_bytes

pytestmark = pytest.mark.gpu
DEV = "cuda"
STATE = 66 * 512 * 4


@pytest.mark.parametrize("H,Nq,tiles,parts", [
    (1, 1, 4, 4),            # the fewest tiles that are divided (the other join)
    (1, 64, 7, 7),           # one part too few for it
    (1, 64, 8, 8),           # one part to a wavefront
    (1, 33, 9, 9),           # a second wavefront of queries with one of them
    (2, 300, 24, 24),        # two blocks of queries per head, the second with 44
    (8, 64, 32, 32),         # the most blocks
    (9, 64, 28, 28),         # one more (the other join)
    (1, 40, 65, 65),         # more than eight parts to a wavefront
    (1, 40, 256, 256),       # as many as the chip holds, a tile each
])
def test_split_join(H, Nq, tiles, parts):
    L = 1024
    n = tiles * 64 - 5
    kc, vc = _filled_caches(H, L, -(-n // L), n, 16, 64, 1)
    assert _scratch_bytes(H, Nq, n, L) == parts * H * -(-Nq // 256) * STATE
    q = synth.queries(CONFIGS["cfg2_window21"], H, Nq, DEV)
    g = torch.Generator().manual_seed(tiles)
    lens = torch.randint(0, n + 1, (Nq,), generator=g, dtype=torch.int32)
    lens[-1], lens[0] = 0, min(n, 64 * 7 + 1)
    khat, vhat = B.decode(kc), B.decode(vc)
    for ql in (None, lens.to(DEV)):
        out, lse = B.attn_decode(q, kc, vc, want_lse=True, n_kv=n, q_kv_len=ql)
        f32 = B.attn_decode(q, kc, vc, n_kv=n, q_kv_len=ql, f32_out=True)
        torch.cuda.synchronize()
        assert torch.equal(f32.to(torch.bfloat16), out)
        for h in sorted({0, H - 1}):
            kb, vb = P.to_np_u16(khat[h, :n]), P.to_np_u16(vhat[h, :n])
            for i in sorted({0, Nq // 2, max(Nq - 2, 0), Nq - 1}):
                seen = n if ql is None else int(lens[i])
                if seen == 0:
                    assert not out[h, i].any() and lse[h, i] == -float("inf")
                    continue
                want, lse_w = O.attention(bf16_bits(q[h, i:i + 1]), kb[:seen], vb[:seen], want_lse=True)
                ok, max_abs, worst = P.attn_tolerance_ok(P.to_np_u16(out[h, i:i + 1]), want)
                assert ok, (h, i, seen, max_abs, worst)
                assert abs(float(lse[h, i]) - lse_w[0]) < 2e-3
