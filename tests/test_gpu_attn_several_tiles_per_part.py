"""Divided attention whose parts have several tiles each, the last ones fewer: every kernel and stored format against the
oracle, the join of few and of many parts, with prefix lengths that end in the first, the second and the last round of
tiles."""
import pytest
import torch

from oracle import qvg_oracle as O
from paper_2602_02958_amd import binding as B
from paper_2602_02958_amd import synth
from paper_2602_02958_amd.configs import CONFIGS
from conftest import bf16_bits
import parity_util as P
from test_gpu_attn_integration import _filled_caches, _rope_table
from test_gpu_attn_parts import _scratch_bytes

pytestmark = pytest.mark.gpu
DEV = "cuda"
STATE = 66 * 512 * 4


def _check(H, Nq, L, n, parts, kc, vc, forms, rope=False):
    tiles = n // L * -(-L // 64) + -(-(n % L) // 64)
    assert _scratch_bytes(H, Nq, n, L) == parts * H * -(-Nq // 256) * STATE
    assert tiles > parts and tiles % parts != 0
    q = synth.queries(CONFIGS["cfg2_window21"], H, Nq, DEV)
    khat, vhat = B.decode(kc), B.decode(vc)
    lens = torch.randint(-2, n + 3, (Nq,), generator=torch.Generator().manual_seed(tiles), dtype=torch.int32)
    first, second, last = 64 * (parts // 2) + 7, 64 * (parts + parts // 3) + 1, n - 3
    for i, v in enumerate((first, second, last, 0)):
        lens[i * Nq // 4] = min(v, n)
    table = _rope_table(n).to(DEV)
    for ql, tab in ((None, None), (lens.to(DEV), None)) + (((None, table),) if rope else ()):
        got = [B.attn_decode(q, kc, vc, want_lse=True, n_kv=n, q_kv_len=ql, k_rope=tab, workspace=ws) for ws in forms]
        f32 = B.attn_decode(q, kc, vc, n_kv=n, q_kv_len=ql, k_rope=tab, f32_out=True)
        torch.cuda.synchronize()
        out, lse = got[0]
        assert all(torch.equal(o, out) and torch.equal(l, lse) for o, l in got)
        assert torch.equal(f32.to(torch.bfloat16), out)
        for h in (0, H - 1):
            kb, vb = P.to_np_u16(khat[h, :n]), P.to_np_u16(vhat[h, :n])
            if tab is not None:
                kb = O.rope_keys(kb, P.to_np_u16(table))
            for i in sorted({j * Nq // 4 for j in range(4)} | {Nq // 3, Nq - 1}):
                seen = n if ql is None else min(max(int(lens[i]), 0), n)
                if seen == 0:
                    assert not out[h, i].any() and lse[h, i] == -float("inf")
                    continue
                want, lse_w = O.attention(bf16_bits(q[h, i:i + 1]), kb[:seen], vb[:seen], want_lse=True)
                ok, max_abs, worst = P.attn_tolerance_ok(P.to_np_u16(out[h, i:i + 1]), want)
                assert ok, (h, i, seen, max_abs, worst)
                assert abs(float(lse[h, i]) - lse_w[0]) < 2e-3


@pytest.mark.parametrize("H,Nq,L,n,parts,T,Bg,S,bits,fmt,K", [
    (40, 1, 520, 1173, 6, 2, 64, 1, 2, B.SCALE_F16, 16),       # 21 tiles
    (40, 64, 520, 1173, 6, 3, 32, 1, 2, B.SCALE_F16, 64),      # staged kernel
    (36, 33, 516, 1100, 7, 2, 64, 1, 2, B.SCALE_F16, 16),      # general kernel, 20 tiles
    (30, 256, 40, 753, 5, 2, 64, 1, 2, B.SCALE_F16, 16),       # chunks of one short tile, 19
    (32, 70, 520, 1100, 7, 1, 16, 4, 2, B.SCALE_E4M3, 64),     # four smoothing stages, 19
    (24, 300, 520, 1033, 5, 1, 64, 1, 4, B.SCALE_E4M3, 64),    # two query blocks, 4-bit levels, 18
    (12, 520, 200, 1333, 6, 5, 128, 1, 2, B.SCALE_F16, 16),    # three query blocks: a tile workspace by default, 27
    (24, 300, 136, 816, 5, 1, 64, 1, 2, B.SCALE_E4M3, 300),    # 16-bit ids, 18
])
def test_formats(H, Nq, L, n, parts, T, Bg, S, bits, fmt, K):
    kc, vc = _filled_caches(H, L, -(-n // L), n, K, Bg, T, S=S, bits=bits, fmt=fmt)
    # whatever is chosen; lent, too small: one kernel; lent
    forms = [None, torch.empty(0, dtype=torch.uint8, device=DEV), B.attn_workspace(H, Nq, L, 1, DEV)]
    _check(H, Nq, L, n, parts, kc, vc, forms, rope=True)


@pytest.mark.parametrize("H,Nq,tiles,parts", [(8, 64, 33, 17), (8, 64, 65, 22), (1, 40, 299, 150), (2, 300, 131, 44), (9, 64, 65, 16)])
def test_joins(H, Nq, tiles, parts):
    L, n = 1024, tiles * 64 - 5
    kc, vc = _filled_caches(H, L, -(-n // L), n, 16, 64, 1)
    _check(H, Nq, L, n, parts, kc, vc, [None])
