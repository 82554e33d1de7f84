"""The C entry points that take no scratch (qvg_attn_decode_ex, _causal, _f32) walk the whole cache with one
workgroup per query block, over many tiles too; attn_decode takes that form when torch has no memory
for the parts.  Against the oracle, and with a tile workspace bit for bit."""
import numpy as np
import pytest
import torch

from oracle import qvg_oracle as O
from paper_2602_02958_amd import binding as B
from paper_2602_02958_amd import synth
from paper_2602_02958_amd.configs import CONFIGS
from conftest import bf16_bits
import parity_util as P
from test_gpu_attn_integration import _filled_caches, _rope_table, _check_against_oracle

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _call(entry, q, k, v, n_kv, rope=None, lens=None, ws=None):
    H, Nq, d = q.shape
    T, G = k.codes.shape[2], k.scales.shape[3]
    p = B.make_params(H, k.centroids.shape[-2], d // G, T, n_smooth_stages=k.n_smooth, bits=k.bits, scale_format=k.scale_format)
    out = torch.empty(H, Nq, d, dtype=torch.float32 if entry == "f32" else torch.bfloat16, device=DEV)
    lse = torch.empty(H, Nq, dtype=torch.float32, device=DEV)
    ptr = lambda t: None if t is None else t.data_ptr()
    args = [B.C.byref(p), Nq, ptr(q), n_kv, k.chunk_len, k.ids.shape[1]] + \
        [ptr(t) for c in (k, v) for t in (c.centroids, c.ids, c.codes, c.scales)] + [ptr(rope)]
    tail = [d ** -0.5, ptr(out), ptr(lse)]
    lent = [ptr(ws), 0 if ws is None else ws.numel()]
    s = [torch.cuda.current_stream().cuda_stream]
    if entry == "ex":
        st = B.lib().qvg_attn_decode_ex(*args, *tail, *lent, *s)
    elif entry == "causal":
        st = B.lib().qvg_attn_decode_causal(*args, ptr(lens), *tail, *lent, *s)
    else:
        st = B.lib().qvg_attn_decode_f32(*args, ptr(lens), *tail, *s)
    assert st == 0
    return out, lse


@pytest.mark.parametrize("L,T,Bg,S,bits,fmt,K", [
    (520, 3, 32, 1, 2, B.SCALE_F16, 64),      # staged kernel
    (516, 2, 64, 1, 2, B.SCALE_F16, 16),      # general kernel
    (1040, 1, 16, 4, 2, B.SCALE_E4M3, 64),    # general kernel, four smoothing stages
    (40, 2, 64, 1, 2, B.SCALE_F16, 16),       # chunks of one short tile
])
@pytest.mark.parametrize("Nq", [33, 300, 600])
def test_undivided_calls_over_many_tiles(L, T, Bg, S, bits, fmt, K, Nq):
    H, n = 2, 2333                                         # 37 tiles and more
    kc, vc = _filled_caches(H, L, -(-n // L), n, K, Bg, T, S=S, bits=bits, fmt=fmt)
    q = synth.queries(CONFIGS["cfg2_window21"], H, Nq, DEV)
    rope = _rope_table(n).to(DEV)
    khat, vhat = B.decode(kc), B.decode(vc)
    lens = torch.arange(Nq, dtype=torch.int32, device=DEV) * 7 % (n + 1)
    lens[0], lens[1] = n, 65
    ws = B.attn_workspace(H, Nq, L, 2, DEV)
    for table in (None, rope):
        out, lse = _call("ex", q, kc, vc, n, rope=table)
        f32, lse32 = _call("f32", q, kc, vc, n, rope=table)
        slab, lses = _call("ex", q, kc, vc, n, rope=table, ws=ws)
        qout, qlse = _call("causal", q, kc, vc, n, rope=table, lens=lens)
        qslab, qlses = _call("causal", q, kc, vc, n, rope=table, lens=lens, ws=ws)
        torch.cuda.synchronize()
        assert torch.equal(out, slab) and torch.equal(lse, lses)
        assert torch.equal(f32.to(torch.bfloat16), out) and torch.equal(lse32, lse)
        assert torch.equal(qout, qslab) and torch.equal(qlse, qlses)
        assert torch.equal(qout[:, 0], out[:, 0])          # its prefix is the whole cache
        for h in range(H):
            kb, vb = P.to_np_u16(khat[h, :n]), P.to_np_u16(vhat[h, :n])
            if table is not None:
                kb = O.rope_keys(kb, rope.cpu().view(torch.int16).numpy().view(np.uint16))
            _check_against_oracle(q, out, lse, kb, vb, h)
            for i in (1, Nq // 2, Nq - 1):
                m = int(lens[i])
                if m == 0:
                    continue
                want, lse_w = O.attention(bf16_bits(q[h, i:i + 1]), kb[:m], vb[:m], want_lse=True)
                ok, max_abs, worst = P.attn_tolerance_ok(P.to_np_u16(qout[h, i:i + 1]), want)
                assert ok, (h, i, m, max_abs, worst)
                assert abs(float(qlse[h, i]) - lse_w[0]) < 2e-3
