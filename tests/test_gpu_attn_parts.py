"""Attention of few query blocks: the cache's tiles are dealt to several workgroups per query block and
their partial results joined.  Against the oracle at the existing bound, with chunks of one tile and parts that lie behind
every prefix (most with a tile to a part; several tiles to a part: test_gpu_attn_several_tiles_per_part.py);
equal bits with a tile workspace, without one and in the fp32 result; NaN stays in its row."""
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


def _scratch_bytes(H, Nq, n_kv, L):
    need = B.C.c_size_t()
    p = B.make_params(H, 16, 64, 1)
    assert B.lib().qvg_attn_scratch_bytes(B.C.byref(p), Nq, n_kv, L, B.C.byref(need)) == 0
    return need.value


@pytest.mark.parametrize("H,Nq,L,chunks,n_kv,T,Bg,S,bits,fmt,K", [
    (1, 1, 520, 1, 511, 2, 64, 1, 2, B.SCALE_F16, 16),       # eight tiles, eight parts, the last tile one short
    (1, 64, 520, 3, 1173, 3, 32, 1, 2, B.SCALE_F16, 64),     # staged kernel, chunks of 8 tiles + 8 tokens
    (2, 33, 516, 2, 1000, 2, 64, 1, 2, B.SCALE_F16, 16),     # general kernel
    (3, 256, 40, 20, 793, 2, 64, 1, 2, B.SCALE_F16, 16),     # chunks of one short tile
    (2, 70, 520, 2, 1040, 1, 16, 4, 2, B.SCALE_E4M3, 64),    # four smoothing stages
    (1, 300, 520, 2, 1033, 1, 64, 1, 4, B.SCALE_E4M3, 64),   # two query blocks
    (1, 520, 200, 5, 933, 5, 128, 1, 2, B.SCALE_F16, 16),    # three query blocks: a tile workspace by default
    (2, 300, 136, 6, 816, 1, 64, 1, 2, B.SCALE_E4M3, 300),   # 16-bit ids
])
def test_parts_against_the_oracle(H, Nq, L, chunks, n_kv, T, Bg, S, bits, fmt, K):
    assert _scratch_bytes(H, Nq, n_kv, L) > 0
    kc, vc = _filled_caches(H, L, chunks, min(n_kv + 5, L * chunks), K, Bg, T, S=S, bits=bits, fmt=fmt)
    q = synth.queries(CONFIGS["cfg2_window21"], H, Nq, DEV)
    khat, vhat = B.decode(kc), B.decode(vc)
    g = torch.Generator().manual_seed(3)
    lens = torch.randint(-2, n_kv + 3, (Nq,), generator=g)
    lens[:min(Nq, 34)] = 65                          # a wavefront (and a query block of 33) that ends in the second tile
    lens[0] = 0
    none = torch.empty(0, dtype=torch.uint8, device=DEV)             # lent, too small: one kernel
    rope = _rope_table(n_kv).to(DEV)
    for ql, table in ((None, None), (lens.to(torch.int32).to(DEV), None), (None, rope)):
        kw = dict(n_kv=n_kv, q_kv_len=ql, k_rope=table)
        out, lse = B.attn_decode(q, kc, vc, want_lse=True, **kw)
        one, lse1 = B.attn_decode(q, kc, vc, want_lse=True, workspace=none, **kw)
        ws = B.attn_workspace(H, Nq, L, 1, DEV)
        slab, lses = B.attn_decode(q, kc, vc, want_lse=True, workspace=ws, **kw)
        f32 = B.attn_decode(q, kc, vc, f32_out=True, **kw)
        torch.cuda.synchronize()
        assert torch.equal(out, one) and torch.equal(lse, lse1)
        assert torch.equal(out, slab) and torch.equal(lse, lses)
        assert torch.equal(f32.to(torch.bfloat16), out)
        eff = (lens.clamp(0, n_kv) if ql is not None else torch.full((Nq,), n_kv)).numpy()
        for h in range(H):
            kb, vb = P.to_np_u16(khat[h, :n_kv]), P.to_np_u16(vhat[h, :n_kv])
            if table is not None:
                kb = O.rope_keys(kb, rope.cpu().view(torch.int16).numpy().view(np.uint16))
            if ql is None:
                _check_against_oracle(q, out, lse, kb, vb, h)
                continue
            for i in sorted({0, 1 % Nq, 33 % Nq, Nq // 2, Nq - 1, int(eff.argmax()), int(eff.argmin())}):
                n = int(eff[i])
                if n == 0:
                    assert not out[h, i].any() and lse[h, i] == -float("inf")
                    continue
                want, lse_w = O.attention(bf16_bits(q[h, i:i + 1]), kb[:n], vb[:n], want_lse=True)
                ok, max_abs, worst = P.attn_tolerance_ok(P.to_np_u16(out[h, i:i + 1]), want)
                assert ok, (h, i, n, max_abs, worst)
                assert abs(float(lse[h, i]) - lse_w[0]) < 2e-3


def test_parts_keep_a_nan_query_in_its_row():
    H, Nq, L, n_kv = 2, 70, 520, 1000
    kc, vc = _filled_caches(H, L, 2, n_kv, 16, 64, 2)
    q = synth.queries(CONFIGS["cfg2_window21"], H, Nq, DEV)
    clean = B.attn_decode(q, kc, vc, n_kv=n_kv)
    q[1, 5, 17] = float("nan")
    out = B.attn_decode(q, kc, vc, n_kv=n_kv)
    torch.cuda.synchronize()
    assert out[1, 5].isnan().all()
    out[1, 5] = clean[1, 5]
    assert torch.equal(out, clean)


def _constant_cache(H, n, L, ids, table):
    """A cache whose tokens decode to the constant rows `table[id]` (all scales zero)."""
    e = B.alloc_cache(H, n, L, len(table), 64, 1, 128, DEV)
    e.centroids.copy_(torch.tensor(table, device=DEV).to(torch.bfloat16)[None, None, :, None].expand_as(e.centroids))
    e.ids.copy_(ids.to(DEV, torch.uint8)[None].expand_as(e.ids))
    e.codes.zero_()
    e.scales.zero_()
    return e


@pytest.mark.parametrize("Nq,L,lend", [(64, 520, False), (33, 516, False), (300, 520, True), (300, 520, False)])
@pytest.mark.parametrize("seen", [0, 100, 999])
def test_scores_that_overflow_weigh_nothing(Nq, L, lend, seen):
    """Finite queries and keys whose product is below fp32's range: those tokens have weight zero, also
    where every token of a part (or of the first tile) is one of them.  Token `seen` is the only other."""
    H, n = 2, 1000
    ids = torch.zeros(n, dtype=torch.int64)
    ids[seen] = 1
    k = _constant_cache(H, n, L, ids, [-2e19, 0.0])
    v = _constant_cache(H, n, L, ids, [-3.0, 1.5])
    assert _scratch_bytes(H, Nq, n, L) > 0
    q = torch.full((H, Nq, 128), 2e19, dtype=torch.bfloat16, device=DEV)
    ws = B.attn_workspace(H, Nq, L, 1, DEV) if lend else torch.empty(0, dtype=torch.uint8, device=DEV)
    lens = torch.full((Nq,), n, dtype=torch.int32, device=DEV)
    lens[::2] = seen + 1
    for ql in (None, lens):
        out, lse = B.attn_decode(q, k, v, want_lse=True, workspace=ws, q_kv_len=ql)
        torch.cuda.synchronize()
        assert (out == 1.5).all(), (ql is None, out.flatten()[:4])
        assert (lse == 0.0).all()                                  # one token of score 0


def _decode_parts(q, k, v, lens, scratch, ws=None):
    """qvg_attn_decode_parts (or, without scratch, the undivided call) on caches of one format."""
    H, Nq, d = q.shape
    out = torch.empty_like(q)
    T, G = k.codes.shape[2], k.scales.shape[3]
    p = B.make_params(H, k.centroids.shape[-2], d // G, T, n_smooth_stages=k.n_smooth, bits=k.bits, scale_format=k.scale_format)
    ptr = lambda t: None if t is None else t.data_ptr()
    st = B.lib().qvg_attn_decode_parts(
        B.C.byref(p), Nq, ptr(q), k.ids.shape[1], k.chunk_len, 0, ptr(k.centroids), ptr(k.ids), ptr(k.codes), ptr(k.scales),
        ptr(v.centroids), ptr(v.ids), ptr(v.codes), ptr(v.scales), None, ptr(lens), d ** -0.5, ptr(out), None, None,
        ptr(ws), 0 if ws is None else ws.numel(), ptr(scratch), 0 if scratch is None else scratch.numel(),
        torch.cuda.current_stream().cuda_stream)
    assert st == 0
    return out


@pytest.mark.parametrize("Nq,L,lend", [(64, 520, False), (33, 516, False), (300, 520, True)])
@pytest.mark.parametrize("longest", [0, 1, 65, 700])
def test_parts_behind_every_prefix_leave_no_state(Nq, L, lend, longest):
    """A call of short prefixes over a long cache costs what its prefixes cost: the parts that lie behind
    the longest one write no state, and the join does not read it."""
    H, n = 2, 4160
    kc, vc = _filled_caches(H, L, -(-n // L), n, 16, 64, 2)
    kc, vc = (B.Encoded(c.centroids, c.ids[:, :n].contiguous(), c.codes[:, :n].contiguous(), c.scales[:, :n].contiguous(),
                        c.chunk_len) for c in (kc, vc))
    q = synth.queries(CONFIGS["cfg2_window21"], H, Nq, DEV)
    need = _scratch_bytes(H, Nq, n, L)
    state = 66 * 512 * 4                                   # of a query block (256 queries)
    blocks = H * -(-Nq // 256)
    parts = need // (blocks * state)
    assert parts > 12
    scratch = torch.full((need,), 0x7F, dtype=torch.uint8, device=DEV)      # as floats: 3.4e38
    lens = torch.full((Nq,), longest, dtype=torch.int32, device=DEV)
    lens[::3] = min(longest, 2)
    ws = B.attn_workspace(H, Nq, L, 2, DEV) if lend else None
    out = _decode_parts(q, kc, vc, lens, scratch, ws)
    one = _decode_parts(q, kc, vc, lens, None, ws)
    torch.cuda.synchronize()
    full, rest = divmod(longest, L)
    tiles = full * -(-L // 64) + -(-rest // 64)
    touched = (scratch.view(parts, blocks * state) != 0x7F).any(1)
    assert touched[:tiles].all() and not touched[max(tiles, 1):].any()
    if longest == 0:
        assert not out.any()
    # one output's rounding and the order of the sums apart
    assert (out.float() - one.float()).abs().max() <= 2 ** -8 * one.float().abs().max() + 2e-3


@pytest.mark.parametrize("H,tiles,parts", [(16, 63, 15), (16, 64, 16), (17, 64, 15)])
def test_join_of_few_and_many_blocks_and_parts(H, tiles, parts):
    """Each side of the rules that choose the join's form; with lengths, some of which only the first parts see."""
    L, Nq = 1024, 200
    n = tiles * 64
    kc, vc = _filled_caches(H, L, 4, n, 16, 64, 1)
    assert _scratch_bytes(H, Nq, n, L) == parts * H * 66 * 512 * 4
    q = synth.queries(CONFIGS["cfg2_window21"], H, Nq, DEV)
    lens = torch.full((Nq,), n, dtype=torch.int32)
    lens[:32], lens[32:64], lens[64], lens[65] = 130, 65 * parts, 0, 1
    khat, vhat = B.decode(kc), B.decode(vc)
    for ql in (None, lens.to(DEV)):
        out, lse = B.attn_decode(q, kc, vc, want_lse=True, n_kv=n, q_kv_len=ql)
        f32 = B.attn_decode(q, kc, vc, n_kv=n, q_kv_len=ql, f32_out=True)
        torch.cuda.synchronize()
        assert torch.equal(f32.to(torch.bfloat16), out)
        for h in (0, H - 1):
            kb, vb = P.to_np_u16(khat[h, :n]), P.to_np_u16(vhat[h, :n])
            for i in (0, 40, 64, 65, 199):
                seen = n if ql is None else int(lens[i])
                if seen == 0:
                    assert not out[h, i].any() and lse[h, i] == -float("inf")
                    continue
                want, lse_w = O.attention(bf16_bits(q[h, i:i + 1]), kb[:seen], vb[:seen], want_lse=True)
                ok, max_abs, worst = P.attn_tolerance_ok(P.to_np_u16(out[h, i:i + 1]), want)
                assert ok, (h, i, seen, max_abs, worst)
                assert abs(float(lse[h, i]) - lse_w[0]) < 2e-3
