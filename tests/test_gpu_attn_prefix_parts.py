"""A prefix length per query and more than 128 query blocks: blocks of long prefixes are divided, the others taken whole.
Sizes at the rule's edges: prefixes around 96 and 144 tiles (two and three parts), a first query that sees as much as the
others, a last block of a few queries; equal bits with a tile workspace (one slab or several), without one and in fp32."""
import pytest
import torch

from oracle import qvg_oracle as O
from paper_2602_02958_amd import binding as B
from paper_2602_02958_amd import synth
from paper_2602_02958_amd.configs import CONFIGS
from conftest import bf16_bits
import parity_util as P
from test_gpu_attn_integration import _filled_caches
from test_gpu_attn_parts import _decode_parts

pytestmark = pytest.mark.gpu
DEV = "cuda"
H, L = 43, 1000                                        # chunks of 16 tiles


def _bytes(Nq, n):
    need = B.C.c_size_t()
    assert B.lib().qvg_attn_scratch_bytes_causal(B.C.byref(B.make_params(H, 16, 64, 1)), Nq, n, L, B.C.byref(need)) == 0
    return need.value


@pytest.fixture(scope="module")
def caches():
    return _filled_caches(H, L, 13, 12500, 16, 64, 1)


@pytest.mark.parametrize("Nq,n,prefixes,divided", [
    (516, 12500, (0, 5935, 12500), (1, 1, 3)),           # 95 tiles, 200; a last block of four queries
    (700, 12500, (1, 5999, 8901), (1, 2, 2)),            # 96 tiles and 143
    (769, 12500, (64, 9000, 40, 12500), (1, 3, 1, 3)),   # 144 tiles; lengths not in order; a last block of one query
    (520, 12500, (12000, 12500, 12500), (1, 1, 1)),      # all about the same: nothing is divided
    (516, 11990, (0, 5999, 11990), None),                # 192 tiles: the shortest cache that is divided
    (516, 11900, (0, 5999, 11900), (1, 1, 1)),           # 191
])
def test_blocks_of_long_prefixes_are_divided(caches, Nq, n, prefixes, divided):
    kc, vc = (B.Encoded(c.centroids, c.ids, c.codes, c.scales, c.chunk_len) for c in caches)
    blocks = -(-Nq // 256)
    state = 66 * 512 * 4 * H * blocks
    assert _bytes(Nq, n) == (0 if n == 11900 else 3 * state)
    q = synth.queries(CONFIGS["cfg2_window21"], H, Nq, DEV)
    lens = torch.cat([torch.full((256,), v, dtype=torch.int32) for v in prefixes])[:Nq]
    lens[3::7] -= torch.arange(len(lens[3::7]), dtype=torch.int32) % 40
    lens = lens.to(DEV)
    out, lse = B.attn_decode(q, kc, vc, want_lse=True, n_kv=n, q_kv_len=lens)
    for chunks in (1, 5, 13):
        ws = B.attn_workspace(H, Nq, L, chunks, DEV)
        lent, lse_lent = B.attn_decode(q, kc, vc, want_lse=True, n_kv=n, q_kv_len=lens, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(out, lent) and torch.equal(lse, lse_lent), chunks
    f32 = B.attn_decode(q, kc, vc, n_kv=n, q_kv_len=lens, f32_out=True)
    assert torch.equal(f32.to(torch.bfloat16), out)
    if n == 12500 and divided:
        # the call without scratch: equal bits where the block is taken whole, one output's rounding and the order of the
        # sums elsewhere
        kd, vd = (B.Encoded(c.centroids[:, :13].contiguous(), c.ids[:, :n].contiguous(), c.codes[:, :n].contiguous(),
                            c.scales[:, :n].contiguous(), c.chunk_len) for c in (kc, vc))
        one = _decode_parts(q, kd, vd, lens, None)
        scratch = torch.full((3 * state,), 0x7F, dtype=torch.uint8, device=DEV)
        assert torch.equal(_decode_parts(q, kd, vd, lens, scratch), out)
        torch.cuda.synchronize()
        touched = (scratch.view(3, H, blocks, -1) != 0x7F).any(-1).all(1).cpu()
        for b in range(blocks):
            assert int(touched[:, b].sum()) == (0 if divided[b] == 1 else divided[b])
            rows = slice(256 * b, min(Nq, 256 * b + 256))
            if divided[b] == 1:
                assert torch.equal(out[:, rows], one[:, rows])
        assert (out.float() - one.float()).abs().max() <= 2 ** -8 * one.float().abs().max() + 2e-3
    khat, vhat = B.decode(kc), B.decode(vc)
    for h in (0, H - 1):
        kb, vb = P.to_np_u16(khat[h, :n]), P.to_np_u16(vhat[h, :n])
        for i in (1, 255, 300, Nq - 1):
            seen = max(int(lens[i]), 0)
            if seen == 0:
                assert not out[h, i].any() and lse[h, i] == -float("inf")
                continue
            want, lse_w = O.attention(bf16_bits(q[h, i:i + 1]), kb[:seen], vb[:seen], want_lse=True)
            ok, max_abs, worst = P.attn_tolerance_ok(P.to_np_u16(out[h, i:i + 1]), want)
            assert ok, (h, i, seen, max_abs, worst)
            assert abs(float(lse[h, i]) - lse_w[0]) < 2e-3


def _lengths_call(caches, q, lens, n):
    """The result, and which parts' states the divided call left: [3, H, blocks]."""
    kd, vd = (B.Encoded(c.centroids[:, :13].contiguous(), c.ids[:, :n].contiguous(), c.codes[:, :n].contiguous(),
                        c.scales[:, :n].contiguous(), c.chunk_len) for c in caches)
    blocks = q.shape[1] // 256
    scratch = torch.full((3 * 66 * 512 * 4 * H * blocks,), 0x7F, dtype=torch.uint8, device=DEV)
    out = _decode_parts(q, kd, vd, lens.to(DEV), scratch)
    torch.cuda.synchronize()
    return out, (scratch.view(3, H, blocks, -1) != 0x7F).any(-1).cpu(), _decode_parts(q, kd, vd, lens.to(DEV), None)


def test_lengths_that_fall_are_divided_as_those_that_rise(caches):
    n, blocks = 12500, 3
    q = synth.queries(CONFIGS["cfg2_window21"], H, 256 * blocks, DEV)
    lens = torch.tensor([40, 5935, 12500], dtype=torch.int32)[:, None] - torch.arange(256, dtype=torch.int32) % 40
    out, touched, _ = _lengths_call(caches, q, lens.flatten(), n)
    assert touched.all(1).sum(0).tolist() == [0, 0, 3]
    fell, touched, _ = _lengths_call(caches, q.view(H, blocks, 256, 128).flip(1).reshape(q.shape).contiguous(), lens.flip(0).flatten(), n)
    assert touched.all(1).sum(0).tolist() == [3, 0, 0]
    assert torch.equal(fell.view(H, blocks, 256, 128).flip(1).reshape(q.shape), out)


@pytest.mark.parametrize("first,last", [(12500, 12500), (12500, 11000), (10940, 12500)])
def test_lengths_about_the_same_are_not_divided(caches, first, last):
    q = synth.queries(CONFIGS["cfg2_window21"], H, 768, DEV)
    lens = torch.full((768,), 12500, dtype=torch.int32)
    lens[:256], lens[-1] = first, last
    out, touched, one = _lengths_call(caches, q, lens, 12500)
    assert not touched.any() and torch.equal(out, one)
