"""The encoder that runs all Lloyd iterations in one launch, at the sizes where its division of the work has edges:
blocks of 256 tokens, more workgroups than blocks, more than 64 rows per workgroup, lists summed by a wavefront and by a
workgroup (with sums that depend on the order), 16-bit ids, several stages; and the same calls done by fewer workgroups
than a unit has, down to one.  Stored arrays against the oracle, bit for bit."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import qvg_oracle as O
from paper_2602_02958_amd import binding as B
from paper_2602_02958_amd import synth
from conftest import bf16_bits

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _inputs(H, N, K, S, seed, wide=False):
    g = torch.Generator().manual_seed(seed)
    centres = torch.randn(H, 24, 128, generator=g)
    pick = torch.randint(0, 24, (H, N), generator=g)
    pick[:, N // 3:] = torch.where(torch.rand(H, N - N // 3, generator=g) < 0.6, 3, pick[:, N // 3:])       # one cluster with most tokens
    x = torch.gather(centres, 1, pick[:, :, None].expand(-1, -1, 128)) + 0.3 * torch.randn(H, N, 128, generator=g)
    if wide:                                       # a channel whose sums round in fp64, so that the order matters
        x[:, ::4, 0] *= 1.0e18
        x[:, 2::4, 0] *= 1.0e-9
    x = x.to(torch.bfloat16)
    inits, r = [], x
    for s in range(S):
        inits.append(synth.cold_start_centroids(r, K, seed=seed + s))
        r = (r.float() - inits[-1].float().mean(1, keepdim=True)).to(torch.bfloat16)
    return x, torch.stack(inits, 1) if S > 1 else inits[0]


def _oracle(x, init, K, Bg, T, I, S, bits, fp8, units):
    return O.encode_batch(bf16_bits(x[units]), bf16_bits(init[units]), K, Bg, T, I, S=S, bits=bits, scale_fmt=int(fp8))


def _bytes(enc, units):
    c = enc.centroids[units].cpu().view(torch.uint8).numpy()
    return c, enc.ids[units].cpu().numpy(), enc.codes[units].cpu().numpy(), enc.scales[units].cpu().view(torch.uint8).numpy()


def _check(enc, ref, units):
    c, ids, codes, scales = _bytes(enc, units)
    assert np.array_equal(c.ravel(), np.ascontiguousarray(ref["cent"]).view(np.uint8).ravel()), "centroids"
    assert np.array_equal(ids.ravel().astype(np.int64) & 0xffff, np.moveaxis(np.asarray(ref["ids"]), 1, 2).ravel().astype(np.int64)), "ids"         # [H][S][N] there
    assert np.array_equal(codes.ravel(), np.asarray(ref["codes"]).view(np.uint8).ravel()), "codes"
    if enc.scale_format == B.SCALE_F16:
        scales = scales.view(np.uint16)
    assert np.array_equal(scales.ravel().astype(np.int64), np.asarray(ref["scales"]).ravel().astype(np.int64)), "scales"


# H, N, K, S, I, T, B, bits, E4M3, wide range
SHAPES = [
    (1, 1, 1, 1, 1, 1, 64, 2, False, False),
    (3, 40, 1, 1, 2, 2, 64, 2, False, False),
    (1, 256, 64, 1, 3, 1, 64, 2, False, False),
    (2, 257, 17, 1, 3, 4, 64, 2, False, True),
    (9, 2048, 52, 1, 2, 3, 32, 2, False, False),        # eight blocks, the most of a small launch
    (2, 2047, 256, 1, 3, 1, 16, 2, True, True),
    (10, 300, 256, 1, 2, 1, 64, 4, True, False),        # more workgroups than blocks
    (40, 1536, 512, 1, 1, 1, 64, 2, False, False),      # 86 rows per workgroup, 16-bit ids
    (24, 5121, 16, 1, 2, 2, 64, 2, False, True),        # 21 blocks; the longest lists
    (16, 6144, 96, 1, 1, 5, 128, 2, False, False),      # the most blocks
    (5, 700, 256, 4, 2, 1, 16, 2, True, False),         # four stages
    (3, 600, 300, 2, 2, 2, 64, 2, False, True),         # two, 16-bit ids
]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(str(v) for v in s))
def test_one_launch_encode_equals_the_oracle(shape):
    H, N, K, S, I, T, Bg, bits, fp8, wide = shape
    x, init = _inputs(H, N, K, S, 7 * N + K, wide)
    enc = B.encode_chunk(x.to(DEV), init.to(DEV), Bg, T, I, bits=bits, scale_format=B.SCALE_E4M3 if fp8 else B.SCALE_F16)
    torch.cuda.synchronize()
    units = sorted({0, H // 2, H - 1})
    _check(enc, _oracle(x, init, K, Bg, T, I, S, bits, fp8, units), units)


@pytest.mark.parametrize("shape", [s for s in SHAPES if s[1] > 256 and s[1] < 3000], ids=lambda s: "x".join(str(v) for v in s))
def test_units_given_up_by_their_workgroups_are_done_over(shape):
    H, N, K, S, I, T, Bg, bits, fp8, wide = shape
    x, init = _inputs(H, N, K, S, 7 * N + K, wide)
    x, init = x.to(DEV), init.to(DEV)
    fmt = B.SCALE_E4M3 if fp8 else B.SCALE_F16
    want = B.encode_chunk(x, init, Bg, T, I, bits=bits, scale_format=fmt)
    got = B.alloc_cache(H, N, N, K, Bg, T, device=DEV, n_smooth=S, bits=bits, scale_format=fmt)
    for t in (got.centroids, got.ids, got.codes, got.scales):
        t.view(torch.uint8).fill_(0xA5)
    p = B.make_params(H, K, Bg, T, I, bits=bits, n_smooth_stages=S, scale_format=fmt)
    ws = torch.full((B.workspace_bytes(p, B.ENTRY_ENCODE, N),), 0x5A, dtype=torch.uint8, device=DEV)
    ptr = lambda t: C.c_void_p(t.data_ptr())
    i64 = C.c_int64
    st = B.lib().qvg_encode_chunk_wait(C.byref(p), i64(N), ptr(x), i64(x.stride(0)), i64(128), ptr(init), ptr(got.centroids), i64(0),
                                       ptr(got.ids), ptr(got.codes), ptr(got.scales), i64(0), ptr(ws), C.c_size_t(ws.numel()),
                                       C.c_void_p(torch.cuda.current_stream().cuda_stream), C.c_uint32(0))
    torch.cuda.synchronize()
    assert st == 0
    # the units' words, behind the norms and the first table: the top bit says that a unit's team was closed
    r256 = lambda v: -(-v // 256) * 256
    norms = r256(H * (-(-K // 64) * 64) * 8)
    at = norms * S + r256(H * 4) + norms + r256(H * K * 256)
    words = ws[at:at + H * 256].view(torch.int32).reshape(H, 64)[:, 0]
    assert int((words < 0).sum()) > 0
    for a, b in zip(_bytes(got, slice(None)), _bytes(want, slice(None))):
        assert np.array_equal(a, b)


def test_start_tables_that_the_result_overwrites():
    """init_centroids inside the output cache (a caller that keeps one table per unit): the launches of their own."""
    H, N, K = 2, 600, 64
    x, init = _inputs(H, N, K, 1, 5)
    want = B.encode_chunk(x.to(DEV), init.to(DEV), 64, 1, 2)
    cache = B.alloc_cache(H, N, N, K, 64, 1, device=DEV)
    cache.centroids[:, 0].copy_(init.to(DEV))
    B.encode_chunk(x.to(DEV), cache.centroids[:, 0], 64, 1, 2, cache=cache)
    torch.cuda.synchronize()
    for a, b in zip(_bytes(cache, slice(None)), _bytes(want, slice(None))):
        assert np.array_equal(a, b)


def test_graph_replays_equal_the_eager_call():
    H, N, K = 6, 1000, 64
    x, init = _inputs(H, N, K, 1, 11)
    x, init = x.to(DEV), init.to(DEV)
    want = B.encode_chunk(x, init, 64, 2, 3)
    cache = B.alloc_cache(H, N, N, K, 64, 2, device=DEV)
    p = B.make_params(H, K, 64, 2, 3)
    ws = torch.empty(B.workspace_bytes(p, B.ENTRY_ENCODE, N), dtype=torch.uint8, device=DEV)
    B.encode_chunk(x, init, 64, 2, 3, cache=cache, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.encode_chunk(x, init, 64, 2, 3, cache=cache, workspace=ws)
    for _ in range(3):
        for t in (cache.centroids, cache.ids, cache.codes, cache.scales):
            t.view(torch.uint8).zero_()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip(_bytes(cache, slice(None)), _bytes(want, slice(None))):
            assert np.array_equal(a, b)


def _team_call(shape, wanted):
    """The encode with units that wait for `wanted` workgroups -> (cache, the units' words: arrived | members << 16, top bit:
    closed).  The words lie behind the norms and the first table."""
    H, N, K, S, I, T, Bg, bits, fp8, wide = shape
    x, init = (t.to(DEV) for t in _inputs(H, N, K, S, 7 * N + K, wide))
    fmt = B.SCALE_E4M3 if fp8 else B.SCALE_F16
    got = B.alloc_cache(H, N, N, K, Bg, T, device=DEV, n_smooth=S, bits=bits, scale_format=fmt)
    for t in (got.centroids, got.ids, got.codes, got.scales):
        t.view(torch.uint8).fill_(0xA5)
    p = B.make_params(H, K, Bg, T, I, bits=bits, n_smooth_stages=S, scale_format=fmt)
    ws = torch.full((B.workspace_bytes(p, B.ENTRY_ENCODE, N),), 0x5A, dtype=torch.uint8, device=DEV)
    ptr = lambda t: C.c_void_p(t.data_ptr())
    i64 = C.c_int64
    st = B.lib().qvg_encode_chunk_wait(C.byref(p), i64(N), ptr(x), i64(x.stride(0)), i64(128), ptr(init), ptr(got.centroids), i64(0),
                                       ptr(got.ids), ptr(got.codes), ptr(got.scales), i64(0), ptr(ws), C.c_size_t(ws.numel()),
                                       C.c_void_p(torch.cuda.current_stream().cuda_stream), C.c_uint32(wanted))
    torch.cuda.synchronize()
    assert st == 0
    r256 = lambda v: -(-v // 256) * 256
    norms = r256(H * (-(-K // 64) * 64) * 8)
    at = norms * S + r256(H * 4) + norms + r256(H * K * 256)
    words = ws[at:at + H * 256].view(torch.int32).reshape(H, 64)[:, 0]
    return B.encode_chunk(x, init, Bg, T, I, bits=bits, scale_format=fmt), got, words.cpu()


TEAMS = SHAPES + [(24, 1200, 256, 4, 3, 1, 16, 2, True, False), (26, 3000, 64, 3, 3, 2, 64, 2, False, True)]


@pytest.mark.parametrize("wanted", [2, 3, 5, 1000])
@pytest.mark.parametrize("shape", [s for s in TEAMS if 512 < s[1]], ids=lambda s: "x".join(str(v) for v in s))
def test_teams_of_fewer_workgroups_make_the_same_bits(shape, wanted):
    """A team of two, three and five (blocks and rows dealt anew, tokens not kept in registers, residuals of several stages
    read back), and one closed by the clock because the last of the wanted does not exist."""
    want, got, words = _team_call(shape, wanted)
    closed = words < 0
    if wanted < 5 or wanted == 1000:
        assert bool(closed.all())
    members = (words[closed] >> 16) & 0x7fff
    assert bool((members >= 1).all() if wanted == 1000 else (members == wanted).all())
    for a, b in zip(_bytes(got, slice(None)), _bytes(want, slice(None))):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("shape", [(24, 4680, 256, 1, 3, 4, 64, 2, False, False), (24, 2000, 64, 4, 3, 1, 16, 2, True, False)],
                         ids=lambda s: "x".join(str(v) for v in s))
def test_beside_a_kernel_that_holds_most_of_the_chip(shape):
    """An attention of 200 workgroups on another stream: units whose workgroups have no place are done by those that have."""
    from test_gpu_attn_integration import _filled_caches
    from paper_2602_02958_amd.configs import CONFIGS
    H, N, K, S, I, T, Bg, bits, fp8, wide = shape
    x, init = (t.to(DEV) for t in _inputs(H, N, K, S, 3, wide))
    fmt = B.SCALE_E4M3 if fp8 else B.SCALE_F16
    want = B.encode_chunk(x, init, Bg, T, I, bits=bits, scale_format=fmt)
    kc, vc = _filled_caches(20, 4680, 4, 18720, 64, 64, 1)
    q = synth.queries(CONFIGS["cfg2_window21"], 20, 2560, DEV)
    B.attn_decode(q, kc, vc)
    torch.cuda.synchronize()
    one, two = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(one):
        outs = [B.attn_decode(q, kc, vc) for _ in range(3)]
    with torch.cuda.stream(two):
        got = [B.encode_chunk(x, init, Bg, T, I, bits=bits, scale_format=fmt) for _ in range(3)]
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[2])
    for g in got:
        for a, b in zip(_bytes(g, slice(None)), _bytes(want, slice(None))):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("shape", [(2, 6200, 256, 4, 2, 1, 16, 2, True, False),     # one block too many for the launch
                                   (2, 2500, 300, 3, 2, 2, 64, 2, False, True)],     # too few workgroups; 16-bit ids
                         ids=lambda s: "x".join(str(v) for v in s))
def test_stages_in_launches_of_their_own(shape):
    """Several stages with Lloyd iterations where the one launch is not taken: residuals, start norms and ids by stage."""
    H, N, K, S, I, T, Bg, bits, fp8, wide = shape
    x, init = _inputs(H, N, K, S, N + K, wide)
    enc = B.encode_chunk(x.to(DEV), init.to(DEV), Bg, T, I, bits=bits, scale_format=B.SCALE_E4M3 if fp8 else B.SCALE_F16)
    torch.cuda.synchronize()
    _check(enc, _oracle(x, init, K, Bg, T, I, S, bits, fp8, slice(None)), slice(None))


@pytest.mark.parametrize("H,N,K,one_launch", [(24, 5100, 64, False), (16, 5100, 16, False), (24, 5376, 83, False), (20, 5100, 19, True),
                                              (24, 5376, 84, True), (24, 5100, 16, True), (24, 4864, 64, True), (16, 6144, 95, False)])
def test_long_lists_of_many_blocks_keep_launches_of_their_own(H, N, K, one_launch):
    """Which form a call takes: with one iteration only the one launch writes the second table's place, where its units meet;
    same bytes as the oracle in both."""
    got, words = _team_call((H, N, K, 1, 1, 1, 64, 2, False, False), 2)[1:]
    assert bool((words < 0).all()) == one_launch and bool((words == 0x5A5A5A5A).all()) != one_launch
    x, init = _inputs(H, N, K, 1, 7 * N + K)
    units = [0, H - 1]
    ref = _oracle(x, init, K, 64, 1, 1, 1, 2, False, units)
    _check(got, ref, units)
