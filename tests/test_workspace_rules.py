"""Host-side size rules, without a GPU."""
import pytest

from paper_2602_02958_amd import binding as B


@pytest.mark.parametrize("entry", [B.ENTRY_ENCODE, B.ENTRY_KMEANS_UPDATE, B.ENTRY_KMEANS_ASSIGN])
@pytest.mark.parametrize("K,S", [(512, 1), (256, 1), (16, 2), (64, 4)])
def test_a_workspace_serves_every_smaller_call(entry, K, S):
    """A caller sizes one workspace for its chunk length and its units: fewer tokens, fewer units or
    fewer iterations never need more."""
    def need(H, n, iters=3):
        return B.workspace_bytes(B.make_params(H, K, 64, 1, kmeans_iters=iters, n_smooth_stages=S), entry, n)
    for H in (1, 3, 40, 80, 81, 400, 1500):
        ns = sorted({n + d for n in (256, 1024, 4096, 13056, 13312, 26368, 26624, 65536, 131072, 262144, 1 << 19, (1 << 20) - 1)
                     for d in (-255, -1, 0, 1, 256)} | {256 * s for s in range(1, 220)})
        sizes = [need(H, n) for n in ns]
        assert all(a <= b for a, b in zip(sizes, sizes[1:])), H
        assert all(need(H, n, 0) <= need(H, n) for n in ns)
    for n in (1, 300, 4680, 13312, 26624, 131072, 1 << 20):
        sizes = [need(H, n) for H in range(1, 500)]
        assert all(a <= b for a, b in zip(sizes, sizes[1:])), n


@pytest.mark.parametrize("heads", [1, 12, 40, 128])
@pytest.mark.parametrize("n_q", [513, 1560, 4680, 10800, 100000])
def test_the_attention_s_own_workspace_stays_within_its_bounds(heads, n_q):
    """What attn_decode takes when it is lent none: at most 256 MiB of tiles and 256 MiB of state, no state
    where one slab holds the cache, and never less than one chunk with the state."""
    state = heads * -(-n_q // 256) * 66 * 512 * 4
    taken = 0
    for chunk_len in (1, 64, 200, 1560, 4680, 10800, 1 << 20, (1 << 63) - 1):
        one = heads * -(-chunk_len // 64) * 64 * 512
        for n_chunks in (1, 2, 3, 8, 160):
            b = B._tile_scratch_bytes(heads, n_q, chunk_len, n_chunks)
            taken += b > 0
            if one * n_chunks <= 256 << 20:
                assert b == one * n_chunks
            elif b:
                assert state <= 256 << 20 and (b - state) % one == 0 and one <= b - state <= 256 << 20
                assert B.workspace_bytes(B.make_params(heads, 16, 64, 1), B.ENTRY_ATTN, 0, n_q) == state
    assert taken > 0


def test_a_cache_that_is_not_asked_about_is_not_divided():
    need = B.C.c_size_t()
    asked = 0
    for chunk_len in (1, 8, 40, 64, 65, 100, 520, 4680, 1 << 40):
        for n_kv in range(1, 600):
            assert B.lib().qvg_attn_scratch_bytes(B.C.byref(B.make_params(1, 16, 64, 1)), 1, n_kv, chunk_len, B.C.byref(need)) == 0
            asked += B._may_divide(n_kv, chunk_len)
            assert need.value == 0 or B._may_divide(n_kv, chunk_len)
    assert asked > 0
