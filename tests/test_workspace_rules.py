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
