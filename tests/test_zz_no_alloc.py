"""qvg_encode_chunk_static (the entry point for callers that cannot allocate device memory: its
workspace is a static device array inside the library) against qvg_encode_chunk on the same
inputs: every stored array bit-equal, on two calls in a row, the second with a smaller input, so
that what the first call left in the shared array is seen not to leak into the second."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2602_02958_amd import binding as B
from paper_2602_02958_amd import synth
from paper_2602_02958_amd.configs import CONFIGS

pytestmark = pytest.mark.gpu


def _encode_both(x, init, Bg, T, I):
    """-> (arrays from qvg_encode_chunk with a caller workspace, arrays from the static-scratch entry)."""
    H, N, d = x.shape
    K = init.shape[-2]
    outs = []
    for static in (False, True):
        cache = B.alloc_cache(H, N, N, K, Bg, T, d, x.device)
        for t in (cache.centroids, cache.ids, cache.codes, cache.scales):
            t.view(torch.uint8).fill_(0xA5)                       # stale bytes must all be overwritten
        B.encode_chunk(x, init, Bg, T, I, cache=cache, static_scratch=static)
        torch.cuda.synchronize()
        outs.append([t.view(torch.uint8).cpu().numpy().copy() for t in (cache.centroids, cache.ids, cache.codes, cache.scales)])
    return outs


def test_static_scratch_encode_equals_workspace_encode_twice_in_a_row():
    wl = CONFIGS["cfg3_dit_small"]
    dev = "cuda"
    st = synth.MixtureStream(wl, 6, 0, dev)
    # first call: 6 units x 3000 tokens, K = 256, Lloyd iterations (assignment scratch, both tables,
    # permutation and offsets all live in the static array)
    x1 = st.next_chunk(3000)
    i1 = synth.cold_start_centroids(x1, 256)
    a, b = _encode_both(x1, i1, 64, 2, 3)
    for u, v, name in zip(a, b, ("centroids", "ids", "codes", "scales")):
        assert np.array_equal(u, v), f"first call: {name} differ"
    # second call, smaller in every size (fewer units, fewer tokens with a ragged tail, fewer
    # centroids, other group size and round count): the array still holds the first call's data
    x2 = st.next_chunk(777)[:3]
    i2 = synth.cold_start_centroids(x2, 40)
    a, b = _encode_both(x2, i2, 32, 3, 2)
    for u, v, name in zip(a, b, ("centroids", "ids", "codes", "scales")):
        assert np.array_equal(u, v), f"second call: {name} differ"
    # and a single pass (no Lloyd iteration: only the assignment scratch is used)
    a, b = _encode_both(x2, i2, 64, 1, 0)
    for u, v, name in zip(a, b, ("centroids", "ids", "codes", "scales")):
        assert np.array_equal(u, v), f"third call: {name} differ"


def test_static_scratch_encode_refuses_sizes_beyond_its_array():
    dev = "cuda"
    H, N, K = 720, 4680, 256                                       # two 47 MB tables: beyond the 16 MiB limit
    p = B.make_params(H, K, 64, 2, kmeans_iters=3)
    assert B.workspace_bytes(p, B.ENTRY_ENCODE, N) > (16 << 20)
    x = torch.zeros(1, 8, 128, dtype=torch.bfloat16, device=dev)   # never read: the call fails first
    st = B.lib().qvg_encode_chunk_static(C.byref(p), N, C.c_void_p(x.data_ptr()), N * 128, 128,
                                         C.c_void_p(x.data_ptr()), C.c_void_p(x.data_ptr()), 0,
                                         C.c_void_p(x.data_ptr()), C.c_void_p(x.data_ptr()), C.c_void_p(x.data_ptr()), 0, None)
    assert st == -7
    torch.cuda.synchronize()
