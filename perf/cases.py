"""The work whose speed is measured: what a rollout does with its compressed KV cache.

A generation step encodes the new chunk's K and V (all heads of a layer in one call), decodes
cached chunks where the plain bf16 tensors are wanted, and attends to the compressed cache with
the new chunk's queries.  The cases cover these three directions from the smallest call (one head,
where launches and latency are everything) to one layer of the 748800-token configuration, in the
stored formats the package is used with: 1..4 rounds of 2-bit levels with binary16 scales, and the
paper's presets (FP8 E4M3 scales, 2- and 4-bit levels, one or four smoothing stages).  Sizes are
those of paper_2602_02958_amd/configs.py, of the paper's latent frames (1560 tokens), or odd.

Inputs come from the package's synthetic mixture (synth.py), seeded; caches are filled by the
encoder, chunk by chunk with warm starts, as a rollout fills them.
"""
from __future__ import annotations

import math

import torch

from paper_2602_02958_amd import binding as B
from paper_2602_02958_amd import synth
from paper_2602_02958_amd.configs import Workload

D = 128                        # head dimension
DEV = "cuda"
FRAME = 1560                   # latent tokens of one frame


def _case(name, op, **kw):
    """op "encode": one chunk of `units` x `tokens`; "decode": a cache of `units` x `tokens` in chunks;
    "attend": `heads` x `n_q` queries over `tokens` cached tokens per head."""
    c = dict(op=op, K=256, B=64, T=1, S=1, bits=2, fp8=False, scale="lognormal0.5")
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # -- encode: x -> centroids, ids, codes, scales ---------------------------------------
        # the first chunk of a single head: a cold fit, ten Lloyd iterations on little data
        _case("encode_one_head_cold", "encode", units=2, tokens=4096, K=16, T=2, iters=10, scale="outlier4x8"),
        # what every generation step of a 12-head layer does: a 3-frame chunk, warm start
        _case("encode_layer_warm", "encode", units=24, tokens=4680, K=256, T=4, iters=3),
        # the paper's QVG-Pro preset on the same chunk: four smoothing stages
        _case("encode_layer_pro", "encode", units=24, tokens=4680, K=256, B=16, S=4, fp8=True, iters=3),
        # the paper's INT4 preset, a chunk of one frame and an odd rest, few heads
        _case("encode_frame_int4", "encode", units=10, tokens=FRAME + 11, K=256, bits=4, fp8=True, iters=3),
        # one layer of a 40-head model, 10800-token chunks
        _case("encode_wide_layer", "encode", units=80, tokens=10800, K=128, B=32, T=3, iters=3, scale="student_t3"),
        # -- decode: the stored form -> bf16 ------------------------------------------------------
        # one chunk of one layer
        _case("decode_chunk", "decode", units=24, tokens=4680, chunk=4680, K=256, T=2),
        # one layer of the longest rollout
        _case("decode_long_layer", "decode", units=24, tokens=748800, chunk=4680, K=256, T=4),
        # -- attention over the compressed cache ------------------------------------------------
        # a few queries of one head (the tile workspace does not apply)
        _case("attend_one_head", "attend", heads=1, n_q=64, tokens=4096, chunk=4096, K=16, T=2, scale="outlier4x8"),
        # one frame's queries over a cache that is not full, no workspace lent, log-sum-exp wanted
        _case("attend_frame", "attend", heads=12, n_q=FRAME, tokens=31997, chunk=4680, K=64, B=32, T=3, lse=True),
        # the queries of several chunks at once, each chunk seeing the chunks before it
        _case("attend_causal", "attend", heads=12, n_q=4680, tokens=37440, chunk=4680, K=64, B=32, T=3,
              causal=4, ws_chunks=8),
        # QVG-Pro with the rotary embedding of the cached keys, merged with the chunk's own attention
        _case("attend_window_pro", "attend", heads=12, n_q=4680, tokens=37440, chunk=4680, K=256, B=16, S=4,
              fp8=True, rope=True, lse=True, merge=True, ws_chunks=8),
        # one layer of the longest rollout: a chunk's queries over 748800 cached tokens per head
        _case("attend_long_layer", "attend", heads=12, n_q=4680, tokens=748800, chunk=4680, K=256, T=4, ws_chunks=32),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


FORMATS = [                    # (K choices, B, T, S, bits, fp8)
    ((16, 64, 256), 64, 2, 1, 2, False), ((64, 100, 256), 32, 3, 1, 2, False), ((128, 256), 64, 4, 1, 2, False),
    ((64, 256), 64, 1, 1, 2, True), ((256,), 16, 1, 4, 2, True), ((256,), 64, 1, 1, 4, True),
    ((512,), 64, 1, 1, 2, True),
]


def draw(rng):
    Ks, Bg, T, S, bits, fp8 = rng.choice(FORMATS)
    fmt = dict(K=rng.choice(Ks), B=Bg, T=T, S=S, bits=bits, fp8=fp8,
               scale=rng.choice(["lognormal0.5", "outlier4x8", "student_t3"]))
    op = rng.choice(["encode", "decode", "attend", "attend"])
    heads = _log_int(rng, 1, 40)
    if op == "encode":
        return _case(None, op, units=2 * heads, tokens=_log_int(rng, FRAME // 2, 10800), iters=rng.choice([0, 3, 3, 10]), **fmt)
    chunk = 8 * _log_int(rng, FRAME // 8, 10800 // 8)
    most = min(748800, 18_000_000 // (2 * heads))            # tokens of all units together: as the longest layer
    tokens = _log_int(rng, min(FRAME, most), most)
    if op == "decode":
        return _case(None, op, units=2 * heads, tokens=tokens, chunk=chunk, **fmt)
    n_q = _log_int(rng, 64, 10800)
    limit = 5_000_000_000_000 // (4 * D * heads * n_q)        # a quarter of the longest layer's operations
    tokens = max(FRAME, min(tokens, limit))
    ws = rng.choice([0, 8, 32]) if n_q > 256 else 0
    extra = rng.choice([{}, {}, dict(rope=True), dict(causal=rng.randint(2, 6)), dict(lse=True, merge=True)])
    return _case(None, op, heads=heads, n_q=n_q, tokens=tokens, chunk=chunk, ws_chunks=ws, **extra, **fmt)


# ------------------------------------------------------------------------------------- inputs
def _workload(case):
    heads = case.get("heads", case.get("units", 2) // 2)
    return Workload("measured", 1, heads, D, case["tokens"], case.get("chunk", case["tokens"]), case["K"],
                    case["T"], case["B"], case.get("n_q", 0), 64, 0.2, case["scale"], 0.05, 10, 3)


class _Chunks:
    """K and V tokens of all heads, chunk by chunk: [2 * heads, n, 128] bf16, K heads first."""

    def __init__(self, wl, seed):
        self.streams = [synth.MixtureStream(wl, wl.heads, kv, DEV, layer=seed) for kv in (0, 1)]

    def next(self, n):
        return torch.cat([s.next_chunk(n) for s in self.streams], 0)


def _cold_start(x, case, seed):
    """Start centroids of a first chunk: tokens of each stage's own input, [units, K, d] or [units, S, K, d]."""
    S, K = case["S"], case["K"]
    inits, r = [], x
    for s in range(S):
        inits.append(synth.cold_start_centroids(r, K, seed=seed + s))
        if s + 1 < S:
            enc = B.encode_chunk(r, inits[s], case["B"], 1, 3)
            idx = enc.ids.long()[:, :, None].expand(-1, -1, D)
            r = (r.float() - torch.gather(enc.centroids[:, 0], 1, idx).float()).to(torch.bfloat16)
    return torch.stack(inits, 1) if S > 1 else inits[0]


def _new_cache(case, wl, tokens, chunk):
    return B.StreamingCache(wl.heads, tokens, chunk, case["K"], case["B"], case["T"], n_smooth=case["S"],
                            bits=case["bits"], scale_format=B.SCALE_E4M3 if case["fp8"] else B.SCALE_F16,
                            warm_iters=wl.kmeans_iters_warm, cold_iters=wl.kmeans_iters_cold, device=DEV)


def _filled(case, wl, seed):
    chunks = _Chunks(wl, seed)
    sc = _new_cache(case, wl, case["tokens"], case["chunk"])
    while sc.n_tokens < case["tokens"]:
        x = chunks.next(min(case["chunk"], case["tokens"] - sc.n_tokens))
        sc.append(x, init=_cold_start(x, case, seed) if sc.n_tokens == 0 else None)
    return sc


def _rope_table(n):
    freq = 10000.0 ** (-torch.arange(D // 2, dtype=torch.float64, device=DEV) / (D // 2))
    ang = torch.arange(n, dtype=torch.float64, device=DEV)[:, None] * freq[None]
    return torch.stack([ang.cos(), ang.sin()], -1).to(torch.float16).contiguous()


def prepare(case, seed):
    wl = _workload(case)
    if case["op"] == "encode":
        # a warm start is the fit of the chunk before; a cold one (ten iterations) picks tokens
        chunks = _Chunks(wl, seed)
        n = case["tokens"]
        x = chunks.next(n)
        init = _cold_start(x, case, seed)
        sc = _new_cache(case, wl, 2 * n + 8, (n + 7) // 8 * 8)
        if case["iters"] < 10:
            sc.append(x, init=init)
            init = sc.cache.centroids[:, 0].contiguous()
            x = chunks.next(n)
        p = B.make_params(2 * wl.heads, case["K"], case["B"], case["T"], case["iters"], bits=case["bits"],
                          n_smooth_stages=case["S"], scale_format=B.SCALE_E4M3 if case["fp8"] else B.SCALE_F16)
        ws = torch.empty(max(16, B.workspace_bytes(p, B.ENTRY_ENCODE, n)), dtype=torch.uint8, device=DEV)
        return dict(case=case, x=x, init=init, cache=sc.cache, ws=ws)
    sc = _filled(case, wl, seed)
    if case["op"] == "decode":
        out = torch.empty(case["units"], case["tokens"], D, dtype=torch.bfloat16, device=DEV)
        return dict(case=case, sc=sc, out=out)
    H, Nq, n = wl.heads, case["n_q"], case["tokens"]
    st = dict(case=case, sc=sc, q=synth.queries(wl, H, Nq, DEV, step=seed), ws=None, rope=None)
    if case.get("ws_chunks"):
        st["ws"] = B.attn_workspace(H, Nq, case["chunk"], min(case["ws_chunks"], -(-n // case["chunk"])), DEV)
    if case.get("rope"):
        st["rope"] = _rope_table(n)
    if case.get("causal"):
        st["q_len"] = torch.tensor(_causal_lengths(case), dtype=torch.int32, device=DEV)
    if case.get("merge"):
        # the chunk's attention to itself, from the model's own attention kernel
        g = torch.Generator(device=DEV).manual_seed(seed + 17)
        st["own"] = (0.3 * torch.randn(H, Nq, D, generator=g, device=DEV)).to(torch.bfloat16)
        st["own_lse"] = 3.0 + 0.5 * torch.randn(H, Nq, generator=g, device=DEV)
    return st


def _causal_lengths(case):
    """Prefix length of every query: `causal` equal groups, group i sees the first (i + 1)/causal of
    the cache's chunks."""
    Nq, n, L, G = case["n_q"], case["tokens"], case["chunk"], case["causal"]
    chunks = -(-n // L)
    return [min(n, L * max(1, -(-chunks * (i * G // Nq + 1) // G))) for i in range(Nq)]


# ---------------------------------------------------------------------------------------- run
def run(state):
    case = state["case"]
    if case["op"] == "encode":
        # the chunk goes into slot 1 of the cache (slot 0 holds the chunk before)
        e = B.encode_chunk(state["x"], state["init"], case["B"], case["T"], case["iters"], cache=state["cache"],
                           chunk_index=1, workspace=state["ws"])
        a = e.chunk_len
        b = a + case["tokens"]
        return e.centroids[:, 1], e.ids[:, a:b], e.codes[:, a:b], e.scales[:, a:b]
    sc = state["sc"]
    if case["op"] == "decode":
        return sc.decode(out=state["out"])
    if case.get("causal"):
        return B.attn_decode(state["q"], sc.k, sc.v, n_kv=sc.n_tokens, k_rope=state["rope"], q_kv_len=state["q_len"],
                             workspace=state["ws"])
    lse = bool(case.get("lse"))
    out = sc.attend(state["q"], k_rope=state["rope"], want_lse=lse, workspace=state["ws"])
    if case.get("merge"):
        return B.attn_merge(out[0], out[1], state["own"], state["own_lse"], want_lse=True)
    return out


# ----------------------------------------------------------------------------- bounds, tolerance
def _stored_bytes(case, units, tokens, chunk):
    """Bytes of the stored form: ids, codes, scales and one set of tables per chunk."""
    per_token = case["S"] * (2 if case["K"] > 256 else 1) + \
        case["T"] * (D * case["bits"] // 8 + (D // case["B"]) * (1 if case["fp8"] else 2))
    return units * (tokens * per_token + -(-tokens // chunk) * case["S"] * case["K"] * D * 2)


def work(case):
    n = case["tokens"]
    if case["op"] == "encode":
        u, table = case["units"], case["units"] * case["S"] * case["K"] * D * 2
        stored = _stored_bytes(case, u, n, n)
        # every stage: iters + 1 assignments (distances to K centroids), iters sums over the members
        flops = u * n * D * case["S"] * ((case["iters"] + 1) * 2 * case["K"] + case["iters"] + 1)
        flops += u * n * D * case["T"] * 4
        return dict(bytes=u * n * D * 2 + table + stored, flops=flops)
    if case["op"] == "decode":
        u = case["units"]
        return dict(bytes=_stored_bytes(case, u, n, case["chunk"]) + u * n * D * 2,
                    flops=u * n * D * (2 * case["T"] + case["S"]))
    H, Nq = case["heads"], case["n_q"]
    pairs = sum(_causal_lengths(case)) if case.get("causal") else Nq * n
    nbytes = _stored_bytes(case, 2 * H, n, case["chunk"]) + 2 * H * Nq * D * 2
    if case.get("rope"):
        nbytes += n * D * 2
    if case.get("lse"):
        nbytes += H * Nq * 4
    if case.get("merge"):
        nbytes += 3 * H * Nq * (D * 2 + 4)
    return dict(bytes=nbytes, flops=4 * H * pairs * D)


def tolerance(case):
    if case["op"] != "attend":
        return "exact"           # stored integers, their scales, and the decoded bf16 values are defined bit for bit
    # two bf16 results of the same attention, its probabilities rounded to binary16 against different
    # running maxima and its sums taken in another order.  Against the same attention in fp64 on the
    # decoded caches the results show 1.0e-3 .. 1.8e-3 (nearly all of it the rounding of the output),
    # two correct results against each other sqrt(2) times that; four times that is stated.
    return dict(rel=1e-2)
