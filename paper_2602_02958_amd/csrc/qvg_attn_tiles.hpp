// Pieces shared by the attention kernels that read the compressed cache: the tile walk over the
// chunks, what a thread loads for its part of a 64-token tile, the dequantization of Eq. 7 on
// those values, and the epilogue that normalises and stores a query's result.
#pragma once
#include <type_traits>

#include "qvg_internal.hpp"

namespace qvg {

constexpr int kAtThreads = 512;
constexpr int kAtWaves = kAtThreads / 64;
constexpr int kAtQPerBlock = 32 * kAtWaves;     // 256
constexpr int kAtKv = 64;
constexpr int kKtPitch = 136;      // bf16 per row of the K tile (272 B, 16-byte aligned, conflict-free)
constexpr int kVtPitch = 72;       // f16 per row of the transposed V tile (144 B)
constexpr int kKtElems = kAtKv * kKtPitch;
constexpr int kVtElems = kHeadDim * kVtPitch;
constexpr size_t kAtSmem = (size_t)2 * (kKtElems + kVtElems) * sizeof(uint16_t);

// acc + the eight f16 values of v, accumulated in fp32 (v_dot2_f32_f16 against ones)
__device__ __forceinline__ float sum_f16_pairs(const uint4 &v, float acc) {
    const halfx2_t ones = {(_Float16)1.0f, (_Float16)1.0f};
    acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(halfx2_t, v.x), ones, acc, false);
    acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(halfx2_t, v.y), ones, acc, false);
    acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(halfx2_t, v.z), ones, acc, false);
    acc = __builtin_amdgcn_fdot2(__builtin_bit_cast(halfx2_t, v.w), ones, acc, false);
    return acc;
}

struct CacheSide {                 // one of K / V, already offset to this unit
    const bf16_t *cent;            // [n_chunks][K][d]
    const uint8_t *ids; const uint8_t *codes;
    const uint8_t *scales;         // binary16 or E4M3 bytes, per the format
    int wide;                      // ids are 16-bit words (more than 256 centroids)
};

struct Tile {                      // one 64-token tile; tiles never straddle a chunk
    int chunk; int t0, cend; bool valid;     // token indices fit 31 bits (checked by the caller)
};

struct Span {                      // the part of the cache a workgroup walks: tiles part, part + parts, ...
    int64_t chunk_len, n_kv; int n_chunks;
    int part, parts;
};
__host__ __device__ __forceinline__ Span span_of(const AttnArgs &a, int part, int parts) {
    Span s; s.chunk_len = a.chunk_len; s.n_kv = a.n_kv; s.n_chunks = a.n_chunks;
    s.part = part; s.parts = parts;
    return s;
}
__host__ __device__ __forceinline__ Span span_of(const AttnArgs &a, int part) { return span_of(a, part, a.parts); }
__host__ __device__ __forceinline__ int tiles_per_chunk(const Span &a) {
    const int64_t l = a.chunk_len < a.n_kv ? a.chunk_len : a.n_kv;
    return (int)((l + kAtKv - 1) / kAtKv);
}
// Tile `ti` of a chunk, counted on into the following ones.  (Its position is compared in 64 bits: a step past
// the end of a cache of nearly 2^31 tokens does not fit 31.)
__host__ __device__ __forceinline__ Tile place_tile(const Span &a, int chunk, int ti) {
    Tile t;
    const int tpc = tiles_per_chunk(a);
    while (ti >= tpc) { ti -= tpc; ++chunk; }            // a division would take vector registers from the tile loops
    t.valid = chunk < a.n_chunks;
    if (t.valid) {
        const int64_t b = (int64_t)chunk * a.chunk_len, t0 = b + (int64_t)ti * kAtKv;
        const int64_t cend = (b + a.chunk_len < a.n_kv) ? b + a.chunk_len : a.n_kv;
        t.valid = t0 < cend;
        t.chunk = chunk; t.t0 = (int)t0; t.cend = (int)cend;
    }
    if (!t.valid) { t.chunk = a.n_chunks - 1; t.t0 = 0; t.cend = 0; }
    return t;
}
static_assert(kAtKv == 64, "next_tile counts tiles by shifts");
__host__ __device__ __forceinline__ Tile first_tile(const Span &a) { return place_tile(a, 0, a.part); }
// Inside a chunk a step is one comparison and one addition: every tile of the one-kernel forms takes it (placed
// anew by chunk and tile number, 40 heads x 1560 queries took 1.48 instead of 1.44 ms over 16384 tokens, 1.34 instead
// of 1.26 over 8192 in the general kernel)
__host__ __device__ __forceinline__ Tile next_tile(const Span &a, Tile t) {
    const int step = a.parts * kAtKv;
    if (t.cend - t.t0 > step) { t.t0 += step; return t; }
    return place_tile(a, t.chunk, (int)(((int64_t)t.t0 - (int64_t)t.chunk * a.chunk_len) >> 6) + a.parts);
}

// Tiles of the cache's first n tokens.
__device__ __forceinline__ int64_t tiles_of(const AttnArgs &a, int n) {
    const int nk = (int)a.n_kv, clen = a.chunk_len < a.n_kv ? (int)a.chunk_len : nk;
    const int full = n / clen, rest = n - full * clen;
    return (int64_t)full * (((int64_t)clen + kAtKv - 1) / kAtKv) + ((int64_t)rest + kAtKv - 1) / kAtKv;
}

// A call with a prefix length per query (a.part_tiles): what its first and its last query see.  Lengths need not be in
// any order, but where these two see about as much, all blocks are taken to.
struct PrefixEnds {
    int first, last;
    __device__ __forceinline__ explicit PrefixEnds(const AttnArgs &a) {
        const int nk = (int)a.n_kv, f = a.q_len[0], l = a.q_len[a.n_q - 1];
        first = f < 0 ? 0 : (f > nk ? nk : f);
        last = l < 0 ? 0 : (l > nk ? nk : l);
    }
    __device__ __forceinline__ bool covers(int longest) const {          // the shorter one about as long as `longest`
        return (int64_t)(first < last ? first : last) * 8 >= (int64_t)longest * 7;
    }
    __device__ __forceinline__ bool equal() const { return covers(first < last ? last : first); }
};

// A workgroup's unit, query block, part, and the parts of its block.
struct Place {
    int h, qblock, part, parts;
    __device__ __forceinline__ Place uniform() const {                   // (values that went through LDS or a division)
        return Place{__builtin_amdgcn_readfirstlane(h), __builtin_amdgcn_readfirstlane(qblock),
                     __builtin_amdgcn_readfirstlane(part), __builtin_amdgcn_readfirstlane(parts)};
    }
};

// Which query block and part a workgroup has, b: its number.  Workgroups are dealt to the 8 XCDs round-robin; they are
// re-numbered so that the query blocks of one unit run on one XCD, whose L2 then serves the unit's cache to all of them.
// Prefixes of different lengths (a.part_tiles) are dealt the other way, the queries of all units from the end that sees
// more on: what is left when the chip runs empty is short, and the XCDs have equal shares of every length.  The first
// a.whole workgroups (a multiple of 8) have a block each.  False: none.  at.parts: at most.
// FORM: a template parameter, so that what a call does not need takes no registers from its tile loop.
enum BlockForm { kPlain, kLengths, kLengthsParted };                     // no q_len; q_len; q_len, and a.part_tiles may be set
template <int FORM>
__device__ __forceinline__ bool block_of(const AttnArgs &a, int n_qblocks, int n_blocks, int blocks_per_xcd, unsigned b, Place &at) {
    if (FORM == kLengths) {
        const int w = (int)(b % 8u) * blocks_per_xcd + (int)(b / 8u);
        at.h = w / (n_qblocks * a.parts);
        at.qblock = (w - at.h * n_qblocks * a.parts) / a.parts;
        at.part = w % a.parts; at.parts = a.parts;
        return w < n_blocks;
    }
    int parts = a.parts, h, qblock, part;
    if (FORM == kLengthsParted && a.part_tiles) {                        // uniform
        const PrefixEnds ends(a);
        if (!ends.equal()) {
            const int i = (int)(b / (unsigned)a.H), n = i / parts;
            h = (int)(b % (unsigned)a.H); part = i - n * parts; qblock = ends.first < ends.last ? n_qblocks - 1 - n : n;
            at = Place{h, qblock, part, parts}.uniform();
            return (int)b < n_blocks;
        }
        parts = 1; n_blocks = n_qblocks * a.H; blocks_per_xcd = (n_blocks + 7) / 8;
        if ((int)(b / 8u) >= blocks_per_xcd) return false;
    }
    int first = 0;
    if (FORM == kPlain && a.whole) {                                     // uniform
        if (b < (unsigned)a.whole) { parts = 1; blocks_per_xcd = a.whole / 8; n_blocks = a.whole; }
        else { first = a.whole; b -= (unsigned)a.whole; }
    }
    const int w = (int)(b % 8u) * blocks_per_xcd + (int)(b / 8u), wq = w / parts, block = first + wq;
    h = block / n_qblocks; qblock = block - h * n_qblocks; part = w - wq * parts;
    at = Place{h, qblock, part, parts}.uniform();
    return w < n_blocks;
}

// Parts of a block whose longest prefix is `longest` tokens.  Dividing blocks that all see about as much only costs (228
// blocks of 592 tiles each 1102 us, in two parts 1180, in three 1240).
__device__ __forceinline__ int block_parts(const AttnArgs &a, int longest) {
    if (!a.part_tiles || a.parts == 1) return a.parts;
    const int64_t n = tiles_of(a, longest) / a.part_tiles;
    const PrefixEnds ends(a);
    if (n < 2 || ends.equal() || ends.covers(longest)) return 1;
    return n < a.parts ? (int)n : a.parts;
}

// Running state of a workgroup's 256 queries, [kStateFloats][512] floats: per thread its 64 output
// values (unnormalised), the maximum and the lane's share of the normaliser.
constexpr int kStateFloats = 66;
// The running maximum before any score.  Finite: finite queries and keys can have a product below fp32's
// range, and where all scores of a tile, or of a part, are -inf, exp2(-inf - (-inf)) would be NaN.
// From here their weights are exp2(-inf) = 0, and a part that holds nothing else joins with weight 0.
constexpr float kNoScore = -3.402823466e38f;
__device__ __forceinline__ void store_state(float *st, const floatx16_t (&O)[4], float m, float l) {
#pragma unroll
    for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) st[(mb * 16 + r) * kAtThreads] = O[mb][r];
    st[64 * kAtThreads] = m;
    st[65 * kAtThreads] = l;
}
// the state of query block `qblock` of unit h as part `part` leaves it
__device__ __forceinline__ float *part_state_of(const AttnArgs &a, int n_qblocks, int h, int qblock, int part) {
    const int64_t block = (int64_t)h * n_qblocks + qblock - a.whole, blocks = (int64_t)a.H * n_qblocks - a.whole;
    return a.part_state + (part * blocks + block) * kStateFloats * kAtThreads + threadIdx.x;
}

// A kernel's arguments (the first parameter), read anew where they are called for, the workgroup's block and
// part, which wait in LDS, and the thread's query, worked out anew: what only the end of the kernel needs
// would otherwise be carried through the tile loop, and registers spill there (general kernel, 40 heads x 1560 queries over
// 8192 tokens with prefix lengths, 1.30 ms instead of 1.20 with the arguments alone carried).
__device__ __forceinline__ const AttnArgs &late_args() {
    auto p = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const AttnArgs *)p;
}
__device__ __forceinline__ int late_thread() {
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}
template <int FORM>
__device__ __forceinline__ Place late_place(const AttnArgs &a, int n_qblocks, int blocks_per_xcd) {
    unsigned b = blockIdx.x;
    asm volatile("" : "+s"(b));
    Place at;
    block_of<FORM>(a, n_qblocks, 0, blocks_per_xcd, b, at);
    return at;
}

// Normalise and store one query's result: the lane holds channels 32*mb + 8*g + 4*half + 0..3 of its
// query.  bf16 (round to nearest even), or fp32 when a.out_f32 is set.  A query that saw no token
// at all (prefix length 0) gets a zero row and a log-sum-exp of -inf, which qvg_attn_merge takes
// as a weightless partial result.
__device__ __forceinline__ void store_result(const AttnArgs &a, int h, int64_t qrow, bool seen, bool qvalid,
                                             int half, const floatx16_t (&O)[4], float m, float l) {
    const float ltot = l + __shfl_xor(l, 32, 64);
    if (!qvalid) return;
    const float inv = seen ? 1.0f / ltot : 0.0f;
    const int64_t row = ((int64_t)h * a.n_q + qrow) * kHeadDim + half * 4;
    if (a.out_f32) {
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                float4 o;
                o.x = seen ? O[mb][4 * gq + 0] * inv : 0.0f; o.y = seen ? O[mb][4 * gq + 1] * inv : 0.0f;
                o.z = seen ? O[mb][4 * gq + 2] * inv : 0.0f; o.w = seen ? O[mb][4 * gq + 3] * inv : 0.0f;
                *reinterpret_cast<float4 *>(a.out_f32 + row + mb * 32 + gq * 8) = o;
            }
    } else {
        bf16_t *op = a.out + row;
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
            for (int gq = 0; gq < 4; ++gq) {
                const uint2 o = seen ? make_uint2(
                    pack_bf16x2(O[mb][4 * gq + 0] * inv, O[mb][4 * gq + 1] * inv),
                    pack_bf16x2(O[mb][4 * gq + 2] * inv, O[mb][4 * gq + 3] * inv)) : make_uint2(0u, 0u);
                *reinterpret_cast<uint2 *>(op + mb * 32 + gq * 8) = o;
            }
    }
    if (a.lse && half == 0)
        a.lse[(int64_t)h * a.n_q + qrow] = seen ? (m + __builtin_log2f(ltot)) * 0.6931471805599453f : -INFINITY;
}

// SM: how the smoothing stages are handled.  1: a single stage; 0: several, their number known at
// run time only (the rows are added as they arrive, which waits for every load where it is
// issued); 2..kMaxSmooth: that many stages, fixed at compile time (the rows stay packed in
// registers while the loads are in flight and are added, in stage order, when the tile is decoded).
template <int TM, int SM = 1>
struct Raw {                       // what one thread loads for its 2 tokens x 8 channels of one side
    uint32_t code[2][TM], sc[2][TM];
    uint4 cen[2];                  // one smoothing stage: the centroid row (8 bf16)
    float ci[2][8];                // SM == 0: the rows added in stage order (fp32)
    uint4 rows[2][SM > 1 ? SM : 1];     // SM > 1: the stages' rows
};

// ids of this thread's two tokens of a tile (0 for tokens past the chunk end / an invalid tile);
// with S smoothing stages a token has S id bytes, stage s in byte s of the result
// (ids of 16 bits, for tables of more than 256 rows: one stage here; with several stages the
// run-time-count path of load_raw reads them itself)
// The ids of a thread's two tokens, as stored: one load per token (the S id bytes of a token
// are contiguous; 1, 2 or 4 of them are one load when the array is aligned for it) and no
// arithmetic on what it returns.  The clamp to the table's last row is applied where the id is
// used (load_raw): applied here, every tile waited for the ids right after requesting them,
// and, the load counter being in order, for the codes, scales and rows requested just before.
// A token that does not exist reads the unit's token 0 instead (it exists), so that the load
// needs no branch; load_raw never uses such an id.
__device__ __forceinline__ void load_ids(const CacheSide &s, const Tile &t, int tp, int S,
                                         int wide, uint32_t id[2]) {
    const bool al = ((uintptr_t)s.ids & (uintptr_t)(S - 1)) == 0;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int n0 = t.t0 + 2 * tp + e;
        const int64_t n = (t.valid && n0 < t.cend) ? n0 : 0;
        if (wide) id[e] = load_id(s.ids, n, 1);
        else if (S == 1) id[e] = s.ids[n];
        else if (S == 2 && al) id[e] = *reinterpret_cast<const uint16_t *>(s.ids + n * 2);
        else if (S == 4 && al) id[e] = *reinterpret_cast<const uint32_t *>(s.ids + n * 4);
        else {
            id[e] = 0u;
            for (int st = 0; st < S; ++st) id[e] |= (uint32_t)s.ids[n * S + st] << (8 * st);
        }
    }
}

// FMT: stored format (kFmt* bits); with 4-bit levels a thread's 8 channels of a round are one
// 32-bit word, else one 16-bit word
template <int T_, int TM, int SM, int FMT>
__device__ __forceinline__ void load_raw(const CacheSide &s, const Tile &t, int tp, int c8, int T,
                                         int G, int g, int K, int S, const uint32_t id[2], Raw<TM, SM> &r) {
    const bf16_t *cent = s.cent + (int64_t)t.chunk * S * K * kHeadDim;      // [S][K][d] of this chunk
    const uint32_t kmax = (uint32_t)K - 1u;        // ids are clamped to the table's last row
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int n = t.t0 + 2 * tp + e;
        const bool ok = t.valid && n < t.cend;
#pragma unroll
        for (int k = 0; k < TM; ++k) { r.code[e][k] = 0u; r.sc[e][k] = 0u; }
        r.cen[e] = make_uint4(0u, 0u, 0u, 0u);
        if (SM == 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) r.ci[e][i] = 0.0f;
        }
        if (SM > 1) {
#pragma unroll
            for (int st = 0; st < SM; ++st) r.rows[e][st] = make_uint4(0u, 0u, 0u, 0u);
        }
        if (ok) {
            constexpr bool FP8 = (FMT & kFmtE4M3) != 0, I4 = (FMT & kFmtInt4) != 0;
            typedef typename std::conditional<I4, uint32_t, uint16_t>::type code_t;
            typedef typename std::conditional<FP8, uint8_t, f16_t>::type scale_t;
            const code_t *cp = reinterpret_cast<const code_t *>(s.codes + (int64_t)n * T * (I4 ? 64 : 32)) + c8;
            const scale_t *sp = reinterpret_cast<const scale_t *>(s.scales) + (int64_t)n * T * G + g;
#pragma unroll
            for (int k = 0; k < TM; ++k)
                if (k < T) { r.code[e][k] = cp[k * 16]; r.sc[e][k] = sp[k * G]; }
            if (SM == 1) {
                r.cen[e] = *reinterpret_cast<const uint4 *>(cent + (int64_t)min(id[e], kmax) * kHeadDim + c8 * 8);
            } else if (SM > 1) {
#pragma unroll
                for (int st = 0; st < SM; ++st)
                    r.rows[e][st] = *reinterpret_cast<const uint4 *>(
                        cent + ((int64_t)st * K + min((id[e] >> (8 * st)) & 0xffu, kmax)) * kHeadDim + c8 * 8);
            } else {
                for (int st = 0; st < S; ++st) {
                    float row[8];
                    // 16-bit ids with several stages do not fit the packed word: read where they are used
                    const uint32_t sid = s.wide ? (uint32_t)reinterpret_cast<const uint16_t *>(s.ids)[(int64_t)n * S + st]
                                                : (id[e] >> (8 * st)) & 0xffu;
                    unpack_bf16x8(*reinterpret_cast<const uint4 *>(
                                      cent + ((int64_t)st * K + min(sid, kmax)) * kHeadDim + c8 * 8), row);
#pragma unroll
                    for (int i = 0; i < 8; ++i) r.ci[e][i] = st ? r.ci[e][i] + row[i] : row[i];
                }
            }
        }
    }
}

// fp32 decoded values of the thread's two tokens (tokens that do not exist decode to zero
// because their codes, scales and centroid were loaded as zero)
template <int T_, int TM, int SM = 1, int FMT = 0>
__device__ __forceinline__ void dequant2x8(const Raw<TM, SM> &r, int T, float *accA, float *accB) {
    if (SM == 0) {
#pragma unroll
        for (int i = 0; i < 8; ++i) { accA[i] = r.ci[0][i]; accB[i] = r.ci[1][i]; }
    } else if (SM > 1) {
        unpack_bf16x8(r.rows[0][0], accA);
        unpack_bf16x8(r.rows[1][0], accB);
#pragma unroll
        for (int st = 1; st < SM; ++st) {
            float ra[8], rb[8];
            unpack_bf16x8(r.rows[0][st], ra);
            unpack_bf16x8(r.rows[1][st], rb);
#pragma unroll
            for (int i = 0; i < 8; ++i) { accA[i] += ra[i]; accB[i] += rb[i]; }
        }
    } else {
        unpack_bf16x8(r.cen[0], accA);
        unpack_bf16x8(r.cen[1], accB);
    }
    if (FMT != 0) {
        constexpr bool FP8 = (FMT & kFmtE4M3) != 0;
#pragma unroll
        for (int t = 0; t < TM; ++t) {
            if (t < T) {
                const float sa = scale_bits_to_f32<FP8>(r.sc[0][t]), sb = scale_bits_to_f32<FP8>(r.sc[1][t]);
                if (FMT & kFmtInt4) {
                    add_stage_int4(accA, r.code[0][t], sa);
                    add_stage_int4(accB, r.code[1][t], sb);
                } else {
                    add_last_stage_of_two_rows(accA, accB, r.code[0][t] | (r.code[1][t] << 16), 0.5f * sa, 0.5f * sb);
                }
            }
        }
        return;
    }
#pragma unroll
    for (int t = 0; t + 1 < TM; t += 2) {
        if (t + 1 < T) {
            add_two_stages(accA, r.code[0][t] | (r.code[0][t + 1] << 16),
                           half_scale(r.sc[0][t]), half_scale(r.sc[0][t + 1]));
            add_two_stages(accB, r.code[1][t] | (r.code[1][t + 1] << 16),
                           half_scale(r.sc[1][t]), half_scale(r.sc[1][t + 1]));
        }
    }
    if (T_ > 0) {
        if (T_ & 1)
            add_last_stage_of_two_rows(accA, accB, r.code[0][TM - 1] | (r.code[1][TM - 1] << 16),
                                       half_scale(r.sc[0][TM - 1]), half_scale(r.sc[1][TM - 1]));
    } else if (T & 1) {
#pragma unroll
        for (int t = 0; t < TM; t += 2)
            if (t == T - 1)
                add_last_stage_of_two_rows(accA, accB, r.code[0][t] | (r.code[1][t] << 16),
                                           half_scale(r.sc[0][t]), half_scale(r.sc[1][t]));
    }
}

// the (cos, sin) pairs of this thread's 8 channels of its two tokens of a tile (zero for tokens
// that do not exist: their decoded value is zero as well)
__device__ __forceinline__ void load_rope(const f16_t *rope, const Tile &t, int tp, int c8, uint4 rp[2]) {
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const int n = t.t0 + 2 * tp + e;
        rp[e] = (t.valid && n < t.cend)
                    ? *reinterpret_cast<const uint4 *>(rope + (int64_t)n * kHeadDim + c8 * 8)
                    : make_uint4(0u, 0u, 0u, 0u);
    }
}

}  // namespace qvg
