// Attention over the compressed cache with the decoded tiles shared by all query blocks.
//
// The fused kernels (qvg_attn.hip) decode every 64-token tile once per workgroup of 256 queries:
// with n_q queries per unit the dequantization of Eq. 7 is repeated ceil(n_q / 256) times, and it
// is what bounds them (vector instructions, not the matrix cores).  When the caller lends a
// workspace, the same work is split at the point where those kernels hand a decoded tile to the
// contractions:
//   slab_decode_kernel   decodes each tile of a slab of chunks ONCE per unit and writes the two
//                        operand images the contractions read: K_hat row-major bf16 [64][128], V_hat
//                        transposed f16 [128][64] with the token permutation of the PV contraction
//                        (the values are exactly those the fused kernels put into LDS);
//   attn_slab_kernel     256 queries per workgroup as before; per tile it copies the two images
//                        (32 KB) into LDS and runs the same S^T = K Q^T, online soft-max and
//                        O^T += V^T P steps.
// A slab is as many whole chunks as the workspace holds; the running soft-max state (maximum,
// normaliser, unnormalised output, fp32) of every query is carried from slab to slab in the
// workspace, so the full-precision cache is never materialised beyond one slab.
#include "qvg_attn_tiles.hpp"

namespace qvg {

constexpr int kImgElems = kAtKv * kHeadDim;             // 16-bit elements of one operand image (16 KB)

struct SlabArgs {
    uint16_t *kimg, *vimg;     // [H][tiles_cap][kImgElems]
    int64_t tiles_cap;         // image slots per unit
    int c0;                    // first chunk of the slab
    int n_tiles;               // tiles of the slab (every one holds at least one token)
    int tpc;                   // tiles per chunk = ceil(chunk_len / 64)
    float *state;              // [workgroup][kStateFloats][512] running state, or nullptr (single slab, or several parts: AttnArgs)
    int first, last;           // first / last slab of the call
};

// tile `i` of the slab (i may be past the end: then invalid)
__device__ __forceinline__ Tile slab_tile(const AttnArgs &a, const SlabArgs &sl, int i) {
    Tile t;
    const int c = i / sl.tpc;
    t.chunk = sl.c0 + c;
    const int64_t b = (int64_t)t.chunk * a.chunk_len;
    t.t0 = (int)(b + (int64_t)(i - c * sl.tpc) * kAtKv);
    t.cend = (int)((b + a.chunk_len < a.n_kv) ? b + a.chunk_len : a.n_kv);
    t.valid = i < sl.n_tiles;
    if (!t.valid) { t.chunk = sl.c0; t.t0 = 0; t.cend = 0; }
    return t;
}

// ---------------------------------------------------------------------------------------------
// Decode a run of tiles of one unit's K or V into the operand images.  512 threads: thread
// (tp, c8) has tokens 2 tp, 2 tp + 1 and channels 8 c8 .. 8 c8 + 7, as in the fused
// kernels.  K rows go straight to memory (16 lanes cover a 256-byte row); V is transposed through
// LDS.  Tokens past the end of a chunk decode to zero.
// ---------------------------------------------------------------------------------------------
// A workgroup decodes ONE side (blockIdx.z: 0 K, 1 V): the kernel is a chain of small dependent loads and lives
// on occupancy, and one side's raw data takes half the registers (three workgroups per CU up to two smoothing
// stages, else two).  32 chunks of 12 heads x 4680 tokens, T = 4: 353 us with both sides in one workgroup, 320 so (364
// and 694 with two and four workgroups per CU); 37440 tokens, S = 4 147 -> 120 us (150 with three), T = 3 86 -> 90.
// 0.92 GB written and 0.57 read in 320 us are 4.7 TB/s, nine tenths of a copy's rate.
template <int T_, int SM, int FMT, bool ROPE>
__global__ __launch_bounds__(kAtThreads, (T_ > 0 && SM <= 2) ? 6 : 4)
void slab_decode_kernel(AttnArgs a, SlabArgs sl, int run) {
    constexpr int TM = T_ > 0 ? T_ : kMaxStages;
    __shared__ __align__(16) uint16_t Vt[kVtElems];                     // [128][72] f16, transposed, swizzled (below)
    const int h = blockIdx.y;
    const int i0 = (int)blockIdx.x * run;
    const int i1 = (i0 + run < sl.n_tiles) ? i0 + run : sl.n_tiles;
    const int tid = threadIdx.x;
    const int T = T_ > 0 ? T_ : a.T, B = a.B, K = a.K;
    const int S = SM > 0 ? SM : a.S;
    const int G = kHeadDim / B;

    const bool vside = blockIdx.z != 0;                                  // uniform
    CacheSide cs;
    constexpr int kCodeBytes = (FMT & kFmtInt4) ? 64 : 32, kScaleBytes = (FMT & kFmtE4M3) ? 1 : 2;
    cs.ids = (vside ? a.v_ids : a.k_ids) + (int64_t)h * a.kv_stride * S * (a.id_wide ? 2 : 1);
    cs.codes = (vside ? a.v_codes : a.k_codes) + (int64_t)h * a.kv_stride * T * kCodeBytes;
    cs.scales = reinterpret_cast<const uint8_t *>(vside ? a.v_scales : a.k_scales) + (int64_t)h * a.kv_stride * T * G * kScaleBytes;
    cs.cent = (vside ? a.v_cent : a.k_cent) + (int64_t)h * a.chunk_stride * S * K * kHeadDim;
    cs.wide = a.id_wide;

    const int c8 = tid & 15, tp = tid >> 4;
    const int g = (c8 * 8) / B;
    const int tok = 2 * tp;
    // position of the token pair in a transposed V row (the order in which a lane's soft-max
    // values feed the PV contraction): token 16 s + 8 a + 4 hh + e sits at 16 s + 8 hh + 4 a + e
    const int v_pos = 16 * (tok >> 4) + 8 * ((tok >> 2) & 1) + 4 * ((tok >> 3) & 1) + (tok & 3);
    uint16_t *img = (vside ? sl.vimg : sl.kimg) + (int64_t)h * sl.tiles_cap * kImgElems;

    uint32_t id[2];
    Raw<TM, SM> r;
    uint4 rp[2];
    auto fetch = [&](const Tile &t) {                                    // ids of `t` are in id
        load_raw<T_, TM, SM, FMT>(cs, t, tp, c8, T, G, g, K, S, id, r);
        if (ROPE && !vside) load_rope(a.rope, t, tp, c8, rp);
    };
    if (i0 >= i1) return;                                                // uniform
    // raw data one tile ahead (requested as soon as the registers are free), ids two tiles ahead
    Tile t = slab_tile(a, sl, i0);
    load_ids(cs, t, tp, S, a.id_wide, id);
    fetch(t);
    Tile tn = slab_tile(a, sl, i0 + 1 < i1 ? i0 + 1 : sl.n_tiles);
    load_ids(cs, tn, tp, S, a.id_wide, id);
    for (int i = i0; i < i1; ++i) {
        float accA[8], accB[8];
        dequant2x8<T_, TM, SM, FMT>(r, T, accA, accB);
        if (ROPE && !vside) { rope_rotate8(accA, rp[0]); rope_rotate8(accB, rp[1]); }
        fetch(tn);                                                       // tile i + 1 (its ids arrived an iteration ago)
        tn = slab_tile(a, sl, i + 2 < i1 ? i + 2 : sl.n_tiles);
        load_ids(cs, tn, tp, S, a.id_wide, id);
        uint16_t *it = img + (int64_t)i * kImgElems;
        if (!vside) {
            *reinterpret_cast<uint4 *>(it + (tok + 0) * kHeadDim + c8 * 8) = pack_bf16x8(accA);
            *reinterpret_cast<uint4 *>(it + (tok + 1) * kHeadDim + c8 * 8) = pack_bf16x8(accB);
            continue;
        }
        // rows 8 c8 .. 8 c8 + 7; the 16-byte group of a row is XOR-ed with (row / 8) & 7 so that the 16
        // lanes that write the same column of 16 different row groups spread over the banks
        uint16_t *vt = Vt + (((v_pos >> 3) ^ (c8 & 7)) * 8 + (v_pos & 7));
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            // round to bf16 (the decoder's output), then to f16 (exact in range): channels e, e+1
            const uint32_t pa = pack_bf16x2(accA[e], accA[e + 1]);
            const uint32_t pb = pack_bf16x2(accB[e], accB[e + 1]);
            *reinterpret_cast<uint32_t *>(vt + (c8 * 8 + e) * kVtPitch) = pack_f16x2_rtz(bf16_lo(pa), bf16_lo(pb));
            *reinterpret_cast<uint32_t *>(vt + (c8 * 8 + e + 1) * kVtPitch) = pack_f16x2_rtz(bf16_hi(pa), bf16_hi(pb));
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int p = tid + k * kAtThreads;                          // 16-byte piece: row p / 8, group p % 8
            *reinterpret_cast<uint4 *>(it + p * 8) =
                *reinterpret_cast<const uint4 *>(Vt + (p >> 3) * kVtPitch + (((p & 7) ^ ((p >> 6) & 7)) * 8));
        }
        __syncthreads();                                                 // Vt is rewritten by the next tile
    }
}

// ---------------------------------------------------------------------------------------------
// The tile loop.  Per wavefront and tile there are 32 contractions (32 cycles of the matrix pipe
// each) and about 120 vector instructions, the 32 exponentials among them costing four times the
// others.  One kind after the other, the two add up: the matrix pipe works beside the vector ALU
// only on contractions issued before, so the kinds have to alternate.  The scores of tile i + 1 and
// the probabilities of tile i do not depend on each other, nor do PV of a tile's first tokens and
// the probabilities of its last:
//   slots  0..15   scores of tile i + 1        beside   probabilities 0 .. kP1 - 1 of tile i
//   slots 16..31   PV of tile i, token order   beside   the other probabilities, then the maxima of tile i + 1
// A slot is one contraction, one operand read (kAhead slots ahead of its use) and its share of the
// vector work; no instruction moves across a slot's end.
// What bounds it is the power cap: 4680 queries x 12 heads x 748800 tokens take 22.5 ms (tile decode 1.75
// of it) against 23.2 ms with the kinds one after the other, but 17.3 against 19.2 ms when all queries are
// zero, and the clock stands at 1.7-1.9 GHz instead of 2.4.  (A large bf16 product on this card:
// 1.58 PFLOP/s, 2.13 on zeros.)  At equal clocks the parks cost most: 2.3 ms when they stand
// together at the end of the tile, half of that spread over slots 9..15.
// ---------------------------------------------------------------------------------------------
constexpr int kAhead = 4;          // operand fragments in flight
constexpr int kP1 = 16;            // probabilities taken beside the scores (12, 20 and 24: 0-2 % slower)
constexpr int kP2Slots = 10;       // slots of PV that carry the others (PV wants them by slots 24 and 28)
constexpr int kSlabKBufs = 3;      // K tiles in LDS: read, next (its first fragments are read before the barrier), being written
constexpr size_t kSlabSmem = ((size_t)kSlabKBufs * kKtElems + 2 * kVtElems) * sizeof(uint16_t);

// probabilities whose exponential is issued by the end of slot k
constexpr int probs_done(int k) {
    return k < 0 ? 0 : k < 16 ? (k + 1) * kP1 / 16 : k >= 15 + kP2Slots ? 32 : kP1 + (k - 15) * (32 - kP1) / kP2Slots;
}
static_assert(probs_done(16 - 3) >= 8 && probs_done(20 - 3) >= 16 && probs_done(24 - 3) >= 24 && probs_done(28 - 3) >= 32,
              "PV would read probabilities that are not there");

// scores of the next tile that have gone into its maximum by the end of slot k: the first block's
// contractions are slots 0..7, the second's 8..15, and a result is there two slots later
constexpr int maxima_done(int k) { return k < 9 ? 0 : k <= 16 ? 2 * (k - 8) : k < 18 ? 16 : k < 26 ? 16 + 2 * (k - 17) : 32; }
constexpr int kMaxSlot = 27;       // the maximum over both lane halves
constexpr int kParkSlot = 9;       // the four pieces of the copy: slots 9, 11, 13, 15

template <int A, int B_, class F>
__device__ __forceinline__ void static_for(F &&f) {
    if constexpr (A < B_) { f(std::integral_constant<int, A>{}); static_for<A + 1, B_>(f); }
}

// No instruction: the value is computed no later than here (it would otherwise move to its first use,
// behind the contractions it is meant to run beside).
template <class T> __device__ __forceinline__ void keep_here(T &v) { asm volatile("" : "+v"(v)); }

// Slot k's share of the probabilities exp2(S scale2 - m): argument, exponential, pair rounded to f16
// and sum each one slot behind the one before, so that nothing waits for a result just issued.
// Probability e belongs to score register e of the lane (two blocks of 16).  The normaliser is the
// sum of the f16 values that the PV contraction uses.
template <int k>
__device__ __forceinline__ void slab_probs(const floatx16_t (&S)[2], float scale2, float m, float (&x)[32],
                                           uint32_t (&p)[16], float &l) {
    constexpr int e0 = probs_done(k - 3), e1 = probs_done(k - 2), e2 = probs_done(k - 1), e3 = probs_done(k), e4 = probs_done(k + 1);
    const halfx2_t ones = {(_Float16)1.0f, (_Float16)1.0f};
#pragma unroll
    for (int e = k == 0 ? 0 : e3; e < e4; ++e) x[e] = __builtin_fmaf(S[e >> 4][e & 15], scale2, -m);
#pragma unroll
    for (int e = e2; e < e3; ++e) { x[e] = __builtin_amdgcn_exp2f(x[e]); keep_here(x[e]); }
#pragma unroll
    for (int j = e1 / 2; j < e2 / 2; ++j) { p[j] = pack_f16x2_rne(x[2 * j], x[2 * j + 1]); keep_here(p[j]); }
#pragma unroll
    for (int j = e0 / 2; j < e1 / 2; ++j) { l = __builtin_amdgcn_fdot2(__builtin_bit_cast(halfx2_t, p[j]), ones, l, false); keep_here(l); }
}

template <int k>
__device__ __forceinline__ void slab_maxima(const floatx16_t (&N)[2], float &nmax) {
#pragma unroll
    for (int e = maxima_done(k - 1); e < maxima_done(k); ++e) nmax = fmaxf(nmax, N[e >> 4][e & 15]);
    if (maxima_done(k - 1) < maxima_done(k)) keep_here(nmax);
}

__device__ __forceinline__ bf16x8_t slab_kfrag(const uint16_t *krow, int i) {          // krow: tile + col * pitch + half * 8
    return *reinterpret_cast<const bf16x8_t *>(krow + (i >> 3) * 32 * kKtPitch + (i & 7) * 16);
}
// i: 16-token step i / 4, channel block i % 4
__device__ __forceinline__ halfx8_t slab_vfrag(const uint16_t *vt, int col, int half, int i) {
    const int mb = i & 3, st = i >> 2;
    return *reinterpret_cast<const halfx8_t *>(vt + (mb * 32 + col) * kVtPitch + (((2 * st + half) ^ (mb * 2)) * 8));
}

// Scores the lane's query must not see: tokens at or beyond `limit` of the tile.
__device__ __forceinline__ void slab_mask(floatx16_t (&S)[2], int half, int limit) {
    limit -= half * 4;
    keep_here(limit);                                                    // the comparisons, and what they need, stay in the rare branch
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (nb * 32 + (r >> 2) * 8 + (r & 3) >= limit) S[nb][r] = -INFINITY;
}

// The running maximum of the lane's query with the lane halves' maxima of a tile (the scale is
// positive: order kept).
__device__ __forceinline__ float slab_new_max(float tmax, float scale2, float m) {
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(tmax), __float_as_uint(tmax), false, false);
    return fmaxf(m, fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1])) * scale2);
}
// What was summed under the old maximum, brought to the new one (skipped when no maximum moved).
__device__ __forceinline__ void slab_rescale(float m_new, float &m, float &l, floatx16_t (&O)[4]) {
    if (__ballot(m_new > m)) {                                           // uniform
        const float alpha = __builtin_amdgcn_exp2f(m - m_new);
        l *= alpha;
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) O[mb][r] *= alpha;
    }
    m = m_new;
}

// The running state of a workgroup's queries between slabs, or behind its part.
template <bool PARTS>
__device__ __forceinline__ float *slab_state(const AttnArgs &a, const SlabArgs &sl, int n_qblocks, const Place &at) {
    if (PARTS) return part_state_of(a, n_qblocks, at.h, at.qblock, at.part);
    return sl.state + ((int64_t)at.h * n_qblocks + at.qblock) * kStateFloats * kAtThreads + threadIdx.x;
}

// One workgroup = 8 wavefronts = 256 queries of one unit, over the tiles of one slab.
// QL: a prefix length per query (a.q_len): scores beyond the lane's prefix are masked in the tiles
// at or past the shortest prefix of the wavefront, and the workgroup stops at the longest prefix
// among its 256 queries.
// PARTS: the tiles are dealt to several workgroups per query block (a.parts).
template <bool QL, bool PARTS>
__device__ __forceinline__ void attend_slab(const AttnArgs &a, const SlabArgs &sl, int n_qblocks, Place at, Place &kept, unsigned char *smem) {
    uint16_t *Kt = reinterpret_cast<uint16_t *>(smem);                  // [3][64][136] bf16
    uint16_t *Vt = Kt + kSlabKBufs * kKtElems;                          // [2][128][72] f16, transposed
    if (threadIdx.x == 0) kept = at;                                    // for the end of the kernel
    const int h = at.h, qblock = at.qblock;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int col = lane & 31, half = lane >> 5;
    const int64_t qrow = (int64_t)qblock * kAtQPerBlock + wave * 32 + col;
    const bool qvalid = qrow < a.n_q;
    // no query: helps with the copy only
    const bool idle = PARTS && !a.whole && (int64_t)qblock * kAtQPerBlock + __builtin_amdgcn_readfirstlane(wave) * 32 >= a.n_q;

    uint4 qa[8];
    {
        const bf16_t *qp = a.q + ((int64_t)h * a.n_q + qrow) * kHeadDim + half * 8;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
            qa[kk] = qvalid ? *reinterpret_cast<const uint4 *>(qp + kk * 16) : make_uint4(0u, 0u, 0u, 0u);
    }
    floatx16_t O[4];
    float m = kNoScore, l = 0.0f;
    if (sl.first) {
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) O[mb][r] = 0.0f;
    } else {
        const float *st = slab_state<PARTS>(a, sl, n_qblocks, at);
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
            for (int r = 0; r < 16; ++r) O[mb][r] = st[(mb * 16 + r) * kAtThreads];
        m = st[64 * kAtThreads];
        l = st[65 * kAtThreads];
    }
    const float scale2 = a.scale * 1.4426950408889634f;
    int qlen = 0x7fffffff, wmin = 0x7fffffff, wgmax = 0x7fffffff;
    if (QL) {
        __shared__ int bmax;
        if (tid == 0) bmax = 0;
        __syncthreads();
        const int nk = (int)a.n_kv;
        qlen = 0;
        if (qvalid) { const int v = a.q_len[qrow]; qlen = v < 0 ? 0 : (v > nk ? nk : v); }
        wmin = qvalid ? qlen : 0x7fffffff;
        int mx = qlen;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const int o = __shfl_xor(wmin, off, 64); wmin = o < wmin ? o : wmin;
            const int p = __shfl_xor(mx, off, 64); mx = p > mx ? p : mx;
        }
        if (lane == 0) atomicMax(&bmax, mx);
        __syncthreads();
        wgmax = bmax;
        wmin = __builtin_amdgcn_readfirstlane(wmin);
        if (PARTS) {                 // a part behind the longest prefix (its first tile is tile `part`): the join does not read it
            at.parts = __builtin_amdgcn_readfirstlane(block_parts(a, wgmax));
            if (at.part >= at.parts || (at.parts > 1 && at.part >= tiles_of(a, wgmax))) return;                 // uniform
            if (tid == 0) kept.parts = at.parts;
        }
    }

    // a thread's four 16-byte pieces of a tile: K pieces tid, tid + 512 (row p / 16, group p % 16),
    // V pieces tid, tid + 512 (row p / 8, group p % 8, XOR-ed with the row's key in LDS)
    const uint16_t *kimg = sl.kimg + (int64_t)h * sl.tiles_cap * kImgElems + tid * 8;
    const uint16_t *vimg = sl.vimg + (int64_t)h * sl.tiles_cap * kImgElems + tid * 8;
    auto k_off = [&](int p) { return (p >> 4) * kKtPitch + (p & 15) * 8; };
    auto v_off = [&](int p) { const int row = p >> 3; return row * kVtPitch + (((p & 7) ^ ((row >> 5) * 2)) * 8); };
    const int koff[2] = {k_off(tid), k_off(tid + kAtThreads)};
    const int voff[2] = {v_off(tid), v_off(tid + kAtThreads)};
    const int n = sl.n_tiles;                                           // >= 1
    // tiles this workgroup attends to: those that start before its longest prefix
    int ne = n;
    if (QL) {
        const int64_t rel = (int64_t)wgmax - (int64_t)sl.c0 * a.chunk_len;
        const int64_t full = rel <= 0 ? 0 : rel / a.chunk_len;
        const int64_t e = rel <= 0 ? 0 : full * sl.tpc + (rel - full * a.chunk_len + kAtKv - 1) / kAtKv;
        ne = e < n ? (int)e : n;
    }
    const int parts = PARTS ? at.parts : 1;
    // this part's share of them: tiles i0, i0 + parts, ... of the slab (part g % parts has tile g of the cache)
    const int i0 = !PARTS ? 0 : (int)(((int64_t)at.part + parts - (int64_t)sl.c0 * sl.tpc % parts) % parts);
    const int count = i0 < ne ? (ne - i0 + parts - 1) / parts : 0;
    // the slab's index of the part's j-th tile; past the end: the last tile (never used)
    auto clampt = [&](int j) { return j < count ? i0 + j * parts : n - 1; };
    uint4 gk0, gk1, gv0, gv1;                                           // the pieces on their way to LDS
    auto fetch_k = [&](int i) {
        const uint16_t *kp = kimg + (int64_t)clampt(i) * kImgElems;
        gk0 = *reinterpret_cast<const uint4 *>(kp);
        gk1 = *reinterpret_cast<const uint4 *>(kp + kAtThreads * 8);
    };
    auto fetch_v = [&](int i) {
        const uint16_t *vp = vimg + (int64_t)clampt(i) * kImgElems;
        gv0 = *reinterpret_cast<const uint4 *>(vp);
        gv1 = *reinterpret_cast<const uint4 *>(vp + kAtThreads * 8);
    };
    auto park_k = [&](uint16_t *kt) {
        *reinterpret_cast<uint4 *>(kt + koff[0]) = gk0;
        *reinterpret_cast<uint4 *>(kt + koff[1]) = gk1;
    };
    auto park_v = [&](uint16_t *vt) {
        *reinterpret_cast<uint4 *>(vt + voff[0]) = gv0;
        *reinterpret_cast<uint4 *>(vt + voff[1]) = gv1;
    };
    // one piece to its place in `tile`, and the same piece (0 or 1) of tile `next` requested
    auto park = [&](uint16_t *tile, int off, const uint16_t *img, uint4 &piece, int next, int half_) {
        *reinterpret_cast<uint4 *>(tile + off) = piece;
        piece = *reinterpret_cast<const uint4 *>(img + (int64_t)clampt(next) * kImgElems + half_ * kAtThreads * 8);
    };
    // the tile whose scores are taken: its first token and the end of its chunk
    const int nkv = (int)a.n_kv, clen = a.chunk_len < a.n_kv ? (int)a.chunk_len : nkv;
    int tb = sl.c0 * clen, ti = i0;                                     // its chunk's first token, its place in the chunk
    int t0, cend;
    auto place = [&]() {
        if (ti >= sl.tpc) { const int c = ti / sl.tpc; tb += c * clen; ti -= c * sl.tpc; }
        t0 = tb + ti * kAtKv;
        cend = nkv - tb < clen ? nkv : tb + clen;
    };
    // scores of the tokens that the tile does not hold or that the lane's query does not see
    auto mask = [&](floatx16_t (&S)[2]) {                               // true: some were
        const bool tail = cend - t0 < kAtKv;                            // uniform: last tile of a chunk
        const bool ends = QL && t0 + kAtKv > wmin;                      // uniform: some query of the wavefront ends here
        if (tail) slab_mask(S, half, cend - t0);
        if (ends) slab_mask(S, half, qlen - t0);
        return tail || ends;
    };
    const uint16_t *krow = Kt + col * kKtPitch + half * 8;
    const floatx16_t zero = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    if (count > 0) {                                                    // uniform
        place();
        fetch_k(0); park_k(Kt);
        fetch_k(1); park_k(Kt + kKtElems);
        fetch_k(2); park_k(Kt + 2 * kKtElems);
        fetch_v(0); park_v(Vt);
        __syncthreads();
        // A wavefront without queries (the last block of a unit) does the copy and the barriers of the steps below only:
        // its SIMD is the other one's, and the energy that it saves is the clock of all (1560 queries, six blocks and 24
        // rows, 12 heads x 31997 tokens 405 -> 392 us; undivided blocks, of which few are such, gain nothing: 4680
        // queries over 748800 tokens 22.48 -> 22.88 ms).
        if (idle) {                                                     // uniform per wavefront
            fetch_v(1);
            fetch_k(3);
            __syncthreads();
            int kb = 0;
            for (int i = 0; i + 1 < count; ++i) {
                uint16_t *vt = Vt + ((i & 1) ^ 1) * kVtElems, *kt = Kt + kb;
                park(vt, voff[0], vimg, gv0, i + 2, 0);
                park(vt, voff[1], vimg, gv1, i + 2, 1);
                park(kt, koff[0], kimg, gk0, i + 4, 0);
                park(kt, koff[1], kimg, gk1, i + 4, 1);
                kb = kb == 2 * kKtElems ? 0 : kb + kKtElems;
                __syncthreads();
            }
            return;
        }
        floatx16_t Sa[2], Sb[2];
        bf16x8_t kf[kAhead];                                            // first fragments of the next tile's scores
#pragma unroll
        for (int i = 0; i < 16; ++i)
            Sa[i >> 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(slab_kfrag(krow, i), __builtin_bit_cast(bf16x8_t, qa[i & 7]),
                                                                (i & 7) ? Sa[i >> 3] : zero, 0, 0, 0);
        mask(Sa);
        float tmax = -INFINITY;
#pragma unroll
        for (int e = 0; e < 32; ++e) tmax = fmaxf(tmax, Sa[e >> 4][e & 15]);
        slab_rescale(slab_new_max(tmax, scale2, m), m, l, O);
        fetch_v(1);
        fetch_k(3);
#pragma unroll
        for (int i = 0; i < kAhead; ++i) kf[i] = slab_kfrag(krow + kKtElems, i);
        __syncthreads();                                                // tile 3 overwrites K tile 0
        // offsets of the K buffers: tile i + 1, i + 2, and the one that takes i + 3
        int kb1 = kKtElems, kb2 = 2 * kKtElems, kb3 = 0;
        // scores of tile i + 1 into N, probabilities (scores S) and PV of tile i
        auto step = [&](int i, floatx16_t (&S)[2], floatx16_t (&N)[2], int vb) {
            ti += parts;
            place();
            const uint16_t *kr = krow + kb1, *vt = Vt + vb * kVtElems;
            float x[32];
            uint32_t p[16];
            bf16x8_t kq[16];
            halfx8_t vq[16];
            float nmax = -INFINITY, m_new = 0.0f;
#pragma unroll
            for (int j = 0; j < kAhead; ++j) kq[j] = kf[j];
            static_for<0, 16>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                N[k >> 3] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kq[k], __builtin_bit_cast(bf16x8_t, qa[k & 7]),
                                                                   (k & 7) ? N[k >> 3] : zero, 0, 0, 0);
                if constexpr (k + kAhead < 16) kq[k + kAhead] = slab_kfrag(kr, k + kAhead);
                else vq[k + kAhead - 16] = slab_vfrag(vt, col, half, k + kAhead - 16);
                slab_probs<k>(S, scale2, m, x, p, l);
                slab_maxima<k>(N, nmax);
                // V tile i - 1 and K tile i were last read an iteration ago: i + 1 and i + 3 take their places,
                // and i + 2 and i + 4 are requested into the registers that become free
                if constexpr (k == kParkSlot) park(Vt + (vb ^ 1) * kVtElems, voff[0], vimg, gv0, i + 2, 0);
                if constexpr (k == kParkSlot + 2) park(Vt + (vb ^ 1) * kVtElems, voff[1], vimg, gv1, i + 2, 1);
                if constexpr (k == kParkSlot + 4) park(Kt + kb3, koff[0], kimg, gk0, i + 4, 0);
                if constexpr (k == kParkSlot + 6) park(Kt + kb3, koff[1], kimg, gk1, i + 4, 1);
                __builtin_amdgcn_sched_barrier(0);
            });
            if (mask(N)) {                                              // uniform
                nmax = -INFINITY;
#pragma unroll
                for (int e = 0; e < maxima_done(15); ++e) nmax = fmaxf(nmax, N[e >> 4][e & 15]);
            }
            static_for<16, 32>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                constexpr int st = (k - 16) >> 2, mb = (k - 16) & 3;
                const uint4 pb = make_uint4(p[4 * st], p[4 * st + 1], p[4 * st + 2], p[4 * st + 3]);
                O[mb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vq[k - 16], __builtin_bit_cast(halfx8_t, pb), O[mb], 0, 0, 0);
                if constexpr (k + kAhead < 32) vq[k + kAhead - 16] = slab_vfrag(vt, col, half, k + kAhead - 16);
                else kf[k + kAhead - 32] = slab_kfrag(krow + kb2, k + kAhead - 32);
                slab_probs<k>(S, scale2, m, x, p, l);
                slab_maxima<k>(N, nmax);
                if constexpr (k == kMaxSlot) m_new = slab_new_max(nmax, scale2, m);
                __builtin_amdgcn_sched_barrier(0);
            });
            slab_rescale(m_new, m, l, O);
            __syncthreads();
            const int kt = kb1;
            kb1 = kb2; kb2 = kb3; kb3 = kt;
        };
        // the last tile: probabilities and PV
        auto finish = [&](floatx16_t (&S)[2], int vb) {
            const uint16_t *vt = Vt + vb * kVtElems;
            uint4 pb[4];
#pragma unroll
            for (int st = 0; st < 4; ++st) {
                float x[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) x[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(S[st >> 1][(st & 1) * 8 + e], scale2, -m));
                pb[st] = make_uint4(pack_f16x2_rne(x[0], x[1]), pack_f16x2_rne(x[2], x[3]),
                                    pack_f16x2_rne(x[4], x[5]), pack_f16x2_rne(x[6], x[7]));
                l = sum_f16_pairs(pb[st], l);
            }
#pragma unroll
            for (int i = 0; i < 16; ++i)
                O[i & 3] = __builtin_amdgcn_mfma_f32_32x32x16_f16(slab_vfrag(vt, col, half, i),
                                                                 __builtin_bit_cast(halfx8_t, pb[i >> 2]), O[i & 3], 0, 0, 0);
        };
        int i = 0;
        for (; i + 2 < count; i += 2) {
            step(i, Sa, Sb, 0);
            step(i + 1, Sb, Sa, 1);
        }
        if (i + 1 < count) {
            step(i, Sa, Sb, 0);
            finish(Sb, 1);
        } else {
            finish(Sa, 0);
        }
    }
    if (count == 0) __syncthreads();                                    // uniform: `kept` has been written
    const Place end = kept.uniform();
    const AttnArgs &e = late_args();
    const int te = late_thread();
    const int64_t row = (int64_t)end.qblock * kAtQPerBlock + (te >> 6) * 32 + (te & 31);
    const bool stored = row < e.n_q;
    if (sl.last && end.parts == 1) store_result(e, end.h, row, stored && (!QL || qlen > 0), stored, (te >> 5) & 1, O, m, l);
    else store_state(slab_state<PARTS>(e, sl, n_qblocks, end), O, m, l);
}

// A whole block takes the form that has no parts (12 heads x 4680 queries that all see 37440 tokens 1090 us, 1126 with parts).
template <bool QL, bool PARTS>
__global__ __launch_bounds__(kAtThreads, 2)
void attn_slab_kernel(AttnArgs a, SlabArgs sl, int n_qblocks, int n_blocks, int blocks_per_xcd) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ Place kept;
    Place at;
    if (!block_of<QL ? kLengthsParted : kPlain>(a, n_qblocks, n_blocks, blocks_per_xcd, blockIdx.x, at)) return;     // uniform, before any barrier
    if (PARTS && at.parts > 1) attend_slab<QL, PARTS>(a, sl, n_qblocks, at, kept, smem);
    else attend_slab<QL, false>(a, sl, n_qblocks, at, kept, smem);
}

// ---- host side ---------------------------------------------------------------------------------
template <int T_, int SM, int FMT>
static hipError_t launch_slab_decode_t(const AttnArgs &a, const SlabArgs &sl, hipStream_t s) {
    // Tiles per workgroup: eight (a workgroup starts with a chain of dependent loads; 16, or as many as
    // fill the chip a whole number of times, make no difference), fewer while the chip is not full once:
    // 600 queries of one head over 4096 tokens 39 -> 34 us
    const int64_t tiles = (int64_t)sl.n_tiles * a.H;
    const int run = tiles >= 8 * 512 ? 8 : (int)((tiles + 511) / 512);
    dim3 grid((unsigned)((sl.n_tiles + run - 1) / run), (unsigned)a.H, 2);
    if (a.rope) hipLaunchKernelGGL((slab_decode_kernel<T_, SM, FMT, true>), grid, dim3(kAtThreads), 0, s, a, sl, run);
    else hipLaunchKernelGGL((slab_decode_kernel<T_, SM, FMT, false>), grid, dim3(kAtThreads), 0, s, a, sl, run);
    return hipGetLastError();
}

// instances with the round and stage counts fixed at compile time for the paper's forms, run-time
// counts for everything else
template <int FMT>
static hipError_t launch_slab_decode_f(const AttnArgs &a, const SlabArgs &sl, hipStream_t s) {
    if (a.S == 1) {
        if constexpr (FMT == 0) {
            switch (a.T) {
                case 1: return launch_slab_decode_t<1, 1, FMT>(a, sl, s);
                case 2: return launch_slab_decode_t<2, 1, FMT>(a, sl, s);
                case 3: return launch_slab_decode_t<3, 1, FMT>(a, sl, s);
                case 4: return launch_slab_decode_t<4, 1, FMT>(a, sl, s);
                default: break;
            }
            return launch_slab_decode_t<0, 1, FMT>(a, sl, s);
        } else {
            if (a.T == 1) return launch_slab_decode_t<1, 1, FMT>(a, sl, s);
            return launch_slab_decode_t<0, 1, FMT>(a, sl, s);
        }
    }
    if (a.T == 1 && a.S == 4 && !a.id_wide) return launch_slab_decode_t<1, 4, FMT>(a, sl, s);
    if (a.T == 1 && a.S == 2 && !a.id_wide) return launch_slab_decode_t<1, 2, FMT>(a, sl, s);
    return launch_slab_decode_t<0, 0, FMT>(a, sl, s);
}

static hipError_t launch_slab_decode(const AttnArgs &a, const SlabArgs &sl, hipStream_t s) {
    switch (a.fmt) {
        case 0: return launch_slab_decode_f<0>(a, sl, s);
        case kFmtE4M3: return launch_slab_decode_f<kFmtE4M3>(a, sl, s);
        case kFmtInt4: return launch_slab_decode_f<kFmtInt4>(a, sl, s);
        default: return launch_slab_decode_f<kFmtInt4 | kFmtE4M3>(a, sl, s);
    }
}

size_t attn_slab_state_bytes(int H, int64_t n_q) {
    const int64_t nqb = (n_q + kAtQPerBlock - 1) / kAtQPerBlock;
    return ((size_t)nqb * H * kStateFloats * kAtThreads * sizeof(float) + 255) / 256 * 256;
}
size_t attn_slab_chunk_bytes(int H, int64_t chunk_len) {
    const int64_t tpc = (chunk_len + kAtKv - 1) / kAtKv;
    return (size_t)H * tpc * 2 * kImgElems * sizeof(uint16_t);
}

// Whether the shared-tile path serves this call with this workspace: more than one query block
// per unit (else nothing is shared) and room for at least one chunk's tiles (plus the running
// state when the cache needs more than one slab).
bool attn_slab_applicable(const AttnArgs &a, const void *ws, size_t ws_bytes) {
    if (!ws || a.n_q <= kAtQPerBlock) return false;
    const size_t chunk = attn_slab_chunk_bytes(a.H, a.chunk_len);
    if (ws_bytes >= chunk * (size_t)a.n_chunks) return true;
    const size_t state = attn_slab_state_bytes(a.H, a.n_q);
    return ws_bytes >= state + chunk;
}

hipError_t launch_attn_slab(const AttnArgs &a, void *ws, size_t ws_bytes, hipStream_t s) {
    const int64_t tpc = (a.chunk_len + kAtKv - 1) / kAtKv;
    const size_t chunk = attn_slab_chunk_bytes(a.H, a.chunk_len);
    const bool single = ws_bytes >= chunk * (size_t)a.n_chunks;
    const size_t state = single ? 0 : attn_slab_state_bytes(a.H, a.n_q);
    int64_t slab_chunks = single ? a.n_chunks : (int64_t)((ws_bytes - state) / chunk);
    if (slab_chunks < 1 || tpc * slab_chunks > 0x7fffffff) return hipErrorInvalidValue;
    if (slab_chunks > a.n_chunks) slab_chunks = a.n_chunks;

    const int form = (a.q_len ? 1 : 0) + (a.parts > 1 ? 2 : 0);
    typedef void (*slab_kernel_t)(AttnArgs, SlabArgs, int, int, int);
    static const slab_kernel_t kernels[4] = {attn_slab_kernel<false, false>, attn_slab_kernel<true, false>,
                                             attn_slab_kernel<false, true>, attn_slab_kernel<true, true>};
    static LdsHighWater lds_limit[4] = {};
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(kernels[form]), kSlabSmem, lds_limit[form]);
    if (e != hipSuccess) return e;
    const int64_t nqb = (a.n_q + kAtQPerBlock - 1) / kAtQPerBlock;
    const int64_t nb = (nqb * a.H - a.whole) * a.parts;                 // beside the whole blocks
    if (nb + a.whole > 0x7fffffff - 8) return hipErrorInvalidValue;
    const int bpx = (int)((nb + 7) / 8);
    if ((int64_t)bpx * 8 > nb + 7) return hipErrorInvalidValue;        // at most 7 surplus workgroups, which return at once

    SlabArgs sl{};
    unsigned char *base = static_cast<unsigned char *>(ws);
    sl.state = single ? nullptr : reinterpret_cast<float *>(base);      // of the blocks that are not divided
    sl.tiles_cap = tpc * slab_chunks;
    sl.kimg = reinterpret_cast<uint16_t *>(base + state);
    sl.vimg = sl.kimg + (size_t)a.H * sl.tiles_cap * kImgElems;
    sl.tpc = (int)tpc;
    for (int64_t c0 = 0; c0 < a.n_chunks; c0 += slab_chunks) {
        const int64_t c1 = (c0 + slab_chunks < a.n_chunks) ? c0 + slab_chunks : a.n_chunks;
        // tiles of chunks c0 .. c1-1: tpc each, fewer in the cache's last chunk when it is short
        const int64_t last_len = ((c1 * a.chunk_len < a.n_kv) ? c1 * a.chunk_len : a.n_kv) - (c1 - 1) * a.chunk_len;
        sl.c0 = (int)c0;
        sl.n_tiles = (int)((c1 - 1 - c0) * tpc + (last_len + kAtKv - 1) / kAtKv);
        sl.first = c0 == 0;
        sl.last = c1 == a.n_chunks;
        if ((e = launch_slab_decode(a, sl, s)) != hipSuccess) return e;
        hipLaunchKernelGGL(kernels[form], dim3((unsigned)(a.whole + bpx * 8)), dim3(kAtThreads), kSlabSmem, s, a, sl, (int)nqb, (int)nb, bpx);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace qvg
