// k-means update step (paper Sec. 4.1: the centroid is the mean of its group).
//
// The mean is defined with a fixed summation order - members in token order, fp64 -
// so that the result does not depend on scheduling.  The assignment leaves the unit's tokens sorted
// by cluster inside blocks of 256..1024 tokens (MemberLists), so that a cluster's members in token
// order are its segments of block 0, 1, ...  One wavefront per centroid adds them in fp64, divides by
// the count, rounds to fp32 and then to bf16: in token order for short lists, in interleaved partial
// sums for long ones (four per wavefront; the longest lists are spread over the wavefronts of the
// block) when a test on the members' exponents shows that no addition can round (then every order
// gives the same bits).  A group without members keeps its previous centroid.  The wavefront also
// leaves the split norm of its new centroid for the next assignment.
//
// A Lloyd iteration is therefore two launches.  A third one, a counting sort of the whole unit by a
// single workgroup (1024 threads), took 6.5 to 8 us of every iteration at 2 to 24 units of 4096 to
// 4680 tokens and 15 us at 80 units of 10800; sorting where the ids are made costs the assignment
// about 1 us.
#include <type_traits>

#include "qvg_kmeans.hpp"

namespace qvg {

// Member lists of ids that come from the caller: one workgroup per block of tokens.
template <bool WIDE>                       // 16-bit ids (more than 256 centroids)
__global__ __launch_bounds__(kAsgThreads)
void member_list_kernel(const uint8_t *ids, int64_t ids_stride, int64_t n_tokens, int K, MemberLists lists) {
    __shared__ uint16_t lid[kMaxTilesPerWave * kAsgThreads];
    __shared__ __align__(16) int scratch[kAsgWaves * kMaxClusters + 8];
    const int h = blockIdx.x;
    const int64_t t0 = (int64_t)blockIdx.y * lists.block;
    for (int i = threadIdx.x; i < lists.block; i += kAsgThreads) {
        uint32_t id = 0xffffu;
        if (t0 + i < n_tokens) { id = load_id(ids, (int64_t)h * ids_stride + t0 + i, WIDE ? 1 : 0); if (id >= (uint32_t)K) id = 0xffffu; }
        lid[i] = (uint16_t)id;
    }
    __syncthreads();
    const int64_t blk = (int64_t)h * lists.n_blocks + blockIdx.y;
    block_member_sort(lid, lists.block / kAsgThreads, K, scratch, lists.perm + blk * lists.block, lists.seg + blk * K);
}

hipError_t launch_member_lists(const uint8_t *ids, int64_t ids_stride, int64_t n_tokens, int H, int K, int id_wide,
                               const MemberLists &lists, hipStream_t s) {
    if (lists.n_blocks == 0) return hipSuccess;
    const dim3 grid((unsigned)H, (unsigned)lists.n_blocks);
    if (id_wide) hipLaunchKernelGGL(member_list_kernel<true>, grid, dim3(kAsgThreads), 0, s, ids, ids_stride, n_tokens, K, lists);
    else hipLaunchKernelGGL(member_list_kernel<false>, grid, dim3(kAsgThreads), 0, s, ids, ids_stride, n_tokens, K, lists);
    return hipGetLastError();
}

constexpr int kMeanWaves = 4;               // wavefronts (and centroids) of a block
constexpr int kMeanWideWaves = 16;          // wavefronts of a block with one centroid and long lists
constexpr int kMeanParallelMin = 96;        // member lists at least this long try the order-free path
constexpr int kMeanCoopMin = 192;           // lists at least this long are summed by the whole block
                                            // (with one centroid per block: every order-free list)
constexpr int kMeanSmallGrid = 2048;        // up to this many centroids in a launch: one block each
// With at most one such block per CU, and lists of 64 members or more on average, the block has 16
// wavefronts: 2 units x 4096 tokens, K = 16, I = 10 195 -> 176 us, 2 x 10800, K = 64, I = 3 80 -> 70 us (24 x 4680,
// K = 64, six blocks to a CU: 92 -> 171 us)
constexpr int kMeanWideGrid = 256, kMeanWideMin = 64;

// A cluster's members in up to 64 consecutive blocks of its unit: lane b holds block b's part.
struct Segments {
    int pre;           // members in the blocks before this one
    int delta;         // member m of this block is entry delta + m of the unit's perm
    int n;             // members in all of these blocks (uniform)
};
struct ListView {      // one unit's lists
    const uint16_t *perm; const uint32_t *seg;
    int block, n_blocks, K, probe;      // probe: first step of the search, the largest power of two below min(n_blocks, 64)
};
__device__ __forceinline__ ListView list_view(const MemberLists &l, int K, int h) {
    ListView v;
    v.perm = l.perm + (int64_t)h * l.n_blocks * l.block;
    v.seg = l.seg + (int64_t)h * l.n_blocks * K;
    v.block = l.block; v.n_blocks = l.n_blocks; v.K = K;
    v.probe = 32;
    while (v.probe > 0 && v.probe >= l.n_blocks) v.probe >>= 1;
    return v;
}
__device__ __forceinline__ Segments load_segments(const ListView &v, int j, int b0, int lane) {
    const int b = b0 + lane;
    const uint32_t w = b < v.n_blocks ? v.seg[(int64_t)b * v.K + j] : 0u;
    const int start = (int)(w & 0xffffu), cnt = (int)(w >> 16) - start;
    const int incl = scan64(cnt);
    Segments s;
    s.pre = incl - cnt;
    s.delta = b * v.block + start - s.pre;
    s.n = __builtin_amdgcn_readlane(incl, 63);
    return s;
}
// token index of member m (0 .. s.n - 1; a larger m gives some valid token) of the blocks b0 ..
__device__ __forceinline__ int member_token(const ListView &v, const Segments &s, int b0, int m) {
    m = m < s.n ? m : s.n - 1;
    int b = 0;                             // last block that starts at or before m: it is not empty
    for (int step = v.probe; step; step >>= 1) {                         // uniform
        const int p = __shfl(s.pre, b + step, 64);
        if (b + step < 64 && p <= m) b += step;
    }
    return (b0 + b) * v.block + (int)v.perm[(int64_t)__shfl(s.delta, b, 64) + m];
}

// Order-free partial sums of a member list: the wavefront takes the groups of 64 members
// first, first + step, .. of the list; lane = member slot (4) x 8 channels, 8 rows in
// flight per lane (ROWS = 16 where registers do not matter).  s: the lane's partial sums of its 8 channels; amax / amin: per 16-bit half the
// largest magnitude bits and the smallest non-zero magnitude bits minus one (0xffff: none).
template <int ROWS>
__device__ __forceinline__ void mean_partial(const bf16_t *xb, int64_t stride_token, const ListView &v, int j,
                                             Segments sg, int first, int step, int lane, double s[8], uint32_t amax[4],
                                             uint32_t amin[4]) {
    const int slot = lane >> 4;
    constexpr bool AHEAD = ROWS > 8;       // member indices requested a group ahead (two more registers)
    for (int b0 = 0;;) {
        int base = 64 * first;
        int nxt = (AHEAD && base < sg.n) ? member_token(v, sg, b0, base + lane) : 0;
        for (; base < sg.n; base += 64 * step) {
            int mine;                                                    // 64 member indices
            if (AHEAD) {
                mine = nxt;
                const int nb = base + 64 * step;
                if (nb < sg.n) nxt = member_token(v, sg, b0, nb + lane);
            } else {
                mine = member_token(v, sg, b0, base + lane);
            }
            const int cntm = (sg.n - base < 64) ? sg.n - base : 64;
            // slot s takes members s, s + 4, s + 8, .. of the group: ROWS rows in flight per lane
            for (int i0 = 0; 4 * i0 < cntm; i0 += ROWS) {
                uint4 row[ROWS];
#pragma unroll
                for (int i = 0; i < ROWS; ++i) {
                    const int u = 4 * (i0 + i) + slot;
                    const int idx = __shfl(mine, u & 63, 64);
                    row[i] = (u < cntm) ? *reinterpret_cast<const uint4 *>(xb + (int64_t)idx * stride_token)
                                        : make_uint4(0u, 0u, 0u, 0u);
                }
#pragma unroll
                for (int i = 0; i < ROWS; ++i) add_row(row[i], s, amax, amin);
            }
        }
        b0 += 64;
        if (b0 >= v.n_blocks) break;                                     // uniform: more than 64 blocks per unit
        sg = load_segments(v, j, b0, lane);
    }
}

// a new centroid's two channels of this lane: rounded to bf16, stored, and the split of its norm
__device__ __forceinline__ void store_centroid(const UpdateArgs &a, int h, int j, int lane, uint32_t packed) {
    *reinterpret_cast<uint32_t *>(a.cent_out + ((int64_t)h * a.K + j) * kHeadDim + lane * 2) = packed;
    if (a.nh3) {                                                         // uniform
        const double lo = (double)bf16_lo(packed), hi = (double)bf16_hi(packed);
        const double n2 = sum64_f64(lo * lo + hi * hi);
        if (lane == 0) a.nh3[(int64_t)h * k_padded(a.K) + j] = split_half_norm(n2);
    }
}

// the defining order: members in token order, two channels per lane
constexpr int kRowsAhead = 16;             // rows in flight (divides 64)
__device__ __forceinline__ uint32_t mean_token_order(const bf16_t *xu, int64_t stride_token, const ListView &v, int j,
                                                     Segments sg, int n, int lane) {
    double s0 = 0.0, s1 = 0.0;
    // bytes between tokens, or 0 where an offset inside the unit may not fit 32 bits
    const uint32_t row_bytes = stride_token * 2 * ((int64_t)v.n_blocks * v.block) < ((int64_t)1 << 31) ? (uint32_t)(stride_token * 2) : 0u;
    for (int b0 = 0;;) {
        for (int base = 0; base < sg.n; base += 64) {
            // 64 member indices at once, then broadcast lane by lane
            const int mine = member_token(v, sg, b0, base + lane);
            const int cntm = (sg.n - base < 64) ? sg.n - base : 64;
            // all lanes of `mine` hold tokens that exist, so that no load needs a predicate; as many rows at a
            // time as there are members, to the next power of two (always sixteen: 400 units x 1024 tokens,
            // K = 512, lists of two, 142 instead of 70 us)
            // (32-bit offsets where the unit's tokens allow them: a 64-bit product per row is eight scalar
            // instructions, and the scalar unit was busier than the vector one)
            auto rows = [&](auto count, auto narrow, int u0) {
                constexpr int R = decltype(count)::value;
                uint32_t wv[R];
#pragma unroll
                for (int u = 0; u < R; ++u) {
                    const int idx = __builtin_amdgcn_readlane(mine, u0 + u);
                    if (decltype(narrow)::value)
                        wv[u] = *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(xu) +
                                                                    (uint32_t)(idx * row_bytes + lane * 4));
                    else
                        wv[u] = *reinterpret_cast<const uint32_t *>(xu + (int64_t)idx * stride_token + lane * 2);
                }
#pragma unroll
                for (int u = 0; u < R; ++u)
                    if (u0 + u < cntm) { s0 += (double)bf16_lo(wv[u]); s1 += (double)bf16_hi(wv[u]); }
            };
            auto group = [&](auto narrow) {
                int u0 = 0;
                for (; u0 + kRowsAhead <= cntm; u0 += kRowsAhead) rows(std::integral_constant<int, kRowsAhead>{}, narrow, u0);
                const int left = cntm - u0;
                if (left > 8) rows(std::integral_constant<int, 16>{}, narrow, u0);
                else if (left > 4) rows(std::integral_constant<int, 8>{}, narrow, u0);
                else if (left > 2) rows(std::integral_constant<int, 4>{}, narrow, u0);
                else if (left > 0) rows(std::integral_constant<int, 2>{}, narrow, u0);
            };
            if (row_bytes) group(std::true_type{}); else group(std::false_type{});
        }
        b0 += 64;
        if (b0 >= v.n_blocks) break;                                     // uniform
        sg = load_segments(v, j, b0, lane);
    }
    const double c = (double)n;
    return pack_bf16x2((float)(s0 / c), (float)(s1 / c));
}

// One wavefront per centroid, CPB = four centroids per block (or CPB = 1, see below).  The defined result is the fp64 sum of
// the members in token order.  Short lists are summed exactly like that.  A long list is
// latency-bound that way (one dependent fp64 add per member), so it is first summed in
// interleaved partial sums, which give the same number whenever no addition rounds: every member
// is an integer multiple of 2^(emin-134) and every partial sum is below n * 256 * 2^(emax-134),
// with emin / emax the smallest / largest exponent field among the non-zero members of the
// channel, so if
//     ceil(log2 n) + 8 + emax - emin <= 53
// all partial sums of any order are exact in fp64.  The exponents are tracked alongside (packed
// 16-bit min / max of the magnitudes' bit patterns); a centroid with a channel that fails the
// test is summed again in token order.  Lists of medium length use the four member slots of their
// own wavefront; the longest ones (one cluster can hold a large share of a unit's tokens, e.g.
// in the later smoothing stages) are split over all wavefronts of the block, whose partial
// results meet in LDS.  Four wavefronts per block and at most 96 registers keep five wavefronts per
// SIMD resident, which is what the common case of many short lists lives on (four with sixteen rows in flight:
// a QVG-Pro chunk 690 against 666 us).  Six, at 80 registers, spill in the order-free sums, which a call
// of short lists hardly takes: there six are better (400 units x 4096 tokens, K = 256 147 -> 135 us, K = 512 202 ->
// 182; 24 x 4680 with K = 256 encoded in 134 instead of 138), but not where a few clusters hold most of a unit
// (that QVG-Pro chunk 848 -> 868, its later stages); eight wavefronts
// per block sum the longest lists faster and everything else slower.  The unit is the fastest
// grid index, as in the assignment: a unit's tokens and lists are then read through one XCD's L2 (the
// other way round that chunk takes 742 us).  A launch with few centroids (one chunk of a few heads) cannot
// fill the chip anyway and is a chain of dependent loads: there a block has ONE centroid (CPB = 1),
// every list long enough for the order-free path is spread over the block's four wavefronts, and
// 16 rows are in flight per lane (ROWS = 16: no occupancy to protect).
template <int CPB, int ROWS, int WAVES, int PER_SIMD>
__global__ __launch_bounds__(WAVES * 64, PER_SIMD)
void kmeans_mean_kernel(UpdateArgs a) {
    constexpr int kCoopMin = CPB == 1 ? kMeanParallelMin : kMeanCoopMin;
    __shared__ double part[WAVES][kHeadDim];
    __shared__ uint32_t pmx[WAVES][kHeadDim / 2], pmn[WAVES][kHeadDim / 2];
    __shared__ int list_len[WAVES];
    const int h = blockIdx.x, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j0 = blockIdx.y * CPB;
    const int j = j0 + wave;
    const int K = a.K;
    const bf16_t *xu = a.x + (int64_t)h * a.stride_head;
    const int slot = lane >> 4, c8 = lane & 15;
    const ListView v = list_view(a.lists, K, h);
    const bool own = wave < CPB && j < K;

    Segments sg = {0, 0, 0};
    int n = 0;                                                           // members of the wavefront's own centroid
    if (own) {
        sg = load_segments(v, j, 0, lane);
        n = sg.n;
        for (int b0 = 64; b0 < v.n_blocks; b0 += 64) n += load_segments(v, j, b0, lane).n;
        if (a.counts_out && lane == 0) a.counts_out[(int64_t)h * K + j] = n;
    }
    // the block's long lists, the same mask in every wavefront; a unit this short has none
    uint32_t coop = 0u;
    int len = 0;
    if (a.n_tokens >= kCoopMin) {                                        // uniform
        if (lane == 0) list_len[wave] = n;
        __syncthreads();
        len = list_len[lane < CPB ? lane : 0];
        coop = (uint32_t)__ballot(lane < CPB && len >= kCoopMin);
    }

    // ---- the wavefront's own centroid, unless its list is left to the whole block ----
    if (own && n < kCoopMin) {
        if (n == 0) {
            store_centroid(a, h, j, lane, *reinterpret_cast<const uint32_t *>(a.cent_prev + (int64_t)h * a.prev_stride + (int64_t)j * kHeadDim + lane * 2));
        } else {
            bool done = false;
            if (CPB > 1 && n >= kMeanParallelMin) {
                double s[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) s[i] = 0.0;
                uint32_t amax[4] = {0u, 0u, 0u, 0u}, amin[4] = {~0u, ~0u, ~0u, ~0u};
                mean_partial<ROWS>(xu + c8 * 8, a.stride_token, v, j, sg, 0, 1, lane, s, amax, amin);
                // the four slots hold partial results of the same channels: lanes l, l^16, l^32, l^48
                int lg = 0;
                while ((1 << lg) < n) ++lg;                                  // ceil(log2 n)
                bool ok = true;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    uint32_t mx = amax[e], mn = amin[e];
#pragma unroll
                    for (int off = 16; off <= 32; off <<= 1) {
                        mx = pk_max_u16(mx, __shfl_xor(mx, off, 64));
                        mn = pk_min_u16(mn, __shfl_xor(mn, off, 64));
                    }
                    ok = ok && mean_exact(mx, mn, lg);
                }
                if (__all(ok)) {
                    // every slot's lanes end up with the total of their 8 channels; lane (slot, c8) keeps
                    // channels 8 c8 + 2 slot, + 1 and hands them to lane 4 c8 + slot
                    uint32_t pk = 0u;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        double t0 = s[2 * e], t1 = s[2 * e + 1];
                        t0 += __shfl_xor(t0, 16, 64); t0 += __shfl_xor(t0, 32, 64);
                        t1 += __shfl_xor(t1, 16, 64); t1 += __shfl_xor(t1, 32, 64);
                        if (slot == e) pk = pack_bf16x2((float)(t0 / (double)n), (float)(t1 / (double)n));
                    }
                    store_centroid(a, h, j, lane, __shfl(pk, (lane & 3) * 16 + (lane >> 2), 64));
                    done = true;
                }
            }
            if (!done) store_centroid(a, h, j, lane, mean_token_order(xu, a.stride_token, v, j, sg, n, lane));
        }
    }

    // ---- the block's longest lists, one after the other, by all wavefronts (every wavefront of
    // the block takes the same branches: the list lengths are read by all of them) ----
    if (coop) for (int t = 0; t < CPB; ++t) {
        if (!(coop >> t & 1)) continue;
        const int nt = __builtin_amdgcn_readlane(len, t);
        const int jt = j0 + t;
        double s[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) s[i] = 0.0;
        uint32_t amax[4] = {0u, 0u, 0u, 0u}, amin[4] = {~0u, ~0u, ~0u, ~0u};
        const Segments st = load_segments(v, jt, 0, lane);
        mean_partial<ROWS>(xu + c8 * 8, a.stride_token, v, jt, st, wave, WAVES, lane, s, amax, amin);
#pragma unroll
        for (int i = 0; i < 8; ++i) {          // harmless if an addition rounds: then the result is discarded
            s[i] += __shfl_xor(s[i], 16, 64);
            s[i] += __shfl_xor(s[i], 32, 64);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
            for (int off = 16; off <= 32; off <<= 1) {
                amax[e] = pk_max_u16(amax[e], __shfl_xor(amax[e], off, 64));
                amin[e] = pk_min_u16(amin[e], __shfl_xor(amin[e], off, 64));
            }
        }
        if (slot == 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) part[wave][c8 * 8 + i] = s[i];
#pragma unroll
            for (int e = 0; e < 4; ++e) { pmx[wave][c8 * 4 + e] = amax[e]; pmn[wave][c8 * 4 + e] = amin[e]; }
        }
        __syncthreads();
        if (wave == t) {                      // the centroid's own wavefront (t < CPB): channels 2*lane, 2*lane+1
            double s0 = 0.0, s1 = 0.0;
            uint32_t mx = 0u, mn = ~0u;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                s0 += part[w][2 * lane];
                s1 += part[w][2 * lane + 1];
                mx = pk_max_u16(mx, pmx[w][lane]);
                mn = pk_min_u16(mn, pmn[w][lane]);
            }
            int lg = 0;
            while ((1 << lg) < nt) ++lg;
            uint32_t pk;
            if (__all(mean_exact(mx, mn, lg))) {
                const double c = (double)nt;
                pk = pack_bf16x2((float)(s0 / c), (float)(s1 / c));
            } else {
                pk = mean_token_order(xu, a.stride_token, v, jt, st, nt, lane);
            }
            store_centroid(a, h, jt, lane, pk);
        }
        __syncthreads();                      // the partial results are overwritten by the next list
    }
}

// Short lists: fewer members than this on average, in a first smoothing stage (what it leaves is centred, and one
// cluster of a later stage can hold most of it)
constexpr int64_t kMeanShort = 32;

hipError_t launch_update(const UpdateArgs &a, hipStream_t s) {
    const int64_t lists = (int64_t)a.K * a.H;
    const dim3 one((unsigned)a.H, (unsigned)a.K), four((unsigned)a.H, (unsigned)((a.K + kMeanWaves - 1) / kMeanWaves));
    if (lists <= kMeanWideGrid && a.n_tokens >= (int64_t)kMeanWideMin * a.K)
        hipLaunchKernelGGL((kmeans_mean_kernel<1, 16, kMeanWideWaves, kMeanWideWaves / 4>), one, dim3(kMeanWideWaves * 64), 0, s, a);
    else if (lists <= kMeanSmallGrid)
        hipLaunchKernelGGL((kmeans_mean_kernel<1, 16, kMeanWaves, kMeanWaves / 4>), one, dim3(kMeanWaves * 64), 0, s, a);
    else if (a.stage == 0 && a.n_tokens < kMeanShort * a.K)
        hipLaunchKernelGGL((kmeans_mean_kernel<kMeanWaves, 8, kMeanWaves, 6>), four, dim3(kMeanWaves * 64), 0, s, a);
    else
        hipLaunchKernelGGL((kmeans_mean_kernel<kMeanWaves, 8, kMeanWaves, 5>), four, dim3(kMeanWaves * 64), 0, s, a);
    return hipGetLastError();
}

}  // namespace qvg
