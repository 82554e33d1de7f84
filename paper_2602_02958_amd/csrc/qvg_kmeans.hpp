// Pieces shared by the assignment and the update kernels: sums and scans over a wavefront by
// data-parallel-primitive moves, and the stable sort of a workgroup's tokens by cluster.
#pragma once
#include "qvg_internal.hpp"

namespace qvg {

constexpr int kAsgThreads = 256;
constexpr int kAsgWaves = kAsgThreads / 64;
constexpr int kAsgTile = 64;                    // tokens per wavefront step (two MFMA column blocks)
constexpr int kMaxTilesPerWave = 4;             // steps of a wavefront: up to 1024 tokens per workgroup

// Sum over each aligned group of 16 lanes, every lane getting the total, by data-parallel-primitive
// moves (VALU; the general lane exchange goes through the LDS pipe and its latency, four times in
// a row per table piece).  Pairings: lane ^ 1, lane ^ 2, then the mirror images inside 8 and
// inside 16 lanes, whose partners hold what lane ^ 4 and lane ^ 8 hold, so the sums are those of
// the xor butterfly bit for bit.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double sum16_f64(double v) {
    v += dpp_f64<0xB1>(v);       // quad_perm [1,0,3,2]
    v += dpp_f64<0x4E>(v);       // quad_perm [2,3,0,1]
    v += dpp_f64<0x141>(v);      // row_half_mirror
    v += dpp_f64<0x140>(v);      // row_mirror
    return v;
}
__device__ __forceinline__ double readlane_f64(double v, int lane) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, lane);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), lane);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double sum64_f64(double v) {          // uniform result
    v = sum16_f64(v);
    return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}
// inclusive prefix sum over the wavefront: shifts inside rows of 16 lanes, then the last lane of row
// 0 / 2 into row 1 / 3 and the last lane of row 1 into rows 2 and 3
__device__ __forceinline__ int scan64(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);     // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);     // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);     // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);     // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);     // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);     // row_bcast:31
    return v;
}

typedef unsigned short ushort2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pk_max_u16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(ushort2_t, a), __builtin_bit_cast(ushort2_t, b)));
}
__device__ __forceinline__ uint32_t pk_min_u16(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(ushort2_t, a), __builtin_bit_cast(ushort2_t, b)));
}

// Two channels of a member into the lane's partial sums; mx / mn as amax / amin below.
__device__ __forceinline__ void add_pair(uint32_t w, double &s0, double &s1, uint32_t &mx, uint32_t &mn) {
    s0 += (double)bf16_lo(w);
    s1 += (double)bf16_hi(w);
    const uint32_t mag = w & 0x7fff7fffu;
    const ushort2_t one = {1, 1};
    mx = pk_max_u16(mx, mag);
    mn = pk_min_u16(mn, __builtin_bit_cast(uint32_t, (ushort2_t)(__builtin_bit_cast(ushort2_t, mag) - one)));   // zero -> 0xffff
}
// A member's 8 channels into the lane's partial sums s; amax / amin: per 16-bit half the largest magnitude bits and
// the smallest non-zero magnitude bits minus one (0xffff: none).
__device__ __forceinline__ void add_row(const uint4 &row, double s[8], uint32_t amax[4], uint32_t amin[4]) {
    const uint32_t w[4] = {row.x, row.y, row.z, row.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) add_pair(w[e], s[2 * e], s[2 * e + 1], amax[e], amin[e]);
}

// no partial sum of n members can round in fp64 when ceil(log2 n) + 8 + emax - emin <= 53; mx /
// mn: the packed largest / smallest-non-zero-minus-one magnitude bits of two channels
__device__ __forceinline__ bool mean_exact(uint32_t mx, uint32_t mn, int lg) {
    bool ok = true;
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
        const uint32_t big = (mx >> (16 * hf)) & 0xffffu, small1 = (mn >> (16 * hf)) & 0xffffu;
        if (small1 == 0xffffu) continue;                     // no non-zero member in this channel: the sum is zero
        const int eb = (int)(big >> 7) > 1 ? (int)(big >> 7) : 1;
        const int es = (int)((small1 + 1u) >> 7) > 1 ? (int)((small1 + 1u) >> 7) : 1;
        if (lg + 8 + eb - es > 53) ok = false;
    }
    return ok;
}

// s / n correctly rounded, r = 1 / n, for a sum s of bf16 numbers in fp64 and a whole n from 1 to 2^13.  q = s r is within 3/2 ulp
// of the quotient; s - n q is a multiple of q's last place below 2^14 of them, so the inner fma is exact, and what the
// outer one rounds is within 2^-52 ulp of s / n.  That rounds alike: s / n is no midpoint between two numbers (n times its 54
// significant bits does not fit s) and differs from each by 1 / 2n ulp at least.
__host__ __device__ __forceinline__ double quotient(double s, double n, double r) {
    const double q = s * r;
    return __builtin_fma(__builtin_fma(-n, q, s), r, q);
}

// Upper bound (one ulp up) of ||c||^2 from the split of -||c||^2 / 2; -0 for a zero row.
__host__ __device__ __forceinline__ float norm_bound(uint2 split) {
    const float hi = __builtin_bit_cast(float, split.x << 16), mid = __builtin_bit_cast(float, split.x & 0xffff0000u);
    const float lo = __builtin_bit_cast(float, split.y << 16);
    return -2.0f * ((hi + mid) + lo) * (1.0f + 0x1p-22f);
}
// A bound as a number that orders like it.  Without the sign: a -0 would be above every norm (64 zero rows of one
// wavefront then hid the table's largest norm from the certification).  Taken off here and not in norm_bound, where
// the assignment with 512 centroids comes out 4 % slower (400 units x 4096 tokens 568 against 589 us).
__host__ __device__ __forceinline__ uint32_t norm_order(float bound) { return __builtin_bit_cast(uint32_t, bound) & 0x7fffffffu; }

// Largest ||c||^2 that can matter to a token of squared norm xn at squared distance d2 from its leader:
// (||x|| + d)^2.  fast_sqrt: a square root good to a few ulp that may flush subnormals.  2^-120 stands
// in for a product below fp32's range (its root, 2^-60, is above the true one's 2^-63), which would
// otherwise halve the result for tokens of norm 2^-32 and less.
template <class F>
__host__ __device__ __forceinline__ float norm_reach(float xn, float d2, F fast_sqrt) {
    return (xn + d2 + 2.0f * fast_sqrt(__builtin_fmaf(xn, d2, 0x1p-120f))) * (1.0f + 0x1p-10f);
}

// LDS of block_member_sort: counters per wavefront and cluster, wavefront totals of the scan
__host__ __device__ inline size_t member_sort_bytes(int K) { return (size_t)(kAsgWaves * k_padded(K) + 8) * sizeof(int); }

// Stable sort of a workgroup's tokens by cluster (see MemberLists).  lid: the tokens' ids in LDS, 256 *
// tiles of them (0xffff: no token, or an id at or above K); scratch: member_sort_bytes(K) of LDS.
// Wavefront w takes the w-th contiguous range, 64 tokens at a time: lanes with equal ids are ranked by
// lane number (ballot-built peer masks), so equal ids keep their token order; after a scan over
// wavefronts and clusters every token knows its place.  Called by all threads, after a barrier that
// follows the last write to lid.
__device__ __forceinline__ void block_member_sort(const uint16_t *lid, int tiles, int K, int *scratch,
                                                  uint16_t *perm_out, uint32_t *seg_out) {
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int Kp = k_padded(K);
    int *cnt = scratch + w * Kp, *wtot = scratch + kAsgWaves * Kp;
    for (int k = lane; k < Kp; k += 64) cnt[k] = 0;
    int my_id[kMaxTilesPerWave], my_pos[kMaxTilesPerWave];
#pragma unroll
    for (int i = 0; i < kMaxTilesPerWave; ++i) {
        my_id[i] = 0xffff; my_pos[i] = 0;
        if (i < tiles) {                                                // uniform
            const int id = lid[(w * tiles + i) * 64 + lane];
            const bool valid = id != 0xffff;
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (int b = 0; b < 9; ++b) {
                if (b == 8 && K <= 256) break;                          // uniform: the ninth bit only with 16-bit ids
                const uint64_t m = __ballot((id >> b) & 1);
                peers &= ((id >> b) & 1) ? m : ~m;
            }
            if (valid) {
                const int rank = __builtin_popcountll(peers & ((1ull << lane) - 1ull));
                const int start = cnt[id];                              // read by all peers before the write below
                my_id[i] = id; my_pos[i] = start + rank;
                if (rank == 0) cnt[id] = start + __builtin_popcountll(peers);
            }
            __builtin_amdgcn_wave_barrier();
        }
    }
    __syncthreads();
    // thread t scans clusters 2 t and 2 t + 1 (K <= 512 = 2 x 256)
    int tot[2] = {0, 0};
    const int k0 = 2 * tid;
    if (k0 < Kp) {
#pragma unroll
        for (int r = 0; r < kAsgWaves; ++r) {
            const int2 c = *reinterpret_cast<const int2 *>(scratch + r * Kp + k0);
            tot[0] += c.x; tot[1] += c.y;
        }
    }
    const int incl = scan64(tot[0] + tot[1]);
    if (lane == 63) wtot[w] = incl;
    __syncthreads();
    int start = incl - tot[0] - tot[1];
#pragma unroll
    for (int r = 0; r < kAsgWaves - 1; ++r) if (r < w) start += wtot[r];
    if (k0 < Kp) {
        int run0 = start, run1 = start + tot[0];
        if (k0 < K) seg_out[k0] = (uint32_t)run0 | (uint32_t)run1 << 16;
        if (k0 + 1 < K) seg_out[k0 + 1] = (uint32_t)run1 | (uint32_t)(run1 + tot[1]) << 16;
#pragma unroll
        for (int r = 0; r < kAsgWaves; ++r) {
            int2 *p = reinterpret_cast<int2 *>(scratch + r * Kp + k0);
            const int2 c = *p;
            *p = make_int2(run0, run1);
            run0 += c.x; run1 += c.y;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kMaxTilesPerWave; ++i)
        if (i < tiles && my_id[i] != 0xffff)
            perm_out[cnt[my_id[i]] + my_pos[i]] = (uint16_t)((w * tiles + i) * 64 + lane);
}

}  // namespace qvg
