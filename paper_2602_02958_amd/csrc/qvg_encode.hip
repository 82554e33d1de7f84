// k-means assignment (paper Sec. 4.1), and the fused encoder pass that follows it:
// centroid subtraction (Eq. 5), T rounds of 2-bit group quantization of the residual
// (Sec. 3.2 Eq. 1-2, applied progressively as in Sec. 4.2) and bit packing.
//
// Assignment = argmin_j ||x - c_j||^2 = argmax_j ( x.c_j - ||c_j||^2 / 2 ).
// The N x K matrix of scores is a dense contraction and runs on the matrix cores
// (v_mfma_f32_32x32x16_bf16; bf16 x bf16 products are exact in fp32), with the centroid
// table of the unit staged once per workgroup in LDS.  The MFMA is issued transposed
// (rows = centroids, columns = tokens) so that one lane owns one token and the argmax over
// centroids is a per-lane running maximum followed by a single exchange between the two
// lane halves.  A wavefront works on 64 tokens at a time: every centroid operand read from
// LDS feeds two MFMAs (two blocks of 32 tokens), which halves the LDS traffic per flop and
// gives two independent accumulation chains.  The term -||c||^2/2 enters through one extra
// MFMA step: a small kernel has split it, per centroid, into three bf16 pieces whose sum is
// the fp32 value exactly, and the matching token operand holds three ones.
//
// Exactness.  The reference result is the argmin of fp64 distances.  The fp32 scores
// carry a rounding error, so the kernel keeps the three largest scores per token
// (cluster index carried in the 7 low mantissa bits) and certifies the winner only
// when it leads by more than a bound on that error,
//     thr = 2^-14 * (||x||^2 / 2 + N),
// N the largest ||c_j||^2 among the centroids that can be the nearest, which covers the 131
// accumulation roundings of half an ulp each plus the index tag for both scores (with more than 256
// centroids the tag has 8 bits and the factor is 1.5 * 2^-14).  Otherwise the candidates are
// re-evaluated in fp64, cooperatively by the wavefront: the two leaders, or, if the third score is
// inside the band as well, every centroid that a second look at the fp32 scores leaves possible.
// Equal fp64 distances go to the lower index.
#include "qvg_kmeans.hpp"

namespace qvg {

constexpr int kCPitch = 136;                    // bf16 elements per LDS centroid row (272 B): 128 + (hi, mid, lo of -||c||^2/2) + 5 zeros
constexpr int kPrepThreads = 256;
constexpr int kPrepRows = kPrepThreads / 16;     // 16 lanes per centroid
constexpr int kScanPairs = 24;                  // candidates up to which fp64 distances are taken two at a time

__device__ __forceinline__ void insert3(float v, int idx, float &b1, float &b2, float &b3,
                                        int &i1, int &i2) {
    if (v > b1) { b3 = b2; b2 = b1; i2 = i1; b1 = v; i1 = idx; }
    else if (v > b2) { b3 = b2; b2 = v; i2 = idx; }
    else if (v > b3) { b3 = v; }
}

__device__ __forceinline__ double shfl_xor_f64(double v, int m) { return __shfl_xor(v, m, 64); }
// acc + a.lo b.lo + a.hi b.hi of two packed bf16 pairs: v_dot2_f32_bf16
__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float acc) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), acc, false);
}
template <bool V> struct BoolK { static constexpr bool value = V; };
// (a & mask) | (b & ~mask): v_bfi_b32
__device__ __forceinline__ uint32_t bfi(uint32_t mask, uint32_t a, uint32_t b) { return (a & mask) | (b & ~mask); }
// a constant the compiler must keep in a vector register (so that the other, scalar operand of a
// three-operand VALU instruction is the only one on the constant bus)
__device__ __forceinline__ uint32_t vgpr_const(uint32_t c) {
    uint32_t v;
    asm volatile("v_mov_b32 %0, %1" : "=v"(v) : "s"(c));
    return v;
}

// ||c||^2 of a row spread over 16 lanes, 8 channels each
__device__ __forceinline__ double row_sumsq(const uint4 &v) {
    double s = 0.0;
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const double lo = (double)bf16_lo(w[e]), hi = (double)bf16_hi(w[e]);
        s += lo * lo; s += hi * hi;
    }
    return sum16_f64(s);
}

// The split norms of start tables (see split_half_norm); the tables of later Lloyd iterations get
// theirs from the update kernel that makes them.  16 lanes per centroid, grid: x = rows, y = table of
// the unit, z = unit.
__global__ __launch_bounds__(kPrepThreads)
void half_norm_kernel(const bf16_t *cent, int64_t cent_stride, int K, int Kpad, uint2 *nh3) {
    const int row = (int)blockIdx.x * kPrepRows + (int)(threadIdx.x >> 4), c16 = threadIdx.x & 15;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (row < K)
        v = *reinterpret_cast<const uint4 *>(cent + (int64_t)blockIdx.z * cent_stride +
                                             ((int64_t)blockIdx.y * K + row) * kHeadDim + c16 * 8);
    const double s = row_sumsq(v);
    if (row < K && c16 == 0)
        nh3[((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * Kpad + row] = split_half_norm(s);
}

hipError_t launch_half_norms(const bf16_t *cent, int64_t cent_stride, int H, int tables, int K, uint2 *nh3, hipStream_t s) {
    hipLaunchKernelGGL(half_norm_kernel, dim3((unsigned)((K + kPrepRows - 1) / kPrepRows), (unsigned)tables, (unsigned)H),
                       dim3(kPrepThreads), 0, s, cent, cent_stride, K, k_padded(K), nh3);
    return hipGetLastError();
}

// T rounds of Eq. 2 (b = 2: scale = max|r|, levels -1, 0, 1) on the 64 residuals r[] a lane
// holds of one token (channels 64*half ..), packed and stored as they are made.
// GL groups of NL elements lie inside the lane (B_ = 128: one group shared with the other half).
// TT > 0: the number of rounds is known at compile time (the loop unrolls, and the last round
// neither updates the residual nor takes the next maximum: a fifth of a round's instructions).
template <int B_, int TT>
__device__ __forceinline__ void quantize_token(float *r, int T, bool valid, int half, uint8_t *codes_tok,
                                               f16_t *scales_tok) {
    constexpr int G = kHeadDim / B_;                 // groups per token
    constexpr int GL = (B_ >= 64) ? 1 : 64 / B_;     // groups held by this lane
    constexpr int NL = (B_ >= 64) ? 64 : B_;         // elements per group in this lane
    auto round = [&](int t, auto last_k) {
        constexpr bool last = decltype(last_k)::value;
        uint32_t word[4];
        uint32_t sh[GL];
#pragma unroll
        for (int g = 0; g < GL; ++g) {
            float *rg = r + g * NL;
            float m = 0.0f;
#pragma unroll
            for (int i = 0; i < NL; i += 2) m = fmaxf(fmaxf(m, fabsf(rg[i])), fabsf(rg[i + 1]));
            if (B_ == 128) m = fmaxf(m, __shfl_xor(m, 32, 64));
            const float s32 = fminf(m, 65504.0f);
            sh[g] = f32_to_f16_bits(s32);
            const float sf = f16_bits_to_f32(sh[g]);
            const float inv = (sf == 0.0f) ? 0.0f : 1.0f / sf;
            // 8 levels -> one 16-bit field group: sum (q_i + 1) 4^i, exact in fp32.
            // |r / sf| <= 1 + 2^-11 unless the scale saturated, so the rounded level is already
            // in [-1, 1]; only a saturated group needs the clamp of Eq. 2.
            auto rounds = [&](auto clamp) {
#pragma unroll
                for (int o = 0; o < NL; o += 8) {
                    float cf = 21845.0f;             // 0x5555: the +1 of every field
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        float q = __builtin_rintf(rg[o + i] * inv);
                        if (decltype(clamp)::value) q = __builtin_amdgcn_fmed3f(q, -1.0f, 1.0f);
                        if (!last) rg[o + i] = __builtin_fmaf(-sf, q, rg[o + i]);
                        cf = __builtin_fmaf(q, (float)(1 << (2 * i)), cf);
                    }
                    const int e = g * NL + o;        // first channel (within the lane) of this field group
                    const uint32_t c16 = (uint32_t)cf;
                    if ((e >> 3) & 1) word[e >> 4] |= c16 << 16; else word[e >> 4] = c16;
                }
            };
            if (m > 65504.0f) rounds(BoolK<true>{}); else rounds(BoolK<false>{});
        }
        if (valid) {
            // word[] holds q + 1 per 2-bit field; the stored form is two's complement:
            // field 00 -> 11, 01 -> 00, 10 -> 01
#pragma unroll
            for (int wi = 0; wi < 4; ++wi) {
                const uint32_t lo = ~word[wi] & 0x55555555u;
                word[wi] = lo | (((~word[wi] >> 1) & lo) << 1);
            }
            *reinterpret_cast<uint4 *>(codes_tok + t * 32 + half * 16) = make_uint4(word[0], word[1], word[2], word[3]);
            f16_t *sp = scales_tok + t * G;
            if (B_ == 128) { if (half == 0) sp[0] = (f16_t)sh[0]; }
            else if (B_ == 64) sp[half] = (f16_t)sh[0];
            else if (B_ == 32)
                *reinterpret_cast<uint32_t *>(sp + half * 2) = sh[0] | (sh[GL - 1] << 16);
            else
                *reinterpret_cast<uint2 *>(sp + half * 4) =
                    make_uint2(sh[0] | (sh[1 % GL] << 16), sh[2 % GL] | (sh[3 % GL] << 16));
        }
    };
    if (TT > 0) {
#pragma unroll
        for (int t = 0; t < TT; ++t) {
            if (t + 1 < TT) round(t, BoolK<false>{}); else round(t, BoolK<true>{});
        }
    } else {
        for (int t = 0; t < T; ++t) round(t, BoolK<false>{});
    }
}

// grid: x = unit, y = block of 256 * tiles_per_wave tokens.  With the unit as the fastest grid
// index and H a multiple of 8, all blocks of a unit run on one XCD and share its table in L2.
// T_: number of quantization rounds of the fused pass when known at compile time (0: a.T)
template <int B_, bool FUSED, int T_>
__global__ __launch_bounds__(kAsgThreads, 2)
void assign_kernel(AssignArgs a, int Kpad, int tiles_per_wave) {
    extern __shared__ __align__(16) unsigned char smem[];
    bf16_t *lc = reinterpret_cast<bf16_t *>(smem);                       // [Kpad][kCPitch]
    bf16_t *lscr = lc + (size_t)Kpad * kCPitch;                          // [waves][128]
    float *lsscr = reinterpret_cast<float *>(lscr + kAsgWaves * kHeadDim);   // [waves][Kpad]

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, col = lane & 31;
    const int h = blockIdx.x;
    const int K = a.K;
    const int64_t N = a.n_tokens;

    // ---- stage the centroid table (rows K.. are zero) and, in each row's padding, the split of its
    // -||c||^2 / 2; rows K..Kpad-1 get a huge negative value so that they never win.  The largest
    // ||c||^2 of the unit (one ulp up) is needed for the error band of the certification.
    __shared__ uint32_t smax;
    if (tid == 0) smax = 0u;
    const bf16_t *cg = a.cent + (int64_t)h * a.cent_stride;
    uint2 nh[kMaxClusters / kAsgThreads];
#pragma unroll
    for (int u = 0; u < kMaxClusters / kAsgThreads; ++u) {
        const int row = tid + u * kAsgThreads;
        nh[u] = make_uint2(__float_as_uint(-3.0e38f) >> 16, 0u);
        if (row < K && a.nh3) nh[u] = a.nh3[(int64_t)h * a.nh3_stride + row];
    }
    const int64_t blk0 = (int64_t)blockIdx.y * tiles_per_wave * (kAsgWaves * kAsgTile);
    const bf16_t *xh = a.x + (int64_t)h * a.stride_head + half * 64;
    // this lane's 64 channels of its two tokens of a step (the MFMA B operands); a token past the
    // end of the chunk reads as zero
    auto load_x = [&](int64_t n0_, uint4 (&dst)[2][8]) {
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            const int64_t nn = n0_ + tb * 32 + col;
            const bf16_t *xp = xh + nn * a.stride_token;
#pragma unroll
            for (int kk = 0; kk < 8; ++kk)
                dst[tb][kk] = (nn < N) ? *reinterpret_cast<const uint4 *>(xp + kk * 8) : make_uint4(0u, 0u, 0u, 0u);
        }
    };
    auto step_start = [&](int k) {
        return k < tiles_per_wave ? blk0 + (int64_t)(k * kAsgWaves + wave) * kAsgTile : N;
    };
    // the first step's tokens are on their way while the table is staged (80 units x 10800 tokens,
    // K = 128, I = 3: 535 -> 490 us)
    uint4 xa[2][8];
    if (step_start(0) < N) load_x(step_start(0), xa);
    // Eight 16-byte pieces per thread are requested before the first is used: taken one at a time
    // (load, store to LDS) every piece waits a whole memory round trip (0.85 us measured),
    // which was most of what a workgroup with a single 256-token step spent on a 256-row table.
    constexpr int kStageBatch = 8;
    for (int i0 = tid; i0 < Kpad * 16; i0 += kAsgThreads * kStageBatch) {      // Kpad*16 is a multiple of the block: whole waves
        uint4 vb[kStageBatch];
#pragma unroll
        for (int u = 0; u < kStageBatch; ++u) {
            const int i = i0 + u * kAsgThreads;
            const int row = i >> 4, c16 = i & 15;
            vb[u] = make_uint4(0u, 0u, 0u, 0u);
            if (i < Kpad * 16 && row < K) vb[u] = *reinterpret_cast<const uint4 *>(cg + (int64_t)row * kHeadDim + c16 * 8);
        }
#pragma unroll
        for (int u = 0; u < kStageBatch; ++u) {
            const int i = i0 + u * kAsgThreads;
            if (i >= Kpad * 16) break;                                  // uniform
            const int row = i >> 4, c16 = i & 15;
            const uint4 v = vb[u];
            if (row < K && a.cent_copy && blockIdx.y == 0)              // the table's way out to the caller, for free
                *reinterpret_cast<uint4 *>(a.cent_copy + (int64_t)h * a.cent_copy_stride + (int64_t)row * kHeadDim + c16 * 8) = v;
            *reinterpret_cast<uint4 *>(lc + row * kCPitch + c16 * 8) = v;
        }
    }
    __syncthreads();                                                    // smax is zero, the rows are in place
    auto place_norm = [&](int row, uint2 n) -> float {                  // returns an upper bound of ||c||^2 in fp32
        *reinterpret_cast<uint4 *>(lc + row * kCPitch + kHeadDim) = make_uint4(n.x, n.y, 0u, 0u);
        return row < K ? norm_bound(n) : 0.0f;
    };
    if (!a.nh3) {                                                       // uniform: a start table of a small launch
        float up = 0.0f;
        const int c16 = tid & 15;
        for (int row = tid >> 4; row < Kpad; row += kAsgThreads / 16) {  // 16 lanes per row, sums as in half_norm_kernel
            const double sq = row_sumsq(*reinterpret_cast<const uint4 *>(lc + row * kCPitch + c16 * 8));
            if (c16 == 0) up = fmaxf(up, place_norm(row, row < K ? split_half_norm(sq) : make_uint2(__float_as_uint(-3.0e38f) >> 16, 0u)));
        }
#pragma unroll
        for (int off = 32; off >= 16; off >>= 1) up = fmaxf(up, __shfl_xor(up, off, 64));
        if (lane == 0) atomicMax(&smax, norm_order(up));
    } else {
#pragma unroll
        for (int u = 0; u < kMaxClusters / kAsgThreads; ++u) {
            const int row = tid + u * kAsgThreads;
            float up = 0.0f;
            if (row < Kpad) up = place_norm(row, nh[u]);
            if (u * kAsgThreads < Kpad) {                               // uniform
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) up = fmaxf(up, __shfl_xor(up, off, 64));
                if (lane == 0) atomicMax(&smax, norm_order(up));
            }
        }
    }
    __syncthreads();
    const float cmax = __uint_as_float(smax);
    bf16_t *scr = lscr + wave * kHeadDim;
    float *sscr = lsscr + wave * Kpad;
    __shared__ uint16_t lid[FUSED ? 1 : kMaxTilesPerWave * kAsgThreads];    // the tokens' ids, for the member lists
    if (!FUSED && a.lists.perm)
        for (int i = tid; i < tiles_per_wave * kAsgThreads; i += kAsgThreads) lid[i] = 0xffffu;   // tokens of steps past the end; each wavefront clears its own
    // token operand of the extra MFMA step: three ones against (hi, mid, lo), lanes 0..31 only
    // 7 tag bits name a row among 256; with more rows the tag takes 8 (and the band below widens)
    const uint32_t tagbits = K > 256 ? 0xFFu : 0x7Fu;
    const uint32_t tagmask = vgpr_const(~tagbits);
    // +inf kept in a register the compiler cannot see through: med3(a, b, +inf) then stays one
    // instruction (as a constant it is rewritten into max(a, b) plus a NaN-quieting copy)
    const float pinf = __uint_as_float(vgpr_const(0x7f800000u));
    const uint4 ones = half ? make_uint4(0u, 0u, 0u, 0u) : make_uint4(0x3F803F80u, 0x00003F80u, 0u, 0u);

    // fp64 squared distances of the token in `scr` to centroids ja and jb (wave-uniform indices), one
    // per half of the wavefront: two rows of 16 lanes summed by DPP moves, the row sums read as
    // scalars (no exchange through LDS).  Both go through the same operations, so equal rows give
    // equal sums.
    auto pair_dist = [&](int ja, int jb, double &Da, double &Db) {
        const int cand = half ? jb : ja;
        const uint2 xv = *reinterpret_cast<const uint2 *>(scr + col * 4);
        const uint2 cv = *reinterpret_cast<const uint2 *>(lc + cand * kCPitch + col * 4);
        const double e0 = (double)bf16_lo(xv.x) - (double)bf16_lo(cv.x);
        const double e1 = (double)bf16_hi(xv.x) - (double)bf16_hi(cv.x);
        const double e2 = (double)bf16_lo(xv.y) - (double)bf16_lo(cv.y);
        const double e3 = (double)bf16_hi(xv.y) - (double)bf16_hi(cv.y);
        double d = e0 * e0; d += e1 * e1; d += e2 * e2; d += e3 * e3;
        d = sum16_f64(d);
        Da = readlane_f64(d, 0) + readlane_f64(d, 16);
        Db = readlane_f64(d, 32) + readlane_f64(d, 48);
    };
    // Nearest centroid of the token in `scr` when more than two may be: the fp32 scores once more, one
    // centroid per lane, and fp64 distances only for those within `band` of the best (the bound on the
    // error of a score holds for this sum as well: as many roundings, and no tag).  With all K
    // distances in fp64 instead, these tokens were a third of the time of a QVG-Pro encode's later
    // stages: 24 units x 4680 tokens, S = 4, K = 256, I = 3 took 1.06 ms, with this and the band
    // below 0.81.
    auto scan_rows = [&](float band) -> int {
        float best = -INFINITY;
#pragma unroll 1
        for (int j = lane; j < K; j += 64) {
            const bf16_t *cr = lc + j * kCPitch;
            float s0 = 0.0f, s1 = 0.0f;
#pragma unroll 4
            for (int kk = 0; kk < 16; ++kk) {
                const uint4 xv = *reinterpret_cast<const uint4 *>(scr + kk * 8);
                const uint4 cv = *reinterpret_cast<const uint4 *>(cr + kk * 8);
                s0 = dot2(xv.x, cv.x, s0); s1 = dot2(xv.y, cv.y, s1);
                s0 = dot2(xv.z, cv.z, s0); s1 = dot2(xv.w, cv.w, s1);
            }
            const uint2 nh = *reinterpret_cast<const uint2 *>(cr + kHeadDim);
            const float s = (s0 + s1) + ((bf16_lo(nh.x) + bf16_hi(nh.x)) + bf16_lo(nh.y));
            sscr[j] = s;
            best = fmaxf(best, s);
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) best = fmaxf(best, __shfl_xor(best, off, 64));
        // (lane l reads back what lane l wrote; !(a < b): a score that overflowed to NaN stays a candidate)
        double bd = INFINITY; int bj = 0x7fffffff;
        int left = kScanPairs;
#pragma unroll 1
        for (int j0 = 0; j0 < K; j0 += 64) {
            uint64_t cm = __ballot(j0 + lane < K && !(sscr[j0 + lane < K ? j0 + lane : 0] < best - band));
            left -= __builtin_popcountll(cm);
            if (left < 0) break;
            while (cm) {
                const int ja = j0 + __builtin_ctzll(cm);
                cm &= cm - 1;
                const int jb = cm ? j0 + __builtin_ctzll(cm) : ja;
                if (cm) cm &= cm - 1;
                double Da, Db;
                pair_dist(ja, jb, Da, Db);
                if (Da < bd) { bd = Da; bj = ja; }                      // ascending indices: ties keep the lower
                if (Db < bd) { bd = Db; bj = jb; }
            }
        }
        if (left >= 0 && bj < K) return bj;
        bd = INFINITY; bj = 0x7fffffff;
        // many candidates (equal centroids): one per lane, the channels summed in index order
        for (int j = lane; j < K; j += 64) {
            const bf16_t *cr = lc + j * kCPitch;
            double acc = 0.0;
            for (int c = 0; c < kHeadDim; c += 2) {
                const uint32_t xw = *reinterpret_cast<const uint32_t *>(scr + c);
                const uint32_t cw = *reinterpret_cast<const uint32_t *>(cr + c);
                const double f0 = (double)bf16_lo(xw) - (double)bf16_lo(cw);
                acc += f0 * f0;
                const double f1 = (double)bf16_hi(xw) - (double)bf16_hi(cw);
                acc += f1 * f1;
            }
            if (acc < bd) { bd = acc; bj = j; }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            const double od = shfl_xor_f64(bd, off);
            const int oj = __shfl_xor(bj, off, 64);
            if (od < bd || (od == bd && oj < bj)) { bd = od; bj = oj; }
        }
        return bj;
    };
    // One step: 64 tokens.  Measured and left out, each without effect on the time of the pass:
    // requesting the next step's tokens a step ahead into a second register set; fetching the
    // tokens with whole rows per instruction through a staging area in LDS (each lane below reads
    // 16 bytes out of 64 different cache lines per instruction); more or fewer steps per workgroup.
    for (int k = 0; k < tiles_per_wave; ++k) {
        const int64_t n0 = step_start(k);
        if (n0 >= N) break;                                  // uniform per wavefront
        if (k > 0) load_x(n0, xa);
        int64_t n[2];
        bool valid[2];
        float xn[2];
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            n[tb] = n0 + tb * 32 + col;
            valid[tb] = n[tb] < N;
        }
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            float s = 0.0f;
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                const uint32_t w[4] = {xa[tb][kk].x, xa[tb][kk].y, xa[tb][kk].z, xa[tb][kk].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bf16x2_t p = __builtin_bit_cast(bf16x2_t, w[e]);
                    s = __builtin_amdgcn_fdot2_f32_bf16(p, p, s, false);
                }
            }
            xn[tb] = s + __shfl_xor(s, 32, 64);
        }

        // ---- scores on the matrix cores, running top three per lane and token ----
        // Blocks of 32 centroids, software-pipelined: the MFMAs of block jb+1 are issued between
        // the VALU instructions that rank the scores of block jb (an MFMA occupies the matrix
        // pipe for 8 VALU issue slots), so one wavefront keeps both pipes busy.
        float b1[2] = {-INFINITY, -INFINITY}, b2[2] = {-INFINITY, -INFINITY}, b3[2] = {-INFINITY, -INFINITY};
        auto score_block = [&](int jb, floatx16_t (&acc)[2]) {
#pragma unroll
            for (int r = 0; r < 16; ++r) { acc[0][r] = 0.0f; acc[1][r] = 0.0f; }
            const bf16_t *arow = lc + (jb * 32 + col) * kCPitch;
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                const bf16x8_t av = *reinterpret_cast<const bf16x8_t *>(arow + half * 64 + kk * 8);
                acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, __builtin_bit_cast(bf16x8_t, xa[0][kk]), acc[0], 0, 0, 0);
                acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, __builtin_bit_cast(bf16x8_t, xa[1][kk]), acc[1], 0, 0, 0);
            }
            const bf16x8_t av = *reinterpret_cast<const bf16x8_t *>(arow + kHeadDim);
            const bf16x8_t bv = __builtin_bit_cast(bf16x8_t, ones);
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc[1], 0, 0, 0);
        };
        auto rank_block = [&](int jb, const floatx16_t (&acc)[2]) {
            uint32_t tag0 = (uint32_t)jb << 4;
            asm volatile("" : "+s"(tag0));      // opaque: tag0 + r stays scalar arithmetic, the tag insert one v_and_or_b32
#pragma unroll
            for (int tb = 0; tb < 2; ++tb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    // (score & ~0x7F) | tag: one v_and_or_b32, the tag is scalar arithmetic.
                    // max(a, b) is written med3(a, b, +inf): no NaN-quieting copy is needed.
                    const float v = __uint_as_float((__float_as_uint(acc[tb][r]) & tagmask) | (tag0 + r));
                    b3[tb] = __builtin_amdgcn_fmed3f(b2[tb], b3[tb], v);
                    b2[tb] = __builtin_amdgcn_fmed3f(b1[tb], b2[tb], v);
                    b1[tb] = __builtin_amdgcn_fmed3f(b1[tb], v, pinf);
                }
        };
        if (FUSED) {
            // the fused pass has no registers for a second set of accumulators
            floatx16_t acc[2];
            for (int jb = 0; jb < (Kpad >> 5); ++jb) { score_block(jb, acc); rank_block(jb, acc); }
        } else {
            // Software pipeline over groups of three k-steps (a block of 32 centroids is three
            // groups: 8 channel steps and the norm step).  The centroid operands of the NEXT group
            // are requested before the six MFMAs of the current one, whose issue slots are shared
            // with a third of the ranking of the PREVIOUS block; scheduling barriers keep each
            // part where it is written (left alone, the compiler reads every operand right
            // before its use and the LDS latency is exposed once per k-step).
            const int nb = Kpad >> 5;                    // even: Kpad is a multiple of 64
            floatx16_t accA[2], accB[2];
            bf16x8_t av[2][3];
            const bf16x8_t bones = __builtin_bit_cast(bf16x8_t, ones);
            auto load_group = [&](int jb, int g, bf16x8_t (&dst)[3]) {
                const bf16_t *arow = lc + (jb * 32 + col) * kCPitch;
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const int kk = g * 3 + i;
                    dst[i] = *reinterpret_cast<const bf16x8_t *>(kk < 8 ? arow + half * 64 + kk * 8 : arow + kHeadDim);
                }
            };
            auto mfma_group = [&](int g, const bf16x8_t (&src)[3], floatx16_t (&acc)[2]) {
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const int kk = g * 3 + i;
                    if (kk == 0) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) { acc[0][r] = 0.0f; acc[1][r] = 0.0f; }
                    }
                    const bf16x8_t b0 = kk < 8 ? __builtin_bit_cast(bf16x8_t, xa[0][kk < 8 ? kk : 0]) : bones;
                    const bf16x8_t b1 = kk < 8 ? __builtin_bit_cast(bf16x8_t, xa[1][kk < 8 ? kk : 0]) : bones;
                    acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(src[i], b0, acc[0], 0, 0, 0);
                    acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(src[i], b1, acc[1], 0, 0, 0);
                }
            };
            // scores 11 c .. 11 c + 10 (of 32: 16 per token block) of a finished block
            auto rank_part = [&](int jb, const floatx16_t (&acc)[2], int c) {
                uint32_t tag0 = (uint32_t)jb << 4;
                asm volatile("" : "+s"(tag0));  // opaque, see rank_block
#pragma unroll
                for (int sidx = 11 * c; sidx < (c == 2 ? 32 : 11 * c + 11); ++sidx) {
                    const int tb = sidx >> 4, r = sidx & 15;
                    const float v = __uint_as_float((__float_as_uint(acc[tb][r]) & tagmask) | (tag0 + r));
                    b3[tb] = __builtin_amdgcn_fmed3f(b2[tb], b3[tb], v);
                    b2[tb] = __builtin_amdgcn_fmed3f(b1[tb], b2[tb], v);
                    b1[tb] = __builtin_amdgcn_fmed3f(b1[tb], v, pinf);
                }
            };
            auto interleave6 = [&]() {
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);
                }
            };
            // one block: its three groups; `prev` (if any) is ranked in their shadow; the operands
            // of the group after the current one are requested first (next_jb < 0: none)
            auto block_step = [&](int jb, floatx16_t (&acc)[2], int prev_jb, const floatx16_t (&prev)[2],
                                  int parity, bool more) {
#pragma unroll
                for (int g = 0; g < 3; ++g) {
                    const int cur = (parity + g) & 1;
                    if (g < 2) load_group(jb, g + 1, av[cur ^ 1]);
                    else if (more) load_group(jb + 1, 0, av[cur ^ 1]);
                    __builtin_amdgcn_sched_barrier(0);
                    mfma_group(g, av[cur], acc);
                    if (prev_jb >= 0) { rank_part(prev_jb, prev, g); interleave6(); }
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            load_group(0, 0, av[0]);
            block_step(0, accA, -1, accB, 0, true);                 // groups 0..2: parities 0, 1, 0
            for (int jb = 1; jb + 1 < nb; jb += 2) {
                block_step(jb, accB, jb - 1, accA, 1, true);        // groups 3..5: parities 1, 0, 1
                block_step(jb + 1, accA, jb, accB, 0, true);
            }
            block_step(nb - 1, accB, nb - 2, accA, 1, false);
            rank_block(nb - 1, accB);
        }
        // tag -> centroid index: row 8*(r/4) + 4*half + r%4 of block jb
        auto tag_to_idx = [&](float v) {
            const uint32_t t = __float_as_uint(v) & tagbits;
            return (int)((t >> 4) * 32 + ((t >> 2) & 3) * 8 + half * 4 + (t & 3));
        };
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            if (n0 + tb * 32 >= N) break;                        // uniform: second block past the end
            float c1 = b1[tb], c2 = b2[tb], c3 = b3[tb];
            int i1 = tag_to_idx(c1), i2 = tag_to_idx(c2);
            {   // merge with the other half of the wavefront (same token, other centroids)
                const float p1 = __shfl_xor(c1, 32, 64), p2 = __shfl_xor(c2, 32, 64),
                            p3 = __shfl_xor(c3, 32, 64);
                const int q1 = __shfl_xor(i1, 32, 64), q2 = __shfl_xor(i2, 32, 64);
                insert3(p1, q1, c1, c2, c3, i1, i2);
                insert3(p2, q2, c1, c2, c3, i1, i2);
                insert3(p3, 0, c1, c2, c3, i1, i2);
            }
            // Which centroids can matter: one that is at least as near as the leader lies within the
            // leader's distance d of the token, so its norm is at most ||x|| + d.  The band therefore
            // takes min(max ||c||^2, (||x|| + d)^2): with the unit's largest norm alone, one centroid on
            // a few outlying tokens widened the band of every token (student-t data, 80 units x 10800
            // tokens, K = 128, I = 3: 0.88 to 1.68 ms, by the draw, against 0.56 to 0.58).
            // d^2 = ||x||^2 - 2 score, with 2^-10 of slack on both terms for the rounding of the score.
            const float d2 = fmaxf(xn[tb] - 2.0f * c1, 0.0f) * (1.0f + 0x1p-10f) + xn[tb] * 0x1p-10f;
            const float reach = norm_reach(xn[tb], d2, [](float v) { return __builtin_amdgcn_sqrtf(v); });
            // (the last term: the tag of a score that is zero, where all norms are)
            const float thr = (K > 256 ? 0x1.8p-14f : 0x1p-14f) * (0.5f * xn[tb] + fminf(cmax, reach)) + 0x1p-126f;
            int id = i1;
            const bool amb = valid[tb] && (i2 < K) && !(c1 - c2 > thr);
            const bool full = !(c1 - c3 > thr);

            // ---- fp64 re-evaluation of tokens the fp32 scores cannot decide ----
            uint64_t mask = __ballot(amb) & 0xffffffffull;
            while (mask) {
                const int tk = __builtin_ctzll(mask);
                mask &= mask - 1;
                if (col == tk) {
#pragma unroll
                    for (int kk = 0; kk < 8; ++kk)
                        *reinterpret_cast<uint4 *>(scr + half * 64 + kk * 8) = xa[tb][kk];
                }
                __builtin_amdgcn_wave_barrier();
                // the token's lane index is wave-uniform: plain lane reads, no exchange through LDS
                const int d1 = __builtin_amdgcn_readlane(i1, tk), d2i = __builtin_amdgcn_readlane(i2, tk);
                const int fl = __builtin_amdgcn_readlane((int)full, tk);
                int winner;
                if (!fl) {
                    double D1, D2;
                    pair_dist(d1, d2i, D1, D2);
                    winner = (D2 < D1 || (D2 == D1 && d2i < d1)) ? d2i : d1;
                } else {
                    winner = scan_rows(__uint_as_float(__builtin_amdgcn_readlane((int)__float_as_uint(thr), tk)));
                }
                if (col == tk) id = winner;
                __builtin_amdgcn_wave_barrier();
            }

            const int64_t hn = (int64_t)h * a.out_stride + n[tb];
            if (valid[tb] && half == 0) store_id(a.ids, hn * a.ids_step + a.ids_off, a.id_wide, (uint32_t)id);
            if (!FUSED) {
                if (a.lists.perm && half == 0) lid[(k * kAsgWaves + wave) * kAsgTile + tb * 32 + col] = valid[tb] ? (uint16_t)id : 0xffffu;
                if (a.resid && valid[tb]) {                              // Eq. 5, rounded to bf16: the next smoothing stage's input
                    const bf16_t *crow = lc + id * kCPitch + half * 64;
                    bf16_t *rp = a.resid + ((int64_t)h * N + n[tb]) * kHeadDim + half * 64;
#pragma unroll
                    for (int kk = 0; kk < 8; ++kk) {
                        float xf[8], cf[8];
                        unpack_bf16x8(xa[tb][kk], xf);
                        unpack_bf16x8(*reinterpret_cast<const uint4 *>(crow + kk * 8), cf);
#pragma unroll
                        for (int i = 0; i < 8; ++i) xf[i] -= cf[i];
                        *reinterpret_cast<uint4 *>(rp + kk * 8) = pack_bf16x8(xf);
                    }
                }
                continue;
            }

            // ---- Eq. 5: residual against the assigned centroid, then the T rounds ----
            float r[64];
            const bf16_t *crow = lc + id * kCPitch + half * 64;
#pragma unroll
            for (int kk = 0; kk < 8; ++kk) {
                const uint4 cv = *reinterpret_cast<const uint4 *>(crow + kk * 8);
                const uint32_t xw[4] = {xa[tb][kk].x, xa[tb][kk].y, xa[tb][kk].z, xa[tb][kk].w};
                const uint32_t cw[4] = {cv.x, cv.y, cv.z, cv.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    r[kk * 8 + 2 * e] = bf16_lo(xw[e]) - bf16_lo(cw[e]);
                    r[kk * 8 + 2 * e + 1] = bf16_hi(xw[e]) - bf16_hi(cw[e]);
                }
            }
            const int T = T_ > 0 ? T_ : a.T;
            quantize_token<B_, T_>(r, T, valid[tb], half, a.codes + hn * T * 32, a.scales + hn * T * (kHeadDim / B_));
            __builtin_amdgcn_sched_barrier(0);       // keep the two tokens' passes apart: each needs most registers
        }
    }
    if (!FUSED && a.lists.perm) {                    // the member lists of this workgroup's tokens
        __syncthreads();                             // every id is in lid, the table is not needed any more
        const int64_t blk = (int64_t)h * a.lists.n_blocks + blockIdx.y;
        block_member_sort(lid, tiles_per_wave, K, reinterpret_cast<int *>(smem), a.lists.perm + blk * a.lists.block,
                          a.lists.seg + blk * K);
    }
}

static size_t assign_smem_bytes(int Kpad) {
    return (size_t)Kpad * kCPitch * 2 + (size_t)kAsgWaves * (kHeadDim * 2 + Kpad * sizeof(float));
}

// 256-token steps per workgroup: more of them amortise the table staging once there are enough
// workgroups to fill the chip several times over
constexpr int64_t kAsgManyGroups = 2048;
int assign_tiles_per_wave(int H, int64_t n_tokens) {
    const int64_t steps = (n_tokens + kAsgWaves * kAsgTile - 1) / (kAsgWaves * kAsgTile);
    int tpw = 1;
    while (tpw < kMaxTilesPerWave && (steps / (2 * tpw)) * H >= kAsgManyGroups) tpw *= 2;
    return tpw;
}

// The blocks themselves get fewer where the steps per workgroup double, and a workspace sized by them would not
// serve a shorter call.  With one step per workgroup there are at most 2 (kAsgManyGroups - 1) + H blocks, with
// two 2 (kAsgManyGroups - 1) + 2 H, with four the number itself.
int64_t member_blocks_bound(int H, int64_t n_tokens) {
    const int64_t steps = (n_tokens + kAsgWaves * kAsgTile - 1) / (kAsgWaves * kAsgTile), h = H;
    const int64_t fewest = h * ((steps + kMaxTilesPerWave - 1) / kMaxTilesPerWave), most = 2 * (kAsgManyGroups - 1) + 2 * h;
    const int64_t bound = most > fewest ? most : fewest;
    return h * steps < bound ? h * steps : bound;
}

// Start tables of up to 128 centroids: the workgroups of a small launch take the norms themselves from the staged rows,
// which saves a launch (2.5 us of a call that is short enough to be host time).  Each workgroup repeats the sums of its
// unit's rows, in a time that grows with their number, so the limit falls with its square: K = 64 up to 2048 workgroups
// (one unit of 2^20 tokens, no iteration 114.1 -> 112.3 us; 400 x 300 27.2 -> 25.1; at 3200 168.6 -> 172.3), K = 128 up to
// 512 (24 units x 64 tokens 15.3 -> 12.0; 24 x 4680 21.5 -> 21.1; at 1024 37.3 -> 39.4).  With more centroids half_norm_kernel's once per
// unit is faster, however few the workgroups (K = 256, no iteration: 20.4 against 21.4 us at 64 of them, 29.7 against 30.9 at
// 456), unless a unit has one workgroup anyway and the assignment is not the fused pass (one unit of 64 tokens 15.5 ->
// 12.6, 400 18.2 -> 16.9; fused 15.6 -> 16.4).
bool assign_takes_norms(int H, int K, int64_t n_tokens, bool fused) {
    const int64_t block = member_block(H, n_tokens), wgs = (n_tokens + block - 1) / block * H, kp = k_padded(K);
    if (!fused && wgs == H && kp <= 256) return true;
    return kp <= 128 && wgs * kp * kp <= ((int64_t)1 << 23);
}

template <int B_, bool FUSED, int T_>
static hipError_t launch_assign_t(const AssignArgs &a, hipStream_t s) {
    const int Kpad = k_padded(a.K);
    const size_t smem = assign_smem_bytes(Kpad);
    static LdsHighWater lds_limit = {};
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(&assign_kernel<B_, FUSED, T_>), smem, lds_limit);
    if (e != hipSuccess) return e;
    const int tpw = assign_tiles_per_wave(a.H, a.n_tokens);
    const int64_t gy = (a.n_tokens + kAsgThreads * tpw - 1) / (kAsgThreads * tpw);
    if (gy > 65535) return hipErrorInvalidValue;
    if (a.lists.perm && (a.lists.block != kAsgThreads * tpw || a.lists.n_blocks != gy)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((assign_kernel<B_, FUSED, T_>), dim3((unsigned)a.H, (unsigned)gy), dim3(kAsgThreads), smem, s, a,
                       Kpad, tpw);
    return hipGetLastError();
}

// the fused pass with the round count of the measured configurations fixed at compile time
// (group 64: 1, 2 and 4 rounds; group 32: 3), any other count at run time
template <int B_>
static hipError_t launch_fused(const AssignArgs &a, hipStream_t s) {
    if (B_ == 64 && a.T == 1) return launch_assign_t<B_, true, (B_ == 64 ? 1 : 0)>(a, s);
    if (B_ == 64 && a.T == 2) return launch_assign_t<B_, true, (B_ == 64 ? 2 : 0)>(a, s);
    if (B_ == 64 && a.T == 4) return launch_assign_t<B_, true, (B_ == 64 ? 4 : 0)>(a, s);
    if (B_ == 32 && a.T == 3) return launch_assign_t<B_, true, (B_ == 32 ? 3 : 0)>(a, s);
    return launch_assign_t<B_, true, 0>(a, s);
}

hipError_t launch_assign(const AssignArgs &a, hipStream_t s) {
    if (a.n_tokens == 0) return hipSuccess;
    if (!a.fused) return launch_assign_t<64, false, 0>(a, s);
    switch (a.B) {
        case 16: return launch_fused<16>(a, s);
        case 32: return launch_fused<32>(a, s);
        case 64: return launch_fused<64>(a, s);
        default: return launch_fused<128>(a, s);
    }
}

}  // namespace qvg
