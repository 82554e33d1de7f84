// Pieces shared by the assignment kernel and the one-launch Lloyd loop: the search for a token's nearest
// centroid in a table staged in LDS (layout, scores, ranking, certification; qvg_encode.hip describes the method)
// and the rounds of 2-bit quantization.
#pragma once
#include "qvg_kmeans.hpp"

namespace qvg {

constexpr int kCPitch = 136;                    // bf16 elements per LDS centroid row (272 B): 128 + (hi, mid, lo of -||c||^2/2) + 5 zeros
constexpr int kScanPairs = 24;                  // candidates up to which fp64 distances are taken two at a time

// Rows of zeros but the first are taken out of a staged table: of equal rows only the lowest can be a token's nearest.
// The residuals of clusters of one token are zero, so a later smoothing stage has a dozen such rows among its centroids, and
// every token near zero had as many candidates: each a scan of the table and their fp64 distances, one after the
// other (K = 256, four stages: 24 units x 4680 tokens, in one launch, 495 -> 455 us; 6 x 1560 783 -> 295; 80 x 4680, in launches of their
// own, 1492 -> 1354).
__device__ __forceinline__ uint2 never_wins() { return make_uint2(__float_as_uint(-3.0e38f) >> 16, 0u); }      // a norm's split
// zero: an LDS word, kMaxClusters while no row with a norm of zero is known
__device__ __forceinline__ void note_zero_norm(uint2 nh, int row, int *zero) {
    if (!((nh.x | nh.y) & 0x7fff7fffu)) atomicMin(zero, row);
}
// By the whole workgroup (tid: the thread's number; in a loop over tables one that the compiler cannot carry through it), behind a barrier
// after the table, its norms nh (of rows t and t + 256, thread t) and the notes.  A barrier precedes the table's use.
__device__ __forceinline__ void drop_zero_rows(int tid, bf16_t *lc, int K, const uint2 (&nh)[kMaxClusters / kAsgThreads], int *zero) {
    if (*zero >= K) return;                                              // uniform
    bool is_zero[kMaxClusters / kAsgThreads];
#pragma unroll
    for (int k = 0; k < kMaxClusters / kAsgThreads; ++k) {
        const int row = tid + k * kAsgThreads;
        is_zero[k] = row < K && !((nh[k].x | nh[k].y) & 0x7fff7fffu);
        if (!is_zero[k]) continue;                                       // (the norm of a tiny row is zero as well)
        uint32_t any = 0u;
        for (int c16 = 0; c16 < kHeadDim / 8; ++c16) {
            const uint4 v = *reinterpret_cast<const uint4 *>(lc + row * kCPitch + c16 * 8);
            any |= v.x | v.y | v.z | v.w;
        }
        is_zero[k] = !(any & 0x7fff7fffu);
    }
    __syncthreads();
    if (tid == 0) *zero = kMaxClusters;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kMaxClusters / kAsgThreads; ++k) if (is_zero[k]) atomicMin(zero, tid + k * kAsgThreads);
    __syncthreads();
    const int keep = *zero;
    const uint2 never = never_wins();
#pragma unroll
    for (int k = 0; k < kMaxClusters / kAsgThreads; ++k)
        if (is_zero[k] && tid + k * kAsgThreads != keep)
            *reinterpret_cast<uint4 *>(lc + (tid + k * kAsgThreads) * kCPitch + kHeadDim) = make_uint4(never.x, never.y, 0u, 0u);
    __syncthreads();
    if (tid == 0) *zero = kMaxClusters;                                  // (for the next table)
}

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

// The same for one round with E4M3 scales, 2- or 4-bit levels (the rules of qvg_quant.hip).  B_ <= 64.
template <int B_, int BITS>
__device__ __forceinline__ void quantize_token_e4m3(const float *r, bool valid, int half, uint8_t *codes_tok, uint8_t *scales_tok) {
    constexpr int GL = 64 / B_;                      // groups held by this lane
    constexpr float qmax = BITS == 4 ? 7.0f : 1.0f;
    uint32_t word[2 * BITS] = {}, scales = 0u;
#pragma unroll
    for (int g = 0; g < GL; ++g) {
        const float *rg = r + g * B_;
        float m = 0.0f;
#pragma unroll
        for (int i = 0; i < B_; i += 2) m = fmaxf(fmaxf(m, fabsf(rg[i])), fabsf(rg[i + 1]));
        const uint32_t sbits = f32_to_e4m3_bits(m / qmax);
        const float sf = e4m3_bits_to_f32(sbits), inv = (sf == 0.0f) ? 0.0f : 1.0f / sf;
        scales |= sbits << (8 * g);
#pragma unroll
        for (int i = 0; i < B_; ++i) {
            const float q = __builtin_amdgcn_fmed3f(__builtin_rintf(rg[i] * inv), -qmax, qmax);
            const int at = (g * B_ + i) * BITS;
            word[at >> 5] |= ((uint32_t)(int)q & ((1u << BITS) - 1u)) << (at & 31);
        }
    }
    if (!valid) return;
#pragma unroll
    for (int i = 0; i < BITS / 2; ++i)
        *reinterpret_cast<uint4 *>(codes_tok + half * 8 * BITS + i * 16) = make_uint4(word[4 * i], word[4 * i + 1], word[4 * i + 2], word[4 * i + 3]);
    __builtin_memcpy(scales_tok + half * GL, &scales, GL);              // (they may lie at any address)
}

// One wavefront's search of the staged table.  A wavefront works on 64 tokens at a time, lane (col, half) holding
// channels 64 half .. of tokens col and 32 + col (the MFMA B operands).
struct TokenSearch {
    const bf16_t *lc;          // [Kpad][kCPitch]: rows, the split of -||c||^2 / 2 in each row's padding
    bf16_t *scr;               // [128] of the wavefront: one token
    float *sscr;               // [Kpad] of the wavefront: its scores
    float cmax;                // the largest ||c||^2 of the table
    int K, Kpad, lane, half, col;
    uint32_t tagbits, tagmask;
    float pinf;

    __device__ __forceinline__ TokenSearch(const bf16_t *lc_, bf16_t *scr_, float *sscr_, float cmax_, int K_, int Kpad_, int lane_)
        : lc(lc_), scr(scr_), sscr(sscr_), cmax(cmax_), K(K_), Kpad(Kpad_), lane(lane_), half(lane_ >> 5), col(lane_ & 31) {
        // 7 tag bits name a row among 256; with more rows the tag takes 8 (and the band below widens)
        tagbits = K > 256 ? 0xFFu : 0x7Fu;
        tagmask = vgpr_const(~tagbits);
        // +inf kept in a register the compiler cannot see through: med3(a, b, +inf) then stays one
        // instruction (as a constant it is rewritten into max(a, b) plus a NaN-quieting copy)
        pinf = __uint_as_float(vgpr_const(0x7f800000u));
    }

    // fp64 squared distances of the token in `scr` to centroids ja and jb (wave-uniform indices), one
    // per half of the wavefront: two rows of 16 lanes summed by DPP moves, the row sums read as
    // scalars (no exchange through LDS).  Both go through the same operations, so equal rows give
    // equal sums.
    __device__ __forceinline__ void pair_dist(int ja, int jb, double &Da, double &Db) const {
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
    }
    // Nearest centroid of the token in `scr` when more than two may be: the fp32 scores once more, one
    // centroid per lane, and fp64 distances only for those within `band` of the best (the bound on the
    // error of a score holds for this sum as well: as many roundings, and no tag).  With all K
    // distances in fp64 instead, these tokens were a third of the time of a QVG-Pro encode's later
    // stages: 24 units x 4680 tokens, S = 4, K = 256, I = 3 took 1.06 ms, with this and the band
    // below 0.81.
    __device__ __forceinline__ int scan_rows(float band) const {
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
        bd = INFINITY; bj = 0xffff;           // (stays where no distance is a number: near no row, and every list leaves it out)
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
    }

    // ||x||^2 of the lane's two tokens
    __device__ __forceinline__ void token_norms(const uint4 (&xa)[2][8], float (&xn)[2]) const {
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
    }

    // the lane's three largest scores of each of its tokens, the centroid's tag in their low mantissa bits
    template <bool FUSED>
    __device__ __forceinline__ void top_scores(const uint4 (&xa)[2][8], float (&b1)[2], float (&b2)[2], float (&b3)[2]) const {
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) { b1[tb] = -INFINITY; b2[tb] = -INFINITY; b3[tb] = -INFINITY; }
        // token operand of the extra MFMA step: three ones against (hi, mid, lo), lanes 0..31 only
        const uint4 ones = half ? make_uint4(0u, 0u, 0u, 0u) : make_uint4(0x3F803F80u, 0x00003F80u, 0u, 0u);
        // ---- scores on the matrix cores, running top three per lane and token ----
        // Blocks of 32 centroids, software-pipelined: the MFMAs of block jb+1 are issued between
        // the VALU instructions that rank the scores of block jb (an MFMA occupies the matrix
        // pipe for 8 VALU issue slots), so one wavefront keeps both pipes busy.
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
    }

    // the nearest centroid of the lane's token `tb` (both halves get it); called by the whole wavefront
    __device__ __forceinline__ int nearest(const uint4 (&xa)[2][8], int tb, bool valid, float xn, float c1, float c2, float c3) const {
        // tag -> centroid index: row 8*(r/4) + 4*half + r%4 of block jb
        auto tag_to_idx = [&](float v) {
            const uint32_t t = __float_as_uint(v) & tagbits;
            return (int)((t >> 4) * 32 + ((t >> 2) & 3) * 8 + half * 4 + (t & 3));
        };
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
        const float d2 = fmaxf(xn - 2.0f * c1, 0.0f) * (1.0f + 0x1p-10f) + xn * 0x1p-10f;
        const float reach = norm_reach(xn, d2, [](float v) { return __builtin_amdgcn_sqrtf(v); });
        // (the last term: the tag of a score that is zero, where all norms are)
        const float thr = (K > 256 ? 0x1.8p-14f : 0x1p-14f) * (0.5f * xn + fminf(cmax, reach)) + 0x1p-126f;
        int id = i1;
        // Rows K.. and rows of zeros but the first, which score never_wins(), lie below `none` and are no candidates.  But where the best itself
        // does, the scores of all rows that could be have overflowed; and where the band is not finite, those of tokens or rows
        // whose norm fp32 does not hold may be missing from the ranking: both mean the exact distances of all rows.
        constexpr float none = -2.9e38f;
        const bool amb = valid && !(c1 - fmaxf(c2, none) > thr);
        const bool full = !(c1 - fmaxf(c3, none) > thr);

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
        return id;
    }
};

}  // namespace qvg
