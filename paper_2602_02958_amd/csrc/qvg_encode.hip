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
#include "qvg_assign.hpp"

namespace qvg {

constexpr int kPrepThreads = 256;
constexpr int kPrepRows = kPrepThreads / 16;     // 16 lanes per centroid

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

// grid: x = unit, y = block of 256 * tiles_per_wave tokens.  With the unit as the fastest grid
// index and H a multiple of 8, all blocks of a unit run on one XCD and share its table in L2.
// T_: number of quantization rounds of the fused pass when known at compile time (0: a.T)
// ZEROS: a call of several smoothing stages, whose later tables may have several rows of zeros.  (An instance of its own, so that calls of
// one stage stay as they are; for all stages, as a second kernel is cold when it is first launched: 6 units x 2000 tokens, two stages 136.7
// us without the search, 137.7, 139.3 with the first stage's launches left out; 40 x 10800, K = 256 711, 715, 720.  Not with FUSED, one of a
// stage's I + 1 passes.)
template <int B_, bool FUSED, int T_, bool ZEROS>
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
    __shared__ int zero_row;
    if (tid == 0) { smax = 0u; if (ZEROS) zero_row = kMaxClusters; }
    const bf16_t *cg = a.cent + (int64_t)h * a.cent_stride;
    uint2 nh[kMaxClusters / kAsgThreads];
#pragma unroll
    for (int u = 0; u < kMaxClusters / kAsgThreads; ++u) {
        const int row = tid + u * kAsgThreads;
        nh[u] = never_wins();
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
            if (c16 == 0) up = fmaxf(up, place_norm(row, row < K ? split_half_norm(sq) : never_wins()));
        }
#pragma unroll
        for (int off = 32; off >= 16; off >>= 1) up = fmaxf(up, __shfl_xor(up, off, 64));
        if (lane == 0) atomicMax(&smax, norm_order(up));
    } else {
#pragma unroll
        for (int u = 0; u < kMaxClusters / kAsgThreads; ++u) {
            const int row = tid + u * kAsgThreads;
            float up = 0.0f;
            if (row < Kpad) { up = place_norm(row, nh[u]); if (ZEROS) note_zero_norm(nh[u], row, &zero_row); }
            if (u * kAsgThreads < Kpad) {                               // uniform
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) up = fmaxf(up, __shfl_xor(up, off, 64));
                if (lane == 0) atomicMax(&smax, norm_order(up));
            }
        }
    }
    __syncthreads();
    if (ZEROS && a.nh3) drop_zero_rows(tid, lc, K, nh, &zero_row);      // uniform
    const float cmax = __uint_as_float(smax);
    bf16_t *scr = lscr + wave * kHeadDim;
    float *sscr = lsscr + wave * Kpad;
    __shared__ uint16_t lid[FUSED ? 1 : kMaxTilesPerWave * kAsgThreads];    // the tokens' ids, for the member lists
    if (!FUSED && a.lists.perm)
        for (int i = tid; i < tiles_per_wave * kAsgThreads; i += kAsgThreads) lid[i] = 0xffffu;   // tokens of steps past the end; each wavefront clears its own
    const TokenSearch ts(lc, scr, sscr, cmax, K, Kpad, lane);
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
        ts.token_norms(xa, xn);
        float b1[2], b2[2], b3[2];
        ts.top_scores<FUSED>(xa, b1, b2, b3);
#pragma unroll
        for (int tb = 0; tb < 2; ++tb) {
            if (n0 + tb * 32 >= N) break;                        // uniform: second block past the end
            const int id = ts.nearest(xa, tb, valid[tb], xn[tb], b1[tb], b2[tb], b3[tb]);

            const int64_t hn = (int64_t)h * a.out_stride + n[tb];
            if (valid[tb] && half == 0) store_id(a.ids, hn * a.ids_step + a.ids_off, a.id_wide, (uint32_t)id);
            if (!FUSED) {
                if (a.lists.perm && half == 0) lid[(k * kAsgWaves + wave) * kAsgTile + tb * 32 + col] = valid[tb] ? (uint16_t)id : 0xffffu;
                if (a.resid && valid[tb]) {                              // Eq. 5, rounded to bf16: the next smoothing stage's input
                    const bf16_t *crow = lc + (id != 0xffff ? id : 0) * kCPitch + half * 64;
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
            const bf16_t *crow = lc + (id != 0xffff ? id : 0) * kCPitch + half * 64;
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

template <int B_, bool FUSED, int T_, bool ZEROS = false>
static hipError_t launch_assign_t(const AssignArgs &a, hipStream_t s) {
    const int Kpad = k_padded(a.K);
    const size_t smem = assign_smem_bytes(Kpad);
    static LdsHighWater lds_limit = {};
    hipError_t e = ensure_dynamic_lds(reinterpret_cast<const void *>(&assign_kernel<B_, FUSED, T_, ZEROS>), smem, lds_limit);
    if (e != hipSuccess) return e;
    const int tpw = assign_tiles_per_wave(a.H, a.n_tokens);
    const int64_t gy = (a.n_tokens + kAsgThreads * tpw - 1) / (kAsgThreads * tpw);
    if (gy > 65535) return hipErrorInvalidValue;
    if (a.lists.perm && (a.lists.block != kAsgThreads * tpw || a.lists.n_blocks != gy)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((assign_kernel<B_, FUSED, T_, ZEROS>), dim3((unsigned)a.H, (unsigned)gy), dim3(kAsgThreads), smem, s, a,
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
    if (!a.fused) return a.ids_step > 1 ? launch_assign_t<64, false, 0, true>(a, s) : launch_assign_t<64, false, 0>(a, s);
    switch (a.B) {
        case 16: return launch_fused<16>(a, s);
        case 32: return launch_fused<32>(a, s);
        case 64: return launch_fused<64>(a, s);
        default: return launch_fused<128>(a, s);
    }
}

}  // namespace qvg
