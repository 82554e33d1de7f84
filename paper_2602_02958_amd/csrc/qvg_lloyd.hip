// The whole encoder of a chunk in one launch: every smoothing stage's Lloyd iterations (paper Sec. 4.1, 4.3), its
// last assignment and, in the formats of lloyd_fuses, the quantization rounds.
//
// What bounds the launches of qvg_encode.hip / qvg_kmeans.hip on one layer's chunk is not their work: an
// iteration of 24 units x 4680 tokens, K = 256 takes 35 us, of which the tokens' way from memory to the CUs, twice,
// is 11 (nothing stays in the L2s from one launch to the next: 30 MB fetched by each) and the launches themselves 3 to 4.  Here a unit's
// workgroups stay: each keeps its 256 tokens in registers through all iterations, the update's gathers find the
// unit's tokens in the L2 that served the assignment (23 MB fetched by a launch where the L2s hold some from the one before, FETCH_SIZE), and the steps are kept apart by a barrier among the
// workgroups of a UNIT (1.2 us among 16 or 19 of them) instead of the end of a launch.
//
// Every iteration: assign (table staged in LDS, qvg_assign.hpp), publish the tokens' ids; meet; update: a
// workgroup has a contiguous range of the unit's centroids, picks their members out of the unit's ids and sums them
// in the defined order (qvg_kmeans.hip), publishes the new rows; meet.
//
// What workgroups exchange inside the launch goes around the L2s, which are not coherent between XCDs: stores and
// loads at agent scope (64 KB to each of 456 workgroups, barrier included: 5.4 us; with fences, which write back and
// invalidate whole caches, 52).
//
// The barrier.  Only workgroups that run at the same time can meet.  The launch is taken only where the chip holds all of
// them (lloyd_groups), but another stream's work may hold part of it for long.  So the workgroups that arrive at the first
// barrier are the unit's team: all of them, or, where some have not even started in time, those that have arrived by then.
// Such a team is closed; it begins anew, the unit's blocks and rows dealt among its members, and a workgroup that
// arrives later leaves.  What that one has written, the first ids, is not read: a closed team has its ids in the codes' place
// in the output.  Behind the first barrier only members are waited for, and they never wait for anybody else.
// How long the first barrier waits for workgroups that have not started: half of what the run takes with the members
// there are, so that it costs little where none comes and few members do not go on alone where others come soon.
// Beside an attention of 130 / 170 / 200 workgroups on another stream that lasts 3 ms, us (launches per iteration; this; as it was
// when a unit waited 2 ms and one workgroup did it over): 24 units x 4680 tokens, K = 256, T = 4, I = 3 295 / 420 / 760; 350 / 860 / 1255; 359 / - / 3190;
// INT4, 10 x 1571 101 / 116 / 174; 158 / 163 / 370; 143 / - / 2520.  Two streams of encodes, a pair of them: 225, 213, 214; 123, 102, 104.  (A
// wait half as long: 200 workgroups 1070; twice as long 1610.)
#include "qvg_assign.hpp"

namespace qvg {

constexpr int kMeetWords = 64;                   // a 256-byte line per unit
constexpr uint32_t kWaitTicks = 1500;            // of 10 ns: half an iteration over one block per workgroup
constexpr int kLloydMaxBlocks = 24;              // blocks of 256 tokens per unit (lloyd_groups; token numbers have 16 bits)
constexpr int kListLong = 128;                   // lists at least this long are summed by the whole workgroup,
constexpr int kListShared = 32;                  // where it has one or two rows, at least this long
constexpr int kRowsAhead = 16;                   // members in flight (a power of two)
constexpr int kLloydRows = 64;                   // rows that a workgroup makes at a time

typedef uint32_t uint32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t uint32x4_t __attribute__((ext_vector_type(4)));

// ---- memory that other workgroups of the launch write or read -----------------------------------
constexpr int kAgentScope = 16;                  // cache policy of the buffer instructions: sc1
struct Shared {                                  // a buffer of one unit; loads beyond it return zero, stores beyond it are dropped
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ Shared(const void *p, uint32_t bytes)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)bytes, 0x00020000)) {}
    __device__ __forceinline__ uint4 load16(uint32_t off) const {
        const uint32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, kAgentScope);
        return make_uint4(v.x, v.y, v.z, v.w);
    }
    __device__ __forceinline__ uint2 load8(uint32_t off) const {
        const uint32x2_t v = __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, kAgentScope);
        return make_uint2(v.x, v.y);
    }
    __device__ __forceinline__ uint32_t load4(uint32_t off) const {
        return __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, kAgentScope);
    }
    __device__ __forceinline__ void store16(uint32_t off, const uint4 &v) const {
        const uint32x4_t w = {v.x, v.y, v.z, v.w};
        __builtin_amdgcn_raw_buffer_store_b128(w, r, (int)off, 0, kAgentScope);
    }
    __device__ __forceinline__ void store8(uint32_t off, const uint2 &v) const {
        const uint32x2_t w = {v.x, v.y};
        __builtin_amdgcn_raw_buffer_store_b64(w, r, (int)off, 0, kAgentScope);
    }
    __device__ __forceinline__ void store4(uint32_t off, uint32_t v) const {
        __builtin_amdgcn_raw_buffer_store_b32(v, r, (int)off, 0, kAgentScope);
    }
};

// A unit's words: the arrivals at the first barrier (and, once the team is closed, bit 31 and the members from bit 16 on), the
// arrivals at all later ones, and (in a cache line of their own) a byte per workgroup that has started.
constexpr uint32_t kTeamClosed = 0x80000000u, kArrivedMask = 0xffffu;
constexpr int kMembersShift = 16, kLaterWord = 4, kStartedAt = 128;
static_assert(kMaxClusters / 8 <= kMeetWords * 4 - kStartedAt && kLloydMaxBlocks <= kMeetWords * 4 - kStartedAt, "a byte per workgroup");

__device__ __forceinline__ void set_started(uint32_t *words, int g) {
    const Shared s(words, kMeetWords * 4);
    __builtin_amdgcn_raw_buffer_store_b8((unsigned char)1, s.r, kStartedAt + g, 0, kAgentScope);
}
__device__ __forceinline__ bool all_started(const uint32_t *words) {     // (bytes that nobody sets are set from the start)
    const Shared s(words, kMeetWords * 4);
    uint4 v[(kMeetWords * 4 - kStartedAt) / 16];                         // (all requested before the first is looked at)
#pragma unroll
    for (int i = 0; i < (kMeetWords * 4 - kStartedAt) / 16; ++i) v[i] = s.load16((uint32_t)(kStartedAt + i * 16));
    uint32_t all = 0x01010101u;
#pragma unroll
    for (int i = 0; i < (kMeetWords * 4 - kStartedAt) / 16; ++i) all &= v[i].x & v[i].y & v[i].z & v[i].w;
    return all == 0x01010101u;
}
// Thread 0 at the first barrier, which waits for `wanted` workgroups: 0 where all have come, else the members of the closed team, -1
// where this one has come too late.  number: of this one, in the order of arrival.
// ticks: the wait for workgroups that have not started, for each block that a member has.
__device__ __forceinline__ int team_meet(uint32_t *words, int wanted, int groups, int nb, uint32_t ticks, int &number) {
    uint32_t v = __hip_atomic_fetch_add(words, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    number = (int)(v & kArrivedMask);
    if ((v & kTeamClosed) || number >= wanted) return -1;
    ++v;
    uint64_t t0 = 0;
    for (uint32_t polls = 0; ; ++polls) {
        if (v & kTeamClosed) return (int)(v >> kMembersShift) & 0x7fff;
        const int there = (int)(v & kArrivedMask);                       // at least this one
        if (there >= wanted) {                                           // (more: they left)
            if (wanted == groups) return 0;
            __hip_atomic_fetch_or(words, kTeamClosed | (uint32_t)wanted << kMembersShift, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return wanted;
        }
        if (polls % 16 == 15) {                                          // (reading the clock at every poll costs 1.5 us)
            const uint64_t now = __builtin_amdgcn_s_memrealtime();
            if (t0 == 0) t0 = now;
            if (now - t0 >= (uint64_t)ticks * (uint32_t)((nb + there - 1) / there)) {
                t0 = now;
                // (the exchange fails only where another workgroup has arrived or closed the team meanwhile)
                if (!all_started(words) && __hip_atomic_compare_exchange_strong(words, &v, v | kTeamClosed | (uint32_t)there << kMembersShift,
                                                                                __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                    return there;
            }
        }
        __builtin_amdgcn_s_sleep(8);
        v = __hip_atomic_load(words, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// All members of the team: everything stored before is seen by all after.
// `word` counts the arrivals; target: members x barriers so far, this one included.
// fresh: data of this launch is going to be read by plain loads.
__device__ __forceinline__ void meet(uint32_t *word, uint32_t members, uint32_t target, bool fresh) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                     // this wavefront's stores have arrived
    __syncthreads();
    if (threadIdx.x == 0) {
        if (members > 1) {                                               // uniform
            uint32_t v = __hip_atomic_fetch_add(word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;
            while (v < target) {
                __builtin_amdgcn_s_sleep(2);
                v = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        if (fresh) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
}

// LDS of the update, over the staged table
struct UpdateLds {
    double *sums;              // [c][128]: the rows' sums
    double (*part)[64][2];     // [4]: a wavefront's sums, two channels per lane
    uint32_t (*pmx)[64], (*pmn)[64];
    int *cnt;                  // [4][64]: members in a wavefront's quarter of the tokens, then where they go
    uint16_t *ids;             // [nb * 256]: the unit's ids, then
    uint16_t *list;            //             the rows' members, token order
    uint32_t *own;             // [4][nb * 64 + 1]: the members of the workgroup's rows in a wavefront's quarter: token | row << 16
    __host__ __device__ static size_t bytes(int nb, int c) { return (size_t)c * 1024 + 4 * 64 * 24 + 4 * 64 * 4 + (size_t)nb * 1536 + 16; }
    __device__ __forceinline__ UpdateLds(unsigned char *p, int nb, int c) {
        sums = reinterpret_cast<double *>(p); p += c * 1024;
        part = reinterpret_cast<double (*)[64][2]>(p); p += 4 * 64 * 16;
        pmx = reinterpret_cast<uint32_t (*)[64]>(p); p += 4 * 64 * 4;
        pmn = reinterpret_cast<uint32_t (*)[64]>(p); p += 4 * 64 * 4;
        cnt = reinterpret_cast<int *>(p); p += 4 * 64 * 4;
        ids = reinterpret_cast<uint16_t *>(p); list = ids; p += nb * 512;
        own = reinterpret_cast<uint32_t *>(p);
    }
};

// The 8 channels' sums over n, rounded as one division each would be (Markstein's correction).  Infinite sums and NaN
// stay what they are.
__device__ __forceinline__ uint4 mean_row(const double s[8], int n) {
    const double d = (double)n, r = 1.0 / d;
    float m[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        m[e] = (float)(__builtin_fabs(s[e]) < INFINITY ? quotient(s[e], d, r) : s[e]);
    }
    return make_uint4(pack_bf16x2(m[0], m[1]), pack_bf16x2(m[2], m[3]), pack_bf16x2(m[4], m[5]), pack_bf16x2(m[6], m[7]));
}

// The launch's arguments and the thread's number, read anew where a phase begins: what is derived from them would
// otherwise be worked out once, before the loop over the iterations, and carried through all phases (47 to 120 spilled
// vector registers, 117 to 147 scalar ones).
__device__ __forceinline__ const LloydArgs &args_again() {
    auto p = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const LloydArgs *)p;
}
__device__ __forceinline__ int thread_id() {
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// The rows of a unit's new table are dealt in index order by their members, not by their number: a stage's largest
// clusters can hold a tenth of a unit's tokens each (later smoothing stages), and the unit waits for the workgroup that has
// most.  Every workgroup has to see the same members: those of the iteration before, which come with the table, and before the
// first update of a stage they are counted from the ids (2 us).  The first stage's clusters are dealt by number: what the
// dealing takes, 0.8 us an iteration, is not gained back there (24 units x 4680 tokens, K = 256, S = 1: 115.0 -> 115.8 us).
struct DealLds {
    int sums[kMaxClusters / 64];   // weights of 64 rows
    int below[kMaxClusters / 64], upto[kMaxClusters / 64];               // of 64 rows: those before this workgroup's, and with them
    int zero;                      // a row whose norm is zero, kMaxClusters: none
};
constexpr int kRowsPerThread = kMaxClusters / kAsgThreads;

// This workgroup's rows: those whose middle lies in its share of the weight.  members: of rows t and t + 256 (thread t).
// The caller's barrier stands between this and dealt().
__device__ __forceinline__ void deal_rows(const int (&members)[kRowsPerThread], int K, int weight, int g, int groups, DealLds &d) {
    const int tid = thread_id(), lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int v[kRowsPerThread], upto[kRowsPerThread];
#pragma unroll
    for (int k = 0; k < kRowsPerThread; ++k) {
        v[k] = k * kAsgThreads + tid < K ? weight + members[k] : 0;
        upto[k] = scan64(v[k]);
        if (lane == 63) d.sums[k * kAsgWaves + w] = upto[k];
    }
    __syncthreads();
    int all = 0, before[kRowsPerThread] = {};
#pragma unroll
    for (int i = 0; i < kMaxClusters / 64; ++i) {
#pragma unroll
        for (int k = 0; k < kRowsPerThread; ++k) before[k] = i == k * kAsgWaves + w ? all : before[k];
        all += d.sums[i];
    }
#pragma unroll
    for (int k = 0; k < kRowsPerThread; ++k) {
        const int at = v[k] ? (2 * (before[k] + upto[k]) - v[k]) * groups : 0x7fffffff;                // (the products are below 2^23)
        const int below = __builtin_popcountll(__ballot(at < 2 * all * g)), with = __builtin_popcountll(__ballot(at < 2 * all * (g + 1)));
        if (lane == 0) { d.below[k * kAsgWaves + w] = below; d.upto[k * kAsgWaves + w] = with; }
    }
}
__device__ __forceinline__ void dealt(const DealLds &d, int &first, int &end) {
    int a = 0, b = 0;
#pragma unroll
    for (int i = 0; i < kMaxClusters / 64; ++i) { a += d.below[i]; b += d.upto[i]; }
    first = __builtin_amdgcn_readfirstlane(a); end = __builtin_amdgcn_readfirstlane(b);
}

// The workgroup's rows of a unit's new table, `rows` <= 64 at a time.
// count: the members are not known yet.
// x: the unit's tokens, row_bytes apart (below 2^31 bytes in all).
__device__ __forceinline__ void update_rows(const void *x, uint32_t row_bytes, int n_tokens, int nb, int K, int g, int groups, int rows, int weight, bool count,
                                            const Shared &ids_x, const Shared &prev, const Shared &table, const Shared &norms, unsigned char *smem, DealLds &deal) {
    const int tid = thread_id(), lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const UpdateLds u(smem, nb, rows);
    int *cnt = u.cnt + w * 64;
    uint32_t *own = u.own + w * (nb * 64 + 1);
    const uint16_t *my = u.ids + w * nb * 64 + lane;                     // the wavefront's quarter of the tokens
    uint32_t *members = reinterpret_cast<uint32_t *>(u.part);            // [K], of the count
    if (count) for (int i = tid; i < K; i += kAsgThreads) members[i] = 0u;
    for (int j0 = -1, end = 0; ; ) {                                     // uniform; from -1 on: its rows are not known yet
        // ---- the unit's ids, four pieces in flight per thread (again for the next rows: the lists of those before are
        // where the ids were) ----
        for (int i0 = tid; i0 < nb * 32; i0 += 4 * kAsgThreads) {
            uint4 v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = ids_x.load16((uint32_t)(i0 + k * kAsgThreads) * 16u);    // (zero beyond the unit)
#pragma unroll
            for (int k = 0; k < 4; ++k) if (i0 + k * kAsgThreads < nb * 32) *reinterpret_cast<uint4 *>(u.ids + (i0 + k * kAsgThreads) * 8) = v[k];
        }
        cnt[lane] = 0;
        __syncthreads();
        if (j0 < 0) {                                                    // uniform
            if (count) {                                                 // uniform
#pragma unroll 4
                for (int i = 0; i < nb; ++i) {
                    const uint32_t id = my[i * 64];
                    if (id < (uint32_t)K) atomicAdd(&members[id], 1u);   // (0xffff: no token)
                }
                __syncthreads();
                int n[kRowsPerThread];
#pragma unroll
                for (int k = 0; k < kRowsPerThread; ++k) n[k] = k * kAsgThreads + tid < K ? (int)members[k * kAsgThreads + tid] : 0;
                deal_rows(n, K, weight, g, groups, deal);
                __syncthreads();
            }
            dealt(deal, j0, end);
        }
        const int c = end - j0 < rows ? end - j0 : rows;
        if (c <= 0) break;
        // ---- the members of these rows, a wavefront's quarter of the tokens at a time, in token order (no branches: what
        // is no member goes to the place behind the last) ----
        int n_own = 0;                                                       // uniform
        for (int i0 = 0; i0 < nb; i0 += 4) {
            uint32_t key[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = i0 + k < nb ? i0 + k : nb - 1;
                key[k] = ((uint32_t)my[i * 64] | (i0 + k < nb ? 0u : 0xffffu)) - (uint32_t)j0;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bool mine = key[k] < (uint32_t)c;
                const uint64_t m = __ballot(mine);
                const int at = n_own + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
                own[mine ? at : nb * 64] = (uint32_t)((w * nb + i0 + k) * 64 + lane) | key[k] << 16;
                n_own += __builtin_popcountll(m);
            }
        }
        // ---- sorted by row: lanes with the same row are ranked by lane number ----
        auto peers_of = [&](uint32_t key, bool mine) {
            uint64_t peers = __ballot(mine);
            for (int b = 0; (c - 1) >> b; ++b) {                             // uniform
                const uint64_t m = __ballot((key >> b) & 1u);
                peers &= ((key >> b) & 1u) ? m : ~m;
            }
            return peers;
        };
        const uint64_t below = (1ull << lane) - 1ull;
        __builtin_amdgcn_wave_barrier();
        for (int e = 0; e < n_own; e += 64) {                                // uniform
            const bool mine = e + lane < n_own;
            const uint32_t key = mine ? own[e + lane] >> 16 : 0u;
            const uint64_t peers = peers_of(key, mine);
            if (mine && !(peers & below)) atomicAdd(&cnt[key], __builtin_popcountll(peers));
        }
        __syncthreads();
        // lane l: row l's members (len) and the first one's place in the list (start), the same in every wavefront
        int len = 0, mine_from = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) { const int n = u.cnt[r * 64 + lane]; if (r < w) mine_from += n; len += n; }
        const int long_min = c <= 2 ? kListShared : kListLong;
        const bool is_long = lane < c && len >= long_min;                    // the long rows' members come behind the others'
        const int n_short = is_long ? 0 : len, upto = scan64(n_short), all_short = __builtin_amdgcn_readlane(upto, 63);
        const int n_long = is_long ? len : 0, upto_long = scan64(n_long);
        const int start = is_long ? all_short + upto_long - len : upto - n_short;
        __syncthreads();                                                     // every wavefront has read the counts
        cnt[lane] = start + mine_from;
        __builtin_amdgcn_wave_barrier();
        for (int e = 0; e < n_own; e += 64) {                                // uniform
            const bool mine = e + lane < n_own;
            const uint32_t v = mine ? own[e + lane] : 0u, key = v >> 16;
            const uint64_t peers = peers_of(key, mine);
            if (mine) {
                const int rank = __builtin_popcountll(peers & below);
                const int at = cnt[key];                                     // read by all peers before the write below
                u.list[at + rank] = (uint16_t)v;
                if (rank == 0) cnt[key] = at + __builtin_popcountll(peers);
            }
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();

        // ---- the rows' sums: lane = channels 2 lane, 2 lane + 1; a member is one load of the wavefront.  (Four rows at a
        // time, 16 lanes with 8 channels each, takes a quarter of the loads and 6.1 instead of 4.4 us on 24 units x 4680 tokens, K =
        // 256: rows of different lengths wait for each other, and the vector ALU is what a SIMD's two wavefronts share.)
        const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(x), 0, (int)((uint32_t)(n_tokens - 1) * row_bytes + kHeadDim * 2), 0x00020000);
        // members m .. m + kRowsAhead - 1 of the list; those behind the end lie beyond the buffer and read as zero
        auto request = [&](int m, int end, uint32_t (&row)[kRowsAhead]) {
            const int i = m + (lane & (kRowsAhead - 1));
            const int at = i < end ? (int)(u.list[i] * row_bytes) : (int)0x80000000u;
#pragma unroll
            for (int k = 0; k < kRowsAhead; ++k)
                row[k] = __builtin_amdgcn_raw_buffer_load_b32(xr, lane * 4 + __builtin_amdgcn_readlane(at, k), 0, 0);
        };
        auto store_sums = [&](int j, double s0, double s1) {
            u.sums[j * kHeadDim + 2 * lane] = s0; u.sums[j * kHeadDim + 2 * lane + 1] = s1;
        };
        // Short lists, a wavefront each, members in token order; the longest first, dealt to and fro.  The next row's first
        // members are requested while this one's are added.
        {
            const bool is_short = n_short > 0;
            int rank = 0;
            for (int j = 0; j < c; ++j) {                                    // uniform
                const int o = __builtin_amdgcn_readlane(is_short ? len : -1, j);
                rank += o > len || (o == len && j < lane);
            }
            if (is_short) cnt[rank] = lane;                                  // this wavefront's copy of the order
            __builtin_amdgcn_wave_barrier();
            const int order = cnt[lane];
            const int rows = __builtin_popcountll(__ballot(is_short));
            auto rank_of = [&](int i) { return 4 * i + (i & 1 ? 3 - w : w); };       // the wavefront's i-th row
            uint32_t row[kRowsAhead], nxt[kRowsAhead];
            int j_n = 0, from_n = 0, n_n = 0;
            auto first = [&](int i) {
                const int r = rank_of(i);
                n_n = 0;
                if (r < rows) {                                              // uniform
                    j_n = __builtin_amdgcn_readlane(order, r);
                    from_n = __builtin_amdgcn_readlane(start, j_n); n_n = __builtin_amdgcn_readlane(len, j_n);
                    request(from_n, from_n + n_n, nxt);
                }
            };
            first(0);
            for (int i = 0; n_n > 0; ++i) {                                  // uniform
                const int j = j_n, from = from_n, n = n_n;
                double s0 = 0.0, s1 = 0.0;
                for (int m = 0; m < n; m += kRowsAhead) {                    // uniform
#pragma unroll
                    for (int k = 0; k < kRowsAhead; ++k) row[k] = nxt[k];
                    if (m + kRowsAhead < n) request(from + m + kRowsAhead, from + n, nxt); else first(i + 1);
#pragma unroll
                    for (int k = 0; k < kRowsAhead; ++k) {                   // (a row that is not there adds +0)
                        if (k == kRowsAhead / 2 && m + k >= n) break;        // uniform
                        s0 += (double)bf16_lo(row[k]); s1 += (double)bf16_hi(row[k]);
                    }
                }
                store_sums(j, s0, s1);
            }
        }
        // Long lists, one after the other, by all wavefronts: partial sums, exact unless the test on the exponents fails (see
        // qvg_kmeans.hip)
        for (uint64_t longs = __ballot(is_long); longs; longs &= longs - 1) {                               // uniform
            const int j = __builtin_ctzll(longs), from = __builtin_amdgcn_readlane(start, j), n = __builtin_amdgcn_readlane(len, j);
            const int m0 = from + n * w / 4, end = from + n * (w + 1) / 4;   // (n >= 32: none is empty)
            double s0 = 0.0, s1 = 0.0;
            uint32_t mx = 0u, mn = ~0u;
            uint32_t row[kRowsAhead], nxt[kRowsAhead];
            request(m0, end, nxt);
            for (int m = m0; m < end; m += kRowsAhead) {                     // uniform
#pragma unroll
                for (int k = 0; k < kRowsAhead; ++k) row[k] = nxt[k];
                if (m + kRowsAhead < end) request(m + kRowsAhead, end, nxt);
#pragma unroll
                for (int k = 0; k < kRowsAhead; ++k) add_pair(row[k], s0, s1, mx, mn);
            }
            u.part[w][lane][0] = s0; u.part[w][lane][1] = s1;
            u.pmx[w][lane] = mx; u.pmn[w][lane] = mn;
            __syncthreads();
            if (w == (j & 3)) {
                s0 = 0.0; s1 = 0.0; mx = 0u; mn = ~0u;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    s0 += u.part[r][lane][0]; s1 += u.part[r][lane][1];
                    mx = pk_max_u16(mx, u.pmx[r][lane]); mn = pk_min_u16(mn, u.pmn[r][lane]);
                }
                if (!__all(mean_exact(mx, mn, 32 - __builtin_clz(n - 1)))) {
                    s0 = 0.0; s1 = 0.0;
                    for (int m = from; m < from + n; m += kRowsAhead) {
                        request(m, from + n, row);
#pragma unroll
                        for (int k = 0; k < kRowsAhead; ++k) { s0 += (double)bf16_lo(row[k]); s1 += (double)bf16_hi(row[k]); }
                    }
                }
                store_sums(j, s0, s1);
            }
            __syncthreads();                      // the partial results are overwritten by the next list
        }
        // ---- the rows: means and norms, 16 lanes each, 8 channels per lane ----
        if (w == 0) cnt[lane] = len;
        __syncthreads();
        for (int j = tid >> 4; j < c; j += kAsgThreads / 16) {
            const int c8 = tid & 15, n = u.cnt[j];
            uint4 v;
            if (n > 0) {
                double s[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) s[e] = u.sums[j * kHeadDim + c8 * 8 + e];
                v = mean_row(s, n);
            } else {
                v = prev.load16((uint32_t)(j0 + j) * (kHeadDim * 2) + c8 * 16);      // an empty group keeps its centroid
            }
            const double q = row_sumsq(v);
            table.store16((uint32_t)(j0 + j) * (kHeadDim * 2) + c8 * 16, v);
            uint2 nh = split_half_norm(q);
            nh.y |= (uint32_t)n << 16;                                       // and the members
            if (c8 == 0) norms.store8((uint32_t)(j0 + j) * 8u, nh);
        }
        j0 += c;
        if (j0 == end) break;
        __syncthreads();
    }
}

__device__ __forceinline__ Shared table_of(const LloydArgs &a, int h) {
    return Shared(a.table + (int64_t)h * a.K * kHeadDim, (uint32_t)a.K * kHeadDim * 2);
}
__device__ __forceinline__ Shared norms_of(const LloydArgs &a, int h) {
    return Shared(a.norms + (int64_t)h * k_padded(a.K), (uint32_t)a.K * 8);
}
__device__ __forceinline__ Shared init_of(const LloydArgs &a, int h, int stage) {
    return Shared(a.init + ((int64_t)h * a.S + stage) * a.K * kHeadDim, (uint32_t)a.K * kHeadDim * 2);
}
// the unit's ids; apart: those of a closed team
__device__ __forceinline__ Shared ids_of(const LloydArgs &a, int h, bool apart) {
    const void *p = apart ? static_cast<const void *>(a.codes + h * a.codes_stride) : a.ids_x + (int64_t)h * a.n_blocks * kAsgThreads;
    return Shared(p, (uint32_t)a.n_blocks * kAsgThreads * 2);
}
// the stage's input
__device__ __forceinline__ const bf16_t *input_of(const LloydArgs &a, int h, int stage) {
    return stage == 0 ? a.x + (int64_t)h * a.stride_head : a.resid[(stage - 1) & 1] + (int64_t)h * a.n_tokens * kHeadDim;
}
__device__ __forceinline__ void load_tokens(int h, int stage, int blk, uint4 (&xa)[2][8]) {
    const LloydArgs &a = args_again();
    const int tid = thread_id(), half = (tid >> 5) & 1;
    const bf16_t *xu = input_of(a, h, stage);
    const int64_t stt = stage == 0 ? a.stride_token : kHeadDim;
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
        const int n = blk * kAsgThreads + (tid >> 6) * kAsgTile + tb * 32 + (tid & 31);
        const bf16_t *xp = xu + (int64_t)n * stt + half * 64;
#pragma unroll
        for (int kk = 0; kk < 8; ++kk)
            xa[tb][kk] = n < a.n_tokens ? *reinterpret_cast<const uint4 *>(xp + kk * 8) : make_uint4(0u, 0u, 0u, 0u);
    }
}

// The current table (the stage's start table, or the update's) into LDS, rows and norms, eight pieces in flight per
// thread.  out: the table goes to the caller.  smax (zero before): the largest norm.
// Deals the rows of the next update among the unit's workgroups, behind the first stage.  deal.zero is kMaxClusters before and after.
__device__ __forceinline__ void stage_table(int h, int stage, bool start, bool out, int g, int groups, unsigned char *smem, DealLds &deal, uint32_t *smax) {
    const LloydArgs &a = args_again();
    const int tid = thread_id(), K = a.K, Kpad = k_padded(K);
    bf16_t *lc = reinterpret_cast<bf16_t *>(smem);                       // [Kpad][kCPitch]
    const Shared src = start ? init_of(a, h, stage) : table_of(a, h);
    const Shared srcn = start ? Shared(a.init_norms + ((int64_t)h * a.S + stage) * Kpad, (uint32_t)K * 8) : norms_of(a, h);
    bf16_t *dst = a.cent_out + (int64_t)h * a.cent_out_stride + (int64_t)stage * K * kHeadDim;
    uint2 nh[kRowsPerThread];
    int members[kRowsPerThread];                                         // (a start table: none)
#pragma unroll
    for (int k = 0; k < kMaxClusters / kAsgThreads; ++k) {
        const int row = tid + k * kAsgThreads;
        nh[k] = srcn.load8((uint32_t)row * 8u);
        members[k] = (int)(nh[k].y >> 16); nh[k].y &= 0xffffu;
        if (row >= K) nh[k] = never_wins();            // rows K..
    }
    constexpr int kBatch = 8;
    for (int i0 = tid; i0 < Kpad * 16; i0 += kAsgThreads * kBatch) {
        uint4 v[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) v[k] = src.load16((uint32_t)(i0 + k * kAsgThreads) * 16u);    // rows K.. read as zero
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int i = i0 + k * kAsgThreads;
            if (i >= Kpad * 16) break;                                   // uniform
            const int row = i >> 4, c16 = i & 15;
            if (out && row < K) *reinterpret_cast<uint4 *>(dst + (int64_t)row * kHeadDim + c16 * 8) = v[k];
            *reinterpret_cast<uint4 *>(lc + row * kCPitch + c16 * 8) = v[k];
        }
    }
#pragma unroll
    for (int k = 0; k < kMaxClusters / kAsgThreads; ++k) {
        const int row = tid + k * kAsgThreads;
        float up = 0.0f;
        if (row < Kpad) {
            *reinterpret_cast<uint4 *>(lc + row * kCPitch + kHeadDim) = make_uint4(nh[k].x, nh[k].y, 0u, 0u);
            if (row < K) {
                up = norm_bound(nh[k]);
                if (stage > 0) note_zero_norm(nh[k], row, &deal.zero);
            }
        }
        if (k * kAsgThreads < Kpad) {                                    // uniform
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) up = fmaxf(up, __shfl_xor(up, off, 64));
            if ((tid & 63) == 0) atomicMax(smax, norm_order(up));
        }
    }
    if (stage > 0) deal_rows(members, K, a.row_weight, g, groups, deal); // uniform
    __syncthreads();
    if (stage > 0) drop_zero_rows(thread_id(), lc, K, nh, &deal.zero);                // uniform
}

// blockIdx.x -> (unit, workgroup of the unit).  With eight units or more a unit's workgroups are 8 apart, on one
// XCD, whose L2 then holds the unit's tokens; they follow each other there, so that workgroups that start in
// order complete one unit after the other.  Fewer units spread over all XCDs.
// FMT: the stored format of the fused rounds (0, or E4M3 scales with one round)
template <int B_, bool FUSED, int T_, int FMT>
__global__ __launch_bounds__(kAsgThreads, 2)
void lloyd_kernel(LloydArgs a0) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t smax;
    __shared__ int number, members;
    __shared__ DealLds deal;
    const int nb = a0.n_blocks;
    int h, g0;
    if (a0.by_xcd) { const int i = (int)(blockIdx.x >> 3); h = (int)(blockIdx.x & 7u) + 8 * (i / a0.groups); g0 = i % a0.groups; }
    else { h = (int)blockIdx.x / a0.groups; g0 = (int)blockIdx.x % a0.groups; }
    if (h >= a0.H) return;                                               // uniform
    // What a team changes waits in LDS and is read anew where a phase begins, as the arguments are.
    __shared__ int lds_groups, lds_g, lds_apart;                         // members, this one's number, a closed team
    if (threadIdx.x == 0) { lds_groups = a0.groups; lds_g = g0; lds_apart = 0; deal.zero = kMaxClusters; }
    __syncthreads();
    auto groups_now = [&] { return __builtin_amdgcn_readfirstlane(lds_groups); };
    auto g_now = [&] { return __builtin_amdgcn_readfirstlane(lds_g); };
    bool formed = a0.groups == 1;                                        // uniform
    uint32_t met = 0;
    auto meet_unit = [&](bool fresh) {
        ++met;
        const uint32_t groups = (uint32_t)groups_now();
        meet(args_again().meet + (int64_t)h * kMeetWords + kLaterWord, groups, met * groups, fresh);
    };

    uint4 xa[2][8];
begin:
    {
        const int g = g_now();
        if (g < nb) load_tokens(h, 0, g, xa);                            // on their way while the table is staged
        if (thread_id() == 0) {
            smax = 0u;
            set_started(args_again().meet + (int64_t)h * kMeetWords, g);
        }
        const int t = thread_id();
        if (t < kMaxClusters / 64) {                                     // the first stage's rows, in equal shares
            const int groups = groups_now(), K = args_again().K;
            deal.below[t] = t ? 0 : K * g / groups; deal.upto[t] = t ? 0 : K * (g + 1) / groups;
        }
    }
    __syncthreads();
    for (int stage = 0; stage < a0.S; ++stage) {
        for (int it = 0; ; ++it) {
            const bool last = it == args_again().iters;                  // uniform: the stage's final assignment
            stage_table(h, stage, it == 0, last && g_now() == 0, g_now(), groups_now(), smem, deal, &smax);
            // ---- this workgroup's tokens ----
            for (int blk = g_now(), groups = groups_now(); blk < nb; blk += groups) {
                if (groups < nb) load_tokens(h, stage, blk, xa);
                const LloydArgs &a = args_again();
                const int tid = thread_id(), lane = tid & 63, wave = tid >> 6, half = lane >> 5, col = lane & 31;
                const int K = a.K, Kpad = k_padded(K), N = a.n_tokens;
                const bf16_t *lc = reinterpret_cast<const bf16_t *>(smem);
                bf16_t *scr = reinterpret_cast<bf16_t *>(smem) + (size_t)Kpad * kCPitch;                // [waves][128]
                float *sscr = reinterpret_cast<float *>(scr + kAsgWaves * kHeadDim);                    // [waves][Kpad]
                const TokenSearch ts(lc, scr + wave * kHeadDim, sscr + wave * Kpad, __uint_as_float(smax), K, Kpad, lane);
                const int n0 = blk * kAsgThreads + wave * kAsgTile;
                int id[2] = {0xffff, 0xffff};
                if (n0 < N) {                                            // uniform per wavefront
                    float xn[2], b1[2], b2[2], b3[2];
                    ts.token_norms(xa, xn);
                    ts.template top_scores<false>(xa, b1, b2, b3);
#pragma unroll
                    for (int tb = 0; tb < 2; ++tb) {
                        if (n0 + tb * 32 >= N) break;                    // uniform
                        const bool valid = n0 + tb * 32 + col < N;
                        const int near = ts.nearest(xa, tb, valid, xn[tb], b1[tb], b2[tb], b3[tb]);
                        if (valid) id[tb] = near;
                    }
                }
                if (!last) {                                             // uniform
                    // the ids, two per word (16 bits, 0xffff where there is no token): word l is tokens 2 l and 2 l + 1
                    const int from = 2 * (lane & 15);
                    const int p0 = __shfl(id[0], from, 64), p1 = __shfl(id[0], from + 1, 64);
                    const int q0 = __shfl(id[1], from, 64), q1 = __shfl(id[1], from + 1, 64);
                    const uint32_t lo = (uint32_t)(lane & 16 ? q0 : p0), hi = (uint32_t)(lane & 16 ? q1 : p1);
                    if (half == 0) ids_of(a, h, __builtin_amdgcn_readfirstlane(lds_apart) != 0).store4((uint32_t)n0 * 2u + lane * 4u, lo | hi << 16);
                    continue;
                }
#pragma unroll
                for (int tb = 0; tb < 2; ++tb) {
                    const int n = n0 + tb * 32 + col;
                    const bool valid = n < N;
                    const int S = a.S;
                    const int64_t hn = (int64_t)h * a.out_stride + n;
                    if (valid && half == 0) store_id(a.ids, hn * S + stage, a.id_wide, (uint32_t)id[tb]);
                    const bf16_t *crow = lc + (id[tb] != 0xffff ? id[tb] : 0) * kCPitch + half * 64;
                    if (stage + 1 < S) {                                 // Eq. 5, rounded to bf16: the next stage's input
                        const Shared resid(a.resid[stage & 1] + (int64_t)h * N * kHeadDim, (uint32_t)N * kHeadDim * 2);
#pragma unroll
                        for (int kk = 0; kk < 8; ++kk) {
                            float xf[8], cf[8];
                            unpack_bf16x8(xa[tb][kk], xf);
                            unpack_bf16x8(*reinterpret_cast<const uint4 *>(crow + kk * 8), cf);
#pragma unroll
                            for (int i = 0; i < 8; ++i) xf[i] -= cf[i];
                            if (valid) {
                                xa[tb][kk] = pack_bf16x8(xf);
                                resid.store16((uint32_t)n * (kHeadDim * 2) + half * 128 + kk * 16, xa[tb][kk]);
                            }
                        }
                    } else if (FUSED) {                                  // Eq. 5, then the T rounds
                        float r[64];
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
                        if constexpr (FMT != 0) {
                            constexpr int BITS = (FMT & kFmtInt4) ? 4 : 2;
                            quantize_token_e4m3<B_, BITS>(r, valid, half, a.codes + hn * (kHeadDim * BITS / 8), static_cast<uint8_t *>(a.scales) + hn * (kHeadDim / B_));
                        } else quantize_token<B_, T_>(r, T, valid, half, a.codes + hn * T * 32, static_cast<f16_t *>(a.scales) + hn * T * (kHeadDim / B_));
                        __builtin_amdgcn_sched_barrier(0);               // keep the two tokens' passes apart: each needs most registers
                    }
                }
            }
            if (last) break;
            if (!formed) {                                               // uniform: the first barrier of all
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // this wavefront's stores have arrived
                __syncthreads();
                if (threadIdx.x == 0) {
                    const LloydArgs &a = args_again();
                    members = team_meet(a.meet + (int64_t)h * kMeetWords, a.wanted, a.groups, nb, a.wait_ticks, number);
                }
                __syncthreads();
                formed = true;
                const int k = __builtin_amdgcn_readfirstlane(members);
                if (k < 0) return;                                       // uniform
                if (k > 0) {                                             // uniform: a closed team, from the beginning
                    if (threadIdx.x == 0) { lds_groups = k; lds_g = number; lds_apart = 1; }
                    __syncthreads();
                    goto begin;
                }
            } else {
                meet_unit(stage > 0 && it == 0);
            }
            if (threadIdx.x == 0) smax = 0u;
            {
                const LloydArgs &a = args_again();
                update_rows(input_of(a, h, stage), stage == 0 ? (uint32_t)a.stride_token * 2u : kHeadDim * 2u, a.n_tokens, nb, a.K, g_now(), groups_now(),
                            a.rows, a.row_weight, stage > 0 && it == 0,
                            ids_of(a, h, __builtin_amdgcn_readfirstlane(lds_apart) != 0), it == 0 ? init_of(a, h, stage) : table_of(a, h),
                            table_of(a, h), norms_of(a, h), smem, deal);
            }
            meet_unit(false);
        }
        if (stage + 1 < a0.S) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();                                             // the staged table is overwritten by the next stage's
            if (threadIdx.x == 0) smax = 0u;
            if (groups_now() < nb) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            __syncthreads();
        }
    }
}

// A row costs what its members cost and as much as this many.
static int row_weight(int K, int nb) {
    const int mean = nb * kAsgThreads / K;
    return mean < 8 ? 8 : mean > 16 ? 16 : mean;
}
static size_t assign_bytes(int K) {
    const int Kpad = k_padded(K);
    return (size_t)Kpad * kCPitch * 2 + (size_t)kAsgWaves * (kHeadDim * 2 + Kpad * sizeof(float));
}
// Rows that a workgroup makes at a time: as many as can have their middle in one share of the weight, where the LDS holds
// them beside a second workgroup's; never fewer than an equal share.
static int rows_at_once(int K, int groups, int nb) {
    const size_t room = assign_bytes(K) > 65536 ? assign_bytes(K) : 65536;
    const int share = (nb * kAsgThreads / row_weight(K, nb) + K) / groups + 2, fit = (int)((room - UpdateLds::bytes(nb, 0)) / 1024);
    const int equal = (K + groups - 1) / groups, most = share < fit ? share : fit;
    const int c = most > equal ? most : equal, rows = c < K ? c : K;
    return rows < kLloydRows ? rows : kLloydRows;
}
static size_t lloyd_smem_bytes(int K, int rows, int nb) {
    const size_t assign = assign_bytes(K), update = UpdateLds::bytes(nb, rows);
    return assign > update ? assign : update;
}

// Norms of the start tables, and the units' meeting words cleared.  16 lanes per centroid, grid: x = rows, y = stage, z = unit.
__global__ __launch_bounds__(kAsgThreads)
void lloyd_prepare_kernel(const bf16_t *init, int K, int Kpad, uint2 *init_norms, uint32_t *meet, int wanted) {
    const int row = (int)blockIdx.x * 16 + (int)(threadIdx.x >> 4), c16 = threadIdx.x & 15;
    const int64_t t = (int64_t)blockIdx.z * gridDim.y + blockIdx.y;
    if (blockIdx.x == 0 && blockIdx.y == 0 && (int)threadIdx.x < kMeetWords * 4)
        reinterpret_cast<unsigned char *>(meet + (int64_t)blockIdx.z * kMeetWords)[threadIdx.x] = (int)threadIdx.x >= kStartedAt + wanted;
    uint4 v = make_uint4(0u, 0u, 0u, 0u);
    if (row < K) v = *reinterpret_cast<const uint4 *>(init + (t * K + row) * kHeadDim + c16 * 8);
    const double s = row_sumsq(v);
    if (row < K && c16 == 0) init_norms[t * Kpad + row] = split_half_norm(s);
}

template <int B_, bool FUSED, int T_, int FMT = 0>
static hipError_t launch_lloyd_t(LloydArgs a, hipStream_t s) {
    const int Kpad = k_padded(a.K), S = a.S;
    static LdsHighWater lds_limit = {};
    const void *kernel = reinterpret_cast<const void *>(&lloyd_kernel<B_, FUSED, T_, FMT>);
    a.row_weight = row_weight(a.K, a.n_blocks);
    a.rows = rows_at_once(a.K, a.groups, a.n_blocks);
    const size_t smem = lloyd_smem_bytes(a.K, a.rows, a.n_blocks);
    hipError_t e = ensure_dynamic_lds(kernel, smem, lds_limit);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(lloyd_prepare_kernel, dim3((unsigned)((a.K + 15) / 16), (unsigned)S, (unsigned)a.H), dim3(kAsgThreads), 0, s,
                       a.init, a.K, Kpad, const_cast<uint2 *>(a.init_norms), a.meet, a.wanted);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    a.by_xcd = a.H >= 8;
    a.wait_ticks = kWaitTicks * (uint32_t)(a.S * a.iters);
    const int64_t grid = a.by_xcd ? (int64_t)8 * a.groups * ((a.H + 7) / 8) : (int64_t)a.groups * a.H;
    hipLaunchKernelGGL((lloyd_kernel<B_, FUSED, T_, FMT>), dim3((unsigned)grid), dim3(kAsgThreads), smem, s, a);
    return hipGetLastError();
}

// Workgroups of a unit, 0: the call is left to the launches of their own.
//
// All workgroups have to run at the same time: two to a CU by registers and LDS, one with more than 256 centroids.  Then
// the launch is taken where it measured faster (24 units x 4680 tokens, K = 256, I = 3: 131 -> 117 us; 10: 346 -> 294; S = 4: 1004 -> 767, 449 since;
// 80 x 1536, K = 64, I = 10: 269 -> 198; 24 x 780, K = 64: 59 -> 50):
// - the chip is more than half full (300 workgroups; at 190 of them, 10 units x 4680, K = 64, 70 -> 84 us);
// - or a unit has up to eight blocks and its lists are short on average (up to 40 members: 6 units x 2000 tokens, K = 64
//   61 -> 59 us, K = 16 62 -> 70).  Every workgroup looks through its whole unit's ids, and few units with long
//   lists have too few wavefronts for the sums: 2 units x 10800, K = 64 65 -> 84 us.
// For the same reason units of more than 24 blocks are left out (I = 10: 8 units x 10800, K = 16 274 -> 324 us, K = 64 257 -> 284, K = 256
// 304 -> 316), and, where lists have more than 64 members on average, those of more than 19 blocks: I = 10, K = 64: 16 units x 20
// blocks 250 -> 258, 24 x 20 257 -> 277, 24 x 21 265 -> 276, K = 16: 16 x 20 298 -> 331, 16 x 21 268 -> 348; but K = 128: 24 x 20 298
// -> 245, K = 256: 326 -> 290, and 19 blocks, K = 64: 24 units 243 -> 242, 16 224 -> 223.  Three iterations lie on the same side each
// time.  Lists of more than 256 stay where the chip is nearly full (400 workgroups: K = 16, 24 x 20 362 -> 316, 24 x 21 398 -> 354).
// (Left in though slower: 24 x 13, K = 64 224 -> 228 us; 32 x 13 231 -> 216, 24 x 16 232 -> 230; 24 x 13, K = 16 310 -> 250.)
// A workgroup with many rows and few blocks to share them is slower too (80 x 800, K = 256: 64 rows each, 111 -> 119 us; 80 x
// 1536, 43 rows, 142 -> 122).
int lloyd_groups(int H, int K, int64_t n_tokens, int64_t stride_token, int iters) {
    const int64_t nb = (n_tokens + kAsgThreads - 1) / kAsgThreads;
    if (iters < 1 || iters > 4096 || nb < 1 || nb > kLloydMaxBlocks || stride_token > ((int64_t)1 << 29) / n_tokens) return 0;
    static int cus[32] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    int n = dev >= 0 && dev < 32 ? cus[dev] : 0;
    if (!n) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        if (dev >= 0 && dev < 32) cus[dev] = n;
    }
    const int64_t units = H >= 8 ? (H + 7) / 8 * 8 : H;                  // by_xcd: whole rounds of the eight XCDs
    if (units * nb > (int64_t)n * (K > 256 ? 1 : 2)) return 0;
    if (nb > 19 && n_tokens > (int64_t)64 * K && (H * nb < 400 || n_tokens <= (int64_t)256 * K)) return 0;
    if (H * nb < 300 && (nb > 8 || n_tokens > (int64_t)40 * K)) return 0;
    // A chip that is not full: more workgroups than blocks, which take rows of the update only, at least eight of them,
    // and at most one workgroup to a CU in all (10 units x 1571 tokens, K = 256: 78 -> 69 us)
    const int64_t spare = (int64_t)n / units, useful = (K + 7) / 8, more = spare < useful ? spare : useful;
    const int64_t groups = more > nb ? more : nb;
    if (n_tokens < 16) return 1;                                         // (a closed team's ids do not fit the codes of fewer tokens)
    return nb < 6 && K > 31 * groups ? 0 : (int)groups;
}

// The formats whose rounds the launch writes itself: 2-bit levels with binary16 scales, and with E4M3 scales one
// round of 2-bit levels in groups of 64 or 16 or of 4-bit levels in groups of 64: the paper's presets but QVG-Pro INT4 (4
// of 461 us, 24 units x 4680 tokens: not worth one more instance).  The others have quantize_kernel after it, a launch that reads the tokens,
// ids and rows once more.
bool lloyd_fuses(int fmt, int B, int T) {
    if (fmt == 0) return true;
    return T == 1 && ((fmt == kFmtE4M3 && (B == 16 || B == 64)) || (fmt == (kFmtE4M3 | kFmtInt4) && B == 64));
}

hipError_t launch_lloyd(const LloydArgs &a, hipStream_t s) {
    if (!a.fused) return launch_lloyd_t<64, false, 0>(a, s);
    if (a.fmt == kFmtE4M3) return a.B == 16 ? launch_lloyd_t<16, true, 1, kFmtE4M3>(a, s) : launch_lloyd_t<64, true, 1, kFmtE4M3>(a, s);
    if (a.fmt != 0) return launch_lloyd_t<64, true, 1, kFmtE4M3 | kFmtInt4>(a, s);
    switch (a.B) {
        case 16: return launch_lloyd_t<16, true, 0>(a, s);
        case 32: return a.T == 3 ? launch_lloyd_t<32, true, 3>(a, s) : launch_lloyd_t<32, true, 0>(a, s);
        case 64:
            switch (a.T) {
                case 1: return launch_lloyd_t<64, true, 1>(a, s);
                case 2: return launch_lloyd_t<64, true, 2>(a, s);
                case 4: return launch_lloyd_t<64, true, 4>(a, s);
                default: return launch_lloyd_t<64, true, 0>(a, s);
            }
        default: return launch_lloyd_t<128, true, 0>(a, s);
    }
}

}  // namespace qvg
