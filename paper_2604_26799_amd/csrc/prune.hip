// Reserve-ratio pruning: for each keep count k_t, the k_t most important
// Gaussians (equal importance: smaller index first), in ascending index order.
// Paper: section "Gaussians Pruning" (the reserve ratio tau keeps the most
// important tau*N Gaussians and cuts the rest).
//
// Importance maps to a 32-bit key, larger importance to a smaller key (-0 and
// +0 alike).  The kept set of count k is every key below the k-th smallest, and
// of the keys equal to it the first ones in index order.
//
// Large inputs.  The k-th key of every count comes from a radix select over
// three digits: a histogram pass over the importance per digit, each of whose
// blocks first picks the digit before from the finished histogram (redundantly:
// a launch between the passes costs more).  The first digit has 15 bits, so that
// few keys share a k's prefix in the second pass, whose bins are too many for
// the blocks to sum them in LDS: about one global atomic per such key (with 13
// bits a million of 5.3e6 keys, 100 us; with 15 a quarter of that).  A compaction then
// writes each kept set in index order: a wavefront owns 1024 consecutive keys,
// counts them against every threshold (one compare and a mask population count
// for 64 keys), a scan per k turns the counts into positions, and the wavefront
// writes its kept indices behind its own running position, without LDS or
// barriers.  Ties across a threshold are counted beside the smaller keys, and
// the scan gives them out in index order.  At 5.3e6 keys and 32 counts: 156 us,
// of which 75 us write the 356 MB of indices (4.7 TB/s) and the three passes
// take 11, 21 and 14 us, bound by the latency of picking the digits; with
// three more digits for the index, a select launch per digit and an LDS scan per
// (chunk, count) in the write it was 356 us.
//
// Inputs of up to 65,536 take one kernel: one workgroup per k holds all keys in
// registers, selects the k-th in LDS and writes the kept set (30 us at n =
// 50,000 and four counts; the launches of the general path take 52 us, and the
// 17 of the earlier one took 81).
#include <algorithm>
#include <cstring>

#include "common.h"

namespace mgs {
namespace {

constexpr int PR_BITS0 = 15;                 // first digit: sign, exponent, 6 bits of the significand
constexpr int PR_BINS0 = 1 << PR_BITS0;
constexpr int PR_REST = 32 - PR_BITS0;       // bits of the second and third digit
constexpr int PR_BITS1 = 9, PR_BITS2 = PR_REST - PR_BITS1;
constexpr int PR_BINS = 1 << PR_BITS1;       // bins of the wider one
constexpr int PR_LDS_ROWS = 58;              // counts whose histogram fits in LDS (the others add to global bins)
constexpr int PR_THREADS = 1024;             // histogram blocks (one per CU: 128 KB of LDS)
constexpr int PR_WAVES = PR_THREADS / MGS_WAVE;
constexpr int PR_HIST_BLOCKS = 96;           // first pass: fewer blocks flush fewer bins
constexpr int PR_ROUNDS = 16;
constexpr int PR_RUN = PR_ROUNDS * MGS_WAVE; // consecutive keys of a compacting wavefront
constexpr int PR_COMPACT_THREADS = 256;
constexpr int64_t PR_SMALL = 65536;          // largest input of the one-kernel form

// The k-th smallest key of one count, as far as it is known.
struct PruneState {
    uint32_t prefix;  // key bits fixed so far (the others 0)
    uint32_t rem;     // rank (1-based) of the wanted key among those with that prefix
    uint32_t have;    // how many there are (rem < have at the end: a tie across the threshold)
    uint32_t pad;
};

struct PruneArgs {
    const float* imp;
    mgs_status_block* status;
    PruneState* state;   // [3][MGS_MAX_RATIOS] after each digit
    uint32_t* hist0;     // [PR_BINS0]
    uint32_t* hist1;     // [T][PR_BINS]
    uint32_t* hist2;     // [T][PR_BINS]
    uint32_t* cnt;       // [T][nstride] keys below the threshold, then the run's first position
    uint32_t* eqc;       // [T][nstride] keys equal to it, then how many of them the runs before take (tied k only)
    int32_t* kept;
    int64_t n;
    int64_t nrun;
    int64_t nstride;     // nrun rounded up to 8: rows of cnt and eqc start on 32 bytes
    int32_t T;
    int32_t pad;
    int64_t k[MGS_MAX_RATIOS];
    int64_t koff[MGS_MAX_RATIOS];
};

__device__ __forceinline__ uint32_t desc_key(float v) {
    const uint32_t b = __float_as_uint(v + 0.0f);             // -0 -> +0
    // negative values keep their bits, the others have all but the sign flipped
    return b ^ (~(uint32_t)((int32_t)b >> 31) & 0x7FFFFFFFu);
}

// Inclusive prefix sum over the lanes of a wavefront.
__device__ __forceinline__ uint32_t wave_inclusive(uint32_t v, int lane) {
#pragma unroll
    for (int o = 1; o < MGS_WAVE; o <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)v, o, MGS_WAVE);
        if (lane >= o) v += y;
    }
    return v;
}

// Exclusive prefix sum over a block of PR_THREADS; `part`: PR_WAVES words.
__device__ __forceinline__ uint32_t block_exclusive(uint32_t v, uint32_t* part, int lane, int wave, uint32_t* total) {
    const uint32_t incl = wave_inclusive(v, lane);
    if (lane == MGS_WAVE - 1) part[wave] = incl;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < PR_WAVES; ++w) {
        if (w < wave) before += part[w];
        all += part[w];
    }
    __syncthreads();
    if (total) *total = all;
    return before + incl - v;
}

// Calls fn(importance) for this block's share of all keys, in any order
// (16-byte loads, four in flight, where the array is aligned to them).
template <typename F>
__device__ __forceinline__ void for_each_importance(const PruneArgs& a, F fn) {
    const int64_t step = (int64_t)gridDim.x * PR_THREADS, i0 = (int64_t)blockIdx.x * PR_THREADS + threadIdx.x;
    if (((uintptr_t)a.imp & 15) == 0) {
        const float4* v4 = (const float4*)a.imp;
        const int64_t n4 = a.n / 4;
        int64_t i = i0;
        for (; i + 3 * step < n4; i += 4 * step) {
            float4 q[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) q[u] = v4[i + u * step];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                fn(q[u].x);
                fn(q[u].y);
                fn(q[u].z);
                fn(q[u].w);
            }
        }
        for (; i < n4; i += step) {
            const float4 q = v4[i];
            fn(q.x);
            fn(q.y);
            fn(q.z);
            fn(q.w);
        }
        if (i0 < a.n - 4 * n4) fn(a.imp[4 * n4 + i0]);
    } else {
        for (int64_t i = i0; i < a.n; i += step) fn(a.imp[i]);
    }
}

// First digit: histogram over all keys (LDS-privatised).
__global__ __launch_bounds__(PR_THREADS) void prune_hist0_kernel(PruneArgs a) {
    extern __shared__ __align__(16) uint32_t h[];  // [PR_BINS0]
    for (int i = threadIdx.x; i < PR_BINS0 / 4; i += PR_THREADS) ((uint4*)h)[i] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    bool bad = false;
    for_each_importance(a, [&](float v) {
        bad |= !finite_f32(v);
        atomicAdd(&h[desc_key(v) >> PR_REST], 1u);
    });
    if (bad) atomicOr(&a.status->nonfinite, 1u);
    __syncthreads();
    for (int i = threadIdx.x; i < PR_BINS0; i += PR_THREADS)
        if (h[i]) atomicAdd(&a.hist0[i], h[i]);
}

// LDS of the second and third pass.
struct PruneShared {
    uint32_t* hist;      // [min(T, PR_LDS_ROWS)][PR_BINS]
    int8_t* slot;        // [PR_BINS0] the digit's first count (of those that own a histogram), -1: none
    uint32_t* pre;       // [MGS_MAX_RATIOS] prefix of each count
    uint32_t* part;      // [PR_WAVES]
    int8_t* next;        // [MGS_MAX_RATIOS] the next count with the same first digit, -1: none
    uint32_t* sums;      // [PR_THREADS] the first digit's counts, prefix sums of 32 bins each
};
__device__ __forceinline__ PruneShared prune_shared(void* base, int T) {
    PruneShared s;
    s.hist = (uint32_t*)base;
    s.slot = (int8_t*)(s.hist + min(T, PR_LDS_ROWS) * PR_BINS);
    s.pre = (uint32_t*)(s.slot + PR_BINS0);
    s.part = s.pre + MGS_MAX_RATIOS;
    s.next = (int8_t*)(s.part + PR_WAVES);
    s.sums = s.pre + MGS_MAX_RATIOS + PR_WAVES + MGS_MAX_RATIOS / 4;
    return s;
}
constexpr size_t prune_lds(int T) {
    return sizeof(uint32_t) * (size_t)(T < PR_LDS_ROWS ? T : PR_LDS_ROWS) * PR_BINS + PR_BINS0 +
           4 * MGS_MAX_RATIOS + 4 * PR_WAVES + MGS_MAX_RATIOS + 4 * PR_THREADS;
}
static_assert(prune_lds(MGS_MAX_RATIOS) <= 163840, "LDS of a CU");

// One count's digit from a histogram of nbins <= PR_BINS bins, by one
// wavefront (lane l: bins [8 l, 8 l + 8)): the digit that holds the rem-th key.
__device__ __forceinline__ PruneState pick_digit(const uint32_t* h, int nbins, int shift, PruneState st, int lane) {
    constexpr int PER = PR_BINS / MGS_WAVE;
    uint32_t c[PER], mine = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        c[j] = lane * PER + j < nbins ? h[lane * PER + j] : 0u;
        mine += c[j];
    }
    const uint32_t before = wave_inclusive(mine, lane) - mine;
    const bool here = before < st.rem && st.rem <= before + mine;
    uint32_t digit = 0, rem = 0, have = 0, cum = before;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
        if (cum < st.rem && st.rem <= cum + c[j]) {
            digit = (uint32_t)(lane * PER + j);
            rem = st.rem - cum;
            have = c[j];
        }
        cum += c[j];
    }
    const uint64_t m = __builtin_amdgcn_ballot_w64(here);
    const int src = m ? __builtin_ctzll(m) : 0;
    PruneState r{};
    r.prefix = st.prefix | ((uint32_t)__builtin_amdgcn_readlane((int)digit, src) << shift);
    r.rem = (uint32_t)__builtin_amdgcn_readlane((int)rem, src);
    r.have = (uint32_t)__builtin_amdgcn_readlane((int)have, src);
    return r;
}

// Second and third digit (LEVEL 1, 2): picks every count's digit before, then
// counts the keys that share a count's prefix (counts with the same prefix
// share a histogram, that of the first of them).
template <int LEVEL>
__global__ __launch_bounds__(PR_THREADS) void prune_hist_kernel(PruneArgs a) {
    extern __shared__ __align__(16) uint32_t lds[];
    const PruneShared s = prune_shared(lds, a.T);
    const int tid = threadIdx.x, lane = tid & (MGS_WAVE - 1), wave = tid / MGS_WAVE;
    for (int i = tid; i < PR_BINS0 / 4; i += PR_THREADS) ((int32_t*)s.slot)[i] = -1;
    const int rows = min(a.T, PR_LDS_ROWS);
    for (int i = tid; i < rows * PR_BINS; i += PR_THREADS) s.hist[i] = 0u;
    // lane u: count u (T <= 64)
    const uint32_t my_k = lane < a.T ? (uint32_t)a.k[lane] : 0u;
    if (LEVEL == 1) {
        // sums of 32 consecutive bins per thread and their prefix; a wavefront
        // finds its count's sum among the 1024 and then its bin among the 32
        constexpr int PER = PR_BINS0 / PR_THREADS;
        static_assert(PER == 32 && PR_THREADS == 1024, "two lookups by ballots");
        // (loads of consecutive pieces by consecutive lanes; eight lanes hold 32 bins)
        const uint4* h4 = (const uint4*)a.hist0;
        uint4 q[PER / 4];
#pragma unroll
        for (int j = 0; j < PER / 4; ++j) q[j] = h4[j * PR_THREADS + tid];
#pragma unroll
        for (int j = 0; j < PER / 4; ++j) {
            uint32_t sum = (q[j].x + q[j].y) + (q[j].z + q[j].w);
#pragma unroll
            for (int o = 1; o < PER / 4; o <<= 1) sum += (uint32_t)__shfl_xor((int)sum, o, MGS_WAVE);
            if (tid % (PER / 4) == 0) s.sums[(j * PR_THREADS + tid) / (PER / 4)] = sum;
        }
        __syncthreads();
        const uint32_t mine = s.sums[tid];  // (each thread replaces its own)
        s.sums[tid] = block_exclusive(mine, s.part, lane, wave, nullptr) + mine;  // inclusive
        __syncthreads();
        for (int t = wave; t < a.T; t += PR_WAVES) {
            const uint32_t k = (uint32_t)__builtin_amdgcn_readlane((int)my_k, t);
            if (k == 0) continue;
            // the first sum >= k: in which 16 of them, then which one
            const int seg = __popcll(__builtin_amdgcn_ballot_w64(s.sums[lane * 16 + 15] < k));
            const int in = __popcll(__builtin_amdgcn_ballot_w64(lane < 16 && s.sums[seg * 16 + (lane & 15)] < k));
            const int g = seg * 16 + in;
            const uint32_t before = g ? s.sums[g - 1] : 0u;
            const uint32_t c = lane < PER ? a.hist0[g * PER + lane] : 0u;
            const uint32_t incl = before + wave_inclusive(c, lane);
            const int bin = __popcll(__builtin_amdgcn_ballot_w64(lane < PER && incl < k));
            const uint32_t have = (uint32_t)__builtin_amdgcn_readlane((int)c, bin);
            const uint32_t upto = (uint32_t)__builtin_amdgcn_readlane((int)incl, bin);
            const uint32_t prefix = (uint32_t)(g * PER + bin) << PR_REST;
            if (lane == 0) {
                s.pre[t] = prefix;
                if (blockIdx.x == 0) a.state[t] = PruneState{prefix, k - (upto - have), have, 0u};
            }
        }
    } else {
        const uint32_t before = my_k ? a.state[lane].prefix : 0u;
        for (int t = wave; t < a.T; t += PR_WAVES) {
            if (__builtin_amdgcn_readlane((int)my_k, t) == 0) continue;
            const PruneState st = a.state[t];
            // the histogram of the first count with this prefix
            const int own = __builtin_ctzll(__builtin_amdgcn_ballot_w64(my_k && before == st.prefix));
            const PruneState r = pick_digit(a.hist1 + own * PR_BINS, 1 << PR_BITS1, PR_BITS2, st, lane);
            if (lane == 0) {
                s.pre[t] = r.prefix;
                if (blockIdx.x == 0) a.state[MGS_MAX_RATIOS + t] = r;
            }
        }
    }
    __syncthreads();
    // ---- the first count with each prefix owns its histogram; owners with the
    // same first digit form a list (one wavefront, lane u: count u)
    if (wave == 0) {
        // (every lane compares its own with all of them, read from LDS: a chain
        // from count to count, a lane at a time, took 4 us)
        const uint32_t pre = my_k ? s.pre[lane] : 0u;
        const uint64_t any = __builtin_amdgcn_ballot_w64(my_k != 0u);
        uint64_t equal = 0, digit = 0;  // the counts with this lane's prefix, first digit
#pragma unroll 8
        for (int t = 0; t < a.T; ++t) {
            const uint32_t pt = s.pre[t];
            equal |= (uint64_t)(pt == pre) << t;
            digit |= (uint64_t)((pt >> PR_REST) == (pre >> PR_REST)) << t;
        }
        const bool owner = my_k && __builtin_ctzll(equal & any) == lane;
        const uint64_t same = digit & __builtin_amdgcn_ballot_w64(owner);  // owners with this lane's first digit
        if (owner) {
            const uint64_t later = lane < 63 ? same >> (lane + 1) : 0ull;
            s.next[lane] = later ? (int8_t)(lane + 1 + __builtin_ctzll(later)) : (int8_t)-1;
            if (__builtin_ctzll(same) == lane) s.slot[pre >> PR_REST] = (int8_t)lane;
        }
    }
    __syncthreads();
    constexpr int fixed = LEVEL == 1 ? PR_REST : PR_BITS2;  // bits below the prefix
    constexpr int bits = LEVEL == 1 ? PR_BITS1 : PR_BITS2;
    uint32_t* out = LEVEL == 1 ? a.hist1 : a.hist2;
    for_each_importance(a, [&](float v) {
        const uint32_t key = desc_key(v);
        int t = s.slot[key >> PR_REST];
        while (t >= 0) {
            if ((key >> fixed) == (s.pre[t] >> fixed)) {
                const uint32_t bin = (uint32_t)t * PR_BINS + ((key >> (fixed - bits)) & ((1u << bits) - 1u));
                if (t < PR_LDS_ROWS) atomicAdd(&s.hist[bin], 1u);
                else atomicAdd(&out[bin], 1u);
            }
            t = LEVEL == 1 ? -1 : s.next[t];  // (one prefix per first digit at level 1)
        }
    });
    __syncthreads();
    // (each block starts elsewhere, so that they do not meet on the same lines)
    const int total = rows * PR_BINS, first = (int)(blockIdx.x * 37 % (unsigned)rows) * PR_BINS;
    for (int j = tid; j < total; j += PR_THREADS) {
        const int i = first + j < total ? first + j : first + j - total;
        if (s.hist[i]) atomicAdd(&out[i], s.hist[i]);
    }
}

// The last digit of every count, one wavefront each.
__global__ __launch_bounds__(MGS_WAVE) void prune_last_kernel(PruneArgs a) {
    const int t = blockIdx.x, lane = threadIdx.x;
    if (a.k[t] <= 0) return;
    const PruneState* st = a.state + MGS_MAX_RATIOS;
    const bool any = lane < a.T && a.k[min(lane, a.T - 1)] > 0;
    const uint32_t mine = any ? st[lane].prefix : 0u;
    const int own = __builtin_ctzll(__builtin_amdgcn_ballot_w64(any && mine == st[t].prefix));
    const PruneState r = pick_digit(a.hist2 + own * PR_BINS, 1 << PR_BITS2, 0, st[t], lane);
    if (lane == 0) a.state[2 * MGS_MAX_RATIOS + t] = r;
}

// A wavefront's run of keys; past the end the largest key, which no finite
// importance has.
struct PruneRun {
    uint32_t key[PR_ROUNDS];
    __device__ __forceinline__ void load(const PruneArgs& a, int64_t run, int lane) {
        float v[PR_ROUNDS];
#pragma unroll
        for (int r = 0; r < PR_ROUNDS; ++r) v[r] = a.imp[min(run * PR_RUN + r * MGS_WAVE + lane, a.n - 1)];
#pragma unroll
        for (int r = 0; r < PR_ROUNDS; ++r)
            key[r] = run * PR_RUN + r * MGS_WAVE + lane < a.n ? desc_key(v[r]) : 0xFFFFFFFFu;
    }
};

__device__ __forceinline__ PruneState final_state(const PruneArgs& a, int t) {
    typedef const __attribute__((address_space(4))) uint32_t* const_u32;  // (scalar loads)
    const const_u32 p = (const_u32)(a.state + 2 * MGS_MAX_RATIOS + t);
    return PruneState{p[0], p[1], p[2], 0u};
}

// The final states of counts t0 + lane, read from the lanes as scalars.
struct LaneStates {
    uint32_t prefix, rem, have;  // have == 0: a count of 0
    __device__ __forceinline__ LaneStates(const PruneArgs& a, int t0, int lane) {
        const int t = min(t0 + lane, a.T - 1);
        const PruneState st = a.state[2 * MGS_MAX_RATIOS + t];
        prefix = st.prefix;
        rem = st.rem;
        have = a.k[t] > 0 ? st.have : 0u;
    }
    __device__ __forceinline__ PruneState get(int l) const {
        return PruneState{(uint32_t)__builtin_amdgcn_readlane((int)prefix, l),
                          (uint32_t)__builtin_amdgcn_readlane((int)rem, l),
                          (uint32_t)__builtin_amdgcn_readlane((int)have, l), 0u};
    }
};

// The run of a compacting wavefront: blocks go round-robin over the XCDs, each
// of which takes a contiguous piece of the runs, so that the cache lines
// between two runs' indices are written through one L2.  -1: none.
constexpr int PR_XCDS = 8;
__device__ __forceinline__ int64_t compact_run(const PruneArgs& a, int wave) {
    const int64_t per = gridDim.x / PR_XCDS;  // (a whole number of rounds)
    const int64_t b = (int64_t)(blockIdx.x % PR_XCDS) * per + blockIdx.x / PR_XCDS;
    const int64_t run = b * (PR_COMPACT_THREADS / MGS_WAVE) + wave;
    return run < a.nrun ? run : -1;
}

// Compaction, counts: one wavefront per (run, counts [blockIdx.y * tb, + tb)).
__global__ __launch_bounds__(PR_COMPACT_THREADS) void prune_count_kernel(PruneArgs a, int tb) {
    const int lane = threadIdx.x & (MGS_WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / MGS_WAVE);
    const int64_t run = compact_run(a, wave);
    if (run < 0) return;
    PruneRun keys;
    keys.load(a, run, lane);
    const int t0 = blockIdx.y * tb, t1 = min(a.T, t0 + tb);
    uint32_t mine = 0, mine_eq = 0;  // lane t - t0: the count's numbers
    const LaneStates states(a, t0, lane);
    for (int t = t0; t < t1; ++t) {
        const PruneState st = states.get(t - t0);
        if (st.have == 0) continue;  // its numbers are never read
        const bool tied = st.rem < st.have;
        uint32_t c = 0, e = 0;
        if (!tied) {
#pragma unroll
            for (int r = 0; r < PR_ROUNDS; ++r)
                c += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(keys.key[r] <= st.prefix));
        } else {
#pragma unroll
            for (int r = 0; r < PR_ROUNDS; ++r) {
                c += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(keys.key[r] < st.prefix));
                e += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(keys.key[r] == st.prefix));
            }
        }
        if (lane == t - t0) {
            mine = c;
            mine_eq = e;
        }
    }
    if (t0 + lane < t1) {
        a.cnt[(int64_t)(t0 + lane) * a.nstride + run] = mine;
        a.eqc[(int64_t)(t0 + lane) * a.nstride + run] = mine_eq;
    }
}

// Compaction, scan: each run's first position, one block per count.  A tied
// count keeps, of the keys equal to its threshold, the first rem in index order.
__global__ __launch_bounds__(PR_THREADS) void prune_scan_kernel(PruneArgs a) {
    constexpr int PER = 8;
    __shared__ uint32_t part[PR_WAVES];
    const int t = blockIdx.x;
    if (a.k[t] <= 0) return;
    const int lane = threadIdx.x & (MGS_WAVE - 1), wave = threadIdx.x / MGS_WAVE;
    uint32_t* c = a.cnt + (int64_t)t * a.nstride;
    uint32_t* e = a.eqc + (int64_t)t * a.nstride;
    const PruneState st = final_state(a, t);
    const bool tied = st.rem < st.have;
    uint32_t carry = 0, carry_eq = 0;
    // (rows are whole groups of 8; the numbers past nrun are never read)
    for (int64_t b0 = 0; b0 < a.nstride; b0 += PR_THREADS * PER) {
        const int64_t b = b0 + (int64_t)threadIdx.x * PER;
        const bool in = b < a.nstride;
        uint32_t v[PER] = {}, sum = 0, total;
        auto load = [&](const uint32_t* p, uint32_t (&x)[PER]) {
            if (!in) return;
            const uint4 lo = *(const uint4*)(p + b), hi = *(const uint4*)(p + b + 4);
            x[0] = lo.x; x[1] = lo.y; x[2] = lo.z; x[3] = lo.w;
            x[4] = hi.x; x[5] = hi.y; x[6] = hi.z; x[7] = hi.w;
#pragma unroll
            for (int j = 0; j < PER; ++j)
                if (b + j >= a.nrun) x[j] = 0u;
        };
        auto store = [&](uint32_t* p, const uint32_t (&x)[PER]) {
            if (!in) return;
            *(uint4*)(p + b) = make_uint4(x[0], x[1], x[2], x[3]);
            *(uint4*)(p + b + 4) = make_uint4(x[4], x[5], x[6], x[7]);
        };
        load(c, v);
        if (tied) {
            uint32_t q[PER] = {}, sq = 0;
            load(e, q);
#pragma unroll
            for (int j = 0; j < PER; ++j) sq += q[j];
            uint32_t before = carry_eq + block_exclusive(sq, part, lane, wave, &total);
            carry_eq += total;
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                const uint32_t taken = min(before, st.rem);  // by the runs before
                before += q[j];
                v[j] += min(before, st.rem) - taken;
                q[j] = taken;
            }
            store(e, q);
        }
#pragma unroll
        for (int j = 0; j < PER; ++j) sum += v[j];
        uint32_t at = carry + block_exclusive(sum, part, lane, wave, &total);
        carry += total;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const uint32_t x = v[j];
            v[j] = at;
            at += x;
        }
        store(c, v);
    }
}

// The position of a lane among the set lanes of m, behind `base`.
__device__ __forceinline__ uint32_t mask_position(uint64_t m, uint32_t base) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, base));
}

// Writes the kept indices of one run (first index i0) for one count behind
// `base`; for a tied count `eq_taken` of its `rem` equal keys went to earlier runs.
template <int ROUNDS>
__device__ __forceinline__ void write_run(const uint32_t (&key)[ROUNDS], uint32_t th, bool tied, uint32_t rem,
                                          uint32_t base, uint32_t eq_taken, uint32_t k, int32_t* out, uint32_t i0,
                                          int lane, int used = ROUNDS) {
    if (!tied) {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            if (r >= used) continue;
            const bool keep = key[r] <= th;
            const uint64_t m = __builtin_amdgcn_ballot_w64(keep);
            const uint32_t pos = mask_position(m, base);
            if (keep && pos < k) out[pos] = (int32_t)(i0 + r * MGS_WAVE + lane);
            base += (uint32_t)__popcll(m);
        }
    } else {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            if (r >= used) continue;
            uint32_t kr = key[r];
            asm volatile("" : "+v"(kr));  // (a round's masks when it is due: all of them do not fit the scalar registers)
            const bool eq = kr == th;
            const uint64_t me = __builtin_amdgcn_ballot_w64(eq);
            const bool keep = kr < th || (eq && mask_position(me, eq_taken) < rem);
            eq_taken += (uint32_t)__popcll(me);
            const uint64_t m = __builtin_amdgcn_ballot_w64(keep);
            const uint32_t pos = mask_position(m, base);
            if (keep && pos < k) out[pos] = (int32_t)(i0 + r * MGS_WAVE + lane);
            base += (uint32_t)__popcll(m);
        }
    }
}

// Compaction, write.
__global__ __launch_bounds__(PR_COMPACT_THREADS) void prune_write_kernel(PruneArgs a, int tb) {
    const int lane = threadIdx.x & (MGS_WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / MGS_WAVE);
    const int64_t run = compact_run(a, wave);
    if (run < 0) return;
    PruneRun keys;
    keys.load(a, run, lane);
    const int t0 = blockIdx.y * tb, t1 = min(a.T, t0 + tb);
    const LaneStates states(a, t0, lane);
    const int tl = min(t0 + lane, t1 - 1);  // lane t - t0: the run's first position and equal keys taken before
    const uint32_t my_base = a.cnt[(int64_t)tl * a.nstride + run], my_eq = a.eqc[(int64_t)tl * a.nstride + run];
    for (int t = t0; t < t1; ++t) {
        const PruneState st = states.get(t - t0);
        if (st.have == 0) continue;
        const uint32_t base = (uint32_t)__builtin_amdgcn_readlane((int)my_base, t - t0);
        const uint32_t eq = (uint32_t)__builtin_amdgcn_readlane((int)my_eq, t - t0);
        write_run<PR_ROUNDS>(keys.key, st.prefix, st.rem < st.have, st.rem, base, eq, (uint32_t)a.k[t],
                             a.kept + a.koff[t], (uint32_t)(run * PR_RUN), lane);
    }
}

// Inputs of up to 64 * ROUNDS * 16: one block per count, wavefront w holding
// keys [w * 64 ROUNDS, + 64 ROUNDS).  Three digits (13, 10 and 9 bits) in LDS.
//
// What bounds it: the instructions of one CU's 16 wavefronts (64 keys per
// thread).  So the keys that share the first digit, a few hundred, go to a list
// in LDS, and the other digits look at that alone; more than PR_LIST of them
// (ties, or values close together) are counted from the registers.
constexpr int PR_SMALL_BITS[3] = {13, 10, 9};
constexpr int PR_LIST = 4096;
constexpr int PR_CROWD = 8;  // of the first 64 keys in one bin
template <int ROUNDS>
__global__ __launch_bounds__(PR_THREADS) void prune_small_kernel(PruneArgs a) {
    __shared__ __align__(16) uint32_t h[1 << PR_SMALL_BITS[0]];
    __shared__ uint32_t list[PR_LIST];
    __shared__ uint32_t part[PR_WAVES], found[3], below[PR_WAVES], equal[PR_WAVES], nlist;
    const int t = blockIdx.x, tid = threadIdx.x;
    const int lane = tid & (MGS_WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / MGS_WAVE);
    const uint32_t n = (uint32_t)a.n;
    // rounds in use, the same for every wavefront (a round of keys past the end
    // would be one bin's, 64 additions to one address)
    const int used = (int)((n + PR_THREADS - 1) / PR_THREADS);
    const uint32_t i0 = (uint32_t)(wave * used) * MGS_WAVE;
    uint32_t key[ROUNDS];
    {
        float v[ROUNDS], nan = 0.0f;
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) v[r] = r < used ? a.imp[min(i0 + r * MGS_WAVE + lane, n - 1u)] : 0.0f;
        // (past the end the largest key: it ranks behind every finite one, so
        // no pass has to leave it out)
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            nan = __builtin_fmaf(v[r], 0.0f, nan);  // NaN once a value is not finite
            key[r] = r < used && i0 + r * MGS_WAVE + lane < n ? desc_key(v[r]) : 0xFFFFFFFFu;
        }
        // every block sees all keys: the first one sets the status word
        const int any = __syncthreads_or(__builtin_isnan(nan));
        if (t == 0 && tid == 0) a.status->nonfinite = any ? 1u : 0u;
    }
    const uint32_t k = (uint32_t)a.k[t];
    if (k == 0) return;
    uint32_t prefix = 0, rem = k, have = 0;
    // the digit [fixed - bits, fixed) from the histogram just made
    auto pick = [&](int fixed, int bits) {
        const int nbins = 1 << bits, per = nbins > PR_THREADS ? nbins / PR_THREADS : 1;
        __syncthreads();
        uint32_t c[8] = {}, mine = 0;
        if (per == 8) {  // (16-byte reads: single ones, 8 words apart, meet in eight banks)
            const uint4 lo = ((const uint4*)h)[2 * tid], hi = ((const uint4*)h)[2 * tid + 1];
            c[0] = lo.x; c[1] = lo.y; c[2] = lo.z; c[3] = lo.w;
            c[4] = hi.x; c[5] = hi.y; c[6] = hi.z; c[7] = hi.w;
        } else if (tid < nbins) {
            c[0] = h[tid];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) mine += c[j];
        uint32_t cum = block_exclusive(mine, part, lane, wave, nullptr);
        if (cum < rem && rem <= cum + mine) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (cum < rem && rem <= cum + c[j]) {
                    found[0] = (uint32_t)(tid * per + j);
                    found[1] = rem - cum;
                    found[2] = c[j];
                }
                cum += c[j];
            }
        }
        __syncthreads();
        prefix |= found[0] << (fixed - bits);
        rem = found[1];
        have = found[2];
    };
    auto clear = [&](int bits) {
        for (int i = tid; i < 1 << bits; i += PR_THREADS) h[i] = 0u;
        __syncthreads();
    };
    constexpr int F1 = 32 - PR_SMALL_BITS[0], F2 = F1 - PR_SMALL_BITS[1];
    static_assert((1 << PR_SMALL_BITS[0]) == 8 * PR_THREADS && PR_SMALL_BITS[1] <= 10 && PR_SMALL_BITS[2] <= 10, "bins per thread: 8 or 1");
    if (tid == 0) nlist = 0u;
    clear(PR_SMALL_BITS[0]);
    // Where a wavefront's first keys crowd into one bin (many equal ones), it counts
    // that bin by masks: additions to one address take their turns, 33 of the 61 us
    // at 50,000 keys of which nine in ten are 0.
    uint32_t crowd = (uint32_t)__builtin_amdgcn_readlane((int)key[0], 0) >> F1;
    {
        const uint32_t b0 = key[0] >> F1, other = (uint32_t)__builtin_amdgcn_readlane((int)b0, MGS_WAVE / 2);
        const int n1 = __popcll(__builtin_amdgcn_ballot_w64(b0 == crowd));
        const int n2 = __popcll(__builtin_amdgcn_ballot_w64(b0 == other));
        if (n2 > n1) crowd = other;
        if (max(n1, n2) < PR_CROWD) {
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r)
                if (r < used) atomicAdd(&h[key[r] >> F1], 1u);
        } else {
            uint32_t count = 0;
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r) {
                if (r >= used) continue;
                const uint32_t b = key[r] >> F1;
                count += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(b == crowd));
                if (b != crowd) atomicAdd(&h[b], 1u);
            }
            if (lane == 0) atomicAdd(&h[crowd], count);
        }
    }
    pick(32, PR_SMALL_BITS[0]);
    const bool listed = have <= PR_LIST;
    const uint32_t nl = have;
    if (listed) {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r)
            if (r < used && (key[r] >> F1) == (prefix >> F1)) list[atomicAdd(&nlist, 1u) & (PR_LIST - 1)] = key[r];
    }
    clear(PR_SMALL_BITS[1]);
    if (listed) {
        for (uint32_t i = tid; i < nl; i += PR_THREADS)
            atomicAdd(&h[(list[i] >> F2) & ((1u << PR_SMALL_BITS[1]) - 1u)], 1u);
    } else {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r)
            if (r < used && (key[r] >> F1) == (prefix >> F1))
                atomicAdd(&h[(key[r] >> F2) & ((1u << PR_SMALL_BITS[1]) - 1u)], 1u);
    }
    pick(F1, PR_SMALL_BITS[1]);
    clear(PR_SMALL_BITS[2]);
    if (listed) {
        for (uint32_t i = tid; i < nl; i += PR_THREADS)
            if ((list[i] >> F2) == (prefix >> F2)) atomicAdd(&h[list[i] & ((1u << PR_SMALL_BITS[2]) - 1u)], 1u);
    } else {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r)
            if (r < used && (key[r] >> F2) == (prefix >> F2)) atomicAdd(&h[key[r] & ((1u << PR_SMALL_BITS[2]) - 1u)], 1u);
    }
    pick(F2, PR_SMALL_BITS[2]);
    // ---- positions: keys below the threshold (and equal to it) in earlier wavefronts
    const bool tied = rem < have;
    uint32_t lt = 0, eq = 0;
    if (!tied) {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r)
            if (r < used) lt += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(key[r] <= prefix));
    } else {
#pragma unroll
        for (int r = 0; r < ROUNDS; ++r) {
            if (r >= used) continue;
            lt += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(key[r] < prefix));
            eq += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(key[r] == prefix));
        }
    }
    if (lane == 0) {
        below[wave] = lt;
        equal[wave] = eq;
    }
    __syncthreads();
    uint32_t base = 0, taken = 0;
    for (int w = 0; w < wave; ++w) {
        base += below[w];
        taken += equal[w];
    }
    taken = min(taken, rem);
    write_run<ROUNDS>(key, prefix, tied, rem, base + (tied ? taken : 0u), taken, k, a.kept + a.koff[t], i0, lane, used);
}

// Workspace layout.
struct PruneLayout {
    size_t state, hist0, hist1, hist2, cnt, eqc, total;
    int64_t nrun, nstride;
};

PruneLayout prune_layout(int64_t n, int32_t T) {
    PruneLayout L;
    const size_t t = (size_t)std::max(T, 1);
    L.nrun = (n + PR_RUN - 1) / PR_RUN;
    L.nstride = (L.nrun + 7) / 8 * 8;
    size_t o = MGS_STATUS_BYTES;
    L.state = o;
    o += sizeof(PruneState) * 3 * MGS_MAX_RATIOS;
    L.hist0 = o;
    o += sizeof(uint32_t) * PR_BINS0;
    L.hist1 = o;
    o += sizeof(uint32_t) * PR_BINS * t;
    L.hist2 = o;
    o += sizeof(uint32_t) * PR_BINS * t;
    L.cnt = o;
    o += mgs_align_up(sizeof(uint32_t) * (size_t)std::max<int64_t>(L.nstride, 1) * t, 256);
    L.eqc = o;
    o += mgs_align_up(sizeof(uint32_t) * (size_t)std::max<int64_t>(L.nstride, 1) * t, 256);
    L.total = o;
    return L;
}

// (A grid's LDS beyond 64 KB has to be allowed once per kernel and device;
// repeating it is cheap and needs no state.)
template <typename K>
int prune_allow_lds(K kernel, size_t bytes) {
    return mgs_hip_status(hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                              (int)bytes));
}

}  // namespace
}  // namespace mgs

extern "C" size_t mgs_prune_select_ws_bytes(int64_t n, int32_t T) {
    if (n < 0) n = 0;
    if (T < 1) T = 1;
    if (T > MGS_MAX_RATIOS) T = MGS_MAX_RATIOS;
    return mgs::prune_layout(n, T).total;
}

extern "C" int mgs_prune_select(const float* d_imp, int64_t n, const int64_t* h_k, int32_t T,
                                int32_t* d_kept, void* d_ws, size_t ws_bytes, void* stream) {
    using namespace mgs;
    if (n < 0 || n >= ((int64_t)1 << 31) || T < 1 || T > MGS_MAX_RATIOS || !h_k) return MGS_EINVAL;
    int64_t ksum = 0;
    for (int t = 0; t < T; ++t) {
        if (h_k[t] < 0 || h_k[t] > n) return MGS_EINVAL;
        ksum += h_k[t];
    }
    if (n > 0 && !d_imp) return MGS_EINVAL;
    if (ksum > 0 && !d_kept) return MGS_EINVAL;
    PruneLayout L = prune_layout(n, T);
    if (!d_ws || ws_bytes < L.total) return MGS_EWORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    char* ws = (char*)d_ws;
    if (n == 0 || ksum == 0) return mgs_fill<uint32_t>((uint32_t*)ws, 64, 0u, s);
    PruneArgs a;
    std::memset(&a, 0, sizeof(a));
    a.imp = d_imp;
    a.status = (mgs_status_block*)ws;
    a.state = (PruneState*)(ws + L.state);
    a.hist0 = (uint32_t*)(ws + L.hist0);
    a.hist1 = (uint32_t*)(ws + L.hist1);
    a.hist2 = (uint32_t*)(ws + L.hist2);
    a.cnt = (uint32_t*)(ws + L.cnt);
    a.eqc = (uint32_t*)(ws + L.eqc);
    a.kept = d_kept;
    a.n = n;
    a.nrun = L.nrun;
    a.nstride = L.nstride;
    a.T = T;
    int64_t off = 0;
    for (int t = 0; t < T; ++t) {
        a.k[t] = h_k[t];
        a.koff[t] = off;
        off += h_k[t];
    }
    if (n <= PR_SMALL) {
        if (n <= PR_SMALL / 4)
            hipLaunchKernelGGL(prune_small_kernel<16>, dim3(T), dim3(PR_THREADS), 0, s, a);
        else
            hipLaunchKernelGGL(prune_small_kernel<64>, dim3(T), dim3(PR_THREADS), 0, s, a);
        return mgs_last_launch();
    }
    const size_t lds0 = sizeof(uint32_t) * PR_BINS0, lds = prune_lds(T);
    int rc = prune_allow_lds(prune_hist0_kernel, lds0);
    if (!rc) rc = prune_allow_lds(prune_hist_kernel<1>, lds);
    if (!rc) rc = prune_allow_lds(prune_hist_kernel<2>, lds);
    // status, states and histograms, in one piece
    if (!rc) rc = mgs_fill<uint32_t>((uint32_t*)ws, (int64_t)(L.cnt / sizeof(uint32_t)), 0u, s);
    if (rc) return rc;
    const int64_t per_block = (int64_t)PR_THREADS * 16;
    const unsigned hb0 = (unsigned)std::min<int64_t>((n + per_block - 1) / per_block, PR_HIST_BLOCKS);
    const unsigned hb = (unsigned)std::min<int64_t>((n + per_block - 1) / per_block, 256);
    hipLaunchKernelGGL(prune_hist0_kernel, dim3(hb0), dim3(PR_THREADS), lds0, s, a);
    hipLaunchKernelGGL(prune_hist_kernel<1>, dim3(hb), dim3(PR_THREADS), lds, s, a);
    hipLaunchKernelGGL(prune_hist_kernel<2>, dim3(hb), dim3(PR_THREADS), lds, s, a);
    hipLaunchKernelGGL(prune_last_kernel, dim3(T), dim3(MGS_WAVE), 0, s, a);
    // counts per compacting wavefront: about 16384 wavefronts, twice what the
    // chip holds (5.3e6 keys, 32 counts: 161 us in all, 169 with 8192)
    const int64_t groups = std::min<int64_t>(T, std::max<int64_t>(1, 16384 / a.nrun));
    const int tb = (int)((T + groups - 1) / groups);
    const int64_t cblocks = (a.nrun + PR_COMPACT_THREADS / MGS_WAVE - 1) / (PR_COMPACT_THREADS / MGS_WAVE);
    const dim3 cgrid((unsigned)((cblocks + PR_XCDS - 1) / PR_XCDS * PR_XCDS), (unsigned)((T + tb - 1) / tb));
    hipLaunchKernelGGL(prune_count_kernel, cgrid, dim3(PR_COMPACT_THREADS), 0, s, a, tb);
    hipLaunchKernelGGL(prune_scan_kernel, dim3(T), dim3(PR_THREADS), 0, s, a);
    hipLaunchKernelGGL(prune_write_kernel, cgrid, dim3(PR_COMPACT_THREADS), 0, s, a, tb);
    return mgs_last_launch();
}
