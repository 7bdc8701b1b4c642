// Region-Adaptive Hierarchical Transform of the attributes over the
// voxelized positions.  Paper: section "Attribute Transformation",
// paragraph "Region Adaptive Hierarchical Transform" (transform T_1, its 2-D
// example, leaf weight 1, merged weight the sum of the child weights,
// unmatched coefficients passing to the next layer, one DC and N - 1 AC
// coefficients per channel).
//
// Positions are Morton codes (per level: x in bit 0, y in bit 1, z in bit 2),
// strictly increasing.  Step s = 0, 1, ..., 3 * depth - 1 merges, along the
// axis of bit s, every two live nodes whose codes agree above bit s: the one
// with bit s clear (weight w1, value a1) and the one with it set (w2, a2):
//   L = (sqrt(w1) a1 + sqrt(w2) a2) / sqrt(w1 + w2)      (goes up, weight w1 + w2)
//   H = (sqrt(w1) a2 - sqrt(w2) a1) / sqrt(w1 + w2)      (AC coefficient)
// A merged node keeps the slot of its first leaf.  Output per channel:
// coefficient 0 = DC (the root's value), then the AC coefficients in the
// order they are made (step by step, within a step in Morton order).  FP64
// arithmetic in the order above, FP32 storage; a quotient is within half a unit in
// the last place plus 2^-104 of its exact value (see quotients()).  The inverse
// undoes the merges in reverse:  a1 = (sqrt(w1) L - sqrt(w2) H) / sqrt(w1 + w2),
//                         a2 = (sqrt(w2) L + sqrt(w1) H) / sqrt(w1 + w2).
//
// The merge structure follows from the codes alone: every merge joins the
// leaves on the two sides of one boundary i between neighbouring codes (N - 1
// boundaries, N - 1 merges).  With d the highest bit in which code[i] and
// code[i + 1] differ, the merge happens at step d and joins the leaves [L, i]
// and [i + 1, R], the run of codes that agree with code[i] above bit d (every
// boundary inside either side differs lower, so each side is one node by then);
// the weights are i - L + 1 and R - i.  The AC index of the merge is its rank
// in (step, boundary) order: counts per (step, block of leaves), a scan over
// them, and the rank within the block by wavefront ballots.
//
// Most merges are local: a run of 256 neighbouring leaves contains all but
// about eight of its merges whole, so the steps are not run one after the other over
// all nodes.  One wavefront takes a tile of 256 leaves, does every merge whose
// run [L, R] lies inside the tile, in step order, on values in LDS, and hands
// on the nodes that are left: the maximal subtrees of a contiguous run of
// leaves, at most two per step (6 depth), about eight of 256 in a scene.  The
// next level joins 16 such lists in the same way, and so on: five levels reach
// the root of 8 million leaves.  The inverse builds the lists bottom-up without
// values and undoes the merges level by level from the root.
//
// What bounds it, at 5.3e6 x 20 on an MI355X: the leaf level (0.38 ms of 0.49)
// reads and writes every attribute once (0.93 GB by the counters, 0.19 ms at
// the rate of a copy) and adds the structure's and the steps' instructions: its
// vector units are busy 0.7 of the time, its LDS half of it.  A round of 64
// (merge, channel) pairs is 26 vector instructions, 24 rounds per 256 leaves and
// four channels.  With weights looked up inside the round, conditions as
// branches and 40 instructions it took 0.46 ms.  Tiles of 128 leaves and 10 channels measured
// 0.69 ms for the whole against 0.62 then, of 64 leaves and 20 channels 0.84:
// fewer rounds per channel, but twice and four times the nodes for the upper
// levels, which are chains of about 20 steps each (0.12 ms).  Run as one launch
// per step over node values in HBM (42 dependent launches, rows of both nodes
// fetched from all over the array) the forward took 1.95 ms at 5.3e6 x 20 and the
// inverse 0.58 ms at 1e6 x 20, which is 0.17 ms now.
#include <algorithm>
#include <cstring>

#include "common.h"

namespace mgs {
namespace {

constexpr int RH_STEPS = 64;                         // bins of merge steps (3 depth <= 63; 63: never merged)
constexpr int RH_TILE = 256;                         // leaves per wavefront at the leaf level
constexpr int RH_ROUNDS = RH_TILE / MGS_WAVE;
constexpr int RH_WAVES = 8;
constexpr int RH_THREADS = RH_WAVES * MGS_WAVE;
constexpr int RH_SPAN = RH_TILE * RH_WAVES;          // leaves per block of the counts
constexpr int RH_MAX_SPANS = 4096;                   // N - 1 <= RH_SPAN * RH_MAX_SPANS
constexpr int RH_MAX_BLOCKS = RH_MAX_SPANS + 1;       // blocks of RH_SPAN leaves
constexpr int RH_CH = 4;                             // channels in LDS at a time (78.5 KB per block: two per CU)
constexpr int RH_UCH = 4;                            // the same at the upper levels
constexpr int RH_VS = RH_TILE + 1;                   // row stride of the values (channels in different banks)
constexpr int RH_GROUP = 16;                         // lists that an upper level joins
constexpr int RH_UPPER_MIN = 256;                     // threads of a group's block at least
constexpr int RH_UPPER_MAX = 512;                     // and at most
constexpr int RH_UPPER_WAVES = RH_UPPER_MAX / MGS_WAVE;
constexpr int RH_CAP1 = 256;                          // nodes of a group in LDS at the first upper level,
constexpr int RH_CAP2 = 768;                          // and above it (few groups, lists of more nodes)
constexpr int RH_LEVELS = 5;                         // leaf level and up to four above it

// The nodes that a level leaves, per tile (leaf level) or group of 16 lists.
struct RahtLevel {
    int32_t* cnt;     // [lists] nodes in the list
    int32_t* first;   // [lists][stride] first leaf of each node (a node reaches to the next one's first leaf)
    uint64_t* code;   // [lists][stride] its code
    int32_t* ac;      // [lists][stride] AC index of the merge across the boundary after the node
    double* rows;     // [lists][stride][C] values
    int32_t lists;
};

struct RahtArgs {
    const uint64_t* codes;
    int64_t N;
    int32_t C;
    int32_t depth;
    int64_t ld, ld_in;     // of the output and of the input (which may lie in the workspace)
    const float* attr;     // forward input [C][ld_in]
    const float* coef_in;  // inverse input [C][ld_in]
    float* coef;           // forward output [C][ld]
    float* attr_out;       // inverse output [C][ld]
    int32_t* cnt;          // [RH_STEPS][nblk] boundaries per (step, block), then their exclusive prefix in the step
    int32_t* tot;          // [RH_STEPS] boundaries per step
    uint32_t* bad;         // [nblk] codes of the block out of order or range
    // scratch of a group whose lists hold more than RH_TILE nodes, per node of the level below
    uint64_t* big_code;
    int32_t* big_i;        // [RH_BIG_ARRAYS][big_stride]
    int64_t big_stride;
    mgs_status_block* status;
    int32_t nblk;          // blocks of RH_SPAN leaves
    int32_t stride;        // node slots per list
    int32_t top;           // the last level (one list, the root)
    RahtLevel lev[RH_LEVELS];
};

enum { RH_FORWARD = 0, RH_STRUCTURE = 1, RH_INVERSE = 2 };

// The merge step of the boundary between two neighbouring codes.  Codes that
// do not increase or lie outside the grid (flagged by the counting kernel) are
// never merged; every index stays in bounds all the same.
__device__ __forceinline__ int merge_step(uint64_t c0, uint64_t c1, int bits) {
    if (c1 <= c0) return RH_STEPS - 1;
    const int d = 63 - __clzll((long long)(c0 ^ c1));
    return d >= bits ? RH_STEPS - 1 : d;
}

// Lanes (of `valid`) that hold the same bin as this one.
__device__ __forceinline__ uint64_t same_bin(bool valid, int b) {
    uint64_t eq = __builtin_amdgcn_ballot_w64(valid);
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        const uint64_t m = __builtin_amdgcn_ballot_w64(valid && ((b >> k) & 1));
        eq &= ((b >> k) & 1) ? m : ~m;
    }
    return eq;
}

__device__ __forceinline__ uint64_t lanes_below(int lane) { return lane == 0 ? 0ull : (~0ull >> (64 - lane)); }

// Rank of this lane's item among the items of its bin so far (`h`: the
// wavefront's counters, which take this round's items up).
__device__ __forceinline__ int bin_rank(bool valid, int b, uint32_t* h, int lane) {
    const uint64_t eq = same_bin(valid, b);
    const uint64_t below = eq & lanes_below(lane);
    const uint32_t base = valid ? h[b] : 0u;
    wave_order();
    if (valid && below == 0ull) h[b] = base + (uint32_t)__popcll(eq);
    wave_order();
    return (int)base + __popcll(below);
}

// Chunk k of n over C channels: its first channel and their number (at most
// one more in the first chunks than in the others).
__device__ __forceinline__ int chunk_first(int C, int n, int k) { return k * (C / n) + min(k, C % n); }
__device__ __forceinline__ int chunk_size(int C, int n, int k) { return C / n + (k < C % n ? 1 : 0); }

// Exclusive prefix sum over the lanes of a wavefront.
__device__ __forceinline__ int wave_exclusive(int v, int lane) {
    int incl = v;
#pragma unroll
    for (int o = 1; o < MGS_WAVE; o <<= 1) {
        const int y = __shfl_up(incl, o, MGS_WAVE);
        if (lane >= o) incl += y;
    }
    return incl - v;
}

// Boundaries of each step per block of RH_SPAN leaves (boundary i belongs to
// the block of leaf i), and whether codes do not increase or do not lie below
// 2^(3 depth) (the scan raises the status flag, which needs no clearing then).
__global__ __launch_bounds__(RH_THREADS) void raht_count_kernel(RahtArgs a) {
    __shared__ uint32_t h[RH_WAVES][RH_STEPS], flag[RH_WAVES];
    const int lane = threadIdx.x & (MGS_WAVE - 1), wave = threadIdx.x / MGS_WAVE;
    h[wave][lane] = 0u;
    wave_order();
    const int64_t i0 = (int64_t)blockIdx.x * RH_SPAN + wave * RH_TILE + lane;
    uint64_t c0[RH_ROUNDS], c1[RH_ROUNDS];
#pragma unroll
    for (int e = 0; e < RH_ROUNDS; ++e) {
        const int64_t i = i0 + e * MGS_WAVE;
        c0[e] = a.codes[min(i, a.N - 1)];
        c1[e] = a.codes[min(i + 1, a.N - 1)];
    }
    const int bits = 3 * a.depth;
    bool bad = false;
#pragma unroll
    for (int e = 0; e < RH_ROUNDS; ++e) {
        const int64_t i = i0 + e * MGS_WAVE;
        const bool valid = i < a.N - 1;
        bad |= (i < a.N && (c0[e] >> bits) != 0) || (valid && c1[e] <= c0[e]);
        bin_rank(valid, merge_step(c0[e], c1[e], bits), h[wave], lane);
    }
    const bool any = __builtin_amdgcn_ballot_w64(bad) != 0ull;
    if (lane == 0) flag[wave] = any;
    __syncthreads();
    if (threadIdx.x == RH_STEPS) {
        uint32_t f = 0;
        for (int w = 0; w < RH_WAVES; ++w) f |= flag[w];
        a.bad[blockIdx.x] = f;
    }
    if (threadIdx.x < RH_STEPS) {
        uint32_t n = 0;
        for (int w = 0; w < RH_WAVES; ++w) n += h[w][threadIdx.x];
        a.cnt[(int64_t)threadIdx.x * a.nblk + blockIdx.x] = (int32_t)n;
    }
}

// One block per step: exclusive prefix of its counts over the blocks, in place,
// and its total (the leaf level adds the totals of the earlier steps).  The first
// one sets the status word.
constexpr int RH_SCAN_THREADS = 1024;
__global__ __launch_bounds__(RH_SCAN_THREADS) void raht_scan_kernel(RahtArgs a) {
    constexpr int PER = (RH_MAX_BLOCKS + RH_SCAN_THREADS - 1) / RH_SCAN_THREADS;
    constexpr int NW = RH_SCAN_THREADS / MGS_WAVE;
    __shared__ int wsum[NW];
    const int lane = threadIdx.x & (MGS_WAVE - 1), wave = threadIdx.x / MGS_WAVE;
    int32_t* c = a.cnt + (int64_t)blockIdx.x * a.nblk;
    const int per = (a.nblk + RH_SCAN_THREADS - 1) / RH_SCAN_THREADS;  // consecutive blocks per thread (<= PER)
    const int j0 = threadIdx.x * per;
    int v[PER], sum = 0;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        v[e] = e < per && j0 + e < a.nblk ? c[j0 + e] : 0;
        sum += v[e];
    }
    int run = wave_exclusive(sum, lane);
    if (lane == MGS_WAVE - 1) wsum[wave] = run + sum;
    __syncthreads();
    int total = 0;
    for (int w = 0; w < NW; ++w) {
        if (w < wave) run += wsum[w];
        total += wsum[w];
    }
#pragma unroll
    for (int e = 0; e < PER; ++e)
        if (e < per && j0 + e < a.nblk) {
            c[j0 + e] = run;
            run += v[e];
        }
    if (threadIdx.x == 0) a.tot[blockIdx.x] = total;
    if (blockIdx.x == 0) {
        int any = 0;
        for (int j = threadIdx.x; j < a.nblk; j += RH_SCAN_THREADS) any |= (int)a.bad[j];
        any = __syncthreads_or(any);
        if (threadIdx.x == 0) a.status->nonfinite = any ? 4u : 0u;
    }
}

// What a merge needs: the roots of both weights, and 1 / sqrt(w1 + w2) as the
// sum of yh (rounded toward zero, so that yl >= 0) and yl.
struct RahtWeights {
    double s1, s2, yh, yl;
};
__device__ __forceinline__ double2 reciprocal(double s) {
    double yh = 1.0 / s;
    double r = __builtin_fma(-s, yh, 1.0);  // exact
    if (r < 0.0) {
        yh = __longlong_as_double(__double_as_longlong(yh) - 1);
        r = __builtin_fma(-s, yh, 1.0);
    }
    return make_double2(yh, r / s);
}

// n1 / s and n2 / s, s = sqrt(w1 + w2).  n yh + n yl is within 2^-104 of the
// quotient before its one rounding: the division's result but where the quotient
// lies that close to the middle of two doubles, and then one of the two next to it
// (of the weights up to 256, 23 have such numerators, one or two in 2^52 each), in
// two operations instead of its dozen, zeros with their sign included
// (both terms have n's).  Infinities, whose products with a yl of 0 are none,
// and what they could come from take the division (the roots give the weights).
// With two corrections by the FMA remainder (Markstein) in place of yl, five
// operations per quotient, the leaf level at 5.3e6 x 20 took 426 us, now 381.
__device__ __forceinline__ void quotients(double n1, double n2, const RahtWeights& w, double& q1, double& q2) {
    q1 = __builtin_fma(n1, w.yh, n1 * w.yl);
    q2 = __builtin_fma(n2, w.yh, n2 * w.yl);
    const bool odd = !(fmax(fabs(n1), fabs(n2)) < 0x1p900);
    if (__builtin_amdgcn_ballot_w64(odd)) {  // (rare; the empty asm keeps it a branch)
        asm volatile("" : "+v"(n1), "+v"(n2));
        if (odd) {
            const double s = sqrt(__builtin_rint(w.s1 * w.s1) + __builtin_rint(w.s2 * w.s2));
            q1 = n1 / s;
            q2 = n2 / s;
        }
    }
}

// The steps of one wavefront on its channels, as rounds of up to 64 (merge,
// channel) pairs, channel fastest; a step of more merges takes several.  A
// round waits for its values alone: its weights were read a round ahead, its
// nodes two, and what addresses them is made at the end of the round before.
// Lanes without a pair repeat the round's last merge and write nothing.  Lane b
// of mstart and msize: first merge of step b, number of them.  nodes(q): the
// merge's packed nodes; where(q, nodes): the place of its weights, weights(place)
// reads them; slots(nodes, channel, first, second): the places of its values.
typedef __attribute__((address_space(3))) double lds_double;
template <int MODE, class N, class P, class W, class S>
__device__ __forceinline__ void run_steps(uint64_t todo, int mstart, int msize, int nch, int lane, double* val, N nodes,
                                          P where, W weights, S slots) {
    if (!todo) return;
    const int per = MGS_WAVE / nch;  // merges of a round
    const int q0 = lane / nch, cc = lane - q0 * nch;
    struct Round {
        int m0, m;  // first merge, merges left of its step (past the last round: 1, 0)
    };
    auto next = [&](Round r) {
        r.m0 += per;
        r.m -= per;
        if (r.m <= 0) {
            r = Round{1, 0};
            if (todo) {
                const int b = MODE == RH_FORWARD ? __builtin_ctzll(todo) : 63 - __builtin_clzll(todo);
                todo &= ~(1ull << b);
                r.m0 = __builtin_amdgcn_readlane(mstart, b);
                r.m = __builtin_amdgcn_readlane(msize, b);
            }
        }
        return r;
    };
    auto merge_of = [&](Round r) { return r.m0 + min(q0, r.m - 1); };
    Round ra = next(Round{0, 0}), rb = next(ra);
    uint32_t nb = nodes(merge_of(ra));
    lds_double* const v = (lds_double*)val;
    lds_double *pa, *pb;
    // (the empty asm keeps the addresses from being made again where they are used)
    auto slots_of = [&](uint32_t n) {
        int ia, ib;
        slots(n, cc, ia, ib);
        pa = v + ia;
        pb = v + ib;
        asm volatile("" : "+v"(pa), "+v"(pb));
    };
    slots_of(nb);
    RahtWeights wa = weights(where(merge_of(ra), nb)), wb{};
    nb = nodes(merge_of(rb));
    uint2 at = where(merge_of(rb), nb);
    auto round = [&](const RahtWeights& now, RahtWeights& then) {
        lds_double *const va = pa, *const vb = pb;
        const double x1 = *va, x2 = *vb;
        then = weights(at);
        const Round rc = next(rb);
        const uint32_t nc = nodes(merge_of(rc));
        double lo, hi;
        if (MODE == RH_FORWARD)
            quotients(now.s1 * x1 + now.s2 * x2, now.s1 * x2 - now.s2 * x1, now, lo, hi);
        else
            quotients(now.s1 * x1 - now.s2 * x2, now.s2 * x1 + now.s1 * x2, now, lo, hi);
        const bool mine = q0 < min(ra.m, per);
        ra = rb;
        rb = rc;
        slots_of(nb);
        at = where(merge_of(rc), nc);  // (before the stores, which it would wait for)
        asm volatile("" : "+v"(at.x), "+v"(at.y));
        nb = nc;
        if (mine) {
            *va = lo;
            *vb = hi;
        }
        wave_order();
    };
    for (;;) {
        round(wa, wb);
        if (ra.m <= 0) break;
        round(wb, wa);
        if (ra.m <= 0) break;
    }
}

// Blocks go round-robin over the XCDs: each XCD takes a contiguous run of
// them, so that neighbouring blocks, which share the cache lines at the ends of
// their runs of coefficients, share an L2.
constexpr int RH_XCDS = 8;
__device__ __forceinline__ int64_t xcd_block(int64_t nblk) {
    const int64_t per = (nblk + RH_XCDS - 1) / RH_XCDS;
    const int64_t b = (int64_t)(blockIdx.x % RH_XCDS) * per + blockIdx.x / RH_XCDS;
    return blockIdx.x / RH_XCDS < per && b < nblk ? b : -1;
}
unsigned xcd_grid(int64_t nblk) { return (unsigned)((nblk + RH_XCDS - 1) / RH_XCDS * RH_XCDS); }

// Leaf level: one wavefront per tile of RH_TILE leaves.  16 wavefronts per CU
// (LDS and registers allow no more): what only the structure needs (the tile's
// codes, counters, AC indices) lies in the LDS that holds the values later.
template <int MODE>
__global__ __launch_bounds__(RH_THREADS) __attribute__((amdgpu_waves_per_eu(4)))
void raht_leaf_kernel(RahtArgs a) {
    __shared__ struct {
        double2 inv[RH_TILE];  // 1 / sqrt(w) as a sum and sqrt(w), at w - 1 (first: their offsets fit the loads')
        double sq[RH_TILE];
        // the tile's merges in step order: first node's slot, second node's, and
        // their weights less one, a byte each
        uint32_t pk[RH_WAVES][RH_TILE];
        int32_t base[RH_STEPS];  // first AC index of each step in this block
        double val[RH_WAVES][RH_CH * RH_VS];
    } lds;
    auto& sq = lds.sq;
    auto& inv = lds.inv;
    auto& pk = lds.pk;
    auto& base = lds.base;
    auto& val = lds.val;
    const int tid = threadIdx.x;
    const int lane = tid & (MGS_WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / MGS_WAVE);
    uint64_t* cd = (uint64_t*)val[wave];                               // [RH_TILE]
    uint32_t* mcnt = (uint32_t*)(cd + RH_TILE);                        // [RH_STEPS]
    int32_t* ac = (int32_t*)(mcnt + RH_STEPS);                         // [RH_TILE]
    auto hist = [&](int w) { return (uint32_t*)(val[w] + 2 * RH_TILE); };  // [RH_STEPS]
    static_assert(RH_CH * RH_VS >= 2 * RH_TILE + RH_STEPS / 2 && RH_TILE % 64 == 0, "scratch beside the values");
    const int64_t blk = xcd_block(a.nblk);
    if (blk < 0) return;
    const int64_t tile = blk * RH_WAVES + wave;
    const int64_t s = tile * RH_TILE;
    const int n = (int)max((int64_t)0, min((int64_t)RH_TILE, a.N - s));
    const int bits = 3 * a.depth;
    if (MODE != RH_STRUCTURE)
        for (int k = tid; k < RH_TILE; k += RH_THREADS) {
            sq[k] = sqrt((double)(k + 1));
            inv[k] = reciprocal(sq[k]);
        }
    hist(wave)[lane] = 0u;
    mcnt[lane] = 0u;
    uint64_t c[RH_ROUNDS];
#pragma unroll
    for (int e = 0; e < RH_ROUNDS; ++e) c[e] = a.codes[min(s + e * MGS_WAVE + lane, a.N - 1)];
    // forward: the attributes of a chunk of channels, loaded while the tile's
    // structure is made or the chunk before is transformed (channels past the
    // chunk and leaves past the tile repeat the last one)
    const int nchunk = (a.C + RH_CH - 1) / RH_CH;
    float x[RH_CH][RH_ROUNDS];
    auto load_chunk = [&](int k) {
        const int k0 = chunk_first(a.C, nchunk, k), nch = chunk_size(a.C, nchunk, k);
#pragma unroll
        for (int cc = 0; cc < RH_CH; ++cc)
#pragma unroll
            for (int e = 0; e < RH_ROUNDS; ++e)
                x[cc][e] = a.attr[(int64_t)(k0 + min(cc, nch - 1)) * a.ld_in + min(s + e * MGS_WAVE + lane, a.N - 1)];
    };
    if (MODE == RH_FORWARD) load_chunk(0);
    const uint64_t before = a.codes[max(min(s, a.N) - 1, (int64_t)0)];
    const uint64_t after = a.codes[min(s + n, a.N - 1)];
    if (wave == 0) {
        const int t = a.tot[lane];
        base[lane] = wave_exclusive(t, lane) + a.cnt[(int64_t)lane * a.nblk + blk];
    }
#pragma unroll
    for (int e = 0; e < RH_ROUNDS; ++e) cd[e * MGS_WAVE + lane] = c[e];
    wave_order();
    // ---- steps and ranks of the tile's boundaries (the last one leads out of it)
    int d[RH_ROUNDS], rank[RH_ROUNDS];
#pragma unroll
    for (int e = 0; e < RH_ROUNDS; ++e) {
        const int j = e * MGS_WAVE + lane;
        const uint64_t nx = j + 1 < n ? cd[j + 1] : after;
        const bool valid = j + 1 < n || (j + 1 == n && s + n < a.N);
        d[e] = valid ? merge_step(c[e], nx, bits) : RH_STEPS - 1;
        rank[e] = bin_rank(valid, d[e], hist(wave), lane);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < RH_ROUNDS; ++e) {
        int r = base[d[e]] + rank[e];
        for (int w = 0; w < wave; ++w) r += (int)hist(w)[d[e]];
        ac[e * MGS_WAVE + lane] = r;
    }
    __syncthreads();  // every wavefront has read the others' counters
    // ---- the run each boundary's merge joins, by binary search in the tile's
    // codes, and whether it lies inside the tile
    uint32_t run[RH_ROUNDS];
    uint64_t merged[RH_ROUNDS];
    int mrank[RH_ROUNDS];
#pragma unroll
    for (int e = 0; e < RH_ROUNDS; ++e) {
        const int j = e * MGS_WAVE + lane;
        const int sh = d[e] + 1;  // <= 63 for a step that merges
        const uint64_t lo = d[e] < RH_STEPS - 1 ? (c[e] >> sh) << sh : 0ull;
        const uint64_t hi = d[e] < RH_STEPS - 1 ? lo + (1ull << sh) : 0ull;
        int L = min(j, RH_TILE - 1), R = min(j + 1, RH_TILE - 1);
#pragma unroll
        for (int o = RH_TILE / 2; o >= 1; o >>= 1) {
            const int pl = max(L - o, 0), pr = min(R + o, RH_TILE - 1);
            const uint64_t cl = cd[pl], cr = cd[pr];
            if (L - o >= 0 && cl >= lo) L = pl;
            if (R + o < n && cr < hi) R = pr;
        }
        const bool left = L > 0 || s == 0 || before < lo;
        const bool right = R < n - 1 || s + n >= a.N || after >= hi;
        const bool m = j + 1 < n && d[e] < RH_STEPS - 1 && left && right;
        run[e] = (uint32_t)(L & 255) | ((uint32_t)((j + 1) & 255) << 8) | ((uint32_t)((j - L) & 255) << 16) |
                 ((uint32_t)((R - j - 1) & 255) << 24);
        merged[e] = __builtin_amdgcn_ballot_w64(m);
        mrank[e] = bin_rank(m, d[e], mcnt, lane);
    }
    const int msize = (int)mcnt[lane];                    // lane b: merges of step b
    const int mstart = wave_exclusive(msize, lane);
    const uint64_t steps = __builtin_amdgcn_ballot_w64(msize > 0);
    wave_order();
    mcnt[lane] = (uint32_t)mstart;
    wave_order();
#pragma unroll
    for (int e = 0; e < RH_ROUNDS; ++e)
        if ((merged[e] >> lane) & 1ull) pk[wave][mcnt[d[e]] + mrank[e]] = run[e];
    int nm = 0;
#pragma unroll
    for (int e = 0; e < RH_ROUNDS; ++e) nm += __popcll(merged[e]);
    // ---- the nodes that are left: leaf j starts one unless boundary j - 1
    // merged; lane t keeps the first leaf of nodes t and t + 64
    int live = 0;
    int32_t node0 = 0, node1 = 0;
    {
        // (the counters' place is free now: a list of the first leaves)
        uint8_t* leaf_of = (uint8_t*)hist(wave);
        static_assert(RH_TILE <= 4 * RH_STEPS, "one byte per leaf in the counters' place");
        uint64_t carry = 0;
        wave_order();
#pragma unroll
        for (int e = 0; e < RH_ROUNDS; ++e) {
            const int j = e * MGS_WAVE + lane;
            const uint64_t sm = ~((merged[e] << 1) | carry) & __builtin_amdgcn_ballot_w64(j < n);
            carry = merged[e] >> 63;
            const int at = live + __popcll(sm & lanes_below(lane));
            const bool starts = (sm >> lane) & 1ull;
            if (starts) leaf_of[at] = (uint8_t)j;
            if (MODE != RH_INVERSE && tile < a.lev[0].lists) {
                const int64_t o = tile * a.stride;
                if (starts && at < a.stride) {
                    a.lev[0].first[o + at] = (int32_t)(s + j);
                    a.lev[0].code[o + at] = c[e];
                }
                // the node that ends at this boundary
                const int upto = at + (int)starts - 1;
                if (j < n && !((merged[e] >> lane) & 1ull) && upto >= 0 && upto < a.stride)
                    a.lev[0].ac[o + upto] = ac[j];
            }
            live += __popcll(sm);
        }
        wave_order();
        live = min(live, a.stride);  // (<= 128)
        if (lane < live) node0 = leaf_of[lane];
        if (lane + MGS_WAVE < live) node1 = leaf_of[lane + MGS_WAVE];
        if (MODE != RH_INVERSE && lane == 0 && tile < a.lev[0].lists) a.lev[0].cnt[tile] = live;
    }
    if (MODE == RH_STRUCTURE || n == 0) return;
    // lane's merges in step order, RH_ROUNDS of them: the second node's slot
    // (0: none) and the coefficient's column
    int second[RH_ROUNDS];
    int32_t column[RH_ROUNDS];
#pragma unroll
    for (int e = 0; e < RH_ROUNDS; ++e) {
        const int q = e * MGS_WAVE + lane;
        second[e] = q < nm ? (int)((pk[wave][q] >> 8) & 255u) : 0;
        column[e] = q < nm ? 1 + ac[second[e] - 1] : 0;
    }
    // ---- values, RH_CH channels at a time; the rows of the nodes that are left
    // by lanes over (node, channel), whole lines at a time
    double* v = val[wave];
    constexpr int ROWS = MGS_WAVE / RH_CH;
    const int node_of = lane / RH_CH, ch_of = lane % RH_CH;
    auto first_leaf = [&](int node) {  // of every lane's node
        const int j0 = __shfl(node0, node & (MGS_WAVE - 1)), j1 = __shfl(node1, node & (MGS_WAVE - 1));
        return node < MGS_WAVE ? j0 : j1;
    };
    for (int k = 0; k < nchunk; ++k) {
        const int k0 = chunk_first(a.C, nchunk, k), nch = chunk_size(a.C, nchunk, k);
        wave_order();
        if (MODE == RH_FORWARD) {
#pragma unroll
            for (int cc = 0; cc < RH_CH; ++cc)
#pragma unroll
                for (int e = 0; e < RH_ROUNDS; ++e) v[cc * RH_VS + e * MGS_WAVE + lane] = (double)x[cc][e];
            if (k + 1 < nchunk) load_chunk(k + 1);
        } else {
            // each merge's coefficient in the slot of its second node, the
            // nodes' values in theirs (all loads issued before the first is used)
            float hx[RH_CH][RH_ROUNDS];
#pragma unroll
            for (int cc = 0; cc < RH_CH; ++cc) {
                const int ch = k0 + min(cc, nch - 1);
#pragma unroll
                for (int e = 0; e < RH_ROUNDS; ++e) hx[cc][e] = a.coef_in[(int64_t)ch * a.ld_in + column[e]];
            }
            auto row = [&](int t) {
                const int node = min(t + node_of, live - 1), ch = k0 + min(ch_of, nch - 1);
                return a.top == 0 ? (double)a.coef_in[(int64_t)ch * a.ld_in]
                                  : a.lev[0].rows[(tile * a.stride + node) * a.C + ch];
            };
            auto put = [&](int t, double r) {
                const int j = first_leaf(t + node_of);
                if (t + node_of < live) v[ch_of * RH_VS + j] = r;
            };
            const double r0 = row(0);
#pragma unroll
            for (int cc = 0; cc < RH_CH; ++cc)
#pragma unroll
                for (int e = 0; e < RH_ROUNDS; ++e)
                    if (second[e]) v[cc * RH_VS + second[e]] = (double)hx[cc][e];
            put(0, r0);
            for (int t = ROWS; t < live; t += ROWS) put(t, row(t));
        }
        wave_order();
        auto nodes = [&](int q) { return pk[wave][q]; };
        // byte offsets of sqrt(w1) and sqrt(w2); their sum leads to one below w1 + w2
        auto where = [&](int, uint32_t w) { return make_uint2((w >> 13) & (255u << 3), (w >> 21) & (255u << 3)); };
        auto weights = [&](uint2 o) {
            auto at = [](const double* t, uint32_t bytes) { return *(const double*)((const char*)t + bytes); };
            const double2 y = *(const double2*)((const char*)(inv + 1) + 2 * (o.x + o.y));
            return RahtWeights{at(sq, o.x), at(sq, o.y), y.x, y.y};
        };
        auto slots = [&](uint32_t w, int cc, int& ia, int& ib) {
            ia = cc * RH_VS + (int)(w & 255u);
            ib = cc * RH_VS + (int)((w >> 8) & 255u);
        };
        run_steps<MODE>(steps, mstart, msize, nch, lane, v, nodes, where, weights, slots);
        if (MODE == RH_FORWARD) {
            // the next chunk's attributes have had the steps' time to arrive:
            // waited for here, they are not waited for behind the stores below
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
            // coefficients in step order: runs of consecutive AC indices per channel
#pragma unroll
            for (int e = 0; e < RH_ROUNDS; ++e)
                if (second[e]) {
#pragma unroll
                    for (int cc = 0; cc < RH_CH; ++cc)
                        if (cc < nch)
                            a.coef[(int64_t)(k0 + cc) * a.ld + column[e]] = (float)v[cc * RH_VS + second[e]];
                }
            for (int t = 0; t < live; t += ROWS) {
                const int node = t + node_of, j = first_leaf(node);
                if (node < live && ch_of < nch) {
                    const double r = v[ch_of * RH_VS + j];
                    if (a.top == 0) a.coef[(int64_t)(k0 + ch_of) * a.ld] = (float)r;  // the root: DC
                    else a.lev[0].rows[(tile * a.stride + node) * a.C + k0 + ch_of] = r;
                }
            }
        } else {
#pragma unroll
            for (int e = 0; e < RH_ROUNDS; ++e) {
                const int j = e * MGS_WAVE + lane;
                if (j < n)
#pragma unroll
                    for (int cc = 0; cc < RH_CH; ++cc)
                        if (cc < nch) a.attr_out[(int64_t)(k0 + cc) * a.ld + s + j] = (float)v[cc * RH_VS + j];
            }
        }
    }
}

// One group of an upper level: the nodes of RH_GROUP lists of the level below,
// as above but with nodes in place of leaves.  Up to CAP nodes lie in LDS: the
// block's threads take a node each for the structure and for the weights of its
// merge, then every wavefront does all steps on RH_UCH channels of its own.
// More nodes (BIG: codes whose trees are combs) lie in the workspace, with the
// values worked on in place, in the rows of the level below.
struct UpperArrays {
    uint64_t* code;
    int32_t *first, *ac, *row, *left, *right, *order;  // first has one entry more
    int32_t* rank;  // boundary j: (step, rank in it) of its merge, or -1 - slot of the node that starts after it
};
constexpr int RH_BIG_ARRAYS = 7;

template <int MODE, bool BIG, int CAP>
__device__ __forceinline__ void raht_group(const RahtArgs& a, int level, int64_t g, int n, const UpperArrays& u,
                                           int my_pre, uint32_t* h, double* wt, uint32_t* pk, double* v, int vwaves) {
    const RahtLevel& in = a.lev[level - 1];
    const RahtLevel& out = a.lev[level];
    const int tid = threadIdx.x, T = blockDim.x;
    const int lane = tid & (MGS_WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / MGS_WAVE);
    const int bits = 3 * a.depth;
    const bool root = level == a.top;
    constexpr int U = BIG ? 1 : CAP / RH_UPPER_MIN;  // nodes per thread (T >= RH_UPPER_MIN)
    // ---- the lists, one after the other: node j of the group is node
    // j - pre of the list whose prefix covers it
    const int64_t list0 = g * RH_GROUP;
    int64_t span = RH_TILE;  // leaves of a group of this level
    for (int l = 0; l < level; ++l) span *= RH_GROUP;
    const int64_t start = g * span, end = min(a.N, (g + 1) * span);
    const uint64_t before = a.codes[max(start - 1, (int64_t)0)], after = a.codes[min(end, a.N - 1)];
    {
        int pre[RH_GROUP];
#pragma unroll
        for (int t = 0; t < RH_GROUP; ++t) pre[t] = __builtin_amdgcn_readlane(my_pre, t);
        h[wave * RH_STEPS + lane] = 0u;
        for (int j0 = tid; j0 < n; j0 += U * T) {
            int at[U], fi[U], ai[U];
            uint64_t co[U];
#pragma unroll
            for (int e = 0; e < U; ++e) {
                const int j = min(j0 + e * T, n - 1);
                int t = 0, p = 0;
#pragma unroll
                for (int l = 1; l < RH_GROUP; ++l)
                    if (j >= pre[l]) {
                        t = l;
                        p = pre[l];
                    }
                at[e] = (int)((list0 + t) * a.stride) + j - p;
                fi[e] = in.first[at[e]];
                ai[e] = in.ac[at[e]];
                co[e] = in.code[at[e]];
            }
#pragma unroll
            for (int e = 0; e < U; ++e)
                if (j0 + e * T < n) {
                    u.first[j0 + e * T] = fi[e];
                    u.ac[j0 + e * T] = ai[e];
                    u.row[j0 + e * T] = at[e];
                    u.code[j0 + e * T] = co[e];
                }
        }
        if (tid == 0) u.first[n] = (int32_t)end;
    }
    __syncthreads();
    // ---- the wavefront's first channels (in flight during the search)
    const int nchunk = BIG ? 1 : (a.C + RH_UCH - 1) / RH_UCH;
    const int k_first = blockIdx.y * vwaves + wave, k_step = (int)gridDim.y * vwaves;
    double* vw = v + (size_t)wave * (RH_UCH * CAP);  // [node][channel]
    // the rows go by lanes over (node, channel), whole lines at a time
    constexpr int ROWS = MGS_WAVE / RH_UCH;
    const int node_of = lane / RH_UCH, ch_of = lane % RH_UCH;
    auto place = [&](int j, int k0, int nch) { return (int64_t)u.row[j] * a.C + k0 + min(ch_of, nch - 1); };
    // forward: the nodes' values; inverse: the coefficient of the boundary
    // before each node (the nodes that are left get their values over it)
    auto fetch = [&](int k) {
        const int k0 = chunk_first(a.C, nchunk, k), nch = chunk_size(a.C, nchunk, k);
        for (int j0 = 0; j0 < n; j0 += RH_TILE) {
            if (MODE == RH_FORWARD) {
                double r[RH_TILE / ROWS];
#pragma unroll
                for (int e = 0; e < RH_TILE / ROWS; ++e) r[e] = in.rows[place(min(j0 + e * ROWS + node_of, n - 1), k0, nch)];
#pragma unroll
                for (int e = 0; e < RH_TILE / ROWS; ++e) vw[(j0 + e * ROWS) * RH_UCH + lane] = r[e];
            } else {
                float r[RH_ROUNDS][RH_UCH];
#pragma unroll
                for (int e = 0; e < RH_ROUNDS; ++e) {
                    const int j = min(j0 + e * MGS_WAVE + lane, n - 1);
                    const int64_t p = min(1 + (int64_t)u.ac[max(j - 1, 0)], a.N - 1);
#pragma unroll
                    for (int cc = 0; cc < RH_UCH; ++cc)
                        r[e][cc] = a.coef_in[(int64_t)(k0 + min(cc, nch - 1)) * a.ld_in + p];
                }
#pragma unroll
                for (int e = 0; e < RH_ROUNDS; ++e)
#pragma unroll
                    for (int cc = 0; cc < RH_UCH; ++cc)
                        vw[(j0 + e * MGS_WAVE + lane) * RH_UCH + cc] = (double)r[e][cc];
            }
        }
    };
    if (MODE != RH_STRUCTURE && !BIG && wave < vwaves && k_first < nchunk) fetch(k_first);
    // ---- each boundary's run, and whether it lies inside the group
    int top = 1;
    while (2 * top < n) top *= 2;
    for (int j0 = tid; j0 < n; j0 += U * T) {
        int d[U], L[U], R[U];
        uint64_t lo[U], hi[U];
#pragma unroll
        for (int e = 0; e < U; ++e) {
            const int j = min(j0 + e * T, n - 1);
            const uint64_t c0 = u.code[j];
            d[e] = j0 + e * T + 1 < n ? merge_step(c0, u.code[min(j + 1, n - 1)], bits) : RH_STEPS - 1;
            const int sh = d[e] + 1;  // <= 63 for a step that merges
            lo[e] = d[e] < RH_STEPS - 1 ? (c0 >> sh) << sh : 0ull;
            hi[e] = d[e] < RH_STEPS - 1 ? lo[e] + (1ull << sh) : 0ull;
            L[e] = j;
            R[e] = min(j + 1, n - 1);
        }
        for (int o = top; o >= 1; o >>= 1)
#pragma unroll
            for (int e = 0; e < U; ++e) {
                const int pl = max(L[e] - o, 0), pr = min(R[e] + o, n - 1);
                const uint64_t cl = u.code[pl], cr = u.code[pr];
                if (L[e] - o >= 0 && cl >= lo[e]) L[e] = pl;
                if (R[e] + o < n && cr < hi[e]) R[e] = pr;
            }
#pragma unroll
        for (int e = 0; e < U; ++e) {
            const int j = j0 + e * T;
            const bool m = d[e] < RH_STEPS - 1 && (L[e] > 0 || start == 0 || before < lo[e]) &&
                           (R[e] < n - 1 || end >= a.N || after >= hi[e]);
            if (j < n) {
                u.left[j] = L[e];
                u.right[j] = R[e];
                u.rank[j] = m ? d[e] : -1;
            }
        }
    }
    __syncthreads();
    // ---- ranks of the merges in their steps, and the nodes that are left: a
    // node starts at 0 and after every boundary that does not merge here.  Each
    // wavefront counts a piece of the boundaries by itself, then adds what the
    // wavefronts before it counted.
    {
        const int nw = T / MGS_WAVE;
        const int piece = ((n + MGS_WAVE - 1) / MGS_WAVE + nw - 1) / nw * MGS_WAVE;
        const int p0 = wave * piece, p1 = min(n, p0 + piece);
        uint32_t* hw = h + wave * RH_STEPS;
        uint32_t* ended = h + RH_UPPER_WAVES * RH_STEPS;
        int live = 0;
        for (int j0 = p0; j0 < p1; j0 += MGS_WAVE) {
            const int j = j0 + lane;
            const int d = j < p1 ? u.rank[j] : -1;
            const uint64_t ends = __builtin_amdgcn_ballot_w64(j < p1 && d < 0);
            const int r = bin_rank(d >= 0, max(d, 0), hw, lane);
            const int slot = live + __popcll(ends & lanes_below(lane));  // of the node that ends at boundary j
            if (j < p1) u.rank[j] = d >= 0 ? (d << 16) | r : -2 - slot;
            live += __popcll(ends);
        }
        if (lane == 0) ended[wave] = (uint32_t)live;
        __syncthreads();
        int before_bin = 0, before_ends = 0, all_ends = 0;  // lane b: merges of step b before the piece
        for (int w = 0; w < nw; ++w) {
            if (w < wave) {
                before_bin += (int)h[w * RH_STEPS + lane];
                before_ends += (int)ended[w];
            }
            all_ends += (int)ended[w];
        }
        const int64_t o = g * a.stride;
        for (int j0 = p0; j0 < p1; j0 += MGS_WAVE) {
            const int j = j0 + lane;
            const int r = j < p1 ? u.rank[j] : -1;
            const int more = __shfl(before_bin, max(r, 0) >> 16);
            if (j < p1) {
                u.rank[j] = r >= 0 ? r + more : r - before_ends;
                const int slot = -2 - r + before_ends;
                if (MODE != RH_INVERSE && r < 0) {
                    if (slot < a.stride) out.ac[o + slot] = u.ac[j];
                    if (slot + 1 < a.stride && j + 1 < n) {
                        out.first[o + slot + 1] = u.first[j + 1];
                        out.code[o + slot + 1] = u.code[j + 1];
                    }
                }
            }
        }
        if (MODE != RH_INVERSE && tid == 0) {
            out.first[o] = (int32_t)start;
            out.code[o] = u.code[0];
            out.cnt[g] = min(all_ends, a.stride);
        }
    }
    if (MODE == RH_STRUCTURE) return;
    __syncthreads();
    int msize = 0;
    for (int w = 0; w < T / MGS_WAVE; ++w) msize += (int)h[w * RH_STEPS + lane];  // lane b: merges of step b
    const int mstart = wave_exclusive(msize, lane);
    const uint64_t steps = __builtin_amdgcn_ballot_w64(msize > 0);
    const int nm = __builtin_amdgcn_readlane(mstart + msize, MGS_WAVE - 1);
    // slot of the node that starts at j, or -1 where none does
    auto slot_of = [&](int j) {
        const int r = j > 0 ? u.rank[j - 1] : -1;
        return r < 0 ? -1 - r : -1;
    };
    if constexpr (!BIG) {
        // ---- the merges in step order, with their weights (in the place of the
        // codes and runs, which are read before the first is written)
        double w1[U], w2[U];
        int to[U];
        uint32_t nodes[U];
#pragma unroll
        for (int e = 0; e < U; ++e) {
            const int j = tid + e * T;
            const int r = j < n ? u.rank[j] : -1;
            const int m0 = __shfl(mstart, max(r, 0) >> 16);
            to[e] = r >= 0 ? m0 + (r & 0xFFFF) : -1;
            w1[e] = w2[e] = 1.0;
            nodes[e] = 0;
            if (r >= 0) {
                const int L = u.left[j], f = u.first[j + 1];
                w1[e] = (double)(f - u.first[L]);
                w2[e] = (double)(u.first[u.right[j] + 1] - f);
                nodes[e] = (uint32_t)L | (uint32_t)(j + 1) << 16;
            }
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < U; ++e)
            if (to[e] >= 0) {
                double* w = wt + to[e] * 4;
                const double2 y = reciprocal(sqrt(w1[e] + w2[e]));
                w[0] = sqrt(w1[e]);
                w[1] = sqrt(w2[e]);
                w[2] = y.x;
                w[3] = y.y;
                pk[to[e]] = nodes[e];
            }
        __syncthreads();
        if (wave >= vwaves) return;
        for (int k = k_first; k < nchunk; k += k_step) {
            const int k0 = chunk_first(a.C, nchunk, k), nch = chunk_size(a.C, nchunk, k);
            if (k != k_first) {
                wave_order();
                fetch(k);
            }
            if (MODE == RH_INVERSE)
                for (int j0 = 0; j0 < n; j0 += RH_TILE) {
                    constexpr int E = RH_TILE / ROWS;
                    double r[E];
                    int slot[E];
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        const int j = j0 + e * ROWS + node_of, ch = k0 + min(ch_of, nch - 1);
                        slot[e] = j < n ? slot_of(j) : -1;
                        if (slot[e] >= a.stride) slot[e] = -1;
                        r[e] = 0.0;
                        if (slot[e] >= 0)
                            r[e] = root ? (double)a.coef_in[(int64_t)ch * a.ld_in]
                                        : out.rows[(g * a.stride + slot[e]) * a.C + ch];
                    }
#pragma unroll
                    for (int e = 0; e < E; ++e)
                        if (slot[e] >= 0) vw[(j0 + e * ROWS) * RH_UCH + lane] = r[e];
                }
            wave_order();
            auto nodes = [&](int q) { return pk[q]; };
            auto where = [&](int q, uint32_t) { return make_uint2((uint32_t)q * 4, 0u); };
            auto weights = [&](uint2 o) { return RahtWeights{wt[o.x], wt[o.x + 1], wt[o.x + 2], wt[o.x + 3]}; };
            auto slots = [&](uint32_t w, int cc, int& ia, int& ib) {
                ia = (int)(w & 0xFFFFu) * RH_UCH + cc;
                ib = (int)(w >> 16) * RH_UCH + cc;
            };
            run_steps<MODE>(steps, mstart, msize, nch, lane, vw, nodes, where, weights, slots);
            if (MODE == RH_FORWARD) {
                for (int j = node_of; j < n; j += ROWS) {
                    const int slot = slot_of(j);
                    if (slot < 0 || slot >= a.stride || ch_of >= nch) continue;
                    const double r = vw[j * RH_UCH + ch_of];
                    if (root) a.coef[(int64_t)(k0 + ch_of) * a.ld] = (float)r;  // DC
                    else out.rows[(g * a.stride + slot) * a.C + k0 + ch_of] = r;
                }
                for (int q = lane; q < nm; q += MGS_WAVE) {
                    const int j = (int)(pk[q] >> 16);
                    const int64_t p = 1 + (int64_t)u.ac[j - 1];
#pragma unroll
                    for (int cc = 0; cc < RH_UCH; ++cc)
                        if (cc < nch) a.coef[(int64_t)(k0 + cc) * a.ld + p] = (float)vw[j * RH_UCH + cc];
                }
            } else {
                for (int j = node_of; j < n; j += ROWS)
                    if (ch_of < nch) in.rows[place(j, k0, nch)] = vw[j * RH_UCH + ch_of];
            }
        }
    } else {
        // ---- values in place, in the rows of the level below
        for (int j0 = 0; j0 < n; j0 += T) {
            const int j = j0 + tid;
            const int r = j < n ? u.rank[j] : -1;
            const int m0 = __shfl(mstart, max(r, 0) >> 16);
            if (r >= 0) u.order[m0 + (r & 0xFFFF)] = j;
        }
        __syncthreads();
        auto value = [&](int c, int j) -> double& { return in.rows[(int64_t)u.row[j] * a.C + c]; };
        if (MODE == RH_INVERSE) {
            for (int j = tid; j < n; j += T) {
                const int slot = slot_of(j);
                if (slot < 0 || slot >= a.stride) continue;
                for (int c = 0; c < a.C; ++c)
                    value(c, j) = root ? (double)a.coef_in[(int64_t)c * a.ld_in]
                                       : out.rows[(g * a.stride + slot) * a.C + c];
            }
            for (int q = tid; q < nm; q += T) {
                const int j = u.order[q];
                for (int c = 0; c < a.C; ++c) value(c, j + 1) = (double)a.coef_in[(int64_t)c * a.ld_in + 1 + u.ac[j]];
            }
        }
        __syncthreads();
        uint64_t todo = steps;
        while (todo) {
            const int b = MODE == RH_FORWARD ? __builtin_ctzll(todo) : 63 - __builtin_clzll(todo);
            todo &= ~(1ull << b);
            const int m0 = __builtin_amdgcn_readlane(mstart, b);
            const uint32_t pairs = (uint32_t)__builtin_amdgcn_readlane(msize, b) * (uint32_t)a.C;
            for (uint32_t p = tid; p < pairs; p += T) {
                const uint32_t q = p / (uint32_t)a.C;
                const int c = (int)(p - q * (uint32_t)a.C);
                const int j = u.order[m0 + (int)q];
                const int L = u.left[j];
                const double w1 = (double)(u.first[j + 1] - u.first[L]);
                const double w2 = (double)(u.first[u.right[j] + 1] - u.first[j + 1]);
                const double s1 = sqrt(w1), s2 = sqrt(w2), sw = sqrt(w1 + w2);
                double &va = value(c, L), &vb = value(c, j + 1);
                const double x1 = va, x2 = vb;
                if (MODE == RH_FORWARD) {
                    va = (s1 * x1 + s2 * x2) / sw;
                    vb = (s1 * x2 - s2 * x1) / sw;
                } else {
                    va = (s1 * x1 - s2 * x2) / sw;
                    vb = (s2 * x1 + s1 * x2) / sw;
                }
            }
            __syncthreads();
        }
        if (MODE == RH_FORWARD) {
            for (int j = tid; j < n; j += T) {
                const int slot = slot_of(j);
                if (slot < 0 || slot >= a.stride) continue;
                for (int c = 0; c < a.C; ++c) {
                    if (root) a.coef[(int64_t)c * a.ld] = (float)value(c, j);  // DC
                    else out.rows[(g * a.stride + slot) * a.C + c] = value(c, j);
                }
            }
            for (int q = tid; q < nm; q += T) {
                const int j = u.order[q];
                for (int c = 0; c < a.C; ++c) a.coef[(int64_t)c * a.ld + 1 + u.ac[j]] = (float)value(c, j + 1);
            }
        }
    }
}

// Upper levels: one block per group of RH_GROUP lists and `vwaves` chunks of
// RH_UCH channels (blockIdx.y takes the others and builds the structure again).
// What bounds a block is its chain: two dependent loads (2 + 2 us), the search
// (2), the ranks (1), the weights (1), then the steps (5), one LDS round trip and
// four dependent FP64 operations each.  With the weights (three dependent LDS
// reads, three square roots, two divisions) inside the steps, one wavefront per
// group and chunk, a level took 24 to 31 us and the first of 5.3e6 x 20, whose
// 1294 groups fill the chip several times, 89; now 18 to 23 and 66.
template <int MODE, int CAP>
__global__ __launch_bounds__(RH_UPPER_MAX) void raht_upper_kernel(RahtArgs a, int level, int vwaves) {
    static_assert(CAP % RH_UPPER_MIN == 0 && CAP % RH_TILE == 0, "nodes per thread, rounds of loads");
    extern __shared__ double up_lds[];
    const int64_t g = xcd_block(a.lev[level].lists);
    if (g < 0) return;
    const RahtLevel& in = a.lev[level - 1];
    const int64_t list0 = g * RH_GROUP;
    const int lane = threadIdx.x & (MGS_WAVE - 1);
    const int m = lane < RH_GROUP && list0 + lane < in.lists ? in.cnt[list0 + lane] : 0;
    const int my_pre = wave_exclusive(m, lane);  // lane t: nodes of the group before list t
    const int n = __builtin_amdgcn_readlane(my_pre + m, MGS_WAVE - 1);
    // values, then weights and node pairs of the merges (before them, in their
    // place, the codes, runs, first leaves and counters), then what stays
    double* v = up_lds;
    double* wt = v + (size_t)vwaves * (RH_UCH * CAP);
    uint32_t* pk = (uint32_t*)(wt + 4 * CAP);
    int32_t* keep = (int32_t*)(pk + CAP);
    uint64_t* code = (uint64_t*)wt;
    int32_t* tmp = (int32_t*)(code + CAP);
    uint32_t* h = (uint32_t*)(tmp + 3 * CAP + 1);
    static_assert(2 * CAP + 3 * CAP + 1 + RH_UPPER_WAVES * (RH_STEPS + 1) <= 9 * CAP, "what is replaced fits");
    if (n <= CAP) {
        const UpperArrays u{code, tmp + 2 * CAP, keep, keep + CAP, tmp, tmp + CAP, nullptr, keep + 2 * CAP};
        raht_group<MODE, false, CAP>(a, level, g, n, u, my_pre, h, wt, pk, v, vwaves);
    } else if (blockIdx.y == 0) {
        const int64_t o = list0 * a.stride + g;  // one entry more per group
        const int64_t st = a.big_stride;
        const UpperArrays u{a.big_code + o,       a.big_i + o,          a.big_i + st + o,     a.big_i + 2 * st + o,
                            a.big_i + 3 * st + o, a.big_i + 4 * st + o, a.big_i + 5 * st + o, a.big_i + 6 * st + o};
        raht_group<MODE, true, CAP>(a, level, g, n, u, my_pre, h, wt, pk, v, vwaves);
    }
}

struct RahtLayout {
    size_t cnt, tot, bad, big_code, big_i, input, total;
    size_t lcnt[RH_LEVELS], first[RH_LEVELS], code[RH_LEVELS], ac[RH_LEVELS], rows[RH_LEVELS];
    int64_t lists[RH_LEVELS], big_stride;
    int64_t nblk;
    int stride, top;
};

RahtLayout raht_layout(int64_t N, int32_t C, int32_t depth) {
    RahtLayout L;
    std::memset(&L, 0, sizeof(L));
    L.nblk = std::max<int64_t>(1, (N + RH_SPAN - 1) / RH_SPAN);
    // a contiguous run of leaves holds at most two maximal subtrees per step
    // (two nodes per lane at the leaf level)
    L.stride = std::min(2 * MGS_WAVE, 6 * depth + 2);
    size_t o = MGS_STATUS_BYTES;
    auto take = [&](size_t bytes) {
        size_t at = o;
        o += mgs_align_up(bytes, 256);
        return at;
    };
    L.cnt = take(sizeof(int32_t) * RH_STEPS * (size_t)L.nblk);
    L.tot = take(sizeof(int32_t) * RH_STEPS);
    L.bad = take(sizeof(uint32_t) * (size_t)L.nblk);
    int64_t lists = std::max<int64_t>(1, (N + RH_TILE - 1) / RH_TILE);
    L.big_stride = lists * L.stride + (lists + RH_GROUP - 1) / RH_GROUP + 1;
    for (int l = 0; l < RH_LEVELS; ++l) {
        L.lists[l] = lists;
        L.top = l;
        L.lcnt[l] = take(sizeof(int32_t) * (size_t)lists);
        L.first[l] = take(sizeof(int32_t) * (size_t)lists * L.stride);
        L.ac[l] = take(sizeof(int32_t) * (size_t)lists * L.stride);
        L.code[l] = take(sizeof(uint64_t) * (size_t)lists * L.stride);
        if (lists == 1) break;  // the root: its value is the DC coefficient
        L.rows[l] = take(sizeof(double) * (size_t)lists * L.stride * (size_t)C);
        lists = (lists + RH_GROUP - 1) / RH_GROUP;
    }
    L.big_code = take(sizeof(uint64_t) * (size_t)L.big_stride);
    L.big_i = take(sizeof(int32_t) * RH_BIG_ARRAYS * (size_t)L.big_stride);
    L.input = take(sizeof(float) * (size_t)N * (size_t)C);
    L.total = o;
    return L;
}

int raht_setup(RahtArgs& a, RahtLayout& L, const uint64_t* codes, int64_t N, int32_t C, int64_t ld,
               int32_t depth, void* d_ws, size_t ws_bytes) {
    if (N < 1 || N >= ((int64_t)1 << 31) || C < 1 || ld < N || depth < 1 || depth > 21 || !codes)
        return MGS_EINVAL;
    L = raht_layout(N, C, depth);
    if (N - 1 > (int64_t)RH_SPAN * RH_MAX_SPANS) return MGS_EINVAL;
    if (!d_ws || ws_bytes < L.total) return MGS_EWORKSPACE;
    char* ws = (char*)d_ws;
    std::memset(&a, 0, sizeof(a));
    a.codes = codes;
    a.N = N;
    a.C = C;
    a.depth = depth;
    a.ld = ld;
    a.cnt = (int32_t*)(ws + L.cnt);
    a.tot = (int32_t*)(ws + L.tot);
    a.bad = (uint32_t*)(ws + L.bad);
    a.big_code = (uint64_t*)(ws + L.big_code);
    a.big_i = (int32_t*)(ws + L.big_i);
    a.big_stride = L.big_stride;
    a.status = (mgs_status_block*)ws;
    a.nblk = (int32_t)L.nblk;
    a.stride = L.stride;
    a.top = L.top;
    for (int l = 0; l <= L.top; ++l) {
        a.lev[l].cnt = (int32_t*)(ws + L.lcnt[l]);
        a.lev[l].first = (int32_t*)(ws + L.first[l]);
        a.lev[l].ac = (int32_t*)(ws + L.ac[l]);
        a.lev[l].code = (uint64_t*)(ws + L.code[l]);
        a.lev[l].rows = (double*)(ws + L.rows[l]);
        a.lev[l].lists = (int32_t)L.lists[l];
    }
    return MGS_OK;
}

// A call in place (input and output overlap) works on a copy of its input: tiles
// write coefficients to columns that other tiles have yet to read.
__global__ void raht_copy_kernel(const float* __restrict__ src, int64_t ld, float* __restrict__ dst, int64_t N,
                                 int64_t total) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t c = i / N;
        dst[i] = src[c * ld + (i - c * N)];
    }
}
const float* raht_input(RahtArgs& a, const RahtLayout& L, const float* in, const float* out, void* d_ws,
                        hipStream_t s) {
    const uintptr_t i0 = (uintptr_t)in, o0 = (uintptr_t)out;
    const uintptr_t bytes = sizeof(float) * (uintptr_t)((a.C - 1) * a.ld + a.N);
    a.ld_in = a.ld;
    if (i0 >= o0 + bytes || o0 >= i0 + bytes) return in;
    float* copy = (float*)((char*)d_ws + L.input);
    const int64_t total = a.N * a.C;
    a.ld_in = a.N;
    hipLaunchKernelGGL(raht_copy_kernel, dim3((unsigned)std::min<int64_t>((total + 255) / 256, 16384)), dim3(256), 0, s,
                       in, a.ld, copy, a.N, total);
    return copy;
}

// The status word and the AC indices' counts.
int raht_counts(RahtArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(raht_count_kernel, dim3(a.nblk), dim3(RH_THREADS), 0, s, a);
    hipLaunchKernelGGL(raht_scan_kernel, dim3(RH_STEPS), dim3(RH_SCAN_THREADS), 0, s, a);
    return mgs_last_launch();
}

// Chunks of RH_UCH channels go to the wavefronts of a block, as many as its
// LDS holds (eight at the first upper level, four above it), the rest to
// blockIdx.y, evenly.  (The attribute belongs to the device's code object:
// repeating it is cheap and needs no state.)
template <int MODE, int CAP>
int raht_upper_launch(const RahtArgs& a, int level, int most, hipStream_t s) {
    const int chunks = MODE == RH_STRUCTURE ? 0 : (a.C + RH_UCH - 1) / RH_UCH;
    const int blocks = std::max(1, std::min(65535, (chunks + most - 1) / most));
    const int vwaves = std::min(most, (chunks + blocks - 1) / blocks);
    const int threads = std::max(RH_UPPER_MIN, vwaves * MGS_WAVE);
    const size_t lds = (size_t)CAP * (vwaves * RH_UCH * sizeof(double) + 48);
    int rc = mgs_hip_status(hipFuncSetAttribute((const void*)raht_upper_kernel<MODE, CAP>,
                                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    if (rc) return rc;
    hipLaunchKernelGGL((raht_upper_kernel<MODE, CAP>), dim3(xcd_grid(a.lev[level].lists), blocks), dim3(threads),
                       lds, s, a, level, vwaves);
    return mgs_last_launch();
}

template <int MODE>
int raht_upper(const RahtArgs& a, int level, hipStream_t s) {
    return level == 1 ? raht_upper_launch<MODE, RH_CAP1>(a, level, 8, s)
                      : raht_upper_launch<MODE, RH_CAP2>(a, level, 4, s);
}

}  // namespace
}  // namespace mgs

extern "C" size_t mgs_raht_ws_bytes(int64_t N, int32_t C, int32_t depth) {
    if (N < 1 || C < 1 || depth < 1 || depth > 21) return 0;
    return mgs::raht_layout(N, C, depth).total;
}

extern "C" int mgs_raht_forward(const uint64_t* d_codes, int64_t N, int32_t C, int32_t depth, const float* d_attr,
                                int64_t ld, float* d_coef, void* d_ws, size_t ws_bytes, void* stream) {
    using namespace mgs;
    RahtArgs a;
    RahtLayout L;
    int rc = raht_setup(a, L, d_codes, N, C, ld, depth, d_ws, ws_bytes);
    if (rc) return rc;
    if (!d_attr || !d_coef) return MGS_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    a.attr = raht_input(a, L, d_attr, d_coef, d_ws, s);
    a.coef = d_coef;
    rc = raht_counts(a, s);
    if (rc) return rc;
    hipLaunchKernelGGL(raht_leaf_kernel<RH_FORWARD>, dim3(xcd_grid(a.nblk)), dim3(RH_THREADS), 0, s, a);
    rc = mgs_last_launch();
    for (int l = 1; l <= a.top && !rc; ++l) rc = raht_upper<RH_FORWARD>(a, l, s);
    return rc;
}

extern "C" int mgs_raht_inverse(const uint64_t* d_codes, int64_t N, int32_t C, int32_t depth, const float* d_coef,
                                int64_t ld, float* d_attr, void* d_ws, size_t ws_bytes, void* stream) {
    using namespace mgs;
    RahtArgs a;
    RahtLayout L;
    int rc = raht_setup(a, L, d_codes, N, C, ld, depth, d_ws, ws_bytes);
    if (rc) return rc;
    if (!d_attr || !d_coef) return MGS_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    a.coef_in = raht_input(a, L, d_coef, d_attr, d_ws, s);
    a.attr_out = d_attr;
    rc = raht_counts(a, s);
    if (rc) return rc;
    // the lists of every level from the leaves up, then the values from the root down
    if (a.top > 0) hipLaunchKernelGGL(raht_leaf_kernel<RH_STRUCTURE>, dim3(xcd_grid(a.nblk)), dim3(RH_THREADS), 0, s, a);
    rc = mgs_last_launch();
    for (int l = 1; l < a.top && !rc; ++l) rc = raht_upper<RH_STRUCTURE>(a, l, s);
    for (int l = a.top; l >= 1 && !rc; --l) rc = raht_upper<RH_INVERSE>(a, l, s);
    if (rc) return rc;
    hipLaunchKernelGGL(raht_leaf_kernel<RH_INVERSE>, dim3(xcd_grid(a.nblk)), dim3(RH_THREADS), 0, s, a);
    return mgs_last_launch();
}
