// One iteration of mini-batch k-means around the nearest-codeword
// assignment.  Paper: section "Attribute Transformation", paragraph
// "Clustering 1+D SH Coefficients" -- the codebook of the higher-degree SH
// vectors is refined by a batched clustering strategy (Sculley's web-scale
// k-means) over several iterations.
//
// Per iteration, on a batch of sample rows chosen by the caller:
//   1. every batch row goes to its nearest center (the exact rule of
//      mgs_vq_assign: FP64 distance, ties to the smaller index);
//   2. center j, which has absorbed v_j samples so far and gets n_j > 0 rows
//      of this batch, moves to the running mean of all of them:
//        c_j <- (v_j c_j + sum of its batch rows) / (v_j + n_j),  v_j += n_j.
// Sculley's per-sample update (v += 1, eta = 1 / v, c <- (1 - eta) c + eta x,
// applied to the batch's rows in order) reaches the same mean.  The sum of a
// center's rows is taken in FP64 in batch order: the batch positions are
// grouped by center with a stable sort (a counting sort over tiles; for very
// many centers rocPRIM's radix sort), so each center's rows
// form one run in batch order, and one wave per center adds its run
// sequentially (lane d adds dimension d).  The result, rounded to FP32 once,
// is therefore the same on every run, bit for bit.
#include <cstring>

#include <rocprim/device/device_radix_sort.hpp>

#include "common.h"

namespace mgs {
namespace {

struct KmArgs {
    const float* x;
    const int64_t* batch;
    float* xb;          // [B][D] gathered batch rows
    int32_t* assign;    // [B]
    uint32_t* table;    // [T][K] rows of a tile per center, then their first place in pos_s
    uint2* run;         // [K] first place and length of a center's run in pos_s
    uint32_t* keys;     // [B] sort keys: the center, K for rows without one
    uint32_t* keys_s;   // [B] the keys sorted
    int32_t* pos;       // [B] batch positions 0 .. B-1
    int32_t* pos_s;     // [B] batch positions in center order (stable: batch order within a center)
    float* cb;          // [K][D] centers (in place)
    int64_t* counts;    // [K] samples absorbed so far
    mgs_status_block* status;
    uint32_t* cursor;   // rows of the runs placed so far (cleared with the status block)
    const mgs_status_block* vq;  // the assignment's status block
    int64_t N, B;
    int32_t D, K;
    int32_t tile, T;    // rows per tile (a multiple of 64), tiles
    int32_t bits;       // key bits
};

// Batch rows into a contiguous block; an index outside [0, N) raises the
// status flag and gathers zeros.  Bound by the rows' lines (random 64-byte
// pieces): a thread issues the loads of its KG_U indices, then of its KG_U
// values, in units of four floats where rows allow (V = float4).  The row of
// a unit is the block's first row plus a 32-bit quotient.
constexpr int KG_U = 4;
template <class V>
__global__ __launch_bounds__(256) void km_gather_kernel(KmArgs a) {
    const uint32_t W = (uint32_t)a.D / (sizeof(V) / sizeof(float));  // units per row
    const int64_t total = a.B * W;
    const V* x = (const V*)a.x;
    V* xb = (V*)a.xb;
    for (int64_t i0 = (int64_t)blockIdx.x * (256 * KG_U); i0 < total; i0 += (int64_t)gridDim.x * (256 * KG_U)) {
        const int64_t r0 = i0 / W;
        const uint32_t e0 = (uint32_t)(i0 - r0 * W) + threadIdx.x;
        int64_t src[KG_U];
        uint32_t d[KG_U];
        V v[KG_U];
#pragma unroll
        for (int u = 0; u < KG_U; ++u) {
            const uint32_t q = (e0 + u * 256) / W;
            d[u] = e0 + u * 256 - q * W;
            src[u] = i0 + u * 256 + threadIdx.x < total ? a.batch[r0 + q] : 0;
        }
#pragma unroll
        for (int u = 0; u < KG_U; ++u) {
            const int64_t i = i0 + u * 256 + threadIdx.x;
            v[u] = V{};
            if (i < total) {
                if (src[u] >= 0 && src[u] < a.N) v[u] = x[src[u] * W + d[u]];
                else if (d[u] == 0) atomicOr(&a.status->nonfinite, 2u);
            }
        }
#pragma unroll
        for (int u = 0; u < KG_U; ++u) {
            const int64_t i = i0 + u * 256 + threadIdx.x;
            if (i < total) xb[i] = v[u];
        }
    }
}

// ---- Batch positions grouped by center: counting sort over tiles of the batch.
// Three launches, each a few microseconds of latency (262,144 rows over 4096
// centers: 5 + 8 + 10 us; the general radix sort with its keys takes 18 launches
// and 107 us, most of it launches): count the rows of every (tile, center) in LDS; turn a center's
// column of counts into first places; replay each tile in batch order.  The
// runs of the centers are placed in the order in which their blocks arrive:
// within a run the order is the batch's, and nothing depends on the others.
constexpr int KM_LDS_K = 16384;   // centers whose counters fit one block's LDS (64 KB); more: radix sort
constexpr int KM_TILES = 256;     // tiles at most: one per CU, and the table stays within 1 KB per center
constexpr int KM_TILE_MIN = 256;  // rows of a tile at least

__global__ __launch_bounds__(256) void km_count_kernel(KmArgs a) {
    extern __shared__ uint32_t km_lds[];
    const int tid = threadIdx.x;
    if (blockIdx.x == 0 && tid == 0 && a.vq->nonfinite) atomicOr(&a.status->nonfinite, a.vq->nonfinite);
    for (int j = tid; j < a.K; j += 256) km_lds[j] = 0;
    __syncthreads();
    const int64_t r0 = (int64_t)blockIdx.x * a.tile;
    const int64_t end = std::min<int64_t>(a.B, r0 + a.tile);
    for (int64_t r = r0 + tid; r < end; r += 256) {
        const uint32_t j = (uint32_t)a.assign[r];
        if (j < (uint32_t)a.K) atomicAdd(&km_lds[j], 1u);
    }
    __syncthreads();
    uint32_t* row = a.table + (size_t)blockIdx.x * a.K;
    for (int j = tid; j < a.K; j += 256) row[j] = km_lds[j];
}

// 16 centers per block: 16 parts of the tiles by 16 centers.
__global__ __launch_bounds__(256) void km_place_kernel(KmArgs a) {
    __shared__ uint32_t part[16][17], base[16];
    constexpr int P = KM_TILES / 16;
    const int c = threadIdx.x & 15, p = threadIdx.x >> 4;
    const int j = blockIdx.x * 16 + c;
    uint32_t n[P];
    uint32_t sum = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) {
        const int t = p * P + i;
        n[i] = t < a.T && j < a.K ? a.table[(size_t)t * a.K + j] : 0;
    }
#pragma unroll
    for (int i = 0; i < P; ++i) sum += n[i];
    part[p][c] = sum;
    __syncthreads();
    if (threadIdx.x < 16) {  // the lengths of the block's runs, then the place of the first
        uint32_t len = 0;
        for (int q = 0; q < 16; ++q) {
            const uint32_t m = part[q][c];
            part[q][c] = len;
            len += m;
        }
        uint32_t incl = len;
        for (int o = 1; o < 16; o <<= 1) {
            const uint32_t m = __shfl_up(incl, o, 16);
            if (c >= o) incl += m;
        }
        uint32_t first = 0;
        if (c == 15) first = atomicAdd(a.cursor, incl);
        first = __shfl(first, 15, 16) + incl - len;
        base[c] = first;
        if (j < a.K) a.run[j] = make_uint2(first, len);
    }
    __syncthreads();
    uint32_t at = base[c] + part[p][c];
#pragma unroll
    for (int i = 0; i < P; ++i) {
        const int t = p * P + i;
        if (t < a.T && j < a.K) a.table[(size_t)t * a.K + j] = at;
        at += n[i];
    }
}

// A tile is replayed in batch order, 64 rows at a step: lanes of one center
// find each other by ballots over the key bits and take consecutive places,
// the first of them moves the center's place on.  The ballots are the long
// part and need no order, so four waves do KS_U steps each at a time; only
// the places are taken in turns.
constexpr int KS_U = 4;
__global__ __launch_bounds__(256) void km_scatter_kernel(KmArgs a) {
    extern __shared__ uint32_t km_lds[];
    const uint32_t* row = a.table + (size_t)blockIdx.x * a.K;
    for (int j = threadIdx.x; j < a.K; j += 256) km_lds[j] = row[j];
    const int lane = threadIdx.x & (MGS_WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / MGS_WAVE);
    const int64_t r0 = (int64_t)blockIdx.x * a.tile;
    const int64_t end = std::min<int64_t>(a.B, r0 + a.tile);
    const uint64_t below = (1ull << lane) - 1;
    for (int64_t b0 = r0; b0 < end; b0 += 4 * KS_U * MGS_WAVE) {
        const int64_t b = b0 + wave * (KS_U * MGS_WAVE) + lane;
        uint32_t key[KS_U], rank[KS_U], cnt[KS_U];
#pragma unroll
        for (int u = 0; u < KS_U; ++u) {
            const int64_t r = b + u * MGS_WAVE;
            key[u] = r < end ? (uint32_t)a.assign[r] : 0xFFFFFFFFu;
        }
#pragma unroll
        for (int u = 0; u < KS_U; ++u) {
            uint64_t same = __ballot(key[u] < (uint32_t)a.K);
            for (int bit = 0; bit < a.bits; ++bit) {
                const bool one = (key[u] >> bit) & 1u;
                const uint64_t m = __ballot(one);
                same &= one ? m : ~m;
            }
            rank[u] = (uint32_t)__popcll(same & below);
            cnt[u] = (uint32_t)__popcll(same);
        }
        for (int w = 0; w < 4; ++w) {
            __syncthreads();  // the places of the tile are there, or of the waves before
            if (wave != w) continue;
#pragma unroll
            for (int u = 0; u < KS_U; ++u) {
                // the place is read by all lanes of the center before the first
                // of them moves it on, and that before the next rows' lanes read it
                const bool valid = key[u] < (uint32_t)a.K;
                const uint32_t at = valid ? km_lds[key[u]] : 0u;
                wave_order();
                if (valid && rank[u] == 0) km_lds[key[u]] = at + cnt[u];
                wave_order();
                if (valid) a.pos_s[(size_t)at + rank[u]] = (int32_t)(b + u * MGS_WAVE);
            }
        }
    }
}

// Sort keys and batch positions of the batch rows (radix sort).
__global__ void km_keys_kernel(KmArgs a) {
    if (blockIdx.x == 0 && threadIdx.x == 0 && a.vq->nonfinite)
        atomicOr(&a.status->nonfinite, a.vq->nonfinite);
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < a.B;
         r += (int64_t)gridDim.x * blockDim.x) {
        const int j = a.assign[r];
        a.keys[r] = (unsigned)j < (unsigned)a.K ? (uint32_t)j : (uint32_t)a.K;
        a.pos[r] = (int32_t)r;
    }
}

// First index of the sorted keys that is >= key.
__device__ __forceinline__ int64_t lower_bound_u32(const uint32_t* k, int64_t n, uint32_t key) {
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (k[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// One wave per center: its run in pos_s, summed in batch order in FP64
// (lane d: dimension d), then the running-mean update
// c <- (v c + sum) / (v + n) and v += n.  Centers without rows keep their
// value and count.  Bound by the latency of the scattered rows: the places of
// 64 rows come with one load, and the rows of two half-chunks of KC_U are in
// flight while they are added in order (262,144 rows of 36 over 4096 centers:
// 39 us with four in flight, 17 us now).
constexpr int KC_U = 32;
template <bool RADIX>
__global__ __launch_bounds__(256) void km_center_kernel(KmArgs a) {
    const int lane = threadIdx.x & (MGS_WAVE - 1);
    const int64_t wave =
        __builtin_amdgcn_readfirstlane((int)(((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / MGS_WAVE));
    const int64_t nwaves = ((int64_t)gridDim.x * blockDim.x) / MGS_WAVE;
    for (int64_t j = wave; j < a.K; j += nwaves) {
        int64_t lo, n;
        if constexpr (RADIX) {
            lo = lower_bound_u32(a.keys_s, a.B, (uint32_t)j);
            n = lower_bound_u32(a.keys_s, a.B, (uint32_t)j + 1u) - lo;
        } else {
            const uint2 r = a.run[j];
            lo = r.x;
            n = r.y;
        }
        if (n == 0) continue;
        const int64_t v = a.counts[j];
        const int dl = std::min(lane, a.D - 1);  // lanes past the row repeat its last value
        const float* xd = a.xb + dl;
        const int32_t* ps = a.pos_s + lo;
        double s = 0.0;
        float f0[KC_U], f1[KC_U];
        int32_t place = 0;
        // places past the run repeat its last row; what they load is not added
        auto load = [&](float(&g)[KC_U], int half) {
#pragma unroll
            for (int u = 0; u < KC_U; ++u)
                g[u] = xd[(int64_t)__builtin_amdgcn_readlane(place, half * KC_U + u) * a.D];
        };
        auto add = [&](const float(&g)[KC_U], int64_t left) {
            if (left >= KC_U) {
#pragma unroll
                for (int u = 0; u < KC_U; ++u) s += (double)g[u];
            } else {  // adding +0 changes no sum (it is never -0)
#pragma unroll
                for (int u = 0; u < KC_U; ++u) s += (double)(u < left ? g[u] : 0.0f);
            }
        };
        place = ps[std::min<int64_t>(lane, n - 1)];
        load(f0, 0);
        for (int64_t i = 0; i < n; i += MGS_WAVE) {
            const bool second = i + KC_U < n, next = i + MGS_WAVE < n;
            if (second) load(f1, 1);
            if (next) place = ps[std::min<int64_t>(i + MGS_WAVE + lane, n - 1)];
            add(f0, n - i);
            if (next) load(f0, 0);
            if (second) add(f1, n - i - KC_U);
        }
        if (lane < a.D) {
            float* c = a.cb + j * a.D + lane;
            *c = (float)(((double)v * (double)*c + s) / (double)(v + n));
        }
        if (lane == 0) a.counts[j] = v + n;
    }
}

struct KmLayout {
    size_t xb, assign, pos_s, table, run, keys, keys_s, pos, sort, sort_bytes, vq, total;
    int32_t tile, T;
};

// Key bits of the sort: enough for the keys 0 .. K (K marks rows without a center).
int km_key_bits(int32_t K) {
    int bits = 1;
    while (bits < 32 && ((uint64_t)1 << bits) <= (uint64_t)K) ++bits;
    return bits;
}

// The size never falls with B or K, so that a workspace taken for the largest
// batch and codebook serves every smaller one: the table is sized for the most
// tiles that a batch of up to B rows can have (the tiles in use go down where
// the tile grows: 256 of 256 rows at 65,536, 205 of 320 at 65,537), and the
// radix sort's part takes at least what the counting sort of KM_LDS_K centers
// does.
KmLayout km_layout(int64_t B, int32_t D, int32_t K) {
    KmLayout L;
    std::memset(&L, 0, sizeof(L));
    const size_t b = (size_t)std::max<int64_t>(B, 1);
    size_t o = MGS_STATUS_BYTES;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += mgs_align_up(bytes, 256);
        return at;
    };
    L.xb = take(sizeof(float) * b * D);
    L.assign = take(sizeof(int32_t) * b);
    L.pos_s = take(sizeof(int32_t) * b);
    const size_t most = std::min<size_t>(KM_TILES, (b + KM_TILE_MIN - 1) / KM_TILE_MIN);  // tiles
    if (K <= KM_LDS_K) {
        const int64_t even = ((int64_t)b + KM_TILES - 1) / KM_TILES;
        L.tile = (int32_t)std::max<int64_t>(KM_TILE_MIN, (even + MGS_WAVE - 1) / MGS_WAVE * MGS_WAVE);
        L.T = (int32_t)(((int64_t)b + L.tile - 1) / L.tile);
        L.table = take(sizeof(uint32_t) * most * (size_t)K);
        L.run = take(sizeof(uint2) * (size_t)K);
    } else {
        const size_t counting = o + mgs_align_up(sizeof(uint32_t) * most * (size_t)KM_LDS_K, 256) +
                                mgs_align_up(sizeof(uint2) * (size_t)KM_LDS_K, 256);
        L.keys = take(sizeof(uint32_t) * b);
        L.keys_s = take(sizeof(uint32_t) * b);
        L.pos = take(sizeof(int32_t) * b);
        // temporary storage of the radix sort (a size query: no device work)
        (void)rocprim::radix_sort_pairs(nullptr, L.sort_bytes, (const uint32_t*)nullptr, (uint32_t*)nullptr,
                                        (const int32_t*)nullptr, (int32_t*)nullptr, (unsigned)b, 0,
                                        km_key_bits(K));
        L.sort = take(std::max<size_t>(L.sort_bytes, 1));
        o = std::max(o, counting);
    }
    L.vq = take(mgs_vq_assign_ws_bytes(B, D, K));
    L.total = o;
    return L;
}

unsigned km_blocks(int64_t n) {
    int64_t b = (n + 255) / 256;
    return (unsigned)std::max<int64_t>(1, std::min<int64_t>(b, 8192));
}

}  // namespace
}  // namespace mgs

extern "C" size_t mgs_kmeans_step_ws_bytes(int64_t B, int32_t D, int32_t K) {
    if (B < 0 || D < 1 || D > MGS_MAX_VQ_DIM || K < 1 || K > (1 << 30)) return 0;
    return mgs::km_layout(B, D, K).total;
}

extern "C" int mgs_kmeans_step(const float* d_x, int64_t N, int32_t D, const int64_t* d_batch, int64_t B,
                               float* d_cb, int32_t K, int64_t* d_counts, int32_t* d_assign, void* d_ws,
                               size_t ws_bytes, void* stream) {
    using namespace mgs;
    if (N < 0 || B < 0 || B >= ((int64_t)1 << 31) || D < 1 || D > MGS_MAX_VQ_DIM || K < 1 || K > (1 << 30) ||
        !d_cb ||
        !d_counts)
        return MGS_EINVAL;
    if (B > 0 && (!d_x || !d_batch)) return MGS_EINVAL;
    const KmLayout L = km_layout(B, D, K);
    if (!d_ws || ws_bytes < L.total) return MGS_EWORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    char* ws = (char*)d_ws;
    KmArgs a;
    std::memset(&a, 0, sizeof(a));
    a.x = d_x;
    a.batch = d_batch;
    a.xb = (float*)(ws + L.xb);
    a.assign = d_assign ? d_assign : (int32_t*)(ws + L.assign);
    a.table = (uint32_t*)(ws + L.table);
    a.run = (uint2*)(ws + L.run);
    a.keys = (uint32_t*)(ws + L.keys);
    a.keys_s = (uint32_t*)(ws + L.keys_s);
    a.pos = (int32_t*)(ws + L.pos);
    a.pos_s = (int32_t*)(ws + L.pos_s);
    a.cb = d_cb;
    a.counts = d_counts;
    a.status = (mgs_status_block*)ws;
    a.cursor = (uint32_t*)ws + 63;  // the last word of the block's 256 bytes
    a.N = N;
    a.B = B;
    a.D = D;
    a.K = K;
    a.tile = L.tile;
    a.T = L.T;
    a.bits = km_key_bits(K);
    int rc = mgs_fill<uint32_t>((uint32_t*)ws, 64, 0u, s);
    if (rc) return rc;
    if (B == 0) return MGS_OK;
    const bool vec = D % 4 == 0 && (uintptr_t)d_x % 16 == 0 && (uintptr_t)a.xb % 16 == 0;
    const unsigned gblocks = km_blocks((B * (vec ? D / 4 : D) + KG_U - 1) / KG_U);
    if (vec) hipLaunchKernelGGL(km_gather_kernel<float4>, dim3(gblocks), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(km_gather_kernel<float>, dim3(gblocks), dim3(256), 0, s, a);
    rc = mgs_last_launch();
    if (rc) return rc;
    // nearest centers of the batch rows; its status word (non-finite rows or
    // centers) is folded into this call's by the first kernel after it
    char* vq_ws = ws + L.vq;
    a.vq = (const mgs_status_block*)vq_ws;
    rc = mgs_vq_assign(a.xb, B, D, d_cb, K, a.assign, nullptr, nullptr, vq_ws,
                       mgs_vq_assign_ws_bytes(B, D, K), stream);
    if (rc) return rc;
    // the batch positions grouped by center, batch order kept within a center;
    // then one wave per center (grid-stride over the centers)
    const dim3 cgrid((unsigned)((std::min<int64_t>(K, 1 << 16) + 3) / 4));
    if (K <= KM_LDS_K) {
        const size_t lds = sizeof(uint32_t) * (size_t)K;
        hipLaunchKernelGGL(km_count_kernel, dim3((unsigned)L.T), dim3(256), lds, s, a);
        hipLaunchKernelGGL(km_place_kernel, dim3((unsigned)((K + 15) / 16)), dim3(256), 0, s, a);
        hipLaunchKernelGGL(km_scatter_kernel, dim3((unsigned)L.T), dim3(256), lds, s, a);
        hipLaunchKernelGGL(km_center_kernel<false>, cgrid, dim3(256), 0, s, a);
        return mgs_last_launch();
    }
    hipLaunchKernelGGL(km_keys_kernel, dim3(km_blocks(B)), dim3(256), 0, s, a);
    rc = mgs_last_launch();
    if (rc) return rc;
    size_t sort_bytes = L.sort_bytes;
    if (rocprim::radix_sort_pairs((void*)(ws + L.sort), sort_bytes, (const uint32_t*)a.keys, a.keys_s,
                                  (const int32_t*)a.pos, a.pos_s, (unsigned)B, 0, km_key_bits(K), s) !=
        hipSuccess)
        return MGS_EDEVICE;
    hipLaunchKernelGGL(km_center_kernel<true>, cgrid, dim3(256), 0, s, a);
    return mgs_last_launch();
}

// ------------------------------------------------------------------ retention
// Paper, same paragraph: the budget left after the essential components keeps
// the original SH vectors of the most important Gaussians; they are appended
// to the codebook and coded with it.  Here: the r retained rows (ascending
// Gaussian index, the selection of mgs_prune_select with one count r) are
// copied after the K codewords and their index entries point at them.
namespace mgs {
namespace {

__global__ void vq_retain_kernel(const float* __restrict__ x, int64_t N, int D,
                                 const int32_t* __restrict__ top, int64_t r, float* cb_ext, int K,
                                 int32_t* idx, mgs_status_block* status) {
    const int64_t total = r * D;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t e = i / D;
        const int d = (int)(i - e * D);
        const int64_t g = top[e];
        if (g < 0 || g >= N) {
            if (d == 0 && status) atomicOr(&status->nonfinite, 2u);
            continue;
        }
        cb_ext[((int64_t)K + e) * D + d] = x[g * D + d];
        if (d == 0) idx[g] = (int32_t)(K + e);
    }
}

}  // namespace
}  // namespace mgs

extern "C" int64_t mgs_vq_retain_count(int64_t remaining_bits, int64_t N, int32_t D) {
    if (remaining_bits <= 0 || N <= 0 || D < 1) return 0;
    return std::min<int64_t>(N, remaining_bits / (32 * (int64_t)D));
}

extern "C" int mgs_vq_retain(const float* d_x, int64_t N, int32_t D, const int32_t* d_top, int64_t r,
                             float* d_cb_ext, int32_t K, int32_t* d_idx, void* d_ws, size_t ws_bytes,
                             void* stream) {
    using namespace mgs;
    if (N < 0 || D < 1 || D > MGS_MAX_VQ_DIM || K < 0 || r < 0 || r > N || (int64_t)K + r >= ((int64_t)1 << 31))
        return MGS_EINVAL;
    if (r > 0 && (!d_x || !d_top || !d_cb_ext || !d_idx)) return MGS_EINVAL;
    if (!d_ws || ws_bytes < MGS_STATUS_BYTES) return MGS_EWORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    auto* status = (mgs_status_block*)d_ws;
    int rc = mgs_fill<uint32_t>((uint32_t*)d_ws, 64, 0u, s);
    if (rc || r == 0) return rc;
    hipLaunchKernelGGL(vq_retain_kernel, dim3(km_blocks(r * D)), dim3(256), 0, s, d_x, N, (int)D, d_top, r,
                       d_cb_ext, (int)K, d_idx, status);
    return mgs_last_launch();
}
