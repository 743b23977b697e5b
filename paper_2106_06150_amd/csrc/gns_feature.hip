// Feature gather (paper Section 2.2 steps 2-3: slice the input nodes' rows;
// cached rows are already device resident, Section 3.2) and the weighted mean
// aggregation of one layer (Algorithm 1 bottom-up loop with Section 3.4's
// rescaling).  Both are pure data movement / fp32 FMA streams: a group of
// lanes owns one row and moves it with 128-bit accesses.
#include <algorithm>
#include "gns_internal.h"
#include "gns_device.hpp"
#include <string.h>
#include <stdlib.h>
#include <type_traits>

namespace gns {

// Four consecutive floats at any 4-byte address, moved at once.
typedef float Float4u __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ float4 load_floats(const char* p)
{
    const Float4u v = *reinterpret_cast<const Float4u*>(p);
    return make_float4(v.x, v.y, v.z, v.w);
}

// Output rows are written once and not read again by the writing kernel: a non-temporal store keeps
// them from displacing the rows other waves still want from L2.
__device__ __forceinline__ void store_floats(char* p, const float4& r)
{
    const Float4u v = {r.x, r.y, r.z, r.w};
    __builtin_nontemporal_store(v, reinterpret_cast<Float4u*>(p));
}

// One launch serves a group of mini-batches: blockIdx.y picks the batch.
struct GatherBatch {
    const int32_t* nodes;
    const int32_t* num_nodes_dev;   // if not null the count is read here (num_nodes is then the worst case)
    float* out;
    int32_t num_nodes;
    int32_t pad;
};

struct GatherArgs {
    GatherBatch b[GNS_MAX_GROUP];
    const int32_t* unless_negative;   // if not null and below zero there, nothing is copied
    int64_t n;
    int32_t feat_dim;
    int32_t use_cache;
    const uint64_t* cache_bitmap;
    const int32_t* cache_prefix;
    const float* cache_feat;
    const float* store;          // device store or device-visible pinned host store
};

// kLanes lanes per row, four floats a lane (F >= 4: where F is no multiple of four the last lane's reach back into those before).
// Bound by the copy.  Two things stood in its way or in the aggregation's:
//  - the chain of every row, node -> bitmap -> rank -> row.  A wave looks up the rows of its next kLanes turns at once, one
//    per lane, and a turn is a read and a store.
//  - what the copy left in the caches.  Cached rows are what the input layer's aggregation reads, some dozens of times each: stored
//    plainly they are still there by then.  All other stores pass the caches by, so as not to displace them, and so do the reads
//    (kPastCaches) of a table that the caches do not hold anyway.
// Groups of four, on states that change from call to call, this kernel and the aggregation behind it: 1 M nodes (4 x 90 K rows of
// 512 bytes) 66.5 + 73 -> 68 + 52 us (all stores past the caches 65 + 85, reads plain 61 + 66, all stores plain 65 + 73), with the
// upper layers cache first 34 + 38.5 -> 32 + 31, 40 M nodes 78 + 54 -> 66 + 52; one mini-batch of 90 K rows 21 + 21.5 -> 20.5 + 16.4.
template <int kLanes, bool kPastCaches>
__global__ void __launch_bounds__(kBlock) k_gather(GatherArgs a)
{
    if (a.unless_negative && *a.unless_negative < 0) return;
    constexpr uint32_t kRows = kWave / kLanes;               // rows a wave copies in a turn
    constexpr int32_t kNone = INT32_MIN;
    const GatherBatch q = a.b[blockIdx.y];
    const uint32_t count = (uint32_t) (q.num_nodes_dev ? *q.num_nodes_dev : q.num_nodes);
    const uint32_t wave = blockIdx.x * (kBlock / kWave) + (uint32_t) __builtin_amdgcn_readfirstlane((int) (threadIdx.x >> 6));
    const uint32_t stride = gridDim.x * (kBlock / kWave) * kRows;
    const int64_t F = a.feat_dim;
    for (uint32_t row0 = wave * kRows; row0 < count; row0 += stride * kLanes) {
        const int lane = opaque_lane_id();
        const uint32_t sub = (uint32_t) lane / kLanes;
        // lane l: row l % kRows of turn l / kRows: its node, ~(its place in the cache table), or kNone
        const uint64_t mine = row0 + (uint64_t) (lane / kRows) * stride + lane % kRows;
        int32_t ref = kNone;
        if (mine < count) {
            const int32_t u = q.nodes[mine];
            if (u >= 0 && (int64_t) u < a.n) {
                ref = u;
                if (a.use_cache) {
                    const uint64_t word = a.cache_bitmap[u >> 6], bit = 1ull << (u & 63);
                    if (word & bit) ref = ~(a.cache_prefix[u >> 6] + __popcll(word & (bit - 1ull)));
                }
            }
        }
        const uint32_t turns = (count - row0 + stride - 1) / stride;
        for (uint32_t t = 0; t < turns && t < kLanes; ++t) {
            const int32_t r = __shfl(ref, (int) (t * kRows + sub), kWave);
            const uint32_t row = row0 + t * stride + sub;
            if (row >= count) continue;
            const float* src = r >= 0 ? a.store + (int64_t) r * F : a.cache_feat + (int64_t) ~r * F;
            float* dst = q.out + (int64_t) row * F;
            for (int64_t c = 4 * (lane % kLanes); c < F; c += 4 * kLanes) {
                const int64_t at = c < F - 4 ? c : F - 4;
                Float4u v = {0.f, 0.f, 0.f, 0.f};
                if (r != kNone) {
                    const Float4u* p = reinterpret_cast<const Float4u*>(src + at);
                    if (kPastCaches) v = __builtin_nontemporal_load(p);
                    else             v = *p;
                }
                if (r < 0) {
                    asm volatile("; cached row");            // (the two stores would become one, without the hint)
                    *reinterpret_cast<Float4u*>(dst + at) = v;
                    asm volatile("; cached row");
                } else {
                    __builtin_nontemporal_store(v, reinterpret_cast<Float4u*>(dst + at));
                }
            }
        }
    }
}

// Rows of fewer than four floats, a lane each.
__global__ void __launch_bounds__(kBlock) k_gather_thin(GatherArgs a)
{
    if (a.unless_negative && *a.unless_negative < 0) return;
    const GatherBatch q = a.b[blockIdx.y];
    const int64_t count = q.num_nodes_dev ? *q.num_nodes_dev : q.num_nodes;
    for (int64_t row = (int64_t) blockIdx.x * kBlock + threadIdx.x; row < count; row += (int64_t) gridDim.x * kBlock) {
        const int32_t u = q.nodes[row];
        const bool valid = u >= 0 && (int64_t) u < a.n;
        const float* src = a.store + (int64_t) u * a.feat_dim;
        if (valid && a.use_cache && bitmap_test(a.cache_bitmap, (uint32_t) u))
            src = a.cache_feat + (int64_t) bitmap_rank(a.cache_bitmap, a.cache_prefix, (uint32_t) u) * a.feat_dim;
        for (int i = 0; i < a.feat_dim; ++i) q.out[row * a.feat_dim + i] = valid ? src[i] : 0.f;
    }
}

// Bytes of a feature table (in HBM) that is read through the caches: what the infinity cache (256 MB) keeps from call to call.  us of a gather
// alone, with reads through the caches and past them, and of a whole call (sampling, gather and aggregation of 1024 seeds):
//   100 K nodes, 128 floats (49 MB)        9.0 and 10.3    64.5 and 66.1, four at a time 119.4 and 125.0
//   200 K nodes, 256 floats (195 MB)      18.6 and 21.9    76.7 and 79.6                 188.1 and 194.7
//   1 M nodes, 64 floats (244 MB)          9.0 and 10.9    69.4 and 68.6                 145.7 and 143.9
//   1 M nodes, 128 floats (488 MB)        15.3 and 17.7    82.2 and 81.1                 188.1 and 188.4
//   4 M nodes, 128 floats (1953 MB)       20.0 and 23.2   100.9 and 100.5                274.4 and 268.4
// (Beyond, what the gather loses the aggregation gains.)
constexpr double kKeptTable = 200.0 * 1024 * 1024;

static inline int lanes_for(int64_t units)
{
    int l = 4;
    while (l < 64 && l < units) l <<= 1;
    return l;
}

template <bool kPastCaches>
static void gather_dispatch(int lanes, dim3 blocks, hipStream_t s, const GatherArgs& a)
{
    switch (lanes) {
        case 4:  hipLaunchKernelGGL((k_gather<4, kPastCaches>), blocks, dim3(kBlock), 0, s, a); break;
        case 8:  hipLaunchKernelGGL((k_gather<8, kPastCaches>), blocks, dim3(kBlock), 0, s, a); break;
        case 16: hipLaunchKernelGGL((k_gather<16, kPastCaches>), blocks, dim3(kBlock), 0, s, a); break;
        case 32: hipLaunchKernelGGL((k_gather<32, kPastCaches>), blocks, dim3(kBlock), 0, s, a); break;
        default: hipLaunchKernelGGL((k_gather<64, kPastCaches>), blocks, dim3(kBlock), 0, s, a); break;
    }
}

// count mini-batches (contexts ctxs[0..count) of one family) in one launch.  num_nodes[b] < 0: the input
// nodes of the last batch sampled on ctxs[b], counted on the device.
hipError_t launch_gather(gns_ctx* const* ctxs, int count, const int32_t* const* nodes, const int32_t* num_nodes,
                         float* const* out, int use_cache_gen, hipStream_t s, const int32_t* unless_negative)
{
    gns_ctx* c = ctxs[0];
    const Layout& L = c->lay;
    GatherArgs a;
    memset(&a, 0, sizeof(a));
    a.unless_negative = unless_negative;
    int64_t most = 0;
    for (int b = 0; b < count; ++b) {
        GatherBatch& q = a.b[b];
        q.nodes = nodes[b];
        q.out = out[b];
        q.num_nodes = num_nodes[b];
        if (num_nodes[b] < 0) {
            q.num_nodes_dev = &ctxs[b]->d_state->num_dst[c->config.num_layers];
            q.num_nodes = (int32_t) L.rows[c->config.num_layers];
        }
        if (q.num_nodes > most) most = q.num_nodes;
    }
    if (most == 0) return hipSuccess;
    a.n = c->graph.num_nodes;
    a.feat_dim = c->graph.feat_dim;
    const int gen = use_cache_gen < 0 ? 0 : use_cache_gen;
    a.use_cache = (use_cache_gen >= 0 && c->uses_cache && c->root->cache_valid) ? 1 : 0;
    a.cache_bitmap = cache_ptr<uint64_t>(c, L.cache_bitmap, gen);
    a.cache_prefix = cache_ptr<int32_t>(c, L.cache_prefix, gen);
    a.cache_feat = cache_ptr<float>(c, L.cache_feat, gen);
    a.store = c->graph.feat_dev ? c->graph.feat_dev : c->graph.feat_host_pinned;
    const bool thin = a.feat_dim < 4;
    const int lanes = lanes_for((a.feat_dim + 3) / 4);
    const int64_t rows_per_block = thin ? kBlock : kBlock / lanes;
    int64_t blocks = (most + rows_per_block - 1) / rows_per_block;
    // What is resident together, of all batches; beyond that a group copies several rows (twice or four times as many: the same).  Not one
    // block more: it would begin when the others end, with as much to do as each of them (groups of three and five were 2049 and 2050
    // blocks: calls on 1 M nodes 190.2 and 284.3 us, 182.0 and 268.9 now).
    const int64_t cap = std::max((int64_t) c->num_cus * 8 / count, (int64_t) 1);
    if (blocks > cap) blocks = cap;
    const dim3 grid((unsigned) blocks, (unsigned) count);
    if (thin) hipLaunchKernelGGL(k_gather_thin, grid, dim3(kBlock), 0, s, a);
    else if (c->graph.feat_dev && (double) a.n * a.feat_dim * 4 <= kKeptTable) gather_dispatch<false>(lanes, grid, s, a);
    else                                                                       gather_dispatch<true>(lanes, grid, s, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
struct AggBatch {
    const int32_t* indptr;
    const int32_t* indices;
    const float* weights;
    const float* x_src;
    float* out;
    const int32_t* num_dst_dev;     // if not null the row count is read here
    const int32_t* num_src_dev;
    int32_t num_dst;
    int32_t num_src;                // rows of x_src; an edge whose index lies outside is skipped
};

struct AggGroup {
    AggBatch b[GNS_MAX_GROUP];
    int32_t feat_dim;
    uint32_t first_window;          // windows of columns of the launches before
};

constexpr uint32_t kAggWindow = 1024;      // columns a block takes at most (64 lanes of four times four)

// the view of one batch the kernel body works on
struct AggArgs : AggBatch {
    int32_t feat_dim;
};

// Columns col0 .. col0 + 4 kLanes kPer - 1 of a call's rows (F >= 4): a group of kLanes lanes owns a dst row, lane l accumulates four
// columns from col0 + 4 l on, and from 4 kLanes further on, ... (kPer times).  Any width and any alignment to four bytes: where F is
// no multiple of four the last lane's columns reach back into those before, and two lanes compute and store the same.  Branch-free inner
// loop: the first kSlots lanes of the group hold one edge each (index and weight, one coalesced read), every lane then takes
// edge t from lane t of its group, so the reads of the source rows are issued back to back; in a slot past its
// row's end a lane group stands aside (weight 0 on zeros: the texture addressers only work for lanes that take
// part in a read), rows with more than kSlots edges take further rounds.  All lanes of the wave stay converged: trip counts
// are wave-uniform (the shuffles need every source lane).
// A row is a chain of dependent accesses (row extent -> edges -> source rows -> store); it is software-pipelined
// over the rows a group visits: while the source rows of row i are in flight, the edges of row i+1 and the
// extent of row i+2 are being read.  (What bounds the kernel on 128-float rows is the rate at which the L2s
// deliver scattered 512-byte rows next to the stream of output rows: a loop with no bookkeeping at all -- hashed
// source rows, constant weights -- is within 15 % of it, and lane layout, pipelining and grid size each move it by
// a few percent only.)
// The hardware counts outstanding vector memory operations in order, and the compiler can only leave the
// younger ones in flight across a use of an older one if it knows how many there are: a read or store inside
// a branch makes it wait for everything.  Hence the accesses of the steady state are unconditional -- reads
// of rows or edges that do not exist go to a valid address (the first extent) and their value is replaced,
// and the last trip, in which some groups have no row, stands apart -- and only rare cases (a row with more than
// kSlots edges, slots beyond the fourth) sit in branches.  Lanes past the last column (kRagged) stand aside in the last of the
// kPer reads and stores all the same: what a read costs the texture addressers is more than the wait.  (In the last of several windows lanes
// can be past the last column in the reads before it too; there they repeat the last four columns.)
// kOff32: every byte offset into x_src fits 32 bits and row index and row size fit 24 bits, so an address is
// the uniform base plus one 32-bit vector offset (one multiply-add per load).  Offsets within a row are counted from the
// window's first column: rows of 2^30 floats are 4 GB long.
template <int kLanes, int kPer, bool kRagged, bool kQuotient, bool kOff32>
__device__ __forceinline__ void aggregate_rows(const AggArgs& a, uint32_t col0, uint32_t group, uint32_t num_groups, uint32_t count,
                                               uint32_t num_src)
{
    constexpr int kSlots = kLanes < 8 ? kLanes : 8;                      // edges a round covers (one per lane)
    constexpr int kFlight = kLanes * kPer == 8 ? 6 : kPer >= 3 ? 5 : kSlots;     // source rows read together
    const int lane = (int) (threadIdx.x % kLanes);
    const uint32_t F = (uint32_t) a.feat_dim;
    const uint32_t row_bytes = F * 4u;                                  // (kOff32)
    const uint32_t base = kLanes * kPer * 4 < kAggWindow ? 0u : col0 < F - 4u ? col0 : F - 4u;
    const bool in_last = !kRagged || col0 + 4u * ((uint32_t) lane + (uint32_t) (kPer - 1) * kLanes) < F;
    uint32_t col_bytes[kPer];
#pragma unroll
    for (int p = 0; p < kPer; ++p) {
        const uint32_t c = col0 + 4u * ((uint32_t) lane + (uint32_t) p * kLanes);
        col_bytes[p] = ((c < F - 4u ? c : F - 4u) - base) * 4u;
    }
    const char* x_bytes = reinterpret_cast<const char*>(a.x_src + base);
    const uint32_t trips = (count + num_groups - 1u) / num_groups;       // the same for every group (count > 0)

    // extent of the row this group visits in trip `it` (empty past the end)
    auto extent = [&](uint32_t it, int32_t& b, int32_t& e) {
        const uint32_t row = group + it * num_groups;
        const bool ok = it < trips && row < count;
        const uint32_t r = ok ? row : 0u;
        struct __attribute__((packed, aligned(4))) Pair { int32_t lo, hi; };       // one 8-byte read, 4-byte aligned
        const Pair pr = *reinterpret_cast<const Pair*>(a.indptr + r);
        b = pr.lo;
        e = ok ? pr.hi : pr.lo;
    };
    // the edge this lane holds in the round that starts at entry q0 of a row ending at e
    auto edge = [&](int32_t q0, int32_t e, uint32_t& j, float& w) {
        const bool mine = q0 + lane < e && lane < kSlots;
        const int32_t* pj = mine ? a.indices + (q0 + lane) : a.indptr;
        const float* pw = mine ? a.weights + (q0 + lane) : reinterpret_cast<const float*>(a.indptr);
        const uint32_t jv = (uint32_t) *pj;
        const float wv = *pw;
        j = mine ? jv : 0u;
        w = mine ? wv : 0.f;
    };
    // one round: the edges (my_j, my_w) the group's lanes hold for entries [q0, e) of the row, slots [kFirst, kSlots)
    auto round = [&](int32_t q0, int32_t e, uint32_t my_j, float my_w, float4 (&acc)[kPer], auto&& between) {
        const int32_t here = e - q0 < kSlots ? (e - q0 > 0 ? e - q0 : 0) : kSlots;   // edges of this round
        const bool bad = lane < here && my_j >= num_src;         // an index outside [0, num_src) is skipped
        if (bad) { my_j = 0u; my_w = 0.f; }
        const bool any_bad = __any(bad);
#pragma unroll
        for (int t0 = 0; t0 < kSlots; t0 += kFlight) {
            if (t0 > 0 && !__any(t0 < here)) break;              // no row of this wave has that many edges
            float4 x[kFlight][kPer];
            float w[kFlight];
#pragma unroll
            for (int u = 0; u < kFlight; ++u) {
                const int t = t0 + u;
                w[u] = 0.f;
#pragma unroll
                for (int p = 0; p < kPer; ++p) x[u][p] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (t >= kSlots || (t >= 4 && !__any(t < here))) continue;       // a slot no row of this wave needs
                const uint32_t j = (uint32_t) __shfl((int) my_j, t, kLanes);
                const float wt = __shfl(my_w, t, kLanes);
                // Lanes of rows that have no edge in this slot stand aside: the texture addressers, which bound this
                // kernel, only work for the lanes that take part in a read.
                if (t < here) {
                    w[u] = wt;
#pragma unroll
                    for (int p = 0; p < kPer; ++p) {
                        if (kRagged && p == kPer - 1 && !in_last) continue;
                        if (kOff32) {
                            const uint32_t off = __umul24(j, row_bytes) + col_bytes[p];     // both factors < 2^24
                            x[u][p] = load_floats(x_bytes + off);
                        } else {
                            const uint64_t off = (uint64_t) j * F * 4u + col_bytes[p];
                            x[u][p] = load_floats(x_bytes + off);
                        }
                    }
                }
            }
            if (t0 == 0) between();                              // reads for the rows ahead, behind this row's first reads
            if (any_bad) {
                // rare: a skipped edge must not contribute even a NaN of the row it was redirected to
#pragma unroll
                for (int u = 0; u < kFlight; ++u) {
                    const int t = t0 + u;
                    if (t >= kSlots) continue;
                    if (__shfl((int) bad, t, kLanes)) {
#pragma unroll
                        for (int p = 0; p < kPer; ++p) x[u][p] = make_float4(0.f, 0.f, 0.f, 0.f);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < kFlight; ++u) {                  // edge order, one fma per term
                if (t0 + u >= kSlots || (t0 + u >= 4 && !__any(t0 + u < here))) continue;
#pragma unroll
                for (int p = 0; p < kPer; ++p) {
                    acc[p].x = fmaf(w[u], x[u][p].x, acc[p].x);
                    acc[p].y = fmaf(w[u], x[u][p].y, acc[p].y);
                    acc[p].z = fmaf(w[u], x[u][p].z, acc[p].z);
                    acc[p].w = fmaf(w[u], x[u][p].w, acc[p].w);
                }
            }
        }
    };

    // one row: its first round with the reads for the rows ahead slipped in, further rounds if it has more than
    // kSlots edges, scaling, store
    auto visit = [&](uint32_t row, int32_t b, int32_t e, uint32_t j, float w, auto&& between, auto&& store) {
        float4 acc[kPer];
#pragma unroll
        for (int p = 0; p < kPer; ++p) acc[p] = make_float4(0.f, 0.f, 0.f, 0.f);
        round(b, e, j, w, acc, between);
        if (__any(e - b > kSlots)) {            // read on the spot
            for (int32_t q0 = b + kSlots; __any(q0 < e); q0 += kSlots) {
                uint32_t my_j;
                float my_w;
                edge(q0, e, my_j, my_w);
                round(q0, e, my_j, my_w, acc, []() {});
            }
        }
        const bool some = e > b;                                           // (a row without edges has read nothing: 0)
        const float n = some ? (float) (e - b) : 1.f;
        const float inv_n = some ? 1.0f / n : 0.f;                         // one division per row, then the products
        // kQuotient: x / n to the last bit, from the product and what it leaves (not for infinities, whose product it is; halfway
        // between two numbers below the normal ones either may come out)
        auto mean = [&](float x) {
            const float q = x * inv_n;
            if (!kQuotient) return q;
            const float left = fmaf(-q, n, x);
            return left == left ? fmaf(left, inv_n, q) : q;
        };
        char* o = reinterpret_cast<char*>(a.out + (int64_t) row * F + base);
#pragma unroll
        for (int p = 0; p < kPer; ++p) {
            if (kRagged && p == kPer - 1 && !in_last) continue;
            const float4 r = make_float4(mean(acc[p].x), mean(acc[p].y), mean(acc[p].z), mean(acc[p].w));
            store(o + col_bytes[p], r);
        }
    };

    int32_t b0, e0, b1, e1;
    uint32_t j0;
    float w0;
    extent(0, b0, e0);
    extent(1, b1, e1);
    edge(b0, e0, j0, w0);
    // every group has a row in all trips but the last: nothing conditional there
    for (uint32_t it = 0; it + 1 < trips; ++it) {
        int32_t b2 = 0, e2 = 0;
        uint32_t j1 = 0;
        float w1 = 0.f;
        visit(group + it * num_groups, b0, e0, j0, w0,
              [&]() {
                  extent(it + 2, b2, e2);       // two rows ahead
                  edge(b1, e1, j1, w1);         // one row ahead
              },
              [](char* dst, const float4& r) { store_floats(dst, r); });
        b0 = b1; e0 = e1; b1 = b2; e1 = e2; j0 = j1; w0 = w1;
    }
    const uint32_t row = group + (trips - 1u) * num_groups;
    const bool live = row < count;
    visit(row, b0, e0, j0, w0, []() {}, [&](char* dst, const float4& r) { if (live) store_floats(dst, r); });
}

// Rows of more columns than a block takes at most are visited once per window of columns (blockIdx.z, behind those of the launches before).
template <int kLanes, int kPer, bool kRagged, bool kQuotient>
__global__ void __launch_bounds__(kBlock, kLanes * kPer == 8 ? 6 : 1) k_aggregate(AggGroup g)
{
    AggArgs a;
    static_cast<AggBatch&>(a) = g.b[blockIdx.y];
    a.feat_dim = g.feat_dim;
    const int lane = (int) (threadIdx.x % kLanes);
    const uint32_t groups_per_block = kBlock / kLanes;
    const uint32_t group = blockIdx.x * groups_per_block + threadIdx.x / kLanes;
    const uint32_t num_groups = gridDim.x * groups_per_block;
    const uint32_t F = (uint32_t) a.feat_dim;
    const int64_t rows = a.num_dst_dev ? (int64_t) *a.num_dst_dev : (int64_t) a.num_dst;
    const uint32_t num_src = (uint32_t) (a.num_src_dev ? *a.num_src_dev : a.num_src);
    if (rows <= 0) return;
    const uint32_t count = (uint32_t) rows;
    constexpr uint32_t kWindow = 4 * kLanes * kPer;
    const uint32_t col0 = kWindow == kAggWindow ? (g.first_window + blockIdx.z) * kWindow : 0u;
    if (num_src == 0) {             // no source row to read (and none may be touched): every edge is skipped
        const uint32_t end = col0 + kWindow < F ? col0 + kWindow : F;
        for (int64_t row = group; row < rows; row += num_groups)
            for (uint32_t i = col0 + (uint32_t) lane; i < end; i += kLanes) a.out[row * F + i] = 0.f;
        return;
    }
    const bool off32 = (uint64_t) num_src * F * 4u < ((uint64_t) 1 << 32) && num_src < (1u << 24) && F < (1u << 22);
    if (off32) aggregate_rows<kLanes, kPer, kRagged, kQuotient, true>(a, col0, group, num_groups, count, num_src);
    else       aggregate_rows<kLanes, kPer, kRagged, kQuotient, false>(a, col0, group, num_groups, count, num_src);
}

// Rows of fewer than four floats, a lane per column.
__global__ void __launch_bounds__(kBlock) k_aggregate_thin(AggGroup g)
{
    const AggBatch a = g.b[blockIdx.y];
    const int64_t F = g.feat_dim;
    const int i = (int) (threadIdx.x % 4);
    const int64_t count = a.num_dst_dev ? (int64_t) *a.num_dst_dev : (int64_t) a.num_dst;
    const uint32_t num_src = (uint32_t) (a.num_src_dev ? *a.num_src_dev : a.num_src);
    if (i >= F) return;
    for (int64_t row = (int64_t) blockIdx.x * (kBlock / 4) + threadIdx.x / 4; row < count; row += (int64_t) gridDim.x * (kBlock / 4)) {
        const int32_t b = a.indptr[row], e = a.indptr[row + 1];
        float acc = 0.f;
        for (int32_t q = b; q < e; ++q) {
            const uint32_t j = (uint32_t) a.indices[q];
            if (j < num_src) acc = fmaf(a.weights[q], a.x_src[(int64_t) j * F + i], acc);
        }
        if (e > b) acc /= (float) (e - b);
        a.out[row * F + i] = acc;
    }
}

// Lanes per row and columns (of four floats) per lane, for rows of F4 columns.  A read costs the lanes that take part in it and the
// lines it touches: so few lanes are left over, and as much of a row as possible is read as one piece, unless rows are whole
// lines (F4 % 8 == 0), of which eight lanes read one each time.  us for four mini-batches of 85 K rows (1 M nodes) behind their gather, lanes x columns:
//   F4   8 x 1   8 x 2   8 x 3   8 x 4  16 x 2  16 x 3  16 x 4  32 x 2     one column a lane, no row ahead
//    5    23.8    24.4                                                      29
//    9            31.8    31.0            36.5
//   12            34.0            38.2                                      44
//   17                    45.4    45.4    49.5                              70
//   21                    53.0    56.4    52.5
//   24                    40.4    45.3    49.2                              46
//   25                            59.1    55.4                              72
//   31                            69.2    62.2
//   32                            49.3    53.4
//   33                                            70.2    72.4    81.3
//   40                                            65.5    75.0    80.0
//   48                                            75.2    80.7    83.4      81
//   50                                                    98.7    93.4     129
//   64                                                   101.9    98.0
// Widths that are no multiple of four took 91 (F = 19), 285 (99) and 623 (255) with a float per lane, an edge at a time.
struct AggLanes {
    int lanes, per;
};

static AggLanes aggregate_lanes(int64_t F4)
{
    if (F4 <= 4) return {4, 1};
    if (F4 <= 8) return {8, 1};
    if (F4 <= 16) return {8, 2};
    if (F4 <= 20 || F4 == 24) return {8, 3};
    if (F4 == 32) return {8, 4};
    if (F4 <= 32) return {16, 2};
    if (F4 <= 48) return {16, 3};
    if (F4 <= 64) return {32, 2};
    if (F4 <= 96) return {32, 3};
    if (F4 <= 128) return {32, 4};
    if (F4 <= 192) return {64, 3};
    return {64, 4};
}

static void aggregate_dispatch(AggLanes q, bool full, bool quotient, dim3 grid, hipStream_t s, const AggGroup& a)
{
    using std::integral_constant;
    using Yes = std::true_type;
    using No = std::false_type;
    auto go = [&](auto lanes, auto per, auto ragged, auto quotient) {
        hipLaunchKernelGGL((k_aggregate<decltype(lanes)::value, decltype(per)::value, decltype(ragged)::value, decltype(quotient)::value>), grid,
                           dim3(kBlock), 0, s, a);
    };
    // fills: whether rows that leave no lane over come here and gain by a form of their own (32 lanes: the one for rows that leave lanes
    // over is ahead where none are, 98 us for 105 at F = 256); leaves: whether others do that are not divided
    auto with = [&](auto lanes, auto per, auto fills, auto leaves) {
        if (quotient) go(lanes, per, Yes(), Yes());
        else if constexpr (!decltype(leaves)::value) go(lanes, per, No(), No());
        else if constexpr (!decltype(fills)::value) go(lanes, per, Yes(), No());
        else if (full) go(lanes, per, No(), No());
        else go(lanes, per, Yes(), No());
    };
    if (q.lanes == 4)       with(integral_constant<int, 4>(), integral_constant<int, 1>(), Yes(), Yes());
    else if (q.lanes == 8) {
        if (q.per == 1)      with(integral_constant<int, 8>(), integral_constant<int, 1>(), Yes(), Yes());
        else if (q.per == 2) with(integral_constant<int, 8>(), integral_constant<int, 2>(), Yes(), Yes());
        else if (q.per == 3) with(integral_constant<int, 8>(), integral_constant<int, 3>(), Yes(), Yes());
        else                 with(integral_constant<int, 8>(), integral_constant<int, 4>(), Yes(), No());         // 128 columns only
    } else if (q.lanes == 16) {
        if (q.per == 2)      with(integral_constant<int, 16>(), integral_constant<int, 2>(), No(), Yes());        // 128 columns are not here
        else                 with(integral_constant<int, 16>(), integral_constant<int, 3>(), Yes(), Yes());
    } else if (q.lanes == 32) {
        if (q.per == 2)      with(integral_constant<int, 32>(), integral_constant<int, 2>(), No(), Yes());
        else if (q.per == 3) with(integral_constant<int, 32>(), integral_constant<int, 3>(), No(), Yes());
        else                 with(integral_constant<int, 32>(), integral_constant<int, 4>(), No(), Yes());
    } else {
        if (q.per == 3)      with(integral_constant<int, 64>(), integral_constant<int, 3>(), Yes(), Yes());
        else                 with(integral_constant<int, 64>(), integral_constant<int, 4>(), Yes(), Yes());
    }
}

hipError_t launch_aggregate(gns_ctx* const* ctxs, int count, const gns_block* const* blks, const float* const* x_src,
                            int32_t feat_dim, float* const* out, hipStream_t s)
{
    gns_ctx* c = ctxs[0];
    if (feat_dim == 0) return hipSuccess;
    AggGroup a;
    memset(&a, 0, sizeof(a));
    int64_t most = 0;
    bool aligned = true;
    for (int b = 0; b < count; ++b) {
        const gns_block* blk = blks[b];
        AggBatch& q = a.b[b];
        int32_t rows = blk->num_dst;
        q.num_src = blk->num_src;
        if (rows < 0) {                 // GNS_DEVICE_COUNTS(layer): rows counted on the device
            const int layer = -1 - rows;
            q.num_dst_dev = &ctxs[b]->d_state->num_dst[layer];
            q.num_src_dev = &ctxs[b]->d_state->num_dst[layer + 1];
            rows = (int32_t) c->lay.rows[layer];
        }
        q.indptr = blk->indptr;
        q.indices = blk->indices;
        q.weights = blk->weights;
        q.x_src = x_src[b];
        q.out = out[b];
        q.num_dst = rows;
        if (rows > most) most = rows;
        aligned = aligned && ((reinterpret_cast<uintptr_t>(x_src[b]) | reinterpret_cast<uintptr_t>(out[b])) & 15u) == 0;
    }
    if (most == 0) return hipSuccess;
    a.feat_dim = feat_dim;
    const int64_t F4 = ((int64_t) feat_dim + 3) / 4;
    const bool thin = feat_dim < 4;
    // x / n is rounded once, not as a product with 1 / n (four more instructions a float, up to 6 of 76 us at F = 130):
    // widths and bases that are no multiple of four floats, and wide rows
    const bool quotient = feat_dim % 4 != 0 || !aligned || feat_dim > 1024 || (feat_dim > 256 && F4 % 8 != 0);
    const AggLanes q = aggregate_lanes(F4);
    const int64_t groups_per_block = kBlock / q.lanes;
    int64_t blocks = (most + groups_per_block - 1) / groups_per_block;
    // Beyond that a group visits several rows, which its pipeline wants anyway.  Four blocks a CU, where three or four are resident: a
    // larger grid is no faster alone and 7 % slower next to another stream's kernels.  Rows of one column a lane are over sooner and read
    // from the L2s, and there it is waves that count: as many as are resident, eight of four lanes a row, and six of eight with six source
    // rows read together (five with eight; seven, of five rows, are the same).  One mini-batch of 78 K rows of F floats, four of them, and four
    // of 21 K, on 1 M, 1 M and 100 K nodes, us with four blocks and so: F = 8 6.0 -> 5.1, 13.1 -> 12.1, 7.8 -> 7.8; F = 16 6.2 -> 5.4,
    // 13.5 -> 12.6, 7.8 -> 7.8; F = 20 7.0 -> 6.6, 20.0 -> 19.2, 13.5 -> 10.8; F = 32 6.6 -> 6.5, 18.0 -> 18.1, 12.7 -> 10.8.  (12.6 K rows of
    // up to 15 edges, F = 20 to 32: 4.1 to 4.6 us, 4.3 to 4.9 with six rows together.)
    const int64_t cap = (int64_t) c->num_cus * (thin ? 16 : q.per > 1 ? 4 : q.lanes == 8 ? 6 : 8);
    if (blocks > cap) blocks = cap;
    if (thin) {
        hipLaunchKernelGGL(k_aggregate_thin, dim3((unsigned) blocks, (unsigned) count), dim3(kBlock), 0, s, a);
        return hipGetLastError();
    }
    const int64_t windows = ((int64_t) feat_dim + kAggWindow - 1) / kAggWindow, most_windows = 65535;      // of a grid
    for (int64_t w = 0; w < windows; w += most_windows) {
        a.first_window = (uint32_t) w;
        const dim3 grid((unsigned) blocks, (unsigned) count, (unsigned) std::min(windows - w, most_windows));
        aggregate_dispatch(q, feat_dim == 4 * q.lanes * q.per, quotient, grid, s, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace gns
