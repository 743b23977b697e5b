// Small mini-batches (a node or a few tens of them, as online inference asks for): all layers in one launch, a block per
// mini-batch.
//
// The sequence of launches in gns_sampler.hip and gns_frontier.hip spends its time between launches and on their chains of
// reads when there is next to nothing to sample: what one launch leaves the next finds in memory.  Here a batch's nodes,
// their local ids and the draws stay in the LDS of one block, and only the graph is read from memory: seeds -> extents ->
// (chunk records) -> drawn entries -> extents of the new nodes -> ...  The results are those of the other path: draws
// keyed by (seed, layer, node, slot), rows' edges in CSR order, new nodes in ascending order of their ids.
// No block waits for another.
#include <string.h>
#include "gns_kernels.hpp"

namespace gns {

constexpr int kSmallPer = 4;                     // slots per thread at most
constexpr int kSmallFanout = 16;
constexpr int kSmallFew = 128;                   // new nodes of a layer that are put in order by comparison with one another
constexpr int kSmallBlocks = 48;                 // layers of all mini-batches of a launch

struct SmallSlot {
    DeviceState* st;
    DeviceState* host;
    const int32_t* seeds;
    int32_t num_seeds;
    int32_t bad;                                 // there are more seeds than nodes
    uint32_t key0, key1;
    uint32_t batch_id, stamp;
    int32_t cache_gen;
};

struct SmallArgs {
    SampleArgs s;                                // graph and cache (generation 0); nothing else of it is used
    const void* g_indptr;
    int32_t g_i64;
    int32_t num_layers;
    int64_t num_nodes;
    uint64_t cache_block_bytes;
    int8_t fanout[GNS_MAX_LAYERS];
    int8_t policy[GNS_MAX_LAYERS];
    SmallSlot b[kMaxGroup];
    BlockPtrs blk[kSmallBlocks];                 // batch b's layer i: blk[b * num_layers + i]
};

// What a block of kThreads threads takes: a row per thread, kSmallPer slots, two and a half nodes.
template <int kThreads>
struct SmallLds {
    static constexpr int kRows = kThreads, kSlots = kSmallPer * kThreads, kNodes = 5 * kThreads / 2, kHash = 4 * kThreads, kBuckets = kThreads;
    union {
        alignas(16) uint32_t slot[kSlots];       // Philox words, then the chosen ranks (top bit: of the fill; ~0: none)
        uint32_t sorted[kNodes];                 // when those have been fetched: the new nodes by bucket
    };
    union {
        int64_t place[kSlots];                   // where a slot's entry is read, -1: nowhere
        uint32_t node[kSlots];                   //   and then which node it is
    };
    int64_t start[kRows];                        // CSR extents of the rows
    uint32_t deg[kRows];
    uint32_t key[kHash];                         // node -> local id, open addressing; ~0: empty
    uint32_t list[kNodes];                       // the batch's nodes by local id
    uint32_t first[kRows], here[kRows], tile[kRows];         // CachedList
    float scale[kRows], fill_w[kRows];
    int32_t count[kRows];                        // entries drawn from the list, and in all << 8
    int32_t offset[kRows];                       // the block's indptr
    uint32_t fresh[kNodes];                      // new nodes of the layer as they turn up
    int32_t bucket[kBuckets + 1];
    int32_t sums[kThreads / kWave];
    uint32_t lows[kThreads / kWave], highs[kThreads / kWave];
    uint16_t local[kHash];
    uint16_t fresh_place[kNodes];                // and their places in the hash
    uint16_t edge[kSlots];                       // slot -> edge of the block
    uint16_t edge_place[kSlots];                 // edge -> its node's place in the hash
    int32_t fresh_count;
    int32_t bad;
};
static_assert(sizeof(SmallLds<1024>) <= kLdsBitmapBytes, "one block's LDS");

// Exclusive scan over the block; *total receives the sum in every thread.
template <int kThreads>
__device__ __forceinline__ int32_t small_scan(int32_t v, int32_t* sums, int32_t* total)
{
    constexpr int kWaves = kThreads / kWave;
    const int lane = opaque_lane_id(), wave = opaque((int) (threadIdx.x >> 6));
    const int32_t incl = wave_inclusive_scan(v);
    __syncthreads();                             // sums may still be read from a previous call
    if (lane == kWave - 1) sums[wave] = incl;
    __syncthreads();
    const int32_t mine = sums[lane & (kWaves - 1)];
    int32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const int32_t x = __builtin_amdgcn_readlane(mine, w);
        if (w < wave) before += x;
        all += x;
    }
    *total = all;
    return before + incl - v;
}

// Finds or enters node u; *fresh says whether it was not there.
template <int kHash>
__device__ __forceinline__ uint32_t small_enter(uint32_t* keys, uint32_t u, bool* fresh)
{
    uint32_t h = (u * 0x9E3779B1u) >> 16 & (kHash - 1);
    for (;;) {                                   // a third of the places stay empty
        const uint32_t old = atomicCAS(&keys[h], ~0u, u);
        if (old == ~0u || old == u) { *fresh = old == ~0u; return h; }
        h = (h + 1) & (kHash - 1);
    }
}

// The code is kept short (loops over turns are not unrolled but where their reads have to be in flight together): a launch of
// a dozen microseconds fetches every line of it for the first time.
template <int kThreads>
__global__ void __launch_bounds__(kThreads) k_sample_small(SmallArgs g)
{
    extern __shared__ uint4 small_lds[];
    using Lds = SmallLds<kThreads>;
    Lds& w = *reinterpret_cast<Lds*>(small_lds);
    const SmallSlot q = g.b[blockIdx.x];
    SampleArgs a = g.s;
    if (q.cache_gen) {
        auto shift = [&](auto*& ptr) {
            if (ptr) ptr = reinterpret_cast<std::remove_reference_t<decltype(ptr)>>(reinterpret_cast<uintptr_t>(ptr) + g.cache_block_bytes);
        };
        shift(a.node_inv_pc);
        shift(a.node_slot);
        shift(a.srec);
        shift(a.s_nodes);
        shift(a.s_count);
    }
    const int tid = (int) threadIdx.x;
    auto extent = [&](int64_t u, int64_t* start, uint32_t* deg) {
        const int64_t b = load_off_rt(g.g_indptr, g.g_i64, u), e = load_off_rt(g.g_indptr, g.g_i64, u + 1);
        *start = b;
        *deg = (uint32_t) (e - b);
    };
    // ---- the seeds
    int32_t R = q.num_seeds;
    {
        const int32_t u = tid < R ? q.seeds[tid] : -1;
        const bool valid = u >= 0 && (int64_t) u < g.num_nodes;
        int64_t start = 0;
        uint32_t deg = 0;
        if (valid) extent(u, &start, &deg);
        for (int i = tid; i < Lds::kHash; i += kThreads) w.key[i] = ~0u;
        if (tid == 0) { w.fresh_count = 0; w.bad = q.bad; }
        __syncthreads();
        if (tid < R) {
            w.list[tid] = (uint32_t) u;
            w.start[tid] = start;
            w.deg[tid] = deg;
            bool fresh = false;
            if (valid) {
                const uint32_t h = small_enter<Lds::kHash>(w.key, (uint32_t) u, &fresh);
                if (fresh) w.local[h] = (uint16_t) tid;
            }
            if (!fresh) w.bad = 1;               // out of range, or repeated
        }
        __syncthreads();
    }
    auto publish_state = [&](uint32_t bad_seed) {                // one thread: what later calls read of this batch
        q.st->key0 = q.key0;
        q.st->key1 = q.key1;
        q.st->stamp = q.stamp;
        q.st->batch_id = q.batch_id;
        q.st->cache_gen = q.cache_gen;
        if (bad_seed) q.st->bad_seed = bad_seed;
        q.host->bad_seed = bad_seed ? bad_seed : q.st->bad_seed;
    };
    // Repeated and invalid seeds are rows beside the graph's nodes, for which neither the arrays here nor the block buffers
    // have room: such a batch ends empty.
    if (w.bad) {
        if (tid <= g.num_layers) q.st->num_dst[tid] = q.host->num_dst[tid] = 0;
        if (tid < g.num_layers) q.st->num_edges[tid] = q.host->num_edges[tid] = 0;
        if (tid == 0) publish_state(q.batch_id);
        return;
    }
    for (int layer = 0; layer < g.num_layers; ++layer) {
        const BlockPtrs out = g.blk[(int) blockIdx.x * g.num_layers + layer];
        const int k = g.fanout[layer], k4 = (k + 3) & ~3, blocks = k4 >> 2;
        const int policy = g.policy[layer];
        const bool last = layer == g.num_layers - 1;
        const uint32_t inv_k = 65535u / (uint32_t) k + 1u;       // t / k = t * inv_k >> 16, exact for t < 4096
        a.fanout = k;
        const uint32_t layer_number = (uint32_t) (g.num_layers - layer);
        // ---- rows: what they draw from, and the Philox words of all their slots over all threads
        uint32_t m = 0, others = 0;
        int cnt = 0, fill = 0;
        CachedList c = {0u, 0u, 0u, 0u};
        if (tid < R) {
            others = w.deg[tid];
            if (policy != GNS_UNIFORM) c = cached_list(a, RowExtent{w.start[tid], w.start[tid] + (int64_t) others});
        }
        const int lg = 32 - __builtin_clz((uint32_t) R | 1u);    // R < 1 << lg
        for (int t = tid; t < blocks << lg; t += kThreads) {
            const int r = t & ((1 << lg) - 1), x = t >> lg;
            if (r >= R) continue;
            const Philox4 p = philox4x32_10(w.list[r], (uint32_t) x, layer_number, kTagNeighbor, q.key0, q.key1);
            *reinterpret_cast<uint4*>(&w.slot[r * k4 + 4 * x]) = make_uint4(p.w[0], p.w[1], p.w[2], p.w[3]);
        }
        if (tid < R) {
            m = policy == GNS_UNIFORM ? others : c.count;
            others -= m;
            cnt = m > (uint32_t) k ? k : (int) m;
            const uint32_t room = (uint32_t) (k - cnt);
            fill = policy != GNS_CACHE_FIRST ? 0 : others > room ? (int) room : (int) others;
            w.first[tid] = c.first; w.here[tid] = c.here; w.tile[tid] = c.tile;
            w.scale[tid] = cached_scale(a, m, cnt);
            w.fill_w[tid] = fill_weight(a, others, fill);
            w.count[tid] = cnt | (cnt + fill) << 8;
        }
        int32_t edges;
        const int32_t off = small_scan<kThreads>(cnt + fill, w.sums, &edges);
        // ---- Floyd's draw, a row per thread (see sample_wave_rows)
        if (tid < R) {
            w.offset[tid] = off;
            out.indptr[tid] = off;
            out.row_eligible[tid] = (int32_t) m;
            out.src_nodes[tid] = (int32_t) w.list[tid];
            const uint32_t room = (uint32_t) (k - cnt);
            const bool draw = m > (uint32_t) k, draw_fill = others > room;
            uint32_t chosen[kSmallFanout];
#pragma unroll
            for (int x = 0; x < kSmallFanout / 4; ++x) {
                uint4 q4 = make_uint4(0u, 0u, 0u, 0u);
                if (x < blocks) q4 = *reinterpret_cast<const uint4*>(&w.slot[tid * k4 + 4 * x]);
                chosen[4 * x] = q4.x; chosen[4 * x + 1] = q4.y; chosen[4 * x + 2] = q4.z; chosen[4 * x + 3] = q4.w;
            }
#pragma unroll
            for (int s = 0; s < kSmallFanout; ++s) {
                if (s >= k) { chosen[s] = 0xFFFFFFFFu; continue; }       // (k is the same for all)
                const bool from_fill = s >= cnt;
                const uint32_t i = (uint32_t) (s - cnt);
                const uint32_t j = from_fill ? others - room + i : m - (uint32_t) k + (uint32_t) s, top = from_fill ? 0x80000000u : 0u;
                const uint32_t t = __umulhi(chosen[s], j + 1u) | top;
                bool dup = false;
#pragma unroll
                for (int p = 0; p < s; ++p) dup = dup || chosen[p] == t;
                uint32_t x = dup ? j | top : t;
                if (from_fill ? !draw_fill : !draw) x = from_fill ? i | top : (uint32_t) s;
                chosen[s] = s < cnt + fill ? x : 0xFFFFFFFFu;
            }
#pragma unroll
            for (int x = 0; x < kSmallFanout / 4; ++x)
                if (x < blocks)
                    *reinterpret_cast<uint4*>(&w.slot[tid * k4 + 4 * x]) = make_uint4(chosen[4 * x], chosen[4 * x + 1], chosen[4 * x + 2], chosen[4 * x + 3]);
        }
        __syncthreads();
        // ---- fetch: one drawn entry per thread and turn
        const int items = R * k;
#pragma unroll 1
        for (int t = tid; t < items; t += kThreads) {
            const int r = (int) ((uint32_t) t * inv_k >> 16), s = t - r * k;
            const int counts = w.count[r];
            int64_t place = -1;
            if (s < counts >> 8) {
                const uint32_t rank = w.slot[r * k4 + s];
                int pos = 0;
#pragma unroll
                for (int x = 0; x < kSmallFanout / 4; ++x) {
                    if (x >= blocks) break;
                    const uint4 o = *reinterpret_cast<const uint4*>(&w.slot[r * k4 + 4 * x]);
                    pos += (o.x < rank ? 1 : 0) + (o.y < rank ? 1 : 0) + (o.z < rank ? 1 : 0) + (o.w < rank ? 1 : 0);
                }
                w.edge[t] = (uint16_t) (w.offset[r] + pos);
                if (policy == GNS_UNIFORM) place = w.start[r] + (int64_t) rank;
                else if (s >= (counts & 255)) place = uncached_entry(a, RowExtent{w.start[r], w.start[r] + (int64_t) w.deg[r]}, rank & 0x7FFFFFFFu);
                else if (rank >= w.here[r]) place = later_tile(a, CachedList{w.first[r], w.here[r], 0u, w.tile[r]}, rank);
                else place = (int64_t) (w.first[r] + rank);
            }
            w.place[t] = place;
        }
        uint32_t u[kSmallPer];
        float weight[kSmallPer];
        bool mine[kSmallPer];
#pragma unroll
        for (int i = 0; i < kSmallPer; ++i) {
            const int t = i * kThreads + tid;
            mine[i] = false;
            if (i * kThreads >= items || t >= items) continue;
            const int64_t place = w.place[t];                    // this thread has put it there
            mine[i] = place >= 0;
            const int r = (int) ((uint32_t) t * inv_k >> 16);
            const bool of_row = policy == GNS_UNIFORM || t - r * k >= (w.count[r] & 255);
            if (mine[i]) u[i] = (uint32_t) (of_row ? a.indices : a.s_nodes)[place];
            weight[i] = policy == GNS_UNIFORM ? 1.0f : of_row ? w.fill_w[r] : w.scale[r];
        }
        if (policy != GNS_UNIFORM) {
#pragma unroll
            for (int i = 0; i < kSmallPer; ++i) {
                const int t = i * kThreads + tid;
                if (i * kThreads >= items || !mine[i]) continue;
                const int r = (int) ((uint32_t) t * inv_k >> 16);
                if (t - r * k < (w.count[r] & 255)) weight[i] *= cached_node(a, u[i]).inv_pc;
            }
        }
        __syncthreads();                                         // places and nodes share their memory
#pragma unroll
        for (int i = 0; i < kSmallPer; ++i)
            if (i * kThreads < items && i * kThreads + tid < items) w.node[i * kThreads + tid] = mine[i] ? u[i] : ~0u;
#pragma unroll 1
        for (int t0 = 0; t0 < items; t0 += kThreads) {
            const int t = t0 + tid;
            const uint32_t node = t < items ? w.node[t] : ~0u;
            bool fresh = false;
            uint32_t h = 0u;
            if (node != ~0u) {
                h = small_enter<Lds::kHash>(w.key, node, &fresh);
                w.edge_place[w.edge[t]] = (uint16_t) h;
            }
            const uint64_t all = __ballot(fresh);
            if (all) {
                const int lane = opaque_lane_id(), leader = __builtin_ctzll(all);
                int at = 0;
                if (lane == leader) at = atomicAdd(&w.fresh_count, (int) __popcll(all));
                at = __builtin_amdgcn_readlane(at, leader) + __popcll(all & ((1ull << lane) - 1ull));
                if (fresh) {
                    w.fresh[at] = node;
                    w.fresh_place[at] = (uint16_t) h;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < kSmallPer; ++i)
            if (i * kThreads < items && mine[i]) out.weights[w.edge[i * kThreads + tid]] = weight[i];
        __syncthreads();
        // ---- union: the new nodes in ascending order.  A few by comparison with all, more by buckets of equal ranges of ids and
        // comparison within a bucket.
        const int M = w.fresh_count;
        const bool few = M <= kSmallFew;
        uint32_t low = ~0u;
        int shift = 0;
        if (!few) {
            uint32_t high = 0u;
            for (int j = tid; j < M; j += kThreads) {
                const uint32_t id = w.fresh[j];
                low = id < low ? id : low;
                high = id > high ? id : high;
            }
#pragma unroll
            for (int x = kWave / 2; x > 0; x >>= 1) {
                const uint32_t l = (uint32_t) __shfl_xor((int) low, x, kWave), h = (uint32_t) __shfl_xor((int) high, x, kWave);
                low = l < low ? l : low;
                high = h > high ? h : high;
            }
            if (opaque_lane_id() == 0) { w.lows[tid >> 6] = low; w.highs[tid >> 6] = high; }
            w.bucket[tid] = 0;
            __syncthreads();
#pragma unroll
            for (int x = 0; x < kThreads / kWave; ++x) {
                low = w.lows[x] < low ? w.lows[x] : low;
                high = w.highs[x] > high ? w.highs[x] : high;
            }
            constexpr int kBucketBits = 31 - __builtin_clz((unsigned) Lds::kBuckets);
            const int bits = 32 - __builtin_clz((high - low) | 1u);
            shift = bits > kBucketBits ? bits - kBucketBits : 0;
            int32_t arrival[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const int j = i * kThreads + tid;
                if (j < M) arrival[i] = atomicAdd(&w.bucket[(w.fresh[j] - low) >> shift], 1);
            }
            __syncthreads();
            int32_t all;
            const int32_t begin = small_scan<kThreads>(w.bucket[tid], w.sums, &all);
            w.bucket[tid] = begin;
            if (tid == 0) w.bucket[Lds::kBuckets] = all;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                const int j = i * kThreads + tid;
                if (j < M) w.sorted[w.bucket[(w.fresh[j] - low) >> shift] + arrival[i]] = w.fresh[j];
            }
            __syncthreads();
        }
#pragma unroll 1
        for (int j = tid; j < M; j += kThreads) {
            const uint32_t id = w.fresh[j];
            int64_t start = 0;
            uint32_t deg = 0;
            if (!last) extent((int64_t) id, &start, &deg);       // it is a row of the next layer
            int pos = 0, end = M;
            const uint32_t* with = w.fresh;
            if (!few) {
                const int x = (int) ((id - low) >> shift);
                pos = w.bucket[x];
                end = w.bucket[x + 1];
                with = w.sorted;
            }
#pragma unroll 8
            for (int p = pos; p < end; ++p) pos += with[p] < id ? 1 : 0;
            const int local = R + pos;
            w.local[w.fresh_place[j]] = (uint16_t) local;
            w.list[local] = id;
            out.src_nodes[local] = (int32_t) id;
            if (!last) { w.start[local] = start; w.deg[local] = deg; }
        }
        if (tid == 0) {
            out.indptr[R] = edges;
            q.st->num_dst[layer] = q.host->num_dst[layer] = R;
            q.st->num_edges[layer] = q.host->num_edges[layer] = edges;
        }
        __syncthreads();
        // ---- relabel
        if (tid == 0) w.fresh_count = 0;
        for (int e = tid; e < edges; e += kThreads) out.indices[e] = (int32_t) w.local[w.edge_place[e]];
        R += M;
    }
    if (tid == 0) {
        q.st->num_dst[g.num_layers] = q.host->num_dst[g.num_layers] = R;
        publish_state(0);
    }
}

// Whether the worst case of the group's seeds fits blocks of kThreads threads.  That of distinct seeds, whose batch has no more
// nodes than the graph; of others the kernel enters the seeds only.
template <int kThreads>
static bool small_fits(const Group& g, const BeginDyn& d)
{
    using Lds = SmallLds<kThreads>;
    const gns_ctx* c = g.ctx[0];
    for (int b = 0; b < g.count; ++b) {
        int64_t rows = d.num_seeds[b];
        for (int i = 0; i < c->config.num_layers; ++i) {
            const int k = c->config.fanout[i], k4 = (k + 3) & ~3;
            if (rows > Lds::kRows || rows * k4 > Lds::kSlots) return false;
            rows += rows * k;
            if (rows > c->graph.num_nodes) rows = c->graph.num_nodes;
        }
        if (rows > Lds::kNodes) return false;
    }
    return true;
}

// The line: every layer's rows are a thread each, its slots (fan-outs rounded up to Philox blocks) four, and the batch's
// nodes two and a half: what one CU's LDS holds.  Up to there a block is ahead of the sequence of launches; gns_sample_blocks with fan-outs
// 10, 5 on 10 K nodes takes 26.7 us for one seed (launches: 41.3), 33.5 for 31 (43.4), with 15, 10, 5 and one seed 37.0 on 1 M
// nodes (56.7) and 34.5 on 40 M (58.8).
bool small_batches(const Group& g, const BeginDyn& d)
{
    const gns_ctx* c = g.ctx[0];
    const int nl = c->config.num_layers;
    if (g.count * nl > kSmallBlocks || c->lds_bitmap_limit < kLdsBitmapBytes) return false;
    for (int i = 0; i < nl; ++i)
        if (!direct_layer(c->config, i) || c->config.fanout[i] > kSmallFanout) return false;
    return small_fits<1024>(g, d);
}

hipError_t launch_small(const Group& g, const BeginDyn& d, hipStream_t s)
{
    gns_ctx* c = g.ctx[0];
    const int nl = c->config.num_layers;
    SmallArgs a;
    memset(&a, 0, sizeof(a));
    fill_sample_template(c, 0, &a.s);
    a.g_indptr = c->graph.indptr;
    a.g_i64 = c->graph.indptr_is_i64;
    a.num_layers = nl;
    a.num_nodes = c->graph.num_nodes;
    a.cache_block_bytes = c->uses_cache ? c->lay.cache_block_bytes : 0;
    for (int i = 0; i < nl; ++i) {
        a.fanout[i] = (int8_t) c->config.fanout[i];
        a.policy[i] = (int8_t) c->config.policy[i];
    }
    for (int b = 0; b < g.count; ++b) {
        SmallSlot& q = a.b[b];
        q.st = g.ctx[b]->d_state;
        q.host = g.ctx[b]->h_state_dev;
        q.seeds = d.seeds[b];
        q.num_seeds = d.num_seeds[b];
        q.bad = (int32_t) (d.too_many >> b & 1u);
        q.key0 = d.key0[b];
        q.key1 = d.key1[b];
        q.batch_id = d.batch_id[b];
        q.stamp = d.stamp[b];
        q.cache_gen = d.cache_gen[b];
        for (int i = 0; i < nl; ++i) a.blk[b * nl + i] = block_ptrs(g.blocks[b][i]);
    }
    const dim3 grid((unsigned) g.count);
    if (small_fits<256>(g, d)) hipLaunchKernelGGL(k_sample_small<256>, grid, dim3(256), sizeof(SmallLds<256>), s, a);
    else                       hipLaunchKernelGGL(k_sample_small<1024>, grid, dim3(1024), sizeof(SmallLds<1024>), s, a);
    return hipGetLastError();
}

}  // namespace gns
