// Kernel argument blocks and device bodies shared between the sampler and the frontier kernels.
//
// One launch serves a *group* of up to kMaxGroup independent mini-batches (mini-batches are independent
// given the cache: the paper's sampling workers, Section 3.3): group_block says which of them a block
// works for.  A launch's arguments are one LayerArgs: templates of the per-batch argument structs holding
// everything the batches have in common (graph, cache, layer constants), the offsets of the sections of a
// context's per-batch scratch, and one BatchSlot per batch (where its scratch lies, its block buffers).
// Every kernel first binds the templates to its own batch.
#pragma once
#include <type_traits>
#include "gns_internal.h"
#include "gns_device.hpp"

namespace gns {

constexpr int kMaxGroup = GNS_MAX_GROUP;

// One record per aligned 64-entry chunk of the CSR entry array (GNS_FLAGS_PER_CACHE).
struct alignas(16) ChunkRec {
    uint64_t flags;            // bit e & 63: entry e points into the cache
    uint32_t before;           // place in s_nodes of the first of them
    uint32_t pad;
};

// Which node has which local id in the current mini-batch: one 32-bit entry per node of the graph, the batch's stamp in
// the upper bits and the local id in the lower `shift` ones.  An entry of another batch carries another stamp, so
// nothing is cleared between batches (the host clears the table when the stamps run out), a node is entered with a
// plain store and found with one read.
struct NodeTable {
    uint32_t* entry;           // [n]
    uint32_t stamp;
    int shift;

    __device__ __forceinline__ uint32_t make(uint32_t local) const { return (stamp << shift) | local; }
    __device__ __forceinline__ bool current(uint32_t e) const { return (e >> shift) == stamp; }
    __device__ __forceinline__ uint32_t local(uint32_t e) const { return e & ((1u << shift) - 1u); }
};

// The cache filter in LDS: CacheFilter::groups, then the tags, as they stand in memory.
__device__ __forceinline__ void stage_filter(uint4* lds, const uint32_t* groups)
{
    stage_lds(lds, reinterpret_cast<const uint4*>(groups), kFilterGroups / 128 + kFilterHot / 8);
}

// What it says of nodes u[0 .. N): ~0 cached, 0 not, 1: to be looked up.  All reads first: left to itself the compiler puts the
// second of a node behind the outcome of the first and waits for each.
template <int N>
__device__ __forceinline__ void filter_test(const uint32_t* lds32, uint32_t mult, const uint32_t* u, uint32_t* w)
{
    const uint16_t* tags = reinterpret_cast<const uint16_t*>(lds32 + kFilterGroups / 32);
    uint32_t tag[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        w[i] = lds32[__umulhi(u[i], mult) >> 5];
        tag[i] = tags[u[i] % kFilterHot];
    }
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+v"(w[i]), "+v"(tag[i]));
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] = tag[i] == u[i] / kFilterHot + 1u ? ~0u : (w[i] >> (__umulhi(u[i], mult) & 31u)) & 1u;
}

struct SampleArgs {
    DeviceState* st;
    int layer_index;
    uint32_t layer_number;     // the paper's l = L - layer_index
    int fanout;
    int wmode;
    int policy;                // GNS_CACHE_ONLY or GNS_CACHE_FIRST for the select kernel
    const int32_t* indices;
    const int32_t* dst_nodes;
    RowExtent* row_ext;        // CSR extent of every dst row's node (written when the node joined the batch)
    const float* node_inv_pc;  // 1 / p^C_u for the nodes of the cache, or
    const CachedNode* node_slot;     //   that and their slots (the other is null)
    int by_slot;               // the layer's new nodes are marked in slot_mark
    uint8_t* slot_mark;        // [slots of the cache]
    int32_t* hub_rows;         // rows of the layer whose CSR segment spans more than kHubChunks chunks
    const uint64_t* cache_bitmap;
    int32_t* s_nbr;
    float* s_w;
    int32_t* s_cnt;
    int32_t* sums_rows;        // sampled neighbors of the rows of every block of the sampler
    int32_t* row_eligible;
    int32_t* src_nodes;        // the layer's src list begins with its dst nodes
    uint64_t* mark;
    uint64_t* mark_summary;    // one bit per word of mark, or null (small graphs)
    NodeTable tab;             // holds this layer's dst nodes
    // CACHE_ONLY: per-batch plan and the CSR-aligned membership flags
    int64_t num_entries;
    unsigned long long* plan_sums;   // [row tiles] (tag, chunks of the tile), see sum_before
    int32_t* plan_desc;        // [max_chunks] ids of the aligned chunks to flag
    uint32_t max_chunks;       // what the chunks of distinct rows come to at most
    uint64_t* flags;           // [ceil(nnz / 64)] bit e & 63 of word e >> 6: entry e points into the cache
    int64_t bitmap_words;
    const uint32_t* filter_groups;   // CacheFilter::groups with the tags behind them, and its mult (flag kernel, mode 2)
    uint32_t filter_mult;
    const uint64_t* coarse_bitmap;   // one bit per 2^coarse_shift ids (mode 3)
    int coarse_shift;
    const ChunkRec* srec;      // induced subgraph (GNS_FLAGS_PER_CACHE): chunk records and the cached entries' node ids
    const int32_t* s_nodes;
    const int32_t* s_count;    // cached entries of every tile of 2^s_tile_shift entries
    int s_tile_shift;
};

// Marks of 64 slots, and the marks before them.
struct alignas(16) SlotWord {
    uint64_t bits;
    int32_t before;
    int32_t pad;

    __device__ __forceinline__ int32_t rank(uint32_t slot) const { return before + __popcll(bits & ((1ull << (slot & 63u)) - 1ull)); }
};

struct FinishArgs {
    DeviceState* st;
    int layer_index;
    int fanout;
    double inv_fanout;
    int unit_weights;              // UNIFORM layers: every weight is 1 and s_w is not used
    const int32_t* s_nbr;          // [R x fanout]
    const float* s_w;              // [R x fanout]
    const int32_t* s_cnt;          // [R]
    const int32_t* sums_rows;      // sampled neighbors of every rows_per_sum consecutive rows
    int32_t rows_per_sum;          //   (a power of two up to kTile; 0: the sampler does not leave them)
    unsigned long long* row_sums;  // [row tiles] (tag, sampled neighbors of the tile's rows) for those
    uint64_t* mark;                // [words]
    uint64_t* mark_summary;        // [ceil(words / 64)] or null: bit w & 63 of word w >> 6 says mark[w] != 0
    int marks_seeds;               // first layer sampled in the launch that enters the seeds: it marks them like any node,
    const uint64_t* seed_mark;     //   and this bitmap of the seeds tells them apart (null otherwise)
    int64_t words;
    NodeTable tab;
    unsigned long long* tile_sums; // [mark_tiles] (tag, new nodes of the tile), see sum_before
    int32_t row_tiles_max;         // grid split point: blocks [0, row_tiles_max) work on rows
    int32_t mark_tiles;            // tiles of mark_tile_words bitmap words
    int32_t mark_tile_words;
    int32_t* indptr;               // block outputs
    int32_t* indices;
    float* weights;
    int32_t* src_nodes;
    RowExtent* row_ext;            // [nodes of the batch] the union step appends the new nodes' CSR extents
    const void* g_indptr;          // the graph's offsets
    int g_i64;
    int64_t num_nodes;
    int32_t last_layer;            // its new nodes have no rows to be sampled
    int32_t max_src;               // places of the layer's src list and of row_ext
    int by_slot;                   // the layer's new nodes are marked by slots of the cache
    int32_t slots;                 //   their number, rounded up to whole words of marks
    int32_t slot_tile;             //   slots of a tile (then tiles are of slots, not of bitmap words)
    uint8_t* slot_mark;            //   [slots]
    SlotWord* slot_words;          //   [slots / 64] written by the union step for the relabel
    const int32_t* cache_nodes;    //   the cached nodes by slot
};

// Byte offsets of the sections of a context's per-batch scratch (the same for every context of a family).
struct WsOffsets {
    uint64_t state, mark, mark_summary, seed_mark, seed_copy, row_ext, hub_rows;
    uint64_t table;
    uint64_t s_nbr[2], s_w[2], s_cnt[2];
    uint64_t plan_desc;            // where slot_marks is not 0: the marks by slot
    uint64_t slot_marks;           // bytes of them
    uint64_t sums_rows, tile_sums, row_sums, plan_sums;
    uint64_t cache_block_bytes;    // distance between the two copies of what a cache draw writes
    int32_t uses_cache;
    int32_t has_summary;
    int32_t table_shift;
    int32_t marks_seeds;           // the first layer's launch fills the seed bitmap
};

struct BlockPtrs {
    int32_t* indptr;
    int32_t* indices;
    int32_t* src_nodes;
    int32_t* row_eligible;
    float* weights;
};

static inline BlockPtrs block_ptrs(const gns_block& k)
{
    BlockPtrs p;
    p.indptr = k.indptr; p.indices = k.indices; p.src_nodes = k.src_nodes; p.row_eligible = k.row_eligible; p.weights = k.weights;
    return p;
}

// What differs between the mini-batches of a group.
struct BatchSlot {
    char* ws;                  // the batch's context: its per-batch scratch
    DeviceState* host;         //   and its pinned host mirror
    const int32_t* dst;        // dst nodes of the layer being sampled / finished
    BlockPtrs cur, prev;       // block buffers of that layer and of the one before it
};

struct LayerArgs {
    SampleArgs s;              // template: cache pointers are those of cache generation 0
    FinishArgs f;              // template for the layer the launch finishes or relabels
    WsOffsets off;
    int32_t dealt;             // see group_block
    int32_t blocks;            // blocks of the launch per batch (the first launch's kernels need no such bound)
    BatchSlot b[kMaxGroup];
};

// What changes from one replay of a group's launch sequence to the next (arguments of the first kernel).
struct BeginDyn {
    const int32_t* seeds[kMaxGroup];
    int32_t num_seeds[kMaxGroup];  // no more than the graph has nodes: the buffers have no room for more rows
    uint32_t too_many;             // bit b: there were more, so that some of them are bad
    uint32_t key0[kMaxGroup], key1[kMaxGroup];
    uint32_t batch_id[kMaxGroup];
    uint32_t stamp[kMaxGroup];     // what the batch's entries of the node table carry
    int32_t cache_gen[kMaxGroup];  // which copy of the cache structures it reads
};

// What the words by which the blocks of a launch pass sums on carry (see sum_before): one value per mini-batch and layer.
__device__ __forceinline__ uint32_t launch_tag(const DeviceState* st, int layer_index)
{
    return st->batch_id * GNS_MAX_LAYERS + (uint32_t) layer_index;
}

template <typename T>
__device__ __forceinline__ T* at(char* base, uint64_t off) { return reinterpret_cast<T*>(base + off); }

__device__ __forceinline__ DeviceState* bind_state(const LayerArgs& g, int b)
{
    return at<DeviceState>(g.b[b].ws, g.off.state);
}

__device__ __forceinline__ NodeTable bind_table(const LayerArgs& g, int b, uint32_t stamp)
{
    NodeTable t;
    t.entry = at<uint32_t>(g.b[b].ws, g.off.table);
    t.stamp = stamp;
    t.shift = g.off.table_shift;
    return t;
}

// The sampler's arguments for batch b of the group, given the batch's stamp and cache generation (left in its device
// state by its first kernel, which has them as arguments).
__device__ __forceinline__ SampleArgs bind_sample(const LayerArgs& g, int b, uint32_t stamp, int cache_gen)
{
    SampleArgs a = g.s;
    const BatchSlot& q = g.b[b];
    char* ws = q.ws;
    a.st = at<DeviceState>(ws, g.off.state);
    const uint64_t gen_shift = cache_gen ? g.off.cache_block_bytes : 0;
    const int par = g.s.layer_index & 1;             // sampler scratch is double-buffered by layer parity
    a.dst_nodes = q.dst;
    a.row_ext = at<RowExtent>(ws, g.off.row_ext);
    a.hub_rows = at<int32_t>(ws, g.off.hub_rows);
    a.s_nbr = at<int32_t>(ws, g.off.s_nbr[par]);
    a.s_w = at<float>(ws, g.off.s_w[par]);
    a.s_cnt = at<int32_t>(ws, g.off.s_cnt[par]);
    a.sums_rows = at<int32_t>(ws, g.off.sums_rows);
    a.row_eligible = q.cur.row_eligible;
    a.src_nodes = q.cur.src_nodes;
    a.mark = at<uint64_t>(ws, g.off.mark);
    a.mark_summary = g.off.has_summary ? at<uint64_t>(ws, g.off.mark_summary) : nullptr;
    a.tab = bind_table(g, b, stamp);
    a.plan_sums = at<unsigned long long>(ws, g.off.plan_sums);
    a.plan_desc = at<int32_t>(ws, g.off.plan_desc);
    a.slot_mark = at<uint8_t>(ws, g.off.plan_desc);
    if (g.off.uses_cache) {
        auto shifted = [&](auto* ptr) {
            return ptr ? reinterpret_cast<decltype(ptr)>(reinterpret_cast<uintptr_t>(ptr) + gen_shift) : ptr;
        };
        a.node_inv_pc = shifted(g.s.node_inv_pc);
        a.node_slot = shifted(g.s.node_slot);
        a.cache_bitmap = shifted(g.s.cache_bitmap);
        a.flags = shifted(g.s.flags);
        a.filter_groups = shifted(g.s.filter_groups);
        a.coarse_bitmap = shifted(g.s.coarse_bitmap);
        a.srec = shifted(g.s.srec);
        a.s_nodes = shifted(g.s.s_nodes);
        a.s_count = shifted(g.s.s_count);
    }
    return a;
}

__device__ __forceinline__ SampleArgs bind_sample(const LayerArgs& g, int b)
{
    const DeviceState* st = bind_state(g, b);
    return bind_sample(g, b, st->stamp, st->cache_gen);
}

// The union / relabel arguments of batch b for the layer the template describes: the launch's own layer
// (own_layer) or the one before it (a relabel riding in the next layer's sampler launch).
__device__ __forceinline__ FinishArgs bind_finish(const LayerArgs& g, int b, bool own_layer)
{
    FinishArgs a = g.f;
    const BatchSlot& q = g.b[b];
    char* ws = q.ws;
    a.st = at<DeviceState>(ws, g.off.state);
    const int par = g.f.layer_index & 1;
    const BlockPtrs& blk = own_layer ? q.cur : q.prev;
    a.s_nbr = at<int32_t>(ws, g.off.s_nbr[par]);
    a.s_w = at<float>(ws, g.off.s_w[par]);
    a.s_cnt = at<int32_t>(ws, g.off.s_cnt[par]);
    a.sums_rows = at<int32_t>(ws, g.off.sums_rows);
    a.mark = at<uint64_t>(ws, g.off.mark);
    a.mark_summary = g.off.has_summary ? at<uint64_t>(ws, g.off.mark_summary) : nullptr;
    a.seed_mark = g.f.marks_seeds ? at<uint64_t>(ws, g.off.seed_mark) : nullptr;
    a.tab = bind_table(g, b, a.st->stamp);
    a.tile_sums = at<unsigned long long>(ws, g.off.tile_sums);
    a.row_sums = at<unsigned long long>(ws, g.off.row_sums);
    a.indptr = blk.indptr;
    a.indices = blk.indices;
    a.weights = blk.weights;
    a.src_nodes = blk.src_nodes;
    a.row_ext = at<RowExtent>(ws, g.off.row_ext);
    if (g.f.by_slot) {
        a.slot_mark = at<uint8_t>(ws, g.off.plan_desc);
        a.slot_words = at<SlotWord>(ws, g.off.plan_desc + g.off.slot_marks);
        a.cache_nodes = reinterpret_cast<const int32_t*>(reinterpret_cast<uintptr_t>(a.cache_nodes) + (a.st->cache_gen ? g.off.cache_block_bytes : 0));
    }
    return a;
}

// ---------------------------------------------------------------------------
// What a row's entries are drawn from: its CSR segment (UNIFORM), its cached neighbors in the induced subgraph
// (CACHE_ONLY), or those first and then the rest of its CSR segment (CACHE_FIRST).
enum { kListRow = 0, kListCached = 1, kListCachedFirst = 2 };

__device__ __forceinline__ uint64_t bits_below(int64_t e)
{
    return (1ull << (e & 63)) - 1ull;
}

// The cached neighbors of one row in the induced subgraph: `count` of them, the first `here` from s_nodes[first] on (all
// of them unless the row crosses a tile), the others from the offsets of tiles tile + 1, tile + 2, ... on.
struct CachedList {
    uint32_t first, here, count, tile;
};

__device__ __forceinline__ CachedList cached_list(const SampleArgs& a, const RowExtent& ext)
{
    CachedList r;
    const bool some = ext.end > ext.start;
    const int64_t start = some ? ext.start : 0, last = some ? ext.end - 1 : 0;
    const ChunkRec rs = a.srec[start >> 6];
    const ChunkRec re = a.srec[last >> 6];
    const uint32_t stop = re.before + (uint32_t) __popcll(re.flags & (bits_below(last) * 2 + 1));
    r.first = rs.before + (uint32_t) __popcll(rs.flags & bits_below(start));
    r.tile = (uint32_t) (start >> a.s_tile_shift);
    r.here = r.count = some ? stop - r.first : 0u;
    const uint32_t last_tile = (uint32_t) (last >> a.s_tile_shift);
    if (r.tile != last_tile) {                       // rare: tiles are much longer than rows
        r.here = r.count = (r.tile << a.s_tile_shift) + (uint32_t) a.s_count[r.tile] - r.first;
        for (uint32_t t = r.tile + 1; t < last_tile; ++t) r.count += (uint32_t) a.s_count[t];
        r.count += stop - (last_tile << a.s_tile_shift);
    }
    return r;
}

// Place in s_nodes of the row's cached neighbor of rank `rank`, here <= rank < count.
__device__ __forceinline__ int64_t later_tile(const SampleArgs& a, const CachedList& r, uint32_t rank)
{
    uint32_t left = rank - r.here, t = r.tile + 1;
    for (;; ++t) {
        const uint32_t n = (uint32_t) a.s_count[t];
        if (left < n) return (int64_t) (t << a.s_tile_shift) + left;
        left -= n;
    }
}

// CSR entry of the row [start, end) that is the `rank`-th among those not in the cache (rank is below their number).
__device__ __forceinline__ int64_t uncached_entry(const SampleArgs& a, const RowExtent& ext, uint32_t rank)
{
    const int64_t first = ext.start >> 6, last = (ext.end - 1) >> 6;
    for (int64_t c = first;; ++c) {
        uint64_t open = ~a.srec[c].flags;
        if (c == first) open &= ~bits_below(ext.start);
        if (c == last) open &= bits_below(ext.end - 1) * 2 + 1;
        const uint32_t n = (uint32_t) __popcll(open);
        if (rank < n || c == last) return (c << 6) + select_bit64(open, (int) rank);
        rank -= n;
    }
}

// What is known of cached node u (slot: only where the context marks by slots).
__device__ __forceinline__ CachedNode cached_node(const SampleArgs& a, uint32_t u)
{
    if (a.node_slot) return a.node_slot[u];
    return {a.node_inv_pc[u], 0};
}

// Section 3.4: coefficient p^C_u * k / min(k, N_C(v)), weight = 1 / coefficient (fp32 from the 1/p^C table on); the factor
// of 1/p^C for a row of m cached neighbors of which cnt are drawn.
__device__ __forceinline__ float cached_scale(const SampleArgs& a, uint32_t m, int cnt)
{
    return a.wmode == GNS_W_UNBIASED ? (float) m / (float) (cnt > 0 ? cnt : 1) : (float) cnt / (float) a.fanout;
}

// Fill neighbors: weight 1 (a node-wise sample), or the inverse inclusion probability of a uniform subset of the
// uncached neighbors in the unbiased mode.
__device__ __forceinline__ float fill_weight(const SampleArgs& a, uint32_t others, int fill)
{
    return a.wmode == GNS_W_UNBIASED ? (float) others / (float) (fill > 0 ? fill : 1) : 1.0f;
}

// ---------------------------------------------------------------------------
// Relabel: every sampled edge of a finished layer gets its neighbor's local id (from the scratch slot if the sampler
// already found one, else from the node table) and is compacted to its CSR position.  `block` of `nblocks` blocks of
// kBlock threads, kRelabelUnroll slots per thread in flight.  It only needs that layer's union step, so it shares a
// launch with the next layer's first kernel.
constexpr int kRelabelUnroll = 4;

__device__ __forceinline__ void relabel_body(const FinishArgs& a, int32_t block, int32_t nblocks)
{
    const int32_t R = a.st->num_dst[a.layer_index];
    const int32_t limit = R * a.fanout;                            // below 2^31: checked when the workspace is sized
    const int32_t step = nblocks * kBlock;
    for (int64_t t0 = (int64_t) block * kBlock + threadIdx.x; t0 < limit; t0 += (int64_t) step * kRelabelUnroll) {
        int32_t u[kRelabelUnroll], o[kRelabelUnroll];
        float w[kRelabelUnroll];
        bool ok[kRelabelUnroll];
#pragma unroll
        for (int i = 0; i < kRelabelUnroll; ++i) {
            const int64_t t = t0 + (int64_t) i * step;
            const int32_t q = t < limit ? (int32_t) t : limit - 1;
            const int32_t row = (int32_t) (((double) q + 0.5) * a.inv_fanout);          // q / fanout: exact below 2^31
            const int32_t s = q - row * a.fanout;
            const int32_t cnt = a.s_cnt[row];
            u[i] = a.s_nbr[q];                        // -(local id + 1) if the sampler already knew it, else the global id
            w[i] = a.unit_weights ? 1.0f : a.s_w[q];
            o[i] = a.indptr[row] + s;
            ok[i] = t < limit && s < cnt;
        }
#pragma unroll
        for (int i = 0; i < kRelabelUnroll; ++i) {
            const bool search = ok[i] && u[i] >= 0;
            int32_t local;
            if (a.by_slot) local = R + a.slot_words[search ? u[i] >> 6 : 0].rank((uint32_t) u[i]);
            else           local = (int32_t) a.tab.local(a.tab.entry[search ? u[i] : 0]);
            if (ok[i]) {
                a.indices[o[i]] = search ? local : -1 - u[i];
                a.weights[o[i]] = w[i];
            }
        }
    }
}

// A row whose CSR segment touches more than kHubChunks aligned 64-entry chunks is a hub: the sampler that reads rows' flag
// words gives it a whole wave.
constexpr int kHubChunks = 32;

__device__ __forceinline__ bool is_hub_extent(int64_t start, int64_t end)
{
    return end > start && ((end - 1) >> 6) - (start >> 6) + 1 > kHubChunks;
}

// The batch's scalars, published for its later kernels; one thread of the batch's first kernel.
__device__ __forceinline__ void begin_state(const LayerArgs& g, const BeginDyn& d, int b)
{
    DeviceState* st = bind_state(g, b);
    st->num_dst[0] = d.num_seeds[b];
    if (d.too_many >> b & 1u) st->bad_seed = d.batch_id[b];
    for (int l = 0; l < GNS_MAX_LAYERS; ++l) { st->num_edges[l] = 0; st->num_dst[l + 1] = 0; st->hub_count[l] = 0; }
    st->key0 = d.key0[b];
    st->key1 = d.key1[b];
    st->stamp = d.stamp[b];
    st->batch_id = d.batch_id[b];
    st->cache_gen = d.cache_gen[b];
}

// Clears the marks by slot for the batch: a share of them by every block of its first kernel.
__device__ __forceinline__ void clear_slot_marks(const LayerArgs& g, int b, int32_t block)
{
    if (g.off.slot_marks == 0) return;
    const uint32_t blocks = g.dealt > 1 ? gridDim.x / (uint32_t) g.dealt : gridDim.x;
    uint4* marks = at<uint4>(g.b[b].ws, g.off.plan_desc);
    for (uint32_t i = (uint32_t) block * kBlock + threadIdx.x; i < g.off.slot_marks / 16; i += blocks * kBlock) marks[i] = make_uint4(0, 0, 0, 0);
}

// Seed q of the batch, node u: the CSR extent of its row (empty for an id out of range).
__device__ __forceinline__ RowExtent seed_extent(const LayerArgs& g, int32_t u)
{
    RowExtent ext = {0, 0};
    if (u >= 0 && (int64_t) u < g.f.num_nodes) {
        ext.start = load_off_rt(g.f.g_indptr, g.f.g_i64, u);
        ext.end = load_off_rt(g.f.g_indptr, g.f.g_i64, (int64_t) u + 1);
    }
    return ext;
}

// Seed q enters the batch: its id copied, its extent recorded, its local id entered in the node table; with `mark` also
// its bit in the seed bitmap, for a first layer that is sampled in the same launch.
__device__ __forceinline__ void enter_seed(const LayerArgs& g, const BeginDyn& d, int b, const NodeTable& tab, int32_t q, int32_t u,
                                           const RowExtent& ext, bool mark)
{
    char* ws = g.b[b].ws;
    bool bad = true;
    if (u >= 0 && (int64_t) u < g.f.num_nodes) {
        if (mark) atomicOr(at<unsigned long long>(ws, g.off.seed_mark) + (u >> 6), 1ull << (u & 63));
        bad = tab.current(atomicExch(&tab.entry[u], tab.make((uint32_t) q)));         // a repeated seed
    }
    at<int32_t>(ws, g.off.seed_copy)[q] = u;
    at<RowExtent>(ws, g.off.row_ext)[q] = ext;
    if (bad) bind_state(g, b)->bad_seed = d.batch_id[b];
}

// ---------------------------------------------------------------------------
// Host side: a group of mini-batches and the argument block of one of its launches.
struct Group {
    int count;
    gns_ctx* ctx[kMaxGroup];
    gns_block* blocks[kMaxGroup];    // each: the caller's array of num_layers blocks
    int64_t rows[GNS_MAX_LAYERS + 1];        // what a batch's layers have at most, see bound_rows
};

// Grids and rows per wave go by the rows that the group's own seeds can lead to, where a launch serves this call alone (d); a captured
// one serves calls with any number of seeds.  A context often takes more seeds than a call brings, and blocks without rows are not
// free, nor are waves of many rows.  Batches of 16, 100 and 256 seeds in contexts for 1024 on 1 M nodes 74.7 -> 68.8, 75.0 -> 71.6 and
// 78.3 -> 76.0 us (a call with gather and aggregation), groups of four times 64 and 256 76.0 -> 72.5 and 116.6 -> 112.7, four times 100 on 40 M nodes
// 92.2 -> 87.1.
// (The limit is the lists' length, not the graph's: behind repeated seeds a list can be longer than that.)
inline void bound_rows(Group& g, const BeginDyn* d)
{
    const gns_ctx* c = g.ctx[0];
    const Layout& L = c->lay;
    g.rows[0] = d ? 1 : L.rows[0];
    for (int b = 0; d && b < g.count; ++b)
        if (d->num_seeds[b] > g.rows[0]) g.rows[0] = d->num_seeds[b];
    for (int i = 0; i < c->config.num_layers; ++i) {
        const int64_t next = g.rows[i] * (1 + c->config.fanout[i]);
        g.rows[i + 1] = next < L.rows[i + 1] ? next : L.rows[i + 1];
    }
}

// Blocks per batch of a group's first launch: those that its seeds need, and no fewer than clear the marks by slot in kClearTurns turns
// (blocks without seeds do nothing else).  Grids of the seeds alone cleared 1.1 MB (1.1 M cached nodes) with one block, in front of everything
// else: sampling 64 seeds, fan-outs 20, 5, on 40 M nodes 41.5 -> 33.5 us, fan-outs 15, 10, 5 46.3 -> 44.5 (before there were such marks
// 37.7 and 58.2); 400 K cached nodes 35.3 -> 32.5 and 44.6 -> 44.0.  One, two and four turns are the same.
constexpr int kClearTurns = 2;
inline int64_t first_blocks(const Group& g, int64_t seed_blocks)
{
    constexpr int64_t kBytes = (int64_t) kClearTurns * kBlock * 16;
    const int64_t clearing = (g.ctx[0]->lay.slot_marks + kBytes - 1) / kBytes;
    return seed_blocks > clearing ? seed_blocks : clearing;
}

// f(kOne): calls it with whether the group is a single batch as a compile-time constant.
template <typename F>
inline void with_one(const Group& g, F&& f)
{
    if (g.count == 1) f(std::integral_constant<bool, true>());
    else              f(std::integral_constant<bool, false>());
}
// Grid of a group's launch with `blocks` blocks per batch.
inline dim3 group_grid(const Group& g, const LayerArgs& a, int64_t blocks)
{
    if (a.dealt == 1) return dim3((unsigned) blocks, (unsigned) g.count);
    return dim3((unsigned) ((blocks + kXcds - 1) / kXcds * kXcds * g.count));
}
// Fills the parts of a LayerArgs that do not depend on the layer: offsets and the per-batch scratch bases.
void fill_group_args(const Group& g, LayerArgs* out);
// Points the slots at layer `layer_index` (dst lists and block buffers of that layer and the one before).
void set_group_layer(const Group& g, int layer_index, LayerArgs* out);
// The templates for one layer (sampler side: own layer; finish side: `finish_layer`).
void fill_sample_template(gns_ctx* c, int layer_index, SampleArgs* out);
void fill_finish_template(const Group& g, int finish_layer, FinishArgs* out);
// The fixed arguments of the group's first kernel.
void fill_first_args(const Group& g, LayerArgs* out);
int relabel_grid(const Group& g, int layer_index);
// Whether a layer is sampled without a plan or flag pass in front: UNIFORM, or from the induced subgraph.
bool direct_layer(const gns_config& config, int layer_index);
// Whether the input layer's union and relabel are one launch.
inline bool finishes_at_once(const gns_ctx* c) { return c->lay.slot_marks > 0 && c->lay.slot_marks <= kSlotsMax; }
// Whether the first layer's sampler is also the batch's first kernel (k_batch_begin runs in front of the others).
bool first_layer_enters_seeds(const gns_config& config);
// Rows whose sampled neighbors the layer's sampler sums up (0: it does not, the union step's blocks do).
int rows_per_sum(const Group& g, int layer_index);
// The batch's first launch when the first layer is direct: seeds and sampling in one.
hipError_t launch_first_layer(const Group& g, const BeginDyn& d, hipStream_t s);
// gns_small.hip: whether every mini-batch of the group fits a block of its own, and the one launch that samples them so.
bool small_batches(const Group& g, const BeginDyn& d);
hipError_t launch_small(const Group& g, const BeginDyn& d, hipStream_t s);

}  // namespace gns
