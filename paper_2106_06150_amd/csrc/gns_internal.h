// Host-side internals of the GNS library: context, workspace layout and the
// launch functions each kernel file exports to the API layer.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include "../../include/gns.h"

namespace gns {

// Device-resident scalars the kernels of one call communicate through.  What a
// call reports to the host goes into the same fields of a pinned struct.
struct DeviceState {
    int32_t num_dst[GNS_MAX_LAYERS + 1];  // rows of layer index i (num_dst[i+1] = num_src of layer i)
    int32_t num_edges[GNS_MAX_LAYERS];
    uint32_t key0, key1;                  // Philox key of the current batch (lo32(seed), hi32(seed))
    uint32_t bad_seed;                    // id of the last batch that had a seed out of range or repeated
    int32_t hub_count[GNS_MAX_LAYERS];    // entries of a scanning layer's hub-row list (reset by the batch's first kernel)
    int32_t draw_distinct[2];             // cache draw: nodes in the cache before a chunk (by the chunk's parity)
    int32_t draw_done_chunk;              //   index of the chunk that completed the cache, -1 while incomplete
    int32_t plan_chunks;                  // CACHE_ONLY sampler: aligned chunks in the current work list
    uint32_t stamp;                       // what the current batch's entries of the node table carry (set by its first kernel)
    uint32_t batch_id;                    // id of the current batch (set by its first kernel)
    int32_t cache_gen;                    // which copy of the cache structures it reads (set by its first kernel)
    unsigned long long cut_draw;          // cache draw: stream index of the draw that completed the cache
    unsigned long long walk_total;        // random-walk probability: sum of the weights
    int32_t walk_support;                 //   number of nodes with a non-zero weight
    int32_t walk_error;                   //   1: bad training node, 2: does not fit in 62 bits
};

// LDS a flag-kernel block may fill with a membership bitmap (the chip's 160 KB minus the block's own needs)
constexpr size_t kLdsBitmapBytes = 160 * 1024 - 1024;

// What stands in LDS for a cache bitmap that does not fit there: which groups of neighboring ids have a cached node, one bit
// each, and of every kFilterHot ids' cached nodes the one with the longest row, as a 16-bit tag.  An entry whose node's tag is
// there is cached, one whose group's bit is off is not; only the others ask the exact bitmap.
constexpr int32_t kFilterHot = 16384;
constexpr int32_t kFilterGroups = (int32_t) (kLdsBitmapBytes - 2 * kFilterHot) * 8;
// On large graphs that bitmap is longer than an L2, and what is asked first there is a list of 16 bits per group: the lower
// seven bits of the group's first two cached nodes (of ids that neighbor one another they tell up to 128 apart) and whether
// it has more, which only the bitmap tells.
struct CacheFilter {
    unsigned long long* keys;     // [kFilterHot] (row length, id) of slot (id % kFilterHot)'s node, 0: none
    uint32_t* groups;             // [kFilterGroups / 32] behind them
    uint16_t* tags;               // [kFilterHot] behind them: what stands in LDS for the keys
    uint16_t* pairs;              // [kFilterGroups] behind them, or null; of groups without a cached node stale
    uint32_t mult;                // group of an id: the upper half of id * mult
};
constexpr uint32_t kPairBits = 7, kPairMask = (1u << kPairBits) - 1u, kPairMore = 1u << 14, kPairSet = 1u << 15;
// Graphs of more nodes than this have no filter.  At the line a group has up to 81 ids.
constexpr int64_t kFilterNodes = (int64_t) kLdsBitmapBytes * 8 * 64;
static_assert(kFilterNodes / kFilterGroups + 2 <= 1 << kPairBits, "a pair tells the ids of a group apart");
constexpr size_t kFilterBytes = (size_t) kFilterHot * (8 + 2) + kFilterGroups / 8 + (size_t) kFilterGroups * 2;
// The pass over the entries with the list and without: 40 M nodes (a bitmap of 5 MB) 1020 and 1188 us, 28 M 705 and 749,
// 20 M 813 and 843, 12 M 378 and 358.
constexpr int64_t kFilterPairsNodes = (int64_t) 16 << 20;

// What a layer that draws from the cache looks up of a node, in one read.
struct alignas(8) CachedNode {
    float inv_pc;              // 1 / p^C_u
    int32_t slot;              // its place in the list of cached nodes
};

struct Layout {
    // persistent cache structures
    size_t cache_bitmap, cache_prefix, cache_nodes, cache_feat;
    size_t filter;            // CacheFilter: keys, then groups (graphs whose bitmap does not fit LDS; 0: unused)
    uint32_t filter_mult;
    size_t coarse_bitmap;     // one bit per 2^coarse_shift node ids: "some node of the group is cached" (0: unused)
    int32_t coarse_shift;
    int64_t coarse_words;
    // random-walk cache probability (only with GNS_PROB_WALK): two weight vectors, their prefix, scan partials
    size_t walk_a, walk_b, prob_prefix, walk_tiles, walk_tiles_nz;
    size_t walk_hot;          //   and the hot nodes' table (HotCopy[2])
    size_t node_pc;           // [n] floats: 1 / p^C_u (Section 3.4), filled for the nodes of the current cache; with slot_marks CachedNode
    // cache-draw scratch
    size_t draw_table, draw_slot, draw_sums, index_sums;
    size_t entry_rows;        // row that owns entry 64 * i of the CSR entry array (Eq. (1) draws; filled by gns_create)
    // frontier structures
    size_t mark_bitmap;
    size_t mark_summary;      // one bit per word of the mark bitmap: "this word has a mark" (large graphs only)
    int64_t summary_words;    // 0: no summary
    size_t seed_copy;         // [max_seeds] the batch's seeds, copied by its first kernel
    size_t hub_rows;          // [max_rows] the layer's rows whose CSR segment spans more than kHubChunks chunks
    size_t row_ext;           // [max nodes of a batch] CSR extent of every node of the batch's list (append-only)
    size_t seed_mark;         // bitmap of the batch's seeds (first layer sampled by the lane kernel)
    size_t table;             // [n] node table: local id of every node of the batch, stamped (the last per-batch section)
    int table_shift;          // bits of a local id in a table entry
    uint32_t max_stamp;
    size_t static_table;      // node table of gns_sample_blocks_static where the library's array cannot hold it (shared; 0: none)
    bool lists_hubs;          // some layer scans its rows and gives the hubs among them a wave of their own
    // per-layer sampler scratch (fixed stride fanout)
    size_t s_nbr[2], s_w[2], s_cnt[2];     // double-buffered by layer parity
    // CACHE_ONLY sampler: chunk work list, CSR-aligned membership flags
    size_t plan_desc, edge_flags;
    // GNS_FLAGS_PER_CACHE: the induced subgraph S of Section 3.3 in compact form (see gns_induced.hip).
    size_t srec, s_nodes;
    size_t s_count;
    int s_tile_shift;

    int64_t max_chunks;
    // The input layer's new nodes are marked by their slots of the cache, a byte each: bytes of the marks, in the place of plan_desc
    // (0: they are marked in the bitmap of all nodes), behind them for caches of more than kSlotsMax slots a SlotWord for every 64,
    // and slots of a tile of the union step there
    int64_t slot_marks;
    int32_t slot_tile;
    // scan partials
    size_t sums_rows, tile_sums, row_sums, plan_sums;
    size_t info;              // outcome of the graph validation
    size_t state;
    size_t shared_begin;      // sections at or past this offset are shared with forked contexts
    size_t cache_block_begin; // first of the two copies of what a cache draw writes (bitmap ... 1/p^C table)
    size_t cache_block_bytes; // the second copy lies this many bytes further
    size_t total;
    // sizes
    int64_t words;            // ceil(n / 64)
    int32_t mark_tile_words;  // bitmap words per frontier tile (kMarkTileMin .. kMarkTileMax, a power of two)
    int64_t mark_tiles;       // ceil(words / mark_tile_words)
    int64_t row_tiles;        // ceil(max rows / kTile)
    int64_t plan_tiles;       // ceil(max rows / kBlock)
    int64_t draw_chunk;       // largest number of stream draws processed at a time
    int64_t draw_unit;        // the draw's limits count the stream in pieces of this many draws
    int64_t draw_tiles;
    int64_t index_tiles;
    uint32_t draw_hash_cap;   // power of two
    int64_t max_rows;         // worst-case dst rows of any layer
    int64_t max_edges;        // worst-case edges of any layer
    int64_t rows[GNS_MAX_LAYERS + 1];
    int64_t edges[GNS_MAX_LAYERS];
};

}  // namespace gns

namespace gns {
// Streams one context may enqueue mini-batches on between two cache draws (each gets an event the
// draw after next waits for).
constexpr int kReaderStreams = 4;
struct Group;       // gns_kernels.hpp: the mini-batches one launch sequence serves
struct BeginDyn;    //   the first kernel's per-replay arguments
// Opaque host-side storage for the first kernel's arguments (LayerArgs, BeginDyn).
struct BeginArgsHost {
    alignas(8) unsigned char fixed[3072];
    alignas(8) unsigned char dyn[768];
    int rows_per_wave;                   // k_sample_first's third argument
};
// One captured launch sequence of a group of mini-batches, kept by the group's first context.
struct BatchGraph {
    hipGraph_t graph;
    hipGraphExec_t exec;
    hipGraphNode_t first;            // the k_batch_begin node
    bool valid;
    uint64_t last_use;
    // capture key: the contexts of the group and the caller's block buffers
    int count;
    gns_ctx* ctx[GNS_MAX_GROUP];
    gns_block blocks[GNS_MAX_GROUP][GNS_MAX_LAYERS];
    BeginArgsHost args;              // the first kernel's arguments (the node's parameter list points here)
    void* arg_ptrs[3];
};
constexpr int kGraphsPerContext = 2;
struct ProfileRecord {
    int32_t stage;
    hipEvent_t start, stop;
};
}  // namespace gns

struct gns_ctx {
    gns_graph graph;
    gns_config config;
    gns::Layout lay;
    char* ws;                        // device workspace base (per-batch scratch sections)
    char* shared_ws;                 // base for the shared sections (the root context's workspace)
    gns_ctx* root;                   // owner of the cache; this for a context made by gns_create
    gns::DeviceState* d_state;       // device
    gns::DeviceState* h_state;       // pinned host mirror, written by the last kernel of every mini-batch
    gns::DeviceState* h_state_dev;   //   its address for kernels
    gns::DeviceState* h_draw;        // pinned: where cache draws and the walk probability leave their outcome (mini-batches
                                     //   of this context may be in flight meanwhile, so not the mirror they write)
    bool uses_cache;
    bool cache_valid;
    int cache_gen;                   // root only: which copy of the cache block the mini-batches read
    // Who may still read the copy a draw is about to overwrite: work enqueued before the previous draw.
    // Every draw records an event on the stream each context of the family last used (all that was
    // enqueued there so far) and waits, on the device, for the events the previous draw recorded.
    hipEvent_t gen_event[2][gns::kReaderStreams];   // alternate from draw to draw; one per stream used
    int gen_event_used[2];           // how many of them the draw that overwrites that copy has to wait for
    hipStream_t reader_streams[gns::kReaderStreams];   // where this context enqueued readers of the cache block
    int reader_stream_count;         //   since the last draw became current
    bool had_cache;                  // root only: some draw has been made current (cache_gen is meaningful)
    uint32_t draw_tag;               // root only: of the last launch of a draw that passes sums between its blocks
    // root only: a draw enqueued by gns_sample_cache_async and not yet made current
    bool pending;
    int pending_gen;
    hipEvent_t ready_event[2];       // recorded behind the draw that filled the copy
    uint64_t cache_version;          // bumped when a copy becomes current
    uint64_t seen_version;           // per context: the version its stream has been made to wait for
    bool has_sampled;                // root only: whether some context of the family has enqueued mini-batches yet, and
    hipStream_t last_sampled_on;     //   the stream of the last ones
    gns_ctx* family[64];             // root only: the root itself and its live forks
    uint32_t forks_made;             // root only: so far
    int family_count;
    int64_t cache_draws;
    // cache probability other than Eq. (1): set by gns_cache_walk_probability on the root context
    bool prob_valid;
    const unsigned long long* prob_weights;   // device, [n]
    unsigned long long prob_total;
    int64_t prob_support;            // nodes with non-zero weight
    int64_t nonzero_degree_nodes;
    int num_cus;
    size_t lds_bitmap_limit;         // largest cache bitmap (bytes) the flag kernel stages in LDS
    // The launch sequence of one mini-batch, captured once per (seeds pointer, block buffers) and
    // replayed; only the first kernel's arguments (seed, number of seeds) change between replays.
    hipStream_t cap_stream;          // used for capture only, never for execution
    gns::BatchGraph* bg;             // [kGraphsPerContext] captured launch sequences (least recently used is replaced)
    uint64_t graph_clock;
    uint32_t stamp;                  // of the last mini-batch enqueued on this context, 1 .. lay.max_stamp (0: none yet)
    int union_spins;                 // how often the union step polls another tile's sum before it counts that tile itself
    uint32_t batch_id;               // id of the last mini-batch enqueued on this context (from 1)
    uint32_t bad_reported;           // DeviceState::bad_seed as of the last report to the caller
    gns_ctx* static_child;           // root only: the context of gns_sample_blocks_static (scratch in the library's array)
    char static_err[160];            // root only: why the library's scratch array is unavailable on this device, if it is
    // optional stage timing (benchmarks only)
    uint32_t prof_mask;
    int32_t prof_capacity;
    int32_t prof_count;
    gns::ProfileRecord* prof;
    char err[256];
};

namespace gns {

template <typename T>
static inline T* ws_ptr(const gns_ctx* c, size_t off)
{
    return reinterpret_cast<T*>((off >= c->lay.shared_begin ? c->shared_ws : c->ws) + off);
}

// The node table of a context (see Layout::static_table for the one place where it is not part of the scratch).
static inline uint32_t* ws_ptr_table(const gns_ctx* c) { return reinterpret_cast<uint32_t*>(c->ws + c->lay.table); }

// A section of the cache block in the given generation (off is the section's offset in generation 0).
template <typename T>
static inline T* cache_ptr(const gns_ctx* c, size_t off, int gen)
{
    return reinterpret_cast<T*>(c->shared_ws + off + (gen ? c->lay.cache_block_bytes : 0));
}

// The cache filter in the given generation (null pointers: none).
static inline CacheFilter cache_filter(const gns_ctx* c, int gen)
{
    CacheFilter f = {nullptr, nullptr, nullptr, nullptr, c->lay.filter_mult};
    if (c->lay.filter) {
        f.keys = cache_ptr<unsigned long long>(c, c->lay.filter, gen);
        f.groups = reinterpret_cast<uint32_t*>(f.keys + kFilterHot);
        f.tags = reinterpret_cast<uint16_t*>(f.groups + kFilterGroups / 32);
        if (c->graph.num_nodes > kFilterPairsNodes) f.pairs = f.tags + kFilterHot;
    }
    return f;
}

// The generation the mini-batches enqueued now read.
static inline int active_gen(const gns_ctx* c) { return c->root->cache_gen; }

// Called before a context enqueues kernels that read the cache block on stream s: remembers the stream and,
// the first time after another copy became current, makes the stream wait for the draw that filled it.
static inline hipError_t before_cache_readers(gns_ctx* c, hipStream_t s)
{
    int known = 0;
    while (known < c->reader_stream_count && c->reader_streams[known] != s) ++known;
    if (known == c->reader_stream_count) {
        if (known == kReaderStreams) return hipErrorInvalidValue;     // reported as GNS_ESTATE
        c->reader_streams[c->reader_stream_count++] = s;
    }
    gns_ctx* root = c->root;
    if (!c->uses_cache || !root->cache_valid || c->seen_version == root->cache_version) return hipSuccess;
    c->seen_version = root->cache_version;
    return hipStreamWaitEvent(s, root->ready_event[root->cache_gen], 0);
}

gns_status ctx_fail(gns_ctx* c, gns_status st, const char* what, hipError_t e = hipSuccess);
// gns_api.hip
gns_status enqueue_batch(const Group& g, const BeginDyn& d, hipStream_t s);
// takes the next stamp of every context of the group (enqueues the clearing of a node table whose stamps have run out)
hipError_t next_stamps(const Group& g, hipStream_t s);
void fill_begin_dyn(const Group& g, const uint64_t* seeds, const int32_t* const* seeds_dev, const int32_t* num_seeds,
                    BeginDyn* out);
gns_status check_batch_args(gns_ctx* c, const int32_t* seeds_dev, int32_t num_seeds, const gns_block* blocks);
hipError_t init_batch_scratch(gns_ctx* c, hipStream_t s);
// Where the scratch of a family's `index`-th context begins in its workspace.  Marks are atomics, which are carried out where the
// memory is, and memory changes hands every 4 KB in a period of 32 KB: on a graph of 33 K nodes a batch's bitmap is one such
// piece, and contexts whose workspaces lie alike mark in the same place together.  Layer of 4 x 1776 rows, fan-out 10: all four at
// one place 13.4 us, at four neighboring ones 8.7, at every other one 7.4; so places are given out in bit-reversed order.
constexpr size_t kPlaceBytes = 4096, kPlacesBytes = 8 * kPlaceBytes;       // what a workspace has for it
static inline char* scratch_begin(void* workspace, uint32_t index)
{
    const uintptr_t at = reinterpret_cast<uintptr_t>(workspace) / kPlaceBytes;
    const uint32_t place = (index & 1u) << 2 | (index & 2u) | (index >> 2 & 1u);
    return static_cast<char*>(workspace) + ((place - at) & 7u) * kPlaceBytes;
}
gns_status make_child(gns_ctx* root, void* workspace, bool with_capture_stream, gns_ctx** out);
// gns_static.hip
gns_status static_scratch_setup(gns_ctx* root);
bool compute_layout(const gns_graph* g, const gns_config* cfg, Layout* out, char* err, size_t errlen);

// Brackets a stage's launches with events when that stage is being timed.
struct StageTimer {
    gns_ctx* c;
    hipStream_t s;
    int32_t slot;
    StageTimer(gns_ctx* ctx, int32_t stage, hipStream_t stream, bool enabled = true) : c(ctx), s(stream), slot(-1)
    {
        if (!enabled || !(c->prof_mask & (1u << stage)) || c->prof_count >= c->prof_capacity) return;
        slot = c->prof_count++;
        c->prof[slot].stage = stage;
        (void) hipEventRecord(c->prof[slot].start, s);
    }
    ~StageTimer()
    {
        if (slot >= 0) (void) hipEventRecord(c->prof[slot].stop, s);
    }
};

// gns_dense.hip
hipError_t launch_sage_dense(gns_ctx* c, const float* h_self, int32_t f1, const float* h_neigh, int32_t f2,
                             const float* w, const float* bias, int32_t hdim, int32_t relu, float* out,
                             int32_t num_rows, hipStream_t s);

// gns_walk.hip
size_t walk_hot_bytes();
gns_status run_walk_probability(gns_ctx* c, const int32_t* train_nodes, int64_t num_train, int32_t scale_log2,
                                hipStream_t s);

// gns_cache.hip
// validates the graph and fills Layout::entry_rows
hipError_t launch_count_nonzero_rows(gns_ctx* c, hipStream_t s, int32_t* d_out);
// Draws of the first chunk of a cache draw: half as many again as the cache has nodes, which completes a cache of one
// percent of the nodes on most graphs; further chunks are Layout::draw_chunk long.
constexpr int32_t kDrawTile = 1024;
constexpr int64_t first_draws(int64_t cache_size) { return cache_size + cache_size / 2 + 2048; }
// wait_for_it: enqueue one chunk or two, with what follows a complete cache behind them, and look at the outcome, then two more
// at a time until it is complete or refused; otherwise enqueue a fixed number of chunks (later ones stand down once the cache
// is complete) and return.
gns_status run_sample_cache(gns_ctx* c, uint64_t seed, uint64_t epoch, bool wait_for_it, hipStream_t s);
gns_status activate_cache(gns_ctx* c);
gns_status retire_cache(gns_ctx* c);
gns_status finish_pending_draw(gns_ctx* c);

// gns_induced.hip
int induced_tile_shift(int64_t num_entries);
// done: as IndexArgs::done in gns_cache.hip
hipError_t launch_build_induced(gns_ctx* c, int cache_gen, const int32_t* done, hipStream_t s);

// gns_sampler.hip
// the previous layer's relabel shares this layer's first launch
hipError_t launch_sample_layer(const Group& g, int layer_index, hipStream_t s);

// gns_frontier.hip
hipError_t launch_batch_begin(const Group& g, const BeginDyn& d, hipStream_t s);
hipError_t launch_relabel(const Group& g, int layer_index, hipStream_t s);
hipError_t launch_finish_layer(const Group& g, int layer_index, hipStream_t s);
hipError_t launch_finish_cached(const Group& g, hipStream_t s);
hipError_t launch_fill_u64(unsigned long long* p, size_t n, unsigned long long v, hipStream_t s);
hipError_t launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t s);

// gns_feature.hip
// use_cache_gen < 0: every row comes from the full store (used while a cache's own table is being filled);
// unless_negative: device count below which nothing is copied, or null
hipError_t launch_gather(gns_ctx* const* ctxs, int count, const int32_t* const* nodes, const int32_t* num_nodes,
                         float* const* out, int use_cache_gen, hipStream_t s, const int32_t* unless_negative = nullptr);
hipError_t launch_aggregate(gns_ctx* const* ctxs, int count, const gns_block* const* blks, const float* const* x_src,
                            int32_t feat_dim, float* const* out, hipStream_t s);

}  // namespace gns
