// Frontier union and relabelling (paper Algorithm 1, top-down loop:
// B^{l-1} <- B^{l-1} U N_l(u)), turned into a block CSR per layer.
//
// The sampler leaves, per dst row, up to k neighbor ids at a fixed stride, their number, the sums of those
// numbers over blocks of rows, and one bit per sampled id in a node-indexed mark bitmap.  Here:
//   begin    the batch's first kernel where the first layer's sampler does not do it itself: scalars, seeds
//            with their local ids into the node table, their CSR extents
//   union    row tiles scan the row counts into indptr; bitmap tiles count their marks, learn the counts of
//            the tiles before them and write the marked ids in ascending order behind the dst prefix, one
//            thread per new id, each entered in the node table with its local id, its CSR extent recorded;
//            the bitmap words are cleared for the next layer
//   relabel  every sampled edge looks its neighbor's local id up and is
//            compacted to its CSR position (inside the next layer's first sampler
//            launch; the last layer has a launch of its own, which also writes the counts to the host)
//   finish   union and relabel of an input layer that samples from the cache only (k_finish_cached)
// Sorted order comes from walking the bitmap, so the result does not depend on
// the order in which threads ran.
#include <string.h>
#include "gns_kernels.hpp"

namespace gns {

__global__ void k_fill_u64(unsigned long long* p, size_t n, unsigned long long v)
{
    size_t i = (size_t) blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t) gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

__global__ void k_fill_u32(uint32_t* p, size_t n, uint32_t v)
{
    size_t i = (size_t) blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t) gridDim.x * blockDim.x;
    for (; i < n; i += stride) p[i] = v;
}

static inline unsigned fill_grid(size_t n)
{
    size_t b = (n + kBlock - 1) / kBlock;
    if (b > 4096) b = 4096;
    if (b < 1) b = 1;
    return (unsigned) b;
}

hipError_t launch_fill_u64(unsigned long long* p, size_t n, unsigned long long v, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u64, dim3(fill_grid(n)), dim3(kBlock), 0, s, p, n, v);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u32, dim3(fill_grid(n)), dim3(kBlock), 0, s, p, n, v);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// First kernel of a mini-batch whose first layer has a plan or flag pass in front of its sampler: publishes the
// batch's scalars (number of seeds, Philox key, node table stamp, which copy of the cache structures it reads) in
// the device state, copies the seeds into the context and enters them, with their local ids, in the node table.
// A bad seed is reported by stamping the batch id, so no flag needs resetting while other blocks may be setting it.
__global__ void __launch_bounds__(kBlock) k_batch_begin(LayerArgs g, BeginDyn d)
{
    const auto [b, block] = group_block<false>(g.dealt);
    const int32_t num_seeds = d.num_seeds[b];
    const NodeTable tab = bind_table(g, b, d.stamp[b]);
    const int32_t q = block * kBlock + (int32_t) threadIdx.x;
    if (q == 0) begin_state(g, d, b);
    clear_slot_marks(g, b, block);
    if (q < num_seeds) {
        const int32_t u = d.seeds[b][q];
        enter_seed(g, d, b, tab, q, u, seed_extent(g, u), false);
    }
}

void fill_group_args(const Group& g, LayerArgs* out)
{
    gns_ctx* c = g.ctx[0];
    const Layout& L = c->lay;
    memset(out, 0, sizeof(*out));
    // no launch has more threads per batch than it has rows, but for a few thousand blocks; a grid has fewer than 2^32
    out->dealt = L.max_rows * g.count <= (int64_t) 1 << 31 ? g.count : 1;
    WsOffsets& o = out->off;
    o.mark_summary = L.mark_summary;
    o.has_summary = L.summary_words > 0 ? 1 : 0;
    o.state = L.state; o.mark = L.mark_bitmap; o.seed_mark = L.seed_mark; o.seed_copy = L.seed_copy;
    o.row_ext = L.row_ext; o.hub_rows = L.hub_rows;
    o.table = L.table;
    o.table_shift = L.table_shift;
    for (int p = 0; p < 2; ++p) { o.s_nbr[p] = L.s_nbr[p]; o.s_w[p] = L.s_w[p]; o.s_cnt[p] = L.s_cnt[p]; }
    o.plan_desc = L.plan_desc;
    o.slot_marks = (uint64_t) L.slot_marks;
    o.sums_rows = L.sums_rows; o.tile_sums = L.tile_sums; o.row_sums = L.row_sums; o.plan_sums = L.plan_sums;
    o.cache_block_bytes = L.cache_block_bytes;
    o.uses_cache = c->uses_cache ? 1 : 0;
    o.marks_seeds = first_layer_enters_seeds(c->config) ? 1 : 0;
    for (int b = 0; b < kMaxGroup; ++b) {
        out->b[b].ws = g.ctx[b < g.count ? b : 0]->ws;
        out->b[b].host = g.ctx[b < g.count ? b : 0]->h_state_dev;
    }
}

void set_group_layer(const Group& g, int layer_index, LayerArgs* out)
{
    for (int b = 0; b < g.count; ++b) {
        gns_ctx* c = g.ctx[b];
        BatchSlot& q = out->b[b];
        const int32_t* seed_copy = ws_ptr<int32_t>(c, c->lay.seed_copy);
        const gns_block* blk = g.blocks[b];
        q.dst = layer_index == 0 ? seed_copy : blk[layer_index - 1].src_nodes;
        q.cur = block_ptrs(blk[layer_index]);
        q.prev = block_ptrs(blk[layer_index > 0 ? layer_index - 1 : 0]);
    }
}

// Enqueues the first kernel of a group of mini-batches.
hipError_t launch_batch_begin(const Group& g, const BeginDyn& d, hipStream_t s)
{
    LayerArgs a;
    fill_first_args(g, &a);
    const dim3 grid = group_grid(g, a, first_blocks(g, (g.rows[0] + kBlock - 1) / kBlock));
    hipLaunchKernelGGL(k_batch_begin, grid, dim3(kBlock), 0, s, a, d);
    return hipGetLastError();
}

// Words first .. first + per - 1 of a tile that starts at word `base` (per <= kPerMax consecutive words of one thread).
template <int kPerMax>
__device__ __forceinline__ void load_marks(const FinishArgs& a, int64_t base, int first, int per, int T, uint64_t* word)
{
    const int64_t w0 = base + first;
#pragma unroll
    for (int i = 0; i < kPerMax; ++i) {
        const int64_t w = w0 + i;
        word[i] = i < per && first + i < T && w < a.words ? a.mark[w] : 0ull;
    }
}

// sum of vals[0..count) by the whole block
__device__ __forceinline__ int32_t block_sum_array(const int32_t* vals, int32_t count, int32_t* smem)
{
    int32_t v = 0;
#pragma unroll 4
    for (int32_t t = (int32_t) threadIdx.x; t < count; t += kBlock) v += vals[t];
    return block_sum(v, smem);
}

// New nodes of one bitmap tile, counted from the bitmap by one thread.
__device__ __forceinline__ uint32_t count_tile(const FinishArgs& a, int32_t tile)
{
    uint32_t n = 0;
    const int64_t first = (int64_t) tile * a.mark_tile_words;
    for (int64_t w = first; w < first + a.mark_tile_words && w < a.words; ++w)
        n += (uint32_t) __popcll(a.mark[w] & (a.seed_mark ? ~a.seed_mark[w] : ~0ull));
    return n;
}

// CSR extent of a node that joins the batch's list.  Nodes that join in the last layer are
// no layer's rows: nothing reads their extents, and on a graph whose offsets fit no L2 the read of one is a trip to memory.
__device__ __forceinline__ RowExtent new_extent(const FinishArgs& a, uint32_t node)
{
    RowExtent ext = {0, 0};
    if (a.last_layer) return ext;
    ext.start = load_off_rt(a.g_indptr, a.g_i64, node);
    ext.end = load_off_rt(a.g_indptr, a.g_i64, (int64_t) node + 1);
    return ext;
}

// The same without a branch, in which a read would be waited for: the offsets as four words of 32 bits, of which those of 32-bit offsets
// are two.
__device__ __forceinline__ RowExtent extent_of(const FinishArgs& a, uint32_t node)
{
    const uint64_t at = a.last_layer ? 0u : node;
    const uint32_t* p = reinterpret_cast<const uint32_t*>(a.g_indptr) + (at << a.g_i64);
    const uint32_t start = p[0], end = p[1 << a.g_i64];
    const uint32_t start_hi = p[a.g_i64], end_hi = p[(1 << a.g_i64) + a.g_i64];
    return {(int64_t) ((uint64_t) (a.g_i64 ? start_hi : 0u) << 32 | start), (int64_t) ((uint64_t) (a.g_i64 ? end_hi : 0u) << 32 | end)};
}

// Node `node` joins the batch's list at place `pos`.  Behind repeated or invalid seeds the list can be longer than the graph has nodes; it is
// cut where its buffers end.
__device__ __forceinline__ void emit_new_node(const FinishArgs& a, int32_t pos, uint32_t node, const RowExtent& ext)
{
    if (pos >= a.max_src) return;
    a.src_nodes[pos] = (int32_t) node;
    a.tab.entry[node] = a.tab.make((uint32_t) pos);
    if (!a.last_layer) a.row_ext[pos] = ext;
}

// New node j of those whose words stand in LDS (count of them, the first at bitmap word `base`): its id.
__device__ __forceinline__ uint32_t new_node(const uint64_t* s_word, const int32_t* s_widx, const int32_t* s_off, int32_t count, int64_t base, int32_t j)
{
    int32_t lo = 0, hi = count;                              // the last word whose offset is <= j
    while (hi - lo > 1) {
        const int32_t mid = (lo + hi) >> 1;
        if (s_off[mid] <= j) lo = mid; else hi = mid;
    }
    return (uint32_t) ((base + s_widx[lo]) * 64 + select_bit64(s_word[lo], j - s_off[lo]));
}

// Places of the last of v[0 .. count) that are <= q, where v ascends in LDS and v[0] <= q: kN searches step by step together, whose
// reads one after the other are a chain of 30 and more.  `count` (>= 1) is the same for the whole block.
template <int kN>
__device__ __forceinline__ void last_not_above(const int32_t* v, int32_t count, const int32_t (&q)[kN], int32_t (&at)[kN])
{
    const int32_t end = __builtin_amdgcn_readfirstlane(count) - 1;
#pragma unroll
    for (int i = 0; i < kN; ++i) at[i] = 0;
    for (int32_t step = end > 0 ? 1 << (31 - __clz(end)) : 0; step > 0; step >>= 1)
#pragma unroll
        for (int i = 0; i < kN; ++i) {
            const int32_t m = at[i] + step < end ? at[i] + step : end;
            at[i] = v[m] <= q[i] ? m : at[i];
        }
}

// What a thread reads of its first new nodes while the counts of the tiles before are on their way: a trip to memory behind that
// wait otherwise.  Groups of four, first and second layer: 1 M nodes 8.7 and 13.2 -> 6.4 and 10.5 us, 40 M 14.8 and 22.6 -> 9.4 and 18.9.
// Where the bitmap has a summary, tiles hold more new nodes and their extents are further away: four a turn, looked up together (two,
// one by one: 12.0 and 20.3).  Smaller graphs gain nothing by it, and two launch sequences side by side lose 0.4 %.
constexpr int kAhead = 2, kAheadFar = 4;

struct NewNodes {
    uint32_t node[kAheadFar];
    RowExtent ext[kAheadFar];
};

// New nodes j, j + kBlock, ... (below hi; node 0 beyond it) of those whose words stand in LDS, `count` of them, the first at bitmap
// word `base`.  j begins with the thread's place; the others are the same for the whole block.
__device__ __forceinline__ void find_new(const FinishArgs& a, const uint64_t* s_word, const int32_t* s_widx, const int32_t* s_off, int32_t count,
                                         int64_t base, int32_t j, int32_t hi, NewNodes& f)
{
#pragma unroll
    for (int i = 0; i < kAheadFar; ++i) f.node[i] = 0u;
    auto look_up = [&](auto turns) {
        constexpr int kTurns = decltype(turns)::value;
        int32_t q[kTurns], at[kTurns];
#pragma unroll
        for (int i = 0; i < kTurns; ++i) q[i] = j + i * kBlock < hi ? j + i * kBlock : hi - 1;
        last_not_above(s_off, count, q, at);
#pragma unroll
        for (int i = 0; i < kTurns; ++i) f.node[i] = (uint32_t) ((base + s_widx[at[i]]) * 64 + select_bit64(s_word[at[i]], q[i] - s_off[at[i]]));
    };
    // (a look-up is 60 instructions: 0.6 us of the union step where tiles have fewer new nodes than threads and every thread took four)
    const int32_t left = __builtin_amdgcn_readfirstlane(hi - j + (int32_t) (threadIdx.x & (kWave - 1)));
    if (left > 2 * kBlock)  look_up(std::integral_constant<int, kAheadFar>());
    else if (left > kBlock) look_up(std::integral_constant<int, 2>());
    else if (left > 0)      look_up(std::integral_constant<int, 1>());
#pragma unroll
    for (int i = 0; i < kAheadFar; ++i) f.ext[i] = extent_of(a, f.node[i]);
}

__device__ __forceinline__ void emit_new_nodes(const FinishArgs& a, int32_t rows, int32_t j, int32_t hi, const NewNodes& f)
{
#pragma unroll
    for (int i = 0; i < kAheadFar; ++i)
        if (j + i * kBlock < hi) emit_new_node(a, rows + j + i * kBlock, f.node[i], f.ext[i]);
}

// Nodes of the batch behind the layer: its rows and the new nodes, as many as the list takes.
__device__ __forceinline__ void publish_nodes(const FinishArgs& a, int32_t nodes)
{
    a.st->num_dst[a.layer_index + 1] = nodes < a.max_src ? nodes : a.max_src;
}

// The bitmap side of the union step on graphs whose bitmap has a summary.  A tile has far more words than marks there, so
// the marked words are enumerated from the tile's summary words (bit q of them is found by a search over their counts in
// LDS) and read four per thread together, kMarkCap at a time: one read of the summary and one of the marks in the chain,
// where a thread that looked at 32 words of its own in turn made the layer 21 to 29 us long (groups of four on 40 M nodes;
// 9 to 19 us now, bound by the scattered reads and writes per new node).  Most tiles take one pass; others read their words once more
// when the ids are written.
__device__ __forceinline__ void union_sparse_tile(const FinishArgs& a, int32_t tile, int32_t R, int spins, int32_t* smem,
                                                  uint64_t* s_word, int32_t* s_widx, int32_t* s_off)
{
    __shared__ uint64_t s_sum[kMarkTileMax / 64];
    __shared__ int32_t s_pre[kMarkTileMax / 64];
    constexpr int kPer = kMarkCap / kBlock;
    const int T = a.mark_tile_words, S = T / 64;
    const int64_t base = (int64_t) tile * T;
    const int tid = (int) threadIdx.x;
    // the tile's summary words and the number of marked words before each
    const bool has = tid < S && base / 64 + tid < (a.words + 63) / 64;
    const uint64_t mine = has ? a.mark_summary[base / 64 + tid] : 0ull;
    int32_t words;
    const int32_t words_before = block_exclusive_scan(__popcll(mine), smem, &words);
    if (tid < S) { s_sum[tid] = mine; s_pre[tid] = words_before; }
    __syncthreads();
    // marked words p0 .. p0 + kMarkCap - 1 into LDS, four consecutive ones per thread; returns the new nodes among them
    int32_t widx[kPer];
    const uint64_t* seeds = a.seed_mark ? a.seed_mark : a.mark;
    auto load_pass = [&](int32_t p0, int32_t before) -> int32_t {
        uint64_t w[kPer], seed[kPer];
        int32_t cnt = 0, q[kPer], at[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) q[i] = p0 + tid * kPer + i;
        last_not_above(s_pre, S, q, at);                     // last summary word with no more than q marked words before it
        // (no read in a branch, in which it would be waited for: places past the last word read the tile's first)
#pragma unroll
        for (int i = 0; i < kPer; ++i) widx[i] = q[i] < words ? at[i] * 64 + select_bit64(s_sum[at[i]], q[i] - s_pre[at[i]]) : -1;
#pragma unroll
        for (int i = 0; i < kPer; ++i) w[i] = a.mark[base + (widx[i] >= 0 ? widx[i] : 0)];
#pragma unroll
        for (int i = 0; i < kPer; ++i) seed[i] = seeds[base + (widx[i] >= 0 ? widx[i] : 0)];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            if (a.seed_mark) w[i] &= ~seed[i];               // a marked seed is no new node
            if (widx[i] < 0) w[i] = 0ull;
            cnt += __popcll(w[i]);
        }
        int32_t total;
        int32_t off = before + block_exclusive_scan(cnt, smem, &total);
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int k = tid * kPer + i;
            s_word[k] = w[i];
            s_widx[k] = widx[i];
            s_off[k] = off;                                  // words without new nodes share the offset of the next one
            off += __popcll(w[i]);
        }
        return total;
    };
    int32_t total = 0;
    for (int32_t p0 = 0; p0 < words; p0 += kMarkCap) total += load_pass(p0, total);
    const uint32_t tag = launch_tag(a.st, a.layer_index);
    if (tid == 0) publish_sum(a.tile_sums, tile, tag, (uint32_t) total);
    const bool last = tile == a.mark_tiles - 1;
    const int32_t ahead = words <= kMarkCap ? total : 0;     // nodes known from the words in LDS
    __syncthreads();
    NewNodes f;
    find_new(a, s_word, s_widx, s_off, ahead > 0 ? words : 0, base, tid, ahead, f);
    int32_t before = 0;
    if (total > 0 || last)
        before = sum_before(a.tile_sums, tag, tile, spins, smem, [&](int32_t t) { return count_tile(a, t); });
    if (last && tid == 0) publish_nodes(a, R + before + total);
    // the count is out: from here on the marks may go
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    if (has && mine) a.mark_summary[base / 64 + tid] = 0ull;
    int32_t node_lo = 0;
    for (int32_t p0 = 0; p0 < words; p0 += kMarkCap) {
        int32_t in_pass = total;
        if (words > kMarkCap) {
            __syncthreads();                                 // the pass before is still being read
            in_pass = load_pass(p0, node_lo);
            __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            if (widx[i] >= 0) a.mark[base + widx[i]] = 0ull;                 // ready for the next layer
        const int32_t here = words - p0 < kMarkCap ? words - p0 : kMarkCap;
        const int32_t hi = node_lo + in_pass;
        for (int32_t j = node_lo + tid; j - tid < hi; j += kAheadFar * kBlock) {
            if (ahead == 0 || j != tid) find_new(a, s_word, s_widx, s_off, here, base, j, hi, f);
            emit_new_nodes(a, R + before, j, hi, f);
        }
        node_lo = hi;
    }
}

// Sixteen marks of a byte each, 0 or 1, as bits.
__device__ __forceinline__ uint16_t mark_bits(const uint4& m)
{
    auto four = [](uint32_t v) { return v * 0x10204080u >> 28; };             // the lowest bits of four bytes, in order
    return (uint16_t) (four(m.x) | four(m.y) << 4 | four(m.z) << 8 | four(m.w) << 12);
}

// New nodes lo, lo + step, ... below hi of those that `words` words of marks in LDS hold, with the marks before each word beside it;
// `nodes` are those of their slots.  Calls emit(j, node) by the thread.
template <typename F>
__device__ __forceinline__ void each_marked(const uint64_t* bits, const int32_t* before, int32_t words, const int32_t* nodes, int32_t lo, int32_t hi,
                                            int32_t step, F&& emit)
{
    for (int32_t j = lo; j < hi; j += kAheadFar * step) {
        int32_t q[kAheadFar], at[kAheadFar], node[kAheadFar];
#pragma unroll
        for (int i = 0; i < kAheadFar; ++i) q[i] = j + i * step < hi ? j + i * step : hi - 1;
        last_not_above(before, words, q, at);
#pragma unroll
        for (int i = 0; i < kAheadFar; ++i) node[i] = nodes[at[i] * 64 + select_bit64(bits[at[i]], q[i] - before[at[i]])];
#pragma unroll
        for (int i = 0; i < kAheadFar; ++i)
            if (j + i * step < hi) emit(j + i * step, node[i]);
    }
}

// The bitmap side of the union step for a layer that marks by slots (see k_finish_cached) of a cache too large for that one
// launch.  What is before a word of marks is left for the relabel, 16 bytes for 64 slots; the marks stay (the next mini-batch's
// first kernel clears them).
__device__ __forceinline__ void union_slot_tile(const FinishArgs& a, int32_t tile, int32_t R, int spins, int32_t* smem, uint64_t* s_bits,
                                                int32_t* s_before)
{
    const int tid = (int) threadIdx.x;
    const int32_t T = a.slot_tile, base = tile * T, here = a.slots - base < T ? a.slots - base : T;
    const uint4* marks = reinterpret_cast<const uint4*>(a.slot_mark + base);
    uint16_t* bits16 = reinterpret_cast<uint16_t*>(s_bits);
    const int32_t pieces = here / 16, words = here / 64;
    uint4 m[kSlotReads];
#pragma unroll
    for (int x = 0; x < kSlotReads; ++x) {
        const int32_t i = x * kBlock + tid;
        m[x] = marks[i < pieces ? i : pieces - 1];
    }
#pragma unroll
    for (int x = 0; x < kSlotReads; ++x) {
        const int32_t i = x * kBlock + tid;
        if (i < pieces) bits16[i] = mark_bits(m[x]);
    }
    __syncthreads();
    constexpr int kPer = kSlotTile * kSlotReads / 64 / kBlock;
    uint64_t word[kPer];
    int32_t marked = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        word[i] = tid * kPer + i < words ? s_bits[tid * kPer + i] : 0ull;
        marked += __popcll(word[i]);
    }
    int32_t total;
    int32_t run = block_exclusive_scan(marked, smem, &total);
    const uint32_t tag = launch_tag(a.st, a.layer_index);
    if (tid == 0) publish_sum(a.tile_sums, tile, tag, (uint32_t) total);
    const bool last = tile == a.mark_tiles - 1;
    if (total == 0 && !last) return;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        if (tid * kPer + i < words) s_before[tid * kPer + i] = run;
        run += __popcll(word[i]);
    }
    const int32_t before = sum_before(a.tile_sums, tag, tile, spins, smem, [&](int32_t t) {
        uint32_t n = 0;
        for (int32_t i = t * T; i < (t + 1) * T; i += 16)                    // a full tile: one follows
            n += (uint32_t) __popc((uint32_t) mark_bits(*reinterpret_cast<const uint4*>(a.slot_mark + i)));
        return n;
    });
    if (last && tid == 0) publish_nodes(a, R + before + total);
    __syncthreads();
    for (int32_t i = tid; i < words; i += kBlock) a.slot_words[base / 64 + i] = {s_bits[i], before + s_before[i], 0};
    each_marked(s_bits, s_before, words, a.cache_nodes + base, tid, total, kBlock, [&](int32_t j, int32_t node) {
        if (R + before + j < a.max_src) a.src_nodes[R + before + j] = node;
    });
}

// The union step of one layer.  Latency-bound: every block is a chain of a few dependent reads (tile words -> counts of
// other tiles -> offsets of the new nodes), so it is one launch (two, with the tile counts in a launch of their own,
// cost another 4.6 us each, three times per mini-batch), the tiles are small, and new nodes are spread over threads.
// kPerMax: words of a tile per thread at most; 0: the bitmap has a summary (union_sparse_tile); -1: marks are by slot.
template <int kPerMax, bool kOne>
__global__ void __launch_bounds__(kBlock) k_union(LayerArgs g, int spins)
{
    __shared__ int32_t smem[kBlock / kWave + 1];
    const auto [b, block] = group_block<kOne>(g.dealt);
    if (!kOne && block >= g.blocks) return;
    const FinishArgs a = bind_finish(g, b, true);
    // the tile's marked words, kMarkCap at a time: the word, its index in the tile, the number of marks before it
    __shared__ uint64_t s_word[kMarkCap];
    __shared__ int32_t s_widx[kMarkCap];
    __shared__ int32_t s_off[kMarkCap];
    const int32_t R = a.st->num_dst[a.layer_index];
    if (block < a.row_tiles_max) {
        const int64_t base = (int64_t) block * kTile;
        if (base >= R) return;
        // blocked arrangement: thread t owns rows base + t*kItems .. +kItems
        int32_t c[kItems];
        int32_t sum = 0;
        const int64_t r0 = base + (int64_t) threadIdx.x * kItems;
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            c[i] = a.s_cnt[r0 + i < R ? r0 + i : R - 1];
            if (r0 + i >= R) c[i] = 0;
            sum += c[i];
        }
        int32_t total, before;
        int32_t off = block_exclusive_scan(sum, smem, &total);
        if (a.rows_per_sum) {
            before = block_sum_array(a.sums_rows, block * (kTile / a.rows_per_sum), smem);
        } else {
            const uint32_t tag = launch_tag(a.st, a.layer_index);
            if (threadIdx.x == 0) publish_sum(a.row_sums, block, tag, (uint32_t) total);
            before = sum_before(a.row_sums, tag, block, spins, smem, [&](int32_t t) {
                uint32_t n = 0;
                for (int32_t r = t * kTile; r < (t + 1) * kTile; ++r) n += (uint32_t) a.s_cnt[r];      // a full tile: one follows
                return n;
            });
        }
        off += before;
        if (base + kTile >= R && threadIdx.x == 0) {
            a.st->num_edges[a.layer_index] = before + total;
            a.indptr[R] = before + total;
        }
#pragma unroll
        for (int i = 0; i < kItems; ++i) {
            if (r0 + i < R) a.indptr[r0 + i] = off;
            off += c[i];
        }
    } else if constexpr (kPerMax < 0) {
        union_slot_tile(a, block - a.row_tiles_max, R, spins, smem, s_word, s_off);
    } else if constexpr (kPerMax == 0) {
        union_sparse_tile(a, block - a.row_tiles_max, R, spins, smem, s_word, s_widx, s_off);
    } else {
        const int32_t tile = block - a.row_tiles_max;
        const int T = a.mark_tile_words;
        const int64_t base = (int64_t) tile * T;
        // thread t owns words t*per .. t*per+per-1 of the tile (per = 1 for tiles of up to kBlock words)
        const int per = T > kBlock ? T / kBlock : 1;
        const int first = (int) threadIdx.x * per;
        uint64_t word[kPerMax];
        load_marks<kPerMax>(a, base, first, per, T, word);
        uint64_t seeds[kPerMax];                                         // a marked seed is no new node
#pragma unroll
        for (int i = 0; i < kPerMax; ++i) seeds[i] = 0ull;
        if (a.seed_mark) {
#pragma unroll
            for (int i = 0; i < kPerMax; ++i) {
                const int64_t w = base + first + i;
                if (i < per && first + i < T && w < a.words) seeds[i] = a.seed_mark[w];
            }
        }
        uint32_t marked = 0;                                             // words to clear
        int32_t cnt = 0, nz = 0;
#pragma unroll
        for (int i = 0; i < kPerMax; ++i) {
            if (word[i]) marked |= 1u << i;
            word[i] &= ~seeds[i];
            cnt += __popcll(word[i]);
            nz += word[i] ? 1 : 0;
        }
        int32_t total, total_nz;
        const int32_t off = block_exclusive_scan(cnt, smem, &total);        // marks before this thread's words
        const uint32_t tag = launch_tag(a.st, a.layer_index);
        if (threadIdx.x == 0) publish_sum(a.tile_sums, tile, tag, (uint32_t) total);
        const bool last = tile == a.mark_tiles - 1;
        const int32_t widx = block_exclusive_scan(nz, smem, &total_nz);     // marked words before this thread's words
        // The marked words go through LDS in order, kMarkCap at a time (most tiles need one pass).
        auto fill = [&](int32_t p0) {
            int32_t my = widx, my_off = off;
#pragma unroll
            for (int i = 0; i < kPerMax; ++i) {
                if (word[i]) {
                    if (my >= p0 && my < p0 + kMarkCap) {
                        s_word[my - p0] = word[i];
                        s_widx[my - p0] = first + i;
                        s_off[my - p0] = my_off;
                    }
                    ++my;
                    my_off += __popcll(word[i]);
                }
            }
        };
        fill(0);
        __syncthreads();
        const int tid = (int) threadIdx.x;
        int32_t in_pass = total_nz < kMarkCap ? total_nz : kMarkCap;
        int32_t node_hi = total_nz > 0 ? s_off[in_pass - 1] + __popcll(s_word[in_pass - 1]) : 0;
        uint32_t node[kAhead];
        RowExtent ext[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            const int32_t j = i * kBlock + tid;
            node[i] = node_hi > 0 ? new_node(s_word, s_widx, s_off, in_pass, base, j < node_hi ? j : node_hi - 1) : 0u;
            ext[i] = extent_of(a, node[i]);
        }
        int32_t before = 0;
        if (total > 0 || last) before = sum_before(a.tile_sums, tag, tile, spins, smem, [&](int32_t t) { return count_tile(a, t); });
        if (last && tid == 0) publish_nodes(a, R + before + total);
        // The count is out (its store is older than the reads that sum_before waited for, or than the barriers of the
        // scan above): from here on the marks may go.
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kPerMax; ++i)
            if (marked & (1u << i)) a.mark[base + first + i] = 0ull;         // ready for the next layer
        if (total == 0) return;
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            if (i * kBlock + tid < node_hi) emit_new_node(a, R + before + i * kBlock + tid, node[i], ext[i]);
        // the others, one thread per new node
        for (int32_t p0 = 0, j = kAhead * kBlock + tid;;) {
            for (; j < node_hi; j += kBlock) {
                const uint32_t u = new_node(s_word, s_widx, s_off, in_pass, base, j);
                emit_new_node(a, R + before + j, u, new_extent(a, u));
            }
            p0 += kMarkCap;
            if (p0 >= total_nz) break;
            __syncthreads();
            fill(p0);
            __syncthreads();
            in_pass = total_nz - p0 < kMarkCap ? total_nz - p0 : kMarkCap;
            j = s_off[0] + tid;
            node_hi = s_off[in_pass - 1] + __popcll(s_word[in_pass - 1]);
        }
    }
}

void fill_finish_template(const Group& g, int layer_index, FinishArgs* out)
{
    const gns_ctx* c = g.ctx[0];
    const Layout& L = c->lay;
    FinishArgs& a = *out;
    memset(&a, 0, sizeof(a));
    a.layer_index = layer_index;
    a.fanout = c->config.fanout[layer_index];
    a.words = L.words;
    a.marks_seeds = layer_index == 0 && first_layer_enters_seeds(c->config) ? 1 : 0;
    a.rows_per_sum = rows_per_sum(g, layer_index);
    a.inv_fanout = 1.0 / (double) a.fanout;
    a.unit_weights = c->config.policy[layer_index] == GNS_UNIFORM ? 1 : 0;
    a.row_tiles_max = (int32_t) ((g.rows[layer_index] + kTile - 1) / kTile);
    a.mark_tiles = (int32_t) L.mark_tiles;
    a.mark_tile_words = L.mark_tile_words;
    a.g_indptr = c->graph.indptr;
    a.g_i64 = c->graph.indptr_is_i64;
    a.num_nodes = c->graph.num_nodes;
    a.last_layer = layer_index == c->config.num_layers - 1 ? 1 : 0;
    a.max_src = (int32_t) L.rows[layer_index + 1];
    a.by_slot = L.slot_marks && a.last_layer ? 1 : 0;
    if (a.by_slot) {
        a.slots = (int32_t) L.slot_marks;
        a.slot_tile = L.slot_tile;
        a.mark_tiles = (a.slots + a.slot_tile - 1) / a.slot_tile;
        a.cache_nodes = cache_ptr<int32_t>(c, L.cache_nodes, 0);
    }
}

int relabel_grid(const Group& g, int layer_index)
{
    const gns_ctx* c = g.ctx[0];
    const int64_t max_slots = g.rows[layer_index] * (int64_t) c->config.fanout[layer_index];
    int64_t rb = (max_slots + kBlock * kRelabelUnroll - 1) / (kBlock * kRelabelUnroll);
    if (rb > (int64_t) c->num_cus * 2) rb = (int64_t) c->num_cus * 2;
    if (rb < 1) rb = 1;
    return (int) rb;
}

// The union step of a layer (the relabel rides with the next layer's first kernel).
hipError_t launch_finish_layer(const Group& g, int layer_index, hipStream_t s)
{
    gns_ctx* c = g.ctx[0];
    LayerArgs a;
    fill_group_args(g, &a);
    set_group_layer(g, layer_index, &a);
    fill_finish_template(g, layer_index, &a.f);
    a.blocks = a.f.row_tiles_max + a.f.mark_tiles;
    const dim3 grid = group_grid(g, a, a.blocks);
    // by summary, or by words of a tile per thread: the kernel's loops over them are unrolled for 1, 4 or 32
    const int per = a.f.mark_tile_words / kBlock, spins = c->union_spins;
    with_one(g, [&](auto kOne) {
        constexpr bool one = decltype(kOne)::value;
        if (a.f.by_slot) hipLaunchKernelGGL((k_union<-1, one>), grid, dim3(kBlock), 0, s, a, spins);
        else if (a.off.has_summary) hipLaunchKernelGGL((k_union<0, one>), grid, dim3(kBlock), 0, s, a, spins);
        else if (per <= 1) hipLaunchKernelGGL((k_union<1, one>), grid, dim3(kBlock), 0, s, a, spins);
        else if (per <= 4) hipLaunchKernelGGL((k_union<4, one>), grid, dim3(kBlock), 0, s, a, spins);
        else               hipLaunchKernelGGL((k_union<kMarkTileMax / kBlock, one>), grid, dim3(kBlock), 0, s, a, spins);
    });
    return hipGetLastError();
}

// What the last launch of a batch does besides: the seed bitmap left empty for the next mini-batch, and the counts written to the
// context's pinned host mirror, where gns_sample_blocks_wait finds them.  By one block; `nodes` and `edges` are the last layer's.
__device__ __forceinline__ void clear_seed_marks(const LayerArgs& g, int b, const FinishArgs& a)
{
    char* ws = g.b[b].ws;
    const int32_t* seeds = at<int32_t>(ws, g.off.seed_copy);
    uint64_t* seed_mark = at<uint64_t>(ws, g.off.seed_mark);
    for (int32_t i = (int32_t) threadIdx.x; g.off.marks_seeds && i < a.st->num_dst[0]; i += kBlock)
        if (seeds[i] >= 0 && (int64_t) seeds[i] < a.num_nodes) seed_mark[seeds[i] >> 6] = 0ull;
}

__device__ __forceinline__ void report_counts(const LayerArgs& g, int b, const FinishArgs& a, int32_t nodes, int32_t edges)
{
    DeviceState* host = g.b[b].host;
    const int i = (int) threadIdx.x;
    if (i <= GNS_MAX_LAYERS) host->num_dst[i] = i == a.layer_index + 1 ? nodes : a.st->num_dst[i];
    if (i < GNS_MAX_LAYERS) host->num_edges[i] = i == a.layer_index ? edges : a.st->num_edges[i];
    if (i == 0) host->bad_seed = a.st->bad_seed;
}

// The last layer's relabel has no following sampler to ride with.
template <bool kOne>
__global__ void __launch_bounds__(kBlock) k_relabel_last(LayerArgs g)
{
    const auto [b, block] = group_block<kOne>(g.dealt);
    if (!kOne && block >= g.blocks) return;
    const FinishArgs a = bind_finish(g, b, true);
    relabel_body(a, block, g.blocks);
    if (block == 0) {
        clear_seed_marks(g, b, a);
        report_counts(g, b, a, a.st->num_dst[a.layer_index + 1], a.st->num_edges[a.layer_index]);
    }
}

hipError_t launch_relabel(const Group& g, int layer_index, hipStream_t s)
{
    LayerArgs a;
    fill_group_args(g, &a);
    set_group_layer(g, layer_index, &a);
    fill_finish_template(g, layer_index, &a.f);
    a.blocks = relabel_grid(g, layer_index);
    with_one(g, [&](auto kOne) { hipLaunchKernelGGL(k_relabel_last<decltype(kOne)::value>, group_grid(g, a, a.blocks), dim3(kBlock), 0, s, a); });
    return hipGetLastError();
}

// Union and relabel of an input layer that samples from the cache only, in one launch.  Its new nodes are cached nodes, which the
// sampler has marked by their slots, a byte each with a plain store; slots ascend with node ids.  So a block reads all marks, knows from
// them how many come before each slot, and needs nothing of any other block: it relabels and compacts its kBlock rows, and the blocks
// share out the list of the new nodes.  Latency-bound: rows, edges and marks are read at once, and what follows is in LDS.
// Every block reads all marks, which sets the line for the cache's size (kSlotsMax, 64 KB: a mini-batch of 13 blocks 10.1 us where 35 K
// slots take 9.4 and 10 K 7.2, against 8.7 + 3.2, 5.8 + 3.8 and 5.9 + 4.4 with marks in the bitmap of all nodes and two launches, whose gap
// comes on top); larger caches have union_slot_tile and k_relabel_last.
// Groups of four on 1 M nodes (10 K cached) 9.1 + 9.4 -> 11.2 us and the sampler 37.6 -> 37.6, on 6.5 M nodes (65 K cached) 11.4 + 7.8 ->
// 11.9 and the sampler 39.7 -> 27.0: its marks were atomics, two each, carried out at the memory.  On 40 M nodes (400 K cached)
// sampler, union and relabel 54 + 17.1 + 11.7 -> 45.4 + 10.7 + 9.3.
constexpr int kFinishFlight = 6;                 // edges of a thread on their way

template <bool kOne>
__global__ void __launch_bounds__(kBlock) k_finish_cached(LayerArgs g)
{
    __shared__ uint64_t s_sums[kBlock / kWave];
    __shared__ int32_t s_part[kBlock / kWave];
    __shared__ uint64_t s_bits[kSlotsMax / 64];
    __shared__ int32_t s_before[kSlotsMax / 64];
    __shared__ int32_t s_off[kBlock], s_num[kBlock];
    const auto [b, block] = group_block<kOne>(g.dealt);
    if (!kOne && block >= g.blocks) return;
    const FinishArgs a = bind_finish(g, b, true);
    const int32_t R = a.st->num_dst[a.layer_index];
    const int32_t base = block * kBlock;
    if (base >= R) return;
    const int tid = (int) threadIdx.x;
    const int32_t k = a.fanout, rows = R - base < kBlock ? R - base : kBlock, items = rows * k;
    const int32_t first = base * k;                              // below 2^31: checked when the workspace is sized
    const int32_t num = tid < rows ? a.s_cnt[base + tid] : 0;
    // the batch begins with its seeds: a bit of the seed bitmap per row to clear
    int32_t marked_seed = -1;
    if (g.off.marks_seeds && base + tid < a.st->num_dst[0]) marked_seed = at<int32_t>(g.b[b].ws, g.off.seed_copy)[base + tid];
    if ((int64_t) marked_seed >= a.num_nodes) marked_seed = -1;
    int32_t u[kFinishFlight];
    float w[kFinishFlight];
    auto load = [&](int32_t q0) {
#pragma unroll
        for (int i = 0; i < kFinishFlight; ++i) {
            const int32_t j = (q0 + i) * kBlock + tid, t = first + (j < items ? j : items - 1);
            u[i] = a.s_nbr[t];
            w[i] = a.s_w[t];
        }
    };
    load(0);
    // marks: sixteen slots a read, 0 or 1 each, into bits; a thread's reads are on their way together
    const uint4* marks = reinterpret_cast<const uint4*>(a.slot_mark);
    uint16_t* bits16 = reinterpret_cast<uint16_t*>(s_bits);
    const int32_t pieces = a.slots / 16;
    auto bits_of = [&](auto reads) {
        constexpr int kReads = decltype(reads)::value;
        for (int32_t i0 = tid; i0 < pieces; i0 += kReads * kBlock) {
            uint4 m[kReads];
#pragma unroll
            for (int x = 0; x < kReads; ++x) {
                const int32_t i = i0 + x * kBlock;
                m[x] = marks[i < pieces ? i : pieces - 1];
            }
#pragma unroll
            for (int x = 0; x < kReads; ++x) {
                const int32_t i = i0 + x * kBlock;
                if (i < pieces) bits16[i] = mark_bits(m[x]);
            }
        }
    };
    if (pieces <= kBlock)          bits_of(std::integral_constant<int, 1>());
    else if (pieces <= 3 * kBlock) bits_of(std::integral_constant<int, 3>());
    else                           bits_of(std::integral_constant<int, 8>());
    int32_t part = 0;                                            // samples of the rows before
    for (int32_t t = tid; t < block * (kBlock / a.rows_per_sum); t += kBlock) part += a.sums_rows[t];
    __syncthreads();
    // Places of the rows' edges and of the words' marks by one scan, each a half of 64 bits.
    const int32_t words = a.slots / 64, per = (words + kBlock - 1) / kBlock;
    int32_t marked = 0;
    for (int32_t i = tid * per; i < (tid + 1) * per && i < words; ++i) marked += __popcll(s_bits[i]);
    const int lane = opaque_lane_id(), wave = opaque(tid >> 6);
    const uint64_t own = (uint64_t) (uint32_t) marked << 32 | (uint32_t) num;
    const uint64_t sums = wave_inclusive_scan64(own);
    part = wave_sum(part);
    if (lane == kWave - 1) { s_sums[wave] = sums; s_part[wave] = part; }
    __syncthreads();
    uint64_t all = 0, start = sums - own;
    int32_t before = 0;
#pragma unroll
    for (int x = 0; x < kBlock / kWave; ++x) {
        if (x < wave) start += s_sums[x];
        all += s_sums[x];
        before += s_part[x];
    }
    const int32_t total = (int32_t) (uint32_t) all, fresh = (int32_t) (all >> 32);
    s_off[tid] = (int32_t) (uint32_t) start;
    s_num[tid] = num;
    int32_t run = (int32_t) (start >> 32);
    for (int32_t i = tid * per; i < (tid + 1) * per && i < words; ++i) {
        s_before[i] = run;
        run += __popcll(s_bits[i]);
    }
    __syncthreads();
    if (tid < rows) a.indptr[base + tid] = before + s_off[tid];
    for (int32_t q0 = 0; q0 < k; q0 += kFinishFlight) {
        if (q0 > 0) load(q0);
        // (all that LDS is asked for first, whether or not an edge is there)
        int32_t o[kFinishFlight], local[kFinishFlight];
        bool ok[kFinishFlight];
#pragma unroll
        for (int i = 0; i < kFinishFlight; ++i) {
            const int32_t j = (q0 + i) * kBlock + tid, jc = j < items ? j : items - 1;
            const int32_t row = (int32_t) (((float) jc + 0.5f) * (float) a.inv_fanout);        // jc / k: exact below 2^16
            const int32_t s = jc - row * k, slot = u[i] >= 0 ? u[i] : 0;
            ok[i] = j < items && s < s_num[row];
            o[i] = before + s_off[row] + s;
            const int32_t word = ok[i] ? slot >> 6 : 0;                  // (places without an edge hold anything)
            local[i] = R + s_before[word] + __popcll(s_bits[word] & bits_below(slot));
        }
#pragma unroll
        for (int i = 0; i < kFinishFlight; ++i) {
            if (!ok[i]) continue;
            a.indices[o[i]] = u[i] >= 0 ? local[i] : -1 - u[i];
            a.weights[o[i]] = w[i];
        }
    }
    // the new nodes: a wave per word of marks, or where blocks are few by all their threads
    const int32_t blocks = (R + kBlock - 1) / kBlock, w0 = block * (kBlock / kWave) + wave;
    auto emit = [&](int32_t n, int32_t node) {
        if (R + n < a.max_src) a.src_nodes[R + n] = node;
    };
    if (words <= blocks * (kBlock / kWave)) {
        if (w0 < words && (s_bits[w0] >> lane & 1ull)) emit(s_before[w0] + __popcll(s_bits[w0] & bits_below(lane)), a.cache_nodes[w0 * 64 + lane]);
    } else {
        each_marked(s_bits, s_before, words, a.cache_nodes, base + tid, fresh, blocks * kBlock, emit);
    }
    if (marked_seed >= 0) at<uint64_t>(g.b[b].ws, g.off.seed_mark)[marked_seed >> 6] = 0ull;
    if (base + kBlock >= R) {
        const int32_t nodes = R + fresh < a.max_src ? R + fresh : a.max_src, edges = before + total;
        if (tid == 0) {
            a.indptr[R] = edges;
            a.st->num_edges[a.layer_index] = edges;
            a.st->num_dst[a.layer_index + 1] = nodes;
        }
        report_counts(g, b, a, nodes, edges);
    }
}

hipError_t launch_finish_cached(const Group& g, hipStream_t s)
{
    gns_ctx* c = g.ctx[0];
    const int layer_index = c->config.num_layers - 1;
    LayerArgs a;
    fill_group_args(g, &a);
    set_group_layer(g, layer_index, &a);
    fill_finish_template(g, layer_index, &a.f);
    a.blocks = (int32_t) ((g.rows[layer_index] + kBlock - 1) / kBlock);
    with_one(g, [&](auto kOne) { hipLaunchKernelGGL(k_finish_cached<decltype(kOne)::value>, group_grid(g, a, a.blocks), dim3(kBlock), 0, s, a); });
    return hipGetLastError();
}

}  // namespace gns
