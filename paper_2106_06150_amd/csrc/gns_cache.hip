// The periodic global node cache (paper Section 3.2, Eq. (1); Theorem 1: the
// cache is drawn without replacement and has |C| nodes).
//
// The cache is the set of the first |C| distinct nodes of an i.i.d. stream in
// which node i appears with probability deg(i)/nnz: draw j picks a CSR entry
// uniformly with a Philox word pair and takes the row that owns it.  The
// stream is processed in chunks; a small hash map keeps, per drawn node, the
// smallest stream index at which it appeared (atomicMin), which makes "draw j
// is the first occurrence of its node" a pure function of the stream and
// independent of thread order.  First occurrences are counted with a prefix
// sum over the blocks of one launch; the chunk in which the count reaches |C|
// is cut at exactly that draw.
//
// On graphs of a million nodes a draw is a chain of small launches, so there are few: clear, then two per chunk (draw,
// commit), then the index with the 1/p^C table and on large graphs the filter's groups; and the host looks at the outcome behind
// the first chunk or two and all of it, once for most caches, then behind two more at a time.  What follows an incomplete cache stands down on the device: half of 1 M
// nodes take 358 us, 16 M of 40 M nodes 11.0 ms.
// A draw of 10 K of 1 M nodes with the mini-batch behind it: 228 us, where a launch per phase, a read-back per chunk of 64 K
// draws and searches over all offsets took 50 us more; 400 K of 40 M nodes: 1420 us.
#include "gns_internal.h"
#include "gns_device.hpp"
#include <string.h>

namespace gns {

// ---------------------------------------------------------------------------
// Graph validation at create time: offsets non-decreasing, ids in range, rows
// strictly ascending; also counts the rows with at least one neighbor.
struct ValidateOut {
    int32_t nonzero_rows;
    int32_t bad_offsets;
    int32_t bad_index;
    int32_t unsorted;
};

template <typename OffT>
__global__ void __launch_bounds__(kBlock) k_validate_graph(const void* indptr, const int32_t* indices, int64_t n,
                                                           int64_t nnz, int32_t* entry_rows, ValidateOut* out)
{
    __shared__ int32_t smem[kBlock / kWave + 1];
    int32_t nonzero = 0;
    for (int64_t v = (int64_t) blockIdx.x * blockDim.x + threadIdx.x; v < n; v += (int64_t) gridDim.x * blockDim.x) {
        const int64_t b = load_off<OffT>(indptr, v), e = load_off<OffT>(indptr, v + 1);
        if (b < 0 || e < b || e > nnz || (v == 0 && b != 0) || (v == n - 1 && e != nnz)) { out->bad_offsets = 1; continue; }
        if (e > b) ++nonzero;
        if (entry_rows)
            for (int64_t i = (b + 63) >> 6; (i << 6) < e; ++i) entry_rows[i] = (int32_t) v;
        int32_t prev = -1;
        for (int64_t q = b; q < e; ++q) {
            const int32_t u = indices[q];
            if (u < 0 || (int64_t) u >= n) out->bad_index = 1;
            if (u <= prev) out->unsorted = 1;
            prev = u;
        }
    }
    nonzero = block_sum(nonzero, smem);
    if (threadIdx.x == 0 && nonzero) atomicAdd(&out->nonzero_rows, nonzero);
}

hipError_t launch_count_nonzero_rows(gns_ctx* c, hipStream_t s, int32_t* d_out)
{
    const int64_t n = c->graph.num_nodes;
    int64_t blocks = (n + kBlock - 1) / kBlock;
    if (blocks > (int64_t) c->num_cus * 32) blocks = (int64_t) c->num_cus * 32;
    hipError_t e = launch_fill_u32(reinterpret_cast<uint32_t*>(d_out), 4, 0u, s);
    if (e != hipSuccess) return e;
    ValidateOut* out = reinterpret_cast<ValidateOut*>(d_out);
    int32_t* entry_rows = c->lay.entry_rows ? ws_ptr<int32_t>(c, c->lay.entry_rows) : nullptr;
    if (c->graph.indptr_is_i64)
        hipLaunchKernelGGL((k_validate_graph<int64_t>), dim3((unsigned) blocks), dim3(kBlock), 0, s, c->graph.indptr,
                           c->graph.indices, n, c->graph.num_entries, entry_rows, out);
    else
        hipLaunchKernelGGL((k_validate_graph<int32_t>), dim3((unsigned) blocks), dim3(kBlock), 0, s, c->graph.indptr,
                           c->graph.indices, n, c->graph.num_entries, entry_rows, out);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
struct DrawArgs {
    DeviceState* st;
    DeviceState* host;         // pinned: draw_done_chunk and cut_draw are left here too
    const void* indptr;
    int64_t n;
    uint64_t nnz;
    const int32_t* entry_rows; // row that owns entry 64 * i, or null
    uint32_t key0, key1, epoch;
    uint64_t j0;               // stream index of the chunk's first draw
    int32_t count;             // draws in this chunk
    unsigned long long* table; // draw hash: node in the upper half, smallest stream index seen for it below (~0 = empty)
    uint32_t hmask, hshift;
    int32_t* draw_slot;        // [chunk] slot of the node in the draw hash
    unsigned long long* sums;  // [tiles] (tag, first occurrences of the tile), see sum_before
    uint32_t tag;
    int32_t spins;
    uint64_t* cache_bitmap;
    int64_t words;
    unsigned long long* filter;    // the cache filter's keys, or null
    int64_t cache_size;
    int32_t chunk_index;       // chunks of one draw are numbered from 0
};

// A draw enqueues its chunks without knowing how many it needs: the chunk that completes the cache says
// so in the device state and every later chunk stands down.
__device__ __forceinline__ bool chunk_stands_down(const DrawArgs& a)
{
    const int32_t done = a.st->draw_done_chunk;
    return done >= 0 && done < a.chunk_index;
}

// What a draw begins with: an empty bitmap, an empty hash, nothing drawn.
__global__ void __launch_bounds__(kBlock) k_cache_clear(DrawArgs a)
{
    const int64_t t = (int64_t) blockIdx.x * kBlock + threadIdx.x, stride = (int64_t) gridDim.x * kBlock;
    if (t == 0) {
        a.st->draw_distinct[0] = 0;
        a.st->draw_done_chunk = -1;
        __hip_atomic_store(&a.host->draw_done_chunk, -1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    for (int64_t i = t; i < a.words; i += stride) a.cache_bitmap[i] = 0ull;
    for (int64_t i = t; i <= (int64_t) a.hmask; i += stride) a.table[i] = ~0ull;
    for (int64_t i = t; a.filter && i < kFilterHot; i += stride) a.filter[i] = 0ull;
}

// the unique row i in [lo, hi) with indptr[i] <= e < indptr[i+1]
template <typename OffT>
__device__ __forceinline__ int64_t owner_row(const void* indptr, int64_t lo, int64_t hi, int64_t e)
{
    while (hi - lo > 1) {
        const int64_t mid = lo + ((hi - lo) >> 1);
        if (load_off<OffT>(indptr, mid) <= e) lo = mid; else hi = mid;
    }
    return lo;
}

// Bound by the chain of reads that finds an entry's row: over the whole of the offsets 20 reads on a graph of 1 M nodes and
// 26 on one of 40 M, the last dozen of them to memory.  The table of every 64th entry's row leaves the few rows in between.
template <typename OffT>
__global__ void __launch_bounds__(kBlock) k_cache_draw(DrawArgs a)
{
    const int32_t t = (int32_t) (blockIdx.x * blockDim.x + threadIdx.x);
    if (t >= a.count || chunk_stands_down(a)) return;
    const uint64_t j = a.j0 + (uint64_t) t;
    const Philox4 r = philox4x32_10((uint32_t) j, (uint32_t) (j >> 32), a.epoch, kTagCache, a.key0, a.key1);
    const uint64_t r64 = ((uint64_t) r.w[1] << 32) | (uint64_t) r.w[0];
    const uint64_t e = __umul64hi(r64, a.nnz);                      // uniform CSR entry
    int64_t lo = 0, hi = a.n;
    if (a.entry_rows) {
        const uint64_t i = e >> 6, last = (a.nnz - 1) >> 6;
        lo = a.entry_rows[i];
        if (i < last) hi = (int64_t) a.entry_rows[i + 1] + 1;
    }
    const uint32_t node = (uint32_t) owner_row<OffT>(a.indptr, lo, hi, (int64_t) e);
    const unsigned long long mine = ((unsigned long long) node << 32) | (uint32_t) j;
    uint32_t h = hash_start(node, a.hshift);
    for (uint32_t probe = 0; probe <= a.hmask; ++probe) {
        const unsigned long long old = atomicCAS(&a.table[h], ~0ull, mine);
        if (old == ~0ull) break;
        if ((uint32_t) (old >> 32) == node) {
            if (old > mine) atomicMin(&a.table[h], mine);
            break;
        }
        h = (h + 1) & a.hmask;
    }
    a.draw_slot[t] = (int32_t) h;
}

// The draws of a chunk that are the first of their node, counted in stream order, enter the cache until it is full.
__global__ void __launch_bounds__(kBlock) k_cache_commit(DrawArgs a)
{
    __shared__ int32_t smem[kBlock / kWave + 1];
    constexpr int kPer = kDrawTile / kBlock;
    if (chunk_stands_down(a)) return;
    const int32_t tile = (int32_t) blockIdx.x;
    const int32_t t0 = tile * kDrawTile + (int32_t) threadIdx.x * kPer;
    // node of draw t if it is the node's first, else -1
    auto first_of = [&](int32_t t) -> int32_t {
        if (t >= a.count) return -1;
        const unsigned long long x = a.table[a.draw_slot[t]];
        return (uint32_t) x == (uint32_t) (a.j0 + (uint64_t) t) ? (int32_t) (x >> 32) : -1;
    };
    int32_t node[kPer];
    int32_t sum = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) { node[i] = first_of(t0 + i); sum += node[i] >= 0 ? 1 : 0; }
    int32_t total;
    const int32_t off = block_exclusive_scan(sum, smem, &total);
    if (threadIdx.x == 0) publish_sum(a.sums, tile, a.tag, (uint32_t) total);
    const int32_t before = sum_before(a.sums, a.tag, tile, a.spins, smem, [&](int32_t t) {
        uint32_t c = 0;
        for (int32_t q = t * kDrawTile; q < (t + 1) * kDrawTile; ++q) c += first_of(q) >= 0 ? 1u : 0u;
        return c;
    });
    // how many more the cache takes; this chunk's blocks read one of the two counts, its last block writes the other
    const int64_t have = (int64_t) a.st->draw_distinct[a.chunk_index & 1];
    const int64_t need = a.cache_size - have;
    int64_t g = (int64_t) before + off;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        if (node[i] < 0) continue;
        if (g < need) {
            atomicOr(reinterpret_cast<unsigned long long*>(&a.cache_bitmap[node[i] >> 6]), 1ull << (node[i] & 63));
            if (g == need - 1) {
                a.st->cut_draw = a.j0 + (uint64_t) (t0 + i);
                __hip_atomic_store(&a.host->cut_draw, (unsigned long long) (a.j0 + (uint64_t) (t0 + i)), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_SYSTEM);
            }
        }
        ++g;
    }
    if (tile == (int32_t) gridDim.x - 1 && threadIdx.x == 0) {
        const int64_t all = (int64_t) before + total;
        a.st->draw_distinct[(a.chunk_index + 1) & 1] = (int32_t) (have + (all < need ? all : need));
        if (all >= need) {
            a.st->draw_done_chunk = a.chunk_index;
            __hip_atomic_store(&a.host->draw_done_chunk, a.chunk_index, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        }
    }
}

// ---------------------------------------------------------------------------
// From the finished bitmap: the rank index, the ascending node list, and Section 3.4 for every node of the cache:
// p_u = deg(u)/nnz, p^C_u = 1 - (1 - p_u)^|C| (expm1/log1p keep a tiny p_u exact), stored as 1/p^C_u in fp32.  The table
// is indexed by node id; entries of nodes outside the current cache are stale and never read.
struct IndexArgs {
    const int32_t* done;       // the draw's completing chunk, or null: below zero the cache is incomplete and there is nothing to do
    const uint64_t* bitmap;
    int64_t words;
    unsigned long long* sums;  // [tiles] (tag, nodes of the tile), see sum_before
    uint32_t tag;
    int32_t spins;
    int32_t* word_prefix;
    int32_t* cache_nodes;
    int64_t cache_size;
    const void* prob_prefix;
    int64_t prob_total;
    float* node_inv_pc;        // or
    CachedNode* node_slot;     //   this, and the other null
    CacheFilter filter;        // or null pointers
    int64_t hot_from;          // rows shorter than this stay out of its slots
    const void* g_indptr;      // the graph's offsets (the filter goes by row lengths whatever the probability)
    int g_i64;
};

// A tile is kPer words per thread.  Latency-bound: one word per thread and many blocks while their number stays small
// enough for every block to add up the sums of the others, then the nodes of the tile over all threads.
template <typename OffT, int kPer>
__global__ void __launch_bounds__(kBlock) k_cache_index(IndexArgs a)
{
    __shared__ int32_t smem[kBlock / kWave + 1];
    if (a.done && *a.done < 0) return;
    const int32_t tile = (int32_t) blockIdx.x;
    const int64_t w0 = ((int64_t) tile * kBlock + threadIdx.x) * kPer;
    uint64_t word[kPer];
    int32_t sum = 0;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        word[i] = (w0 + i < a.words) ? a.bitmap[w0 + i] : 0ull;
        sum += __popcll(word[i]);
    }
    int32_t total;
    const int32_t off = block_exclusive_scan(sum, smem, &total);
    if (threadIdx.x == 0) publish_sum(a.sums, tile, a.tag, (uint32_t) total);
    const int32_t before = sum_before(a.sums, a.tag, tile, a.spins, smem, [&](int32_t t) {
        uint32_t c = 0;
        const int64_t first = (int64_t) t * kBlock * kPer;
        for (int64_t w = first; w < first + kBlock * kPer && w < a.words; ++w) c += (uint32_t) __popcll(a.bitmap[w]);
        return c;
    });
    int32_t pos = before + off;
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
        if (w0 + i < a.words) {
            a.word_prefix[w0 + i] = pos;
            uint64_t rest = word[i];
            while (rest) {
                const int bit = __builtin_ctzll(rest);
                rest &= rest - 1;
                a.cache_nodes[pos++] = (int32_t) ((w0 + i) * 64 + bit);
            }
        }
    }
    __syncthreads();                                     // the tile's part of the list is read back by other threads
    for (int32_t i = (int32_t) threadIdx.x; i < total; i += kBlock) {
        const int32_t u = a.cache_nodes[before + i];
        const int64_t deg = load_off<OffT>(a.prob_prefix, (int64_t) u + 1) - load_off<OffT>(a.prob_prefix, u);
        const double p = (double) deg / (double) a.prob_total;
        const double pc = (p >= 1.0) ? 1.0 : -expm1((double) a.cache_size * log1p(-p));
        const float inv_pc = (float) (1.0 / pc);
        if (a.node_slot) a.node_slot[u] = {inv_pc, before + i};
        else             a.node_inv_pc[u] = inv_pc;
        if (a.filter.keys) {
            const int64_t len = load_off_rt(a.g_indptr, a.g_i64, (int64_t) u + 1) - load_off_rt(a.g_indptr, a.g_i64, u);
            const unsigned long long key = ((unsigned long long) (len < 0xFFFFFFFFll ? len : 0xFFFFFFFFll) << 32) | (uint32_t) u;
            unsigned long long* slot = &a.filter.keys[(uint32_t) u % kFilterHot];
            if (len >= a.hot_from && key > *slot) atomicMax(slot, key);
        }
    }
}

template <typename OffT>
static void launch_cache_index(const IndexArgs& a, hipStream_t s)
{
    auto grid = [&](int per) { return dim3((unsigned) ((a.words + (int64_t) kBlock * per - 1) / ((int64_t) kBlock * per))); };
    if (a.words <= 1024 * kBlock / 4)      hipLaunchKernelGGL((k_cache_index<OffT, 1>), grid(1), dim3(kBlock), 0, s, a);
    else if (a.words <= 1024 * kBlock * 4) hipLaunchKernelGGL((k_cache_index<OffT, 4>), grid(4), dim3(kBlock), 0, s, a);
    else                                   hipLaunchKernelGGL((k_cache_index<OffT, 16>), grid(16), dim3(kBlock), 0, s, a);
}

// Coarse companion of the cache bitmap: bit g of the result is set iff some node of
// [g << shift, (g + 1) << shift) is cached.  One lane per coarse bit; a wave's ballot is a coarse word.
__global__ void __launch_bounds__(kBlock) k_cache_coarse(const int32_t* done, const uint64_t* bitmap, int64_t words, int shift,
                                                         uint64_t* coarse, int64_t coarse_words)
{
    if (done && *done < 0) return;
    const int64_t cw = (int64_t) blockIdx.x * (kBlock / kWave) + (threadIdx.x >> 6);
    if (cw >= coarse_words) return;
    const int64_t g = cw * kWave + lane_id();
    bool any = false;
    if (shift >= 6) {
        const int64_t first = g << (shift - 6), last = (g + 1) << (shift - 6);
        for (int64_t w = first; w < last && w < words; ++w) any = any || bitmap[w] != 0ull;
    } else {
        const int64_t w = g >> (6 - shift);
        const uint64_t mask = (1ull << (1 << shift)) - 1ull;
        any = w < words && ((bitmap[w] >> ((g << shift) & 63)) & mask) != 0ull;
    }
    const uint64_t out = __ballot(any);
    if (lane_id() == 0) coarse[cw] = out;
}

// The first id of a group of the cache filter: the smallest whose product with mult has g in its upper half.
__device__ __forceinline__ int64_t group_begin(uint32_t g, uint32_t mult)
{
    const uint64_t x = (uint64_t) g << 32;                     // below 2^53
    uint64_t q = (uint64_t) ((double) x / (double) mult);      // at most one off
    if (q * mult < x) ++q;
    else if (q > 0 && (q - 1) * mult >= x) --q;
    return (int64_t) q;
}

// The groups of the cache filter, the tags of its hot nodes, and, where there is a list of them, the groups' first two nodes.
// One lane per group.  (With the tags made from the keys by every block that stages the filter, that took 1.2 us longer.)
__global__ void __launch_bounds__(kBlock) k_cache_groups(const int32_t* done, const uint64_t* bitmap, int64_t n, CacheFilter f)
{
    if (done && *done < 0) return;
    const uint32_t g = blockIdx.x * kBlock + threadIdx.x;      // the grid is exact
    if (g < kFilterHot) {
        const unsigned long long key = f.keys[g];
        f.tags[g] = key ? (uint16_t) ((uint32_t) key / kFilterHot + 1u) : (uint16_t) 0;
    }
    const int64_t lo = group_begin(g, f.mult), next = group_begin(g + 1u, f.mult), hi = next < n ? next : n;
    uint32_t found = 0, pair = 0;
    for (int64_t w = lo >> 6; w << 6 < hi; ++w) {
        uint64_t word = bitmap[w];
        if (w == lo >> 6) word &= ~0ull << (lo & 63);
        if (hi - (w << 6) < 64) word &= (1ull << (hi - (w << 6))) - 1ull;
        for (; word && found < 3; ++found, word &= word - 1) {
            const uint32_t low = (uint32_t) ((w << 6) + __builtin_ctzll(word)) & kPairMask;
            if (found == 0) pair = low | low << kPairBits;
            if (found == 1) pair = (pair & kPairMask) | low << kPairBits;
        }
    }
    const uint64_t any = __ballot(found > 0);
    if (lane_id() == 0) *reinterpret_cast<uint64_t*>(f.groups + (g >> 5)) = any;
    if (f.pairs && found > 0) f.pairs[g] = (uint16_t) (pair | (found > 2 ? kPairMore : 0u) | kPairSet);
}

// ---------------------------------------------------------------------------
static gns_status fail(gns_ctx* c, gns_status st, const char* what, hipError_t e)
{
    if (e != hipSuccess) snprintf(c->err, sizeof(c->err), "%s: %s", what, hipGetErrorString(e));
    else snprintf(c->err, sizeof(c->err), "%s", what);
    return st;
}

#define GNS_HIP_TRY(expr, what)                                        \
    do {                                                               \
        hipError_t e__ = (expr);                                       \
        if (e__ != hipSuccess) return fail(c, GNS_EHIP, what, e__);    \
    } while (0)

constexpr int kAsyncUnits = 8;      // draws an asynchronous draw enqueues, in Layout::draw_unit (a typical cache needs one or two)

// Records, on the stream every context of the family last used, the end of what may still read the copy
// of the cache block that stops being current now.
static gns_status mark_last_readers(gns_ctx* c, int old_gen)
{
    for (int i = 0; i < c->family_count; ++i) {
        gns_ctx* m = c->family[i];
        for (int i = 0; i < m->reader_stream_count; ++i)
            GNS_HIP_TRY(hipEventRecord(m->gen_event[old_gen][i], m->reader_streams[i]), "event record");
        m->gen_event_used[old_gen] = m->reader_stream_count;
        m->reader_stream_count = 0;          // streams used from now on read the next cache
    }
    return GNS_OK;
}

// The current cache stops being usable without a successor (the cache probability is about to change).
gns_status retire_cache(gns_ctx* c)
{
    const gns_status st = mark_last_readers(c, c->cache_gen);
    if (st != GNS_OK) return st;
    c->cache_valid = false;
    return GNS_OK;
}

// Makes the copy a finished or enqueued draw filled the current one.
gns_status activate_cache(gns_ctx* c)
{
    if (c->cache_valid) {
        const gns_status st = mark_last_readers(c, c->cache_gen);
        if (st != GNS_OK) return st;
    }
    c->cache_gen = c->pending_gen;
    c->cache_valid = true;
    c->had_cache = true;
    c->pending = false;
    c->cache_version += 1;
    return GNS_OK;
}

// Reads the outcome of the last draw back (synchronises behind it).
gns_status finish_pending_draw(gns_ctx* c)
{
    const int gen = c->pending ? c->pending_gen : c->cache_gen;
    GNS_HIP_TRY(hipEventSynchronize(c->ready_event[gen]), "cache draw wait");
    if (c->h_draw->draw_done_chunk < 0)
        return fail(c, GNS_ECAPACITY, "cache draw: the stream did not yield cache_size distinct nodes within the chunks an asynchronous draw enqueues", hipSuccess);
    c->cache_draws = (int64_t) c->h_draw->cut_draw + 1;
    return GNS_OK;
}

// Everything a finished bitmap determines: index, weights, coarse bitmap, induced subgraph, the cached rows' features.
static gns_status fill_cache(gns_ctx* c, int gen, const IndexArgs& x, bool i64, hipStream_t s)
{
    const Layout& L = c->lay;
    if (i64) launch_cache_index<int64_t>(x, s);
    else     launch_cache_index<int32_t>(x, s);
    GNS_HIP_TRY(hipGetLastError(), "cache index launch");
    if (L.filter) {
        hipLaunchKernelGGL(k_cache_groups, dim3(kFilterGroups / kBlock), dim3(kBlock), 0, s, x.done, x.bitmap, c->graph.num_nodes,
                           x.filter);
        GNS_HIP_TRY(hipGetLastError(), "cache filter launch");
    }
    if (L.coarse_shift > 0) {
        const unsigned cb = (unsigned) ((L.coarse_words + kBlock / kWave - 1) / (kBlock / kWave));
        hipLaunchKernelGGL(k_cache_coarse, dim3(cb), dim3(kBlock), 0, s, x.done, x.bitmap, (int64_t) L.words, (int) L.coarse_shift,
                           cache_ptr<uint64_t>(c, L.coarse_bitmap, gen), (int64_t) L.coarse_words);
        GNS_HIP_TRY(hipGetLastError(), "coarse bitmap launch");
    }
    if (c->config.flag_mode == GNS_FLAGS_PER_CACHE) GNS_HIP_TRY(launch_build_induced(c, gen, x.done, s), "induced subgraph");
    if (c->graph.feat_dim > 0) {
        // fill the device table of cached feature rows (slot order) straight from the full store
        const int32_t* fill_nodes = x.cache_nodes;
        const int32_t fill_count = (int32_t) x.cache_size;
        float* fill_out = cache_ptr<float>(c, L.cache_feat, gen);
        GNS_HIP_TRY(launch_gather(&c, 1, &fill_nodes, &fill_count, &fill_out, -1, s, x.done), "cache feature fill");
    }
    return GNS_OK;
}

gns_status run_sample_cache(gns_ctx* c, uint64_t seed, uint64_t epoch, bool wait_for_it, hipStream_t s)
{
    const Layout& L = c->lay;
    const int64_t C = c->config.cache_size;
    // The draw fills the copy of the cache block the mini-batches are not reading.  Whatever was enqueued
    // while that copy was the current one ended with the events recorded when it stopped being current:
    // the device may not have reached all of it yet if the host runs far ahead, so the draw waits for them.
    const int gen = c->had_cache ? (c->cache_gen ^ 1) : 0;
    uint64_t* bitmap = cache_ptr<uint64_t>(c, L.cache_bitmap, gen);
    // Draws share their hash and their outcome, so one begins when the one before has ended, also on another stream: the
    // one that is to be made current still (this one replaces it), or the one that is.
    if (c->pending || c->had_cache)
        GNS_HIP_TRY(hipStreamWaitEvent(s, c->ready_event[c->pending ? c->pending_gen : c->cache_gen], 0), "wait for the draw before");
    for (int i = 0; i < c->family_count; ++i) {
        gns_ctx* m = c->family[i];
        for (int i = 0; i < m->gen_event_used[gen]; ++i)
            GNS_HIP_TRY(hipStreamWaitEvent(s, m->gen_event[gen][i], 0), "wait for the readers of the old cache");
        m->gen_event_used[gen] = 0;
    }
    // The draw picks a uniform integer below the total mass and takes the node whose prefix interval
    // holds it: the CSR offsets for Eq. (1), the prefix of the walk weights for the other probability.
    const bool walk = c->config.cache_probability == GNS_PROB_WALK;
    const void* prob_prefix = walk ? static_cast<const void*>(ws_ptr<int64_t>(c, L.prob_prefix)) : c->graph.indptr;
    const uint64_t prob_total = walk ? (uint64_t) c->prob_total : (uint64_t) c->graph.num_entries;
    const bool i64 = walk || c->graph.indptr_is_i64 != 0;
    auto next_tag = [&]() { return ++c->draw_tag ? c->draw_tag : ++c->draw_tag; };
    DrawArgs a;
    memset(&a, 0, sizeof(a));
    a.st = c->d_state;
    a.host = c->h_state_dev + 1;                        // h_draw, as kernels see it
    a.indptr = prob_prefix;
    a.n = c->graph.num_nodes;
    a.nnz = prob_total;
    a.entry_rows = walk ? nullptr : ws_ptr<int32_t>(c, L.entry_rows);
    a.key0 = (uint32_t) seed;
    a.key1 = (uint32_t) (seed >> 32);
    a.epoch = (uint32_t) epoch;
    a.table = ws_ptr<unsigned long long>(c, L.draw_table);
    a.hmask = L.draw_hash_cap - 1;
    a.hshift = 32u - (uint32_t) __builtin_ctz(L.draw_hash_cap);
    a.draw_slot = ws_ptr<int32_t>(c, L.draw_slot);
    a.sums = ws_ptr<unsigned long long>(c, L.draw_sums);
    a.spins = c->union_spins;
    a.cache_bitmap = bitmap;
    a.words = L.words;
    a.filter = cache_filter(c, gen).keys;
    a.cache_size = C;
    {
        int64_t blocks = ((int64_t) L.draw_hash_cap + kBlock * 4 - 1) / (kBlock * 4);
        if (blocks > (int64_t) c->num_cus * 8) blocks = (int64_t) c->num_cus * 8;
        hipLaunchKernelGGL(k_cache_clear, dim3((unsigned) blocks), dim3(kBlock), 0, s, a);
        GNS_HIP_TRY(hipGetLastError(), "cache draw clear");
    }

    // The draw hash holds every distinct node seen so far: fewer than |C| before the final
    // chunk plus at most one chunk's worth, which is what it was sized for.  Stream indices
    // are kept in 32 bits; a cache that needs more draws than the limit is refused.  How many of a
    // chunk's first occurrences enter the cache, and whether they complete it, is decided on the device
    // (k_cache_commit); the host only needs to know when to stop enqueuing chunks.
    uint64_t draw_limit = 256ull * (uint64_t) C + 64ull * (uint64_t) L.draw_unit;
    if (draw_limit > 0xFFFFFFFFull) draw_limit = 0xFFFFFFFFull;
    draw_limit -= draw_limit % (uint64_t) L.draw_unit;
    const uint64_t ahead = (uint64_t) kAsyncUnits * (uint64_t) L.draw_unit;
    const uint64_t stop = wait_for_it || draw_limit < ahead ? draw_limit : ahead;
    uint64_t drawn = 0;
    auto enqueue_chunk = [&]() -> hipError_t {
        uint64_t count = (uint64_t) (drawn == 0 && first_draws(C) < L.draw_chunk ? first_draws(C) : L.draw_chunk);
        if (count > stop - drawn) count = stop - drawn;
        a.j0 = drawn;
        a.count = (int32_t) count;
        a.tag = next_tag();
        const dim3 draws((unsigned) ((count + kBlock - 1) / kBlock)), tiles((unsigned) ((count + kDrawTile - 1) / kDrawTile));
        if (i64) hipLaunchKernelGGL((k_cache_draw<int64_t>), draws, dim3(kBlock), 0, s, a);
        else     hipLaunchKernelGGL((k_cache_draw<int32_t>), draws, dim3(kBlock), 0, s, a);
        hipLaunchKernelGGL(k_cache_commit, tiles, dim3(kBlock), 0, s, a);
        drawn += count;
        a.chunk_index += 1;
        return hipGetLastError();
    };
    IndexArgs x;
    memset(&x, 0, sizeof(x));
    x.bitmap = bitmap;
    x.words = L.words;
    x.sums = ws_ptr<unsigned long long>(c, L.index_sums);
    x.spins = c->union_spins;
    x.word_prefix = cache_ptr<int32_t>(c, L.cache_prefix, gen);
    x.cache_nodes = cache_ptr<int32_t>(c, L.cache_nodes, gen);
    x.cache_size = C;
    x.prob_prefix = prob_prefix;
    x.prob_total = (int64_t) prob_total;
    x.node_inv_pc = L.slot_marks ? nullptr : cache_ptr<float>(c, L.node_pc, gen);
    x.node_slot = L.slot_marks ? cache_ptr<CachedNode>(c, L.node_pc, gen) : nullptr;
    x.filter = cache_filter(c, gen);
    // Of |C| cached nodes kFilterHot have a slot: nodes that are unlikely to be among them (on a power law the rows of the C-th
    // node are ten times the average, and lengths fall about as ranks grow) stay out of the atomics.
    x.hot_from = c->graph.num_entries / c->graph.num_nodes * 3 * (C / (2 * kFilterHot));
    x.g_indptr = c->graph.indptr;
    x.g_i64 = c->graph.indptr_is_i64;
    if (wait_for_it) {
        // A chunk and what follows it, then a look at the outcome.  While the cache is incomplete (a stream that repeats
        // itself a lot: a large share of the nodes, a concentrated probability) two chunks more are tried, for more than a
        // twentieth of the nodes from the start on: a chunk that stands down is two launches in front of everything else, a
        // second look a wait.  One and two chunks first: 100 of 10 K nodes 39 and 48 us, 10 K of 1 M 81 and 85, 50 K 102 and
        // 105, 100 K 164 and 148.
        const bool one = C <= c->nonzero_degree_nodes / 20;
        x.done = &c->d_state->draw_done_chunk;
        do {
            if (drawn >= stop) {
                c->pending = false;                    // the copy an enqueued draw may have filled is gone
                return fail(c, GNS_ECAPACITY, "cache draw: the stream did not yield cache_size distinct nodes within the draw limit (cache_size too close to the number of nodes with neighbors)", hipSuccess);
            }
            for (int k = drawn == 0 && one ? 1 : 2; k > 0 && drawn < stop; --k) GNS_HIP_TRY(enqueue_chunk(), "cache draw launch");
            x.tag = next_tag();
            const gns_status st = fill_cache(c, gen, x, i64, s);
            if (st != GNS_OK) return st;
            GNS_HIP_TRY(hipStreamSynchronize(s), "cache draw sync");
        } while (c->h_draw->draw_done_chunk < 0);
    } else {
        while (drawn < stop) GNS_HIP_TRY(enqueue_chunk(), "cache draw launch");
        x.tag = next_tag();                            // an incomplete cache has consistent structures too: it may be made current
        const gns_status st = fill_cache(c, gen, x, i64, s);
        if (st != GNS_OK) return st;
    }
    GNS_HIP_TRY(hipEventRecord(c->ready_event[gen], s), "event record");
    c->pending = true;
    c->pending_gen = gen;
    c->cache_draws = -1;                           // read back on demand
    if (!wait_for_it) return GNS_OK;
    c->cache_draws = (int64_t) c->h_draw->cut_draw + 1;
    return activate_cache(c);
}

}  // namespace gns
