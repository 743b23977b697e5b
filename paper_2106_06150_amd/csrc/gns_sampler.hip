// Layer sampler: for every dst row v independently, N_l(v) <- sample(N(v), C)
// (paper Algorithm 1, top-down loop).
//
//   UNIFORM     Section 2.1: min(k, deg(v)) neighbors uniformly without
//               replacement.  Only the k chosen CSR entries are read.
//   CACHE_ONLY  Sections 3.3 and 4.1: the eligible list is the row's entries
//               whose node is in the cache, in CSR order; min(k, N_C(v)) of
//               them are chosen; each carries the Section 3.4 weight.
//   CACHE_FIRST Section 3.3: as CACHE_ONLY; a row with N_C(v) < k then draws the
//               shortfall uniformly from its entries outside the cache.
//
// The without-replacement choice is Robert Floyd's subset algorithm on ranks
// of the eligible list, driven by k Philox words keyed by (seed, layer, node,
// slot); the chosen ranks are emitted in ascending order.  All decisions are
// integer arithmetic, so the sample does not depend on scheduling.
//
// Output per row r (fixed stride k): s_nbr[r*k + i] (the neighbor's local id as -(id+1) if it has
// one, else its global id), s_w[r*k + i] for i < s_cnt[r] (UNIFORM layers: no weights, they are 1),
// row_eligible[r], the dst node as the r-th src node, and the sum of s_cnt over the rows of a block;
// every emitted id that has no local id yet (it is not a dst node of this layer) also sets its bit in
// the node-indexed mark bitmap that the frontier stage turns into the src list.  An input layer that samples from the cache
// only, with the induced subgraph, marks by slots of the cache instead and leaves a new node's slot (see k_finish_cached).
#include <string.h>
#include <stdlib.h>
#include "gns_kernels.hpp"

namespace gns {

// Floyd's subset draw inside a group of G consecutive lanes (G a power of two
// <= 64).  Lane s < k ends up with one chosen rank of {0..m-1} in *val and that
// rank's position in ascending order in *pos.  Requires m > k.  k may differ from
// group to group; k_loop >= every group's k must be the same for the whole wave
// (it bounds the loops that exchange data between lanes).  The word of lane s is
// slot slot0 + s of (layer, node).  Every lane of the wave must call it.
template <int G>
__device__ __forceinline__ void floyd_in_group(uint32_t m, int k, int k_loop, uint32_t key0, uint32_t key1,
                                               uint32_t layer, uint32_t node, int s, uint32_t* val, int* pos,
                                               int slot0 = 0)
{
    s = opaque(s);
    // lane s draws t_s uniform in [0, m-k+s]
    const uint32_t slot = (uint32_t) (slot0 + s);
    const Philox4 r = philox4x32_10(node, slot >> 2, layer, kTagNeighbor, key0, key1);
    const int sel = (int) (slot & 3u);
    const uint32_t word = sel == 0 ? r.w[0] : sel == 1 ? r.w[1] : sel == 2 ? r.w[2] : r.w[3];
    const uint32_t j_own = m - (uint32_t) k + (uint32_t) s;
    const uint32_t t_own = __umulhi(word, j_own + 1u);
    uint32_t chosen = 0xFFFFFFFFu;              // not yet decided
    const int group_base = opaque_lane_id() & ~(G - 1);
    const uint64_t group_mask = (G == 64) ? ~0ull : (((1ull << (G & 63)) - 1ull) << group_base);
    for (int q = 0; q < k_loop; ++q) {
        const uint32_t t_q = __shfl(t_own, q, G);
        // is t_q already among the ranks decided by slots < q ?
        const uint64_t hit = __ballot(s < q && chosen == t_q) & group_mask;
        if (s == q) chosen = hit ? j_own : t_own;
    }
    int rank = 0;
    for (int q = 0; q < k_loop; ++q) {
        const uint32_t c_q = __shfl(chosen, q, G);
        rank += (q < k && c_q < chosen) ? 1 : 0;
    }
    *val = chosen;
    *pos = rank;
}

// A sampled id becomes a new src node unless it already owns a local id.  Returns what the relabel
// step should find in the scratch slot: the node's local id as -(id + 1) if it has one (no second
// lookup then), else the global id (>= 0), whose local id is assigned by the union step.
// Sets node u's bit in the frontier mark bitmap.  (Looking at the bit first, to spare popular nodes'
// words thousands of atomics per batch, measured slower: the extra dependent read costs more than the
// atomics it saves.)
__device__ __forceinline__ void mark_node(const SampleArgs& a, uint32_t u)
{
    atomicOr(reinterpret_cast<unsigned long long*>(&a.mark[u >> 6]), 1ull << (u & 63u));
    if (a.mark_summary)
        atomicOr(reinterpret_cast<unsigned long long*>(&a.mark_summary[u >> 12]), 1ull << ((u >> 6) & 63u));
}

__device__ __forceinline__ int32_t mark_if_new(const SampleArgs& a, uint32_t u)
{
    const uint32_t e = a.tab.entry[u];
    if (a.tab.current(e)) return -1 - (int32_t) a.tab.local(e);
    mark_node(a, u);
    return (int32_t) u;
}

// The same in a layer that marks by slot: what is left for a new node is its slot.
__device__ __forceinline__ int32_t mark_if_new_slot(const SampleArgs& a, uint32_t u, int32_t slot)
{
    const uint32_t e = a.tab.entry[u];
    if (a.tab.current(e)) return -1 - (int32_t) a.tab.local(e);
    a.slot_mark[slot] = 1;
    return slot;
}

// ---------------------------------------------------------------------------
// Direct layers with fan-outs up to 16.  A wave takes W rows (W a power of two up to kWaveRows) in two stages:
//   draw   one row per lane: extent, chunk records, Floyd's draw for the whole row (the loops over the slots are
//          unrolled, the chosen ranks stay in registers and are sorted there: an entry's slot is then its place in the row);
//          the Philox blocks of the W rows are spread over all lanes;
//   fetch  one drawn entry per lane: the W * k (row, slot) pairs are dealt to the lanes in turns of 64, the list's
//          entry -> node table and 1/p^C -> mark, scratch.
// The stages have opposite needs.  The draw is instruction-bound (a Philox block is forty quarter-rate multiplies), and
// with a slot per lane every lane of a row repeats it; the fetch is a chain of scattered reads, and with a row per lane
// half of the slots a lane holds sit in branches that wait for one another.
// The sort (38 instructions a row of 8 slots) takes the place of a count, per entry, of the row's smaller ranks: that read
// the row's slots from LDS for every entry and held 103 registers, four waves per SIMD where 36 let seven or eight run, and
// entries in ascending order share the lines of list and scratch.  With that many waves a lane has one entry on its way at a
// time: five, which few waves needed, are turns that small layers have no entries for (upper layers cache first: 21 us for
// 23.5; input layer on 40 M nodes 55 for 57.5).  Groups of four on the graph of 1 M nodes, three layers (entering
// the seeds included): 9.3 / 25.4 / 36.8 us, with the count (and up to 64 rows per wave) 9.9 / 27 / 41.5, where a lane group
// per row on the upper and a row per lane on the input layer took 15.7 / 28 / 55; on 40 M nodes 9.5 / 22 / 55 for 10 / 24 / 60.
// The input layer is bound by the lines its records and drawn entries pull in (1.3 M L2 misses).
// kFirst: also the batch's first kernel.  No sampled node has a local id yet as far as that launch can know, so every one
// is marked, and the union step takes the seeds out again (seed bitmap).
constexpr int kWaveRows = 32;                    // at most, see wave_rows

template <int K>
struct WaveRows {
    static_assert(K % 4 == 0, "whole Philox blocks");
    static constexpr int kSlots = K;
    uint32_t slot[kWaveRows][kSlots];            // Philox words, then the chosen ranks, ascending (top bit: of the fill; ~0: none)
    int64_t start[kWaveRows], end[kWaveRows];    // CSR extent
    uint32_t first[kWaveRows], here[kWaveRows], tile[kWaveRows];     // CachedList
    int32_t count[kWaveRows];                    // entries drawn from the list, and in all, << 8
    float scale[kWaveRows], fill_w[kWaveRows];
};

// Batcher's odd-even merge sort of a lane's slots, ascending; 19, 42 and 63 exchanges for 8, 12 and 16.
template <int K>
__device__ __forceinline__ void sort_slots(uint32_t (&v)[K])
{
#pragma unroll
    for (int p = 1; p < K; p *= 2) {
#pragma unroll
        for (int q = p; q >= 1; q /= 2) {
#pragma unroll
            for (int i = 0; i + q < K; ++i) {
                if (i >= q % p && (i - q % p) % (2 * q) < q && i / (2 * p) == (i + q) / (2 * p)) {
                    const uint32_t lo = v[i] < v[i + q] ? v[i] : v[i + q];
                    v[i + q] = v[i] < v[i + q] ? v[i + q] : v[i];
                    v[i] = lo;
                }
            }
        }
    }
}

template <int K, int kList, bool kFirst>
__device__ __forceinline__ void sample_wave_rows(const LayerArgs& g, const BeginDyn* d, const SampleArgs& a, int b, int32_t row0,
                                                 int W, int32_t R, uint32_t key0, uint32_t key1, WaveRows<K>& w, int32_t& sum)
{
    const int k = a.fanout;                         // <= K
    const int lane = opaque_lane_id();
    const bool live = lane < W && row0 + lane < R;
    const int32_t row = row0 + lane < R && lane < W ? row0 + lane : R - 1;
    // ---- draw
    RowExtent ext;
    int32_t vi;
    if (kFirst) {
        vi = d->seeds[b][row];
        ext = seed_extent(g, vi);
        if (live) enter_seed(g, *d, b, a.tab, row, vi, ext, true);
    } else {
        ext = a.row_ext[row];
        vi = a.dst_nodes[row];
    }
    const int blocks = (k + 3) >> 2;
    for (int t = lane; t < kWaveRows * blocks; t += kWave) {
        // task t: block t / W of row t % W (tasks past the last repeat nothing of use; the shuffle wants every lane)
        const int r = t & (W - 1), c = t >> __builtin_ctz((unsigned) W);
        if (!__any(c < blocks)) break;
        const uint32_t v = (uint32_t) __shfl(vi, r, kWave);
        if (c < blocks) {
            const Philox4 p = philox4x32_10(v, (uint32_t) c, a.layer_number, kTagNeighbor, key0, key1);
            *reinterpret_cast<uint4*>(&w.slot[r][4 * c]) = make_uint4(p.w[0], p.w[1], p.w[2], p.w[3]);
        }
    }
    const uint32_t deg = (uint32_t) (ext.end - ext.start);
    CachedList cached = {0u, 0u, 0u, 0u};
    if (kList != kListRow) cached = cached_list(a, ext);
    const uint32_t m = kList == kListRow ? deg : cached.count;
    const int cnt = m > (uint32_t) k ? k : (int) m;           // entries drawn from the list
    const uint32_t others = deg - m, room = (uint32_t) (k - cnt);
    const int fill = kList != kListCachedFirst ? 0 : others > room ? (int) room : (int) others;
    const int total = cnt + fill;
    __builtin_amdgcn_wave_barrier();
    if (lane < W) {
        uint32_t word[WaveRows<K>::kSlots];
#pragma unroll
        for (int c = 0; c < WaveRows<K>::kSlots / 4; ++c) {
            const uint4 q = *reinterpret_cast<const uint4*>(&w.slot[lane][4 * c]);
            word[4 * c] = q.x; word[4 * c + 1] = q.y; word[4 * c + 2] = q.z; word[4 * c + 3] = q.w;
        }
        // List ranks, then (kListCachedFirst) ranks among the other neighbors with the top bit set.  A row with no more
        // entries than slots takes them all.
        const bool draw = m > (uint32_t) k, draw_fill = kList == kListCachedFirst && others > room;
        uint32_t chosen[WaveRows<K>::kSlots];
#pragma unroll
        for (int s = 0; s < WaveRows<K>::kSlots; ++s) {
            const uint32_t j = m - (uint32_t) k + (uint32_t) s;
            const uint32_t t = __umulhi(word[s], j + 1u);
            bool dup = false;
#pragma unroll
            for (int q = 0; q < s; ++q) dup = dup || chosen[q] == t;
            uint32_t c = draw ? (dup ? j : t) : (uint32_t) s;
            if (kList == kListCachedFirst) {
                // slot cnt + i draws fill entry i: a Floyd draw of `room` out of `others`
                const uint32_t i = (uint32_t) (s - cnt);
                const uint32_t fj = others - room + i;
                const uint32_t ft = __umulhi(word[s], fj + 1u) | 0x80000000u;
                bool fdup = false;
#pragma unroll
                for (int q = 0; q < s; ++q) fdup = fdup || chosen[q] == ft;
                if (s >= cnt) c = draw_fill ? (fdup ? fj | 0x80000000u : ft) : i | 0x80000000u;
            }
            chosen[s] = s < total ? c : 0xFFFFFFFFu;
        }
        sort_slots(chosen);
#pragma unroll
        for (int c = 0; c < WaveRows<K>::kSlots / 4; ++c)
            *reinterpret_cast<uint4*>(&w.slot[lane][4 * c]) = make_uint4(chosen[4 * c], chosen[4 * c + 1], chosen[4 * c + 2], chosen[4 * c + 3]);
        w.start[lane] = ext.start;
        if (kList == kListCachedFirst) { w.end[lane] = ext.end; w.fill_w[lane] = fill_weight(a, others, fill); }
        if (kList != kListRow) {
            w.first[lane] = cached.first; w.here[lane] = cached.here; w.tile[lane] = cached.tile;
            w.scale[lane] = cached_scale(a, m, cnt);
        }
        w.count[lane] = live ? cnt | total << 8 : 0;
    }
    if (live) {
        a.s_cnt[row] = total;
        a.row_eligible[row] = (int32_t) m;
        a.src_nodes[row] = vi;
        sum += total;
    }
    __builtin_amdgcn_wave_barrier();

    // ---- fetch
    const int items = W * k;
    const uint32_t inv_k = 65535u / (uint32_t) k + 1u;          // j / k = j * inv_k >> 16, exact for j < 4096
    for (int j0 = 0; j0 < items; j0 += kWave) {
        const int j = j0 + lane;
        const int q = j < items ? j : 0;
        const int r = (int) ((uint32_t) q * inv_k >> 16);
        const int s = q - r * k;
        const int counts = w.count[r];
        if (j >= items || s >= counts >> 8) continue;
        const uint32_t rank = w.slot[r][s];
        const bool is_fill = kList == kListCachedFirst && s >= (counts & 255);
        int64_t place;
        if (kList == kListRow)         place = w.start[r] + (int64_t) rank;
        else if (is_fill)              place = uncached_entry(a, RowExtent{w.start[r], w.end[r]}, rank & 0x7FFFFFFFu);
        else if (rank >= w.here[r])    place = later_tile(a, CachedList{w.first[r], w.here[r], 0u, w.tile[r]}, rank);      // rare: the row crosses a tile
        else                           place = (int64_t) (w.first[r] + rank);
        const uint32_t u = (uint32_t) (kList == kListRow || is_fill ? a.indices : a.s_nodes)[place];
        const uint32_t e = kFirst ? 0u : a.tab.entry[u];
        const CachedNode c = kList == kListRow || is_fill ? CachedNode{1.0f, 0} : cached_node(a, u);
        int32_t out = (int32_t) u;
        if (!kFirst && a.tab.current(e)) {
            out = -1 - (int32_t) a.tab.local(e);
        } else if (kList == kListCached && a.by_slot) {
            out = c.slot;
            a.slot_mark[c.slot] = 1;
        } else {
            mark_node(a, u);
        }
        const int64_t at = (int64_t) row0 * k + j;
        a.s_nbr[at] = out;
        if (kList != kListRow) a.s_w[at] = is_fill ? w.fill_w[r] : c.inv_pc * w.scale[r];
    }
    __builtin_amdgcn_wave_barrier();
}

// Blocks of four waves: rows block * 4 * W .. of the batch's layer, whose sampled neighbors are summed for the union step.
template <int K, int kList, bool kFirst>
__device__ __forceinline__ void sample_block_rows(const LayerArgs& g, const BeginDyn* d, const SampleArgs& a, int b, int32_t block,
                                                  int W, int32_t R, uint32_t key0, uint32_t key1, WaveRows<K>* w, int32_t* smem)
{
    const int wave = __builtin_amdgcn_readfirstlane((int) (threadIdx.x >> 6));
    const int32_t row0 = (block * (kBlock / kWave) + wave) * W;
    int32_t sum = 0;
    if (row0 < R) sample_wave_rows<K, kList, kFirst>(g, d, a, b, row0, W, R, key0, key1, w[wave], sum);
    sum = block_sum(sum, smem);
    if (threadIdx.x == 0) a.sums_rows[block] = sum;
}

template <int K, int kList, bool kOne>
__global__ void __launch_bounds__(kBlock) k_sample_rows(LayerArgs g, int W, int relabel_blocks)
{
    // the last relabel_blocks blocks finish the previous layer's block instead (see relabel_body); they are
    // dispatched after this layer's rows, whose dependent loads set the length of the launch
    __shared__ int32_t smem[kBlock / kWave + 1];
    __shared__ WaveRows<K> rows[kBlock / kWave];
    const GroupBlock q = group_block<kOne>(g.dealt);
    if (!kOne && q.block >= g.blocks) return;
    const int32_t nblocks = g.blocks - relabel_blocks;
    if (q.block >= nblocks) {
        relabel_body(bind_finish(g, q.b, false), q.block - nblocks, relabel_blocks);
        return;
    }
    const SampleArgs a = bind_sample(g, q.b);
    const int32_t R = a.st->num_dst[a.layer_index];
    for (int32_t block = q.block; (int64_t) block * (kBlock / kWave) * W < R; block += nblocks)
        sample_block_rows<K, kList, false>(g, nullptr, a, q.b, block, W, R, a.st->key0, a.st->key1, rows, smem);
}

// The first layer of a mini-batch, in the launch that enters its seeds.
template <int K, int kList, bool kOne>
__global__ void __launch_bounds__(kBlock) k_sample_first(LayerArgs g, BeginDyn d, int W)
{
    __shared__ int32_t smem[kBlock / kWave + 1];
    __shared__ WaveRows<K> rows[kBlock / kWave];
    const auto [b, block] = group_block<kOne>(g.dealt);
    const int32_t R = d.num_seeds[b];
    if (block == 0 && threadIdx.x == 0) begin_state(g, d, b);
    if ((int64_t) block * (kBlock / kWave) * W < R) {
        const SampleArgs a = bind_sample(g, b, d.stamp[b], d.cache_gen[b]);
        sample_block_rows<K, kList, true>(g, &d, a, b, block, W, R, d.key0[b], d.key1[b], rows, smem);
    }
    clear_slot_marks(g, b, block);
}

// ---------------------------------------------------------------------------
// Direct layers with fan-outs above 16: a wave per row, one slot per lane.
template <int kList, bool kOne>
__global__ void __launch_bounds__(kBlock) k_sample_wide(LayerArgs g, int relabel_blocks)
{
    __shared__ int32_t smem[kBlock / kWave + 1];
    const GroupBlock q = group_block<kOne>(g.dealt);
    if (!kOne && q.block >= g.blocks) return;
    const int32_t nblocks = g.blocks - relabel_blocks;
    if (q.block >= nblocks) {
        relabel_body(bind_finish(g, q.b, false), q.block - nblocks, relabel_blocks);
        return;
    }
    const SampleArgs a = bind_sample(g, q.b);
    const int32_t R = a.st->num_dst[a.layer_index];
    const uint32_t key0 = a.st->key0, key1 = a.st->key1;
    constexpr int kRows = kBlock / kWave;
    for (int32_t block = q.block; (int64_t) block * kRows < R; block += nblocks) {
        const int k = a.fanout;
        const int s = opaque_lane_id();
        const int32_t my_row = block * kRows + (int32_t) (threadIdx.x >> 6);
        const bool live = my_row < R;
        const int32_t row = live ? my_row : R - 1;
        const RowExtent ext = a.row_ext[row];
        const int32_t vi = a.dst_nodes[row];
        const uint32_t v = (uint32_t) vi, deg = (uint32_t) (ext.end - ext.start);
        CachedList cached = {0u, 0u, 0u, 0u};
        if (kList != kListRow) cached = cached_list(a, ext);
        const uint32_t m = kList == kListRow ? deg : cached.count;
        const int cnt = m > (uint32_t) k ? k : (int) m;           // entries drawn from the list
        const uint32_t others = deg - m, room = (uint32_t) (k - cnt);
        const int fill = kList != kListCachedFirst ? 0 : others > room ? (int) room : (int) others;
        // run the draw with a safe size in every lane, then keep it only where it applies
        uint32_t val;
        int pos;
        floyd_in_group<kWave>(m > (uint32_t) k ? m : (uint32_t) k + 1u, k, k, key0, key1, a.layer_number, v, s, &val, &pos);
        if (m <= (uint32_t) k) { val = (uint32_t) s; pos = s; }
        const bool is_fill = kList == kListCachedFirst && s >= cnt;
        if (kList == kListCachedFirst && __any(fill > 0)) {
            // the shortfall: slots cnt, cnt + 1, ... of the row draw from its entries outside the cache; lane i draws the
            // i-th of them, lane cnt + i emits it
            uint32_t fval;
            int fpos;
            floyd_in_group<kWave>(others > room ? others : room + 1u, (int) room, k, key0, key1, a.layer_number, v, s, &fval, &fpos, cnt);
            if (others <= room) { fval = (uint32_t) s; fpos = s; }
            const int from = s >= cnt ? s - cnt : 0;
            const uint32_t f = (uint32_t) __shfl((int) fval, from, kWave);
            const int fp = __shfl(fpos, from, kWave);
            if (is_fill) { val = f; pos = cnt + fp; }
        }
        if (live && s < cnt + fill) {
            int64_t place;
            if (is_fill)                  place = uncached_entry(a, ext, val);
            else if (kList == kListRow)   place = ext.start + val;
            else if (val >= cached.here)  place = later_tile(a, cached, val);
            else                          place = (int64_t) cached.first + val;
            const uint32_t u = (uint32_t) (kList == kListRow || is_fill ? a.indices : a.s_nodes)[place];
            const int64_t at = (int64_t) row * k + pos;
            CachedNode c = {1.0f, 0};
            if (kList != kListRow && !is_fill) c = cached_node(a, u);
            if (kList != kListRow) a.s_w[at] = is_fill ? fill_weight(a, others, fill) : c.inv_pc * cached_scale(a, m, cnt);
            a.s_nbr[at] = kList == kListCached && a.by_slot ? mark_if_new_slot(a, u, c.slot) : mark_if_new(a, u);
        }
        if (live && s == 0) {
            a.s_cnt[row] = cnt + fill;
            a.row_eligible[row] = (int32_t) m;
            a.src_nodes[row] = vi;
        }
        const int32_t sum = block_sum(live && s == 0 ? cnt + fill : 0, smem);
        if (threadIdx.x == 0) a.sums_rows[block] = sum;
    }
}

// ---------------------------------------------------------------------------
// CACHE_ONLY in two balanced phases.
//
// The CSR entry array is cut into aligned chunks of 64 entries; flags[g] holds, for chunk g,
// one bit per entry: "this neighbor is in the cache".
//   plan     per dst row, the aligned chunks its segment touches; prefix sum; the chunk ids
//            are written out as a flat work list (k_plan)
//   flag     one wave step = a few chunks of the list: coalesced 256-byte index loads, one
//            cache-bitmap test per entry, a ballot per chunk stored as one 64-bit word.  Every
//            chunk costs the same, so the stream is balanced whatever the degree skew
//            (k_flag_chunks; the bitmap is staged in LDS when it fits)
//   select   per dst row (a group of lanes): read the row's flag words, trim the two boundary
//            words to the row, count N_C(v), draw, map the chosen ranks back to CSR positions,
//            emit ids and Section 3.4 weights (k_select_rows)
// A chunk shared by two dst rows is flagged twice with the same value.

__device__ __forceinline__ int32_t chunks_touched(int64_t start, int64_t end)
{
    return end > start ? (int32_t) (((end - 1) >> 6) - (start >> 6) + 1) : 0;
}

// Plan tiles are kPlanTile rows (one row per thread): many small blocks keep the expansion parallel.
constexpr int kPlanTile = kBlock;
constexpr int kPlanFlight = 8;      // entries of a thread that look their rows up together

// One launch: a tile's block passes its number of chunks on to the blocks of later tiles (sum_before), as the union step's
// blocks do with the rows' samples.  Two launches fewer: a mini-batch with a scan of its rows 189 -> 185 us.
// Bound by latency: extents, the sums of the tiles before, and eight dependent reads of LDS per entry of the list, which is why a thread
// looks eight entries up together, the first eight while the sums are on their way (85 K rows with 300 K chunks 14.7 -> 9.5 us).
template <bool kOne>
__global__ void __launch_bounds__(kBlock) k_plan(LayerArgs g, int relabel_blocks, int spins)
{
    __shared__ int32_t smem[kBlock / kWave + 1];
    __shared__ int32_t s_off[kPlanTile];
    __shared__ int32_t s_g0[kPlanTile];
    __shared__ int32_t s_hubs[kBlock / kWave], s_first_hub;
    const auto [b, tile] = group_block<kOne>(g.dealt);
    if (!kOne && tile >= g.blocks) return;
    const int32_t ntiles = g.blocks - relabel_blocks;
    if (tile >= ntiles) {
        relabel_body(bind_finish(g, b, false), tile - ntiles, relabel_blocks);
        return;
    }
    const SampleArgs a = bind_sample(g, b);
    const int32_t R = a.st->num_dst[a.layer_index];
    if (tile >= (R + kPlanTile - 1) / kPlanTile) return;
    const int32_t r = tile * kPlanTile + (int32_t) threadIdx.x;
    RowExtent ext = {0, 0};
    if (r < R) ext = a.row_ext[r];
    s_g0[threadIdx.x] = (int32_t) (ext.start >> 6);
    const bool hub = is_hub_extent(ext.start, ext.end);
    const uint64_t hubs = __ballot(hub);
    if (lane_id() == 0) s_hubs[threadIdx.x >> 6] = __popcll(hubs);
    int32_t total;
    s_off[threadIdx.x] = block_exclusive_scan(chunks_touched(ext.start, ext.end), smem, &total);
    const uint32_t tag = launch_tag(a.st, a.layer_index);
    if (threadIdx.x == 0) publish_sum(a.plan_sums, tile, tag, (uint32_t) total);
    __syncthreads();
    // behind the sum others wait for: the tile's hubs take their places in the layer's list
    int32_t first_hub = 0;
    if (threadIdx.x == 0) {
        int32_t hub_total = 0;
#pragma unroll
        for (int w = 0; w < kBlock / kWave; ++w) hub_total += s_hubs[w];
        if (hub_total) first_hub = atomicAdd(&a.st->hub_count[a.layer_index], hub_total);
    }
    const uint32_t last_chunk = (uint32_t) ((a.num_entries - 1) >> 6);
    // Entries j, j + kBlock, ... of the tile's work list: an entry's row is the last one whose offset is <= it (rows without a chunk
    // have the offset of the row behind them).
    auto entries = [&](int32_t j, uint32_t (&chunk)[kPlanFlight]) {
        int32_t row[kPlanFlight];
#pragma unroll
        for (int i = 0; i < kPlanFlight; ++i) row[i] = 0;
#pragma unroll
        for (int step = kPlanTile / 2; step > 0; step /= 2)
#pragma unroll
            for (int i = 0; i < kPlanFlight; ++i) row[i] += s_off[row[i] + step] <= j + i * kBlock ? step : 0;
#pragma unroll
        for (int i = 0; i < kPlanFlight; ++i) {
            const uint32_t c = (uint32_t) s_g0[row[i]] + (uint32_t) (j + i * kBlock - s_off[row[i]]);
            chunk[i] = c < last_chunk ? c : last_chunk;
        }
    };
    uint32_t chunk[kPlanFlight];
    entries((int32_t) threadIdx.x, chunk);                       // (while the sums of the tiles before are on their way)
    // chunks of all earlier tiles
    const int32_t before = sum_before(a.plan_sums, tag, tile, spins, smem, [&](int32_t t) {
        uint32_t n = 0;
        for (int32_t q = t * kPlanTile; q < (t + 1) * kPlanTile; ++q)            // a full tile: one follows
            n += (uint32_t) chunks_touched(a.row_ext[q].start, a.row_ext[q].end);
        return n;
    });
    // Rows of repeated seeds can have more chunks together than there is room for, or than 32 bits count; what such a batch
    // samples is of no matter, but its list has to end in bounds and hold chunks of the graph.
    if (tile == (R - 1) / kPlanTile && threadIdx.x == 0) {
        const uint32_t chunks = (uint32_t) before + (uint32_t) total;
        a.st->plan_chunks = (int32_t) (chunks < a.max_chunks ? chunks : a.max_chunks);
    }
    if (threadIdx.x == 0) s_first_hub = first_hub;
    __syncthreads();
    if (hub) {
        int32_t place = s_first_hub + __popcll(hubs & ((1ull << lane_id()) - 1ull));
        for (int w = 0; w < (int) (threadIdx.x >> 6); ++w) place += s_hubs[w];
        a.hub_rows[place] = r;
    }
    for (int32_t j = (int32_t) threadIdx.x;;) {
#pragma unroll
        for (int i = 0; i < kPlanFlight; ++i) {
            const uint32_t place = (uint32_t) before + (uint32_t) (j + i * kBlock);
            if (j + i * kBlock < total && place < a.max_chunks) a.plan_desc[place] = (int32_t) chunk[i];
        }
        j += kPlanFlight * kBlock;
        if (j >= total) break;
        entries(j, chunk);
    }
}

constexpr int kFlagUnroll = 32;     // chunks a wave keeps in flight
constexpr int kFlagBatch = 64;      // work-list entries a wave fetches at once (one per lane)

// Membership words of kUnroll chunks, chunk ids in lanes sub .. sub+kUnroll-1 of my_chunk
// (every one a valid chunk id).  Lane l tests entry l of each chunk; the ballot of chunk sub+i
// lands in lane sub+i of (*lo, *hi).  Three passes over the unrolled set -- all index loads, all
// bitmap reads, all tests -- so that the loads of the whole set are in flight together.
//   kCareful: the set may hold the last chunk of the entry array, whose tail lanes lie beyond
//   num_entries; those lanes re-read the last entry and are masked out of the ballot.
//   kMode 0: the bitmap is read from global memory; 1: from LDS; 2: LDS holds the cache filter, and only the entries it
//   leaves open go on to read the exact bitmap; 3: a coarse bitmap (one bit per group of ids) in global memory, small
//   enough to stay in every XCD's L2, does so for those whose group has no cached node.
template <int kMode, int kUnroll, bool kCareful>
__device__ __forceinline__ void flag_chunk_set(const SampleArgs& a, const uint32_t* lds32, int32_t my_chunk, int sub,
                                               int lane, uint32_t* lo, uint32_t* hi)
{
    const int64_t last_chunk = (a.num_entries - 1) >> 6;
    const int last_lanes = (int) (a.num_entries - (last_chunk << 6));          // 1..64 entries in the last chunk
    const int lane_clamped = lane < last_lanes ? lane : last_lanes - 1;
    const uint64_t last_mask = last_lanes == 64 ? ~0ull : ((1ull << last_lanes) - 1ull);
    uint32_t u[kUnroll];
#pragma unroll
    for (int i = 0; i < kUnroll; ++i) {
        const int32_t g = __builtin_amdgcn_readlane(my_chunk, sub + i);
        const int32_t* row = a.indices + ((int64_t) g << 6);                   // wave-uniform base
        const int off = (kCareful && g == last_chunk) ? lane_clamped : lane;
        u[i] = (uint32_t) row[off];
    }
    const uint32_t* exact32 = reinterpret_cast<const uint32_t*>(a.cache_bitmap);
    uint32_t w[kUnroll];
#pragma unroll
    for (int i = 0; kMode != 2 && i < kUnroll; ++i) {
        if (kMode == 1)      w[i] = lds32[u[i] >> 5];
        else if (kMode == 0) w[i] = exact32[u[i] >> 5];
        else                 w[i] = reinterpret_cast<const uint32_t*>(a.coarse_bitmap)[(u[i] >> a.coarse_shift) >> 5];
    }
    if (kMode == 2) {
#pragma unroll
        for (int i = 0; i < kUnroll; i += 8) filter_test<8>(lds32, a.filter_mult, u + i, w + i);
#pragma unroll
        for (int i = 0; i < kUnroll; ++i)
            if (w[i] == 1u) w[i] = exact32[u[i] >> 5];
    }
    if (kMode == 3) {
#pragma unroll
        for (int i = 0; i < kUnroll; ++i) {
            const bool maybe = (w[i] >> ((u[i] >> a.coarse_shift) & 31u)) & 1u;
            w[i] = maybe ? exact32[u[i] >> 5] : 0u;
        }
    }
#pragma unroll
    for (int i = 0; i < kUnroll; ++i) {
        uint64_t ballot = __ballot((w[i] >> (u[i] & 31u)) & 1u);
        if (kCareful && __builtin_amdgcn_readlane(my_chunk, sub + i) == last_chunk) ballot &= last_mask;
        if (lane == sub + i) { *lo = (uint32_t) ballot; *hi = (uint32_t) (ballot >> 32); }
    }
}

// Chunks begin .. end - 1 of a work list (the same for all lanes of a wave), in sets of kUnroll.
template <int kMode, int kUnroll>
__device__ __forceinline__ void flag_list_part(const SampleArgs& a, const uint32_t* lds32, int64_t begin, int64_t end)
{
    const int64_t last_chunk = (a.num_entries - 1) >> 6;
    const bool last_is_partial = (a.num_entries & 63) != 0;
    for (int64_t c0 = begin; c0 < end; c0 += kFlagBatch) {
        const int lane = opaque_lane_id();
        const int here = (int) ((end - c0 < kFlagBatch) ? end - c0 : kFlagBatch);     // scalar, >= 1
        // Lane l holds the chunk id of work-list entry c0 + l; lanes past the share repeat its last
        // entry (their result is not stored), so that every unrolled set is made of valid chunks.
        const int64_t q = c0 + (lane < here ? lane : here - 1);
        const int32_t my_chunk = a.plan_desc[q];
        const bool careful = last_is_partial && __ballot((int64_t) my_chunk == last_chunk) != 0ull;
        uint32_t lo = 0, hi = 0;
        for (int sub = 0; sub < here; sub += kUnroll) {                                // scalar bounds
            if (careful) flag_chunk_set<kMode, kUnroll, true>(a, lds32, my_chunk, sub, lane, &lo, &hi);
            else         flag_chunk_set<kMode, kUnroll, false>(a, lds32, my_chunk, sub, lane, &lo, &hi);
        }
        if (lane < here) a.flags[my_chunk] = ((uint64_t) hi << 32) | lo;
    }
}

// kMode 1 / 2: the cache bitmap / the cache filter is first copied into dynamic LDS (rounded up to
// 16 bytes).  The work lists of the group's `count` mini-batches, which read the same cache, are shared out as one: every wave
// takes an equal part, which may go on from one list to the next.  Each list shared out by itself, one after the other, cost its
// chain of reads every time: lists of four mini-batches 20.5 to 24 us on up to 1.3 M nodes and 37 to 43 on 2 to 20 M, as one 8.5 to 15
// and 14 to 27.
// Short lists ask the exact bitmap in global memory instead, in small sets: staging takes 4 us to 10 us (the filter) whatever the
// lists' length.  Below one chunk per wave 7.5 to 9 us staged (bitmap) or 12.5 to 16 (filter) and 4 to 5 direct.  The direct pass
// grows by 64 requests a chunk at the L2s' rate: at 7 to 8 chunks per wave 8.7 to 10 and 6.1 to 7.3 us (bitmap), 13 to 16 and 9.4 to
// 10.7 (filter), at 10 as long or longer on 1 M nodes and more, for single lists and for groups of two and four.
constexpr int kFlagShortUnroll = 4, kFlagShort = 8;          // chunks: of a set, of a wave at most

template <int kMode>
__global__ void k_flag_chunks(LayerArgs g, int count)
{
    extern __shared__ uint4 lds_bitmap16[];
    const uint32_t* lds32 = reinterpret_cast<const uint32_t*>(lds_bitmap16);
    SampleArgs a = bind_sample(g, 0);                    // the batches differ in their lists only
    const int wave = __builtin_amdgcn_readfirstlane((int) (threadIdx.x >> 6));
    const int64_t waves_per_block = (int64_t) (blockDim.x >> 6), num_waves = (int64_t) gridDim.x * waves_per_block;
    const int lane = lane_id();
    const int32_t chunks = lane < count ? bind_state(g, lane)->plan_chunks : 0;          // lane b: of list b
    int64_t all = 0;
    for (int b = 0; b < count; ++b) all += __builtin_amdgcn_readlane(chunks, b);
    // chunks begin .. end - 1 of all lists
    auto flag = [&](auto mode, auto unroll, int64_t begin, int64_t end) {
        for (int b = 0; b < count && end > 0; ++b) {
            const int64_t Q = __builtin_amdgcn_readlane(chunks, b);
            a.plan_desc = at<int32_t>(g.b[b].ws, g.off.plan_desc);
            flag_list_part<decltype(mode)::value, decltype(unroll)::value>(a, lds32, begin > 0 ? begin : 0, end < Q ? end : Q);
            begin -= Q;
            end -= Q;
        }
    };
    int64_t share = (all + num_waves - 1) / num_waves;
    if ((kMode == 1 || kMode == 2) && share <= kFlagShort) {
        // a list of fewer sets than there are waves is spread over the blocks
        if (share < kFlagShortUnroll) share = kFlagShortUnroll;
        const int64_t begin = ((int64_t) wave * gridDim.x + blockIdx.x) * share;
        flag(std::integral_constant<int, 0>(), std::integral_constant<int, kFlagShortUnroll>(), begin, begin + share);
        return;
    }
    if (kMode == 1) stage_lds(lds_bitmap16, reinterpret_cast<const uint4*>(a.cache_bitmap), (int32_t) ((a.bitmap_words + 1) / 2));
    if (kMode == 2) stage_filter(lds_bitmap16, a.filter_groups);
    if (kMode == 1 || kMode == 2) __syncthreads();
    const int64_t begin = ((int64_t) blockIdx.x * waves_per_block + wave) * share;
    flag(std::integral_constant<int, kMode>(), std::integral_constant<int, kFlagUnroll>(), begin, begin + share);
}

// group-wide helpers for G consecutive lanes (G a power of two)
template <int G>
__device__ __forceinline__ int32_t group_inclusive_scan(int32_t v, int s)
{
#pragma unroll
    for (int d = 1; d < G; d <<= 1) {
        const int32_t up = __shfl_up(v, d, G);
        if (s >= d) v += up;
    }
    return v;
}

constexpr int kHubWords = 4;        // flag words a lane holds per step when the whole wave walks a hub row

// One dst row per group of G consecutive lanes (s = lane within the group): count the row's
// eligible neighbors from its flag words, draw, map the chosen ranks back to CSR positions and
// emit.  A step covers G * W words, lane s holding words s*W .. s*W+W-1 of it,
// so ranks run in lane order.  Every lane of the wave must call it (it exchanges data between
// lanes); `live` says whether this lane's group has a row.
template <int G, int W>
__device__ __forceinline__ void select_row(const SampleArgs& a, int64_t row, bool live, int s, int64_t start,
                                           int64_t end, int32_t vi)
{
    const int k = a.fanout;
    const int32_t nw = live ? chunks_touched(start, end) : 0;     // flag words of this row
    const int64_t g0 = start >> 6;
    const uint64_t head_mask = ~0ull << (start & 63);
    const int tail_bits = (int) (end & 63);
    const uint64_t tail_mask = tail_bits ? ((1ull << tail_bits) - 1ull) : ~0ull;

    auto load_words = [&](int32_t j0, uint64_t* w) -> int32_t {
        int32_t c = 0;
#pragma unroll
        for (int i = 0; i < W; ++i) {
            const int32_t j = j0 + i;
            uint64_t x = 0;
            if (j < nw) {
                x = a.flags[g0 + j];
                if (j == 0) x &= head_mask;
                if (j == nw - 1) x &= tail_mask;
            }
            w[i] = x;
            c += __popcll(x);
        }
        return c;
    };

    // pass 1: N_C(v) = set bits of the row's flag words, trimmed to [start, end)
    uint32_t m = 0;
    uint64_t w_first[W];
    int32_t incl_first = 0;
#pragma unroll
    for (int i = 0; i < W; ++i) w_first[i] = 0;
    for (int32_t it = 0; __any(it * G * W < nw); ++it) {
        uint64_t w[W];
        const int32_t c = load_words((it * G + s) * W, w);
        const int32_t incl = group_inclusive_scan<G>(c, s);
        if (it == 0) {
#pragma unroll
            for (int i = 0; i < W; ++i) w_first[i] = w[i];
            incl_first = incl;
        }
        m += (uint32_t) __shfl(incl, G - 1, G);
    }

    uint32_t val;
    int pos;
    floyd_in_group<G>(m > (uint32_t) k ? m : (uint32_t) k + 1u, k, k, a.st->key0, a.st->key1, a.layer_number,
                      (uint32_t) vi, s, &val, &pos);
    const int cnt = (m > (uint32_t) k) ? k : (int) m;
    if (m <= (uint32_t) k) { val = (uint32_t) s; pos = s; }

    // pass 2: lane s < count finds the lane, then the word, then the bit that holds its rank `want` among
    // the set bits of the row's words (of their complements inside the row when `inverted`)
    auto locate = [&](uint32_t want, int count, bool inverted) -> int64_t {
        int64_t entry = -1;
        uint32_t run = 0;
        for (int32_t it = 0; __any(it * G * W < nw); ++it) {
            uint64_t w[W];
            int32_t incl = incl_first;
#pragma unroll
            for (int i = 0; i < W; ++i) w[i] = w_first[i];
            if (it > 0) incl = group_inclusive_scan<G>(load_words((it * G + s) * W, w), s);   // long rows reload
            if (inverted) {
                // entries of the row that are not flagged: complement inside [start, end)
                int32_t c = 0;
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    const int32_t j = (it * G + s) * W + i;
                    uint64_t valid = (j < nw) ? ~0ull : 0ull;
                    if (j == 0) valid &= head_mask;
                    if (j == nw - 1) valid &= tail_mask;
                    w[i] = ~w[i] & valid;
                    c += __popcll(w[i]);
                }
                incl = group_inclusive_scan<G>(c, s);
            }
            const uint32_t step_total = (uint32_t) __shfl(incl, G - 1, G);
            const bool mine = s < count && entry < 0 && want >= run && want < run + step_total;
            const uint32_t local = want - run;
            // owner = number of lanes whose inclusive count is <= local
            int owner = 0;
            if (G == 64) {
                // the whole wave is one group: one ballot per drawn slot instead of one shuffle per lane
                for (int q = 0; q < k; ++q) {
                    const uint32_t local_q = (uint32_t) __shfl((int) local, q, G);
                    const int below = __popcll(__ballot((uint32_t) incl <= local_q));
                    if (s == q) owner = below;
                }
            } else {
                for (int t = 0; t < G; ++t) owner += ((uint32_t) __shfl(incl, t, G) <= local) ? 1 : 0;
            }
            owner = owner < G ? owner : G - 1;
            uint64_t wo[W];
            int32_t own_total = 0;
#pragma unroll
            for (int i = 0; i < W; ++i) {
                wo[i] = __shfl(w[i], owner, G);
                own_total += __popcll(wo[i]);
            }
            const int32_t incl_owner = __shfl(incl, owner, G);
            if (mine) {
                int32_t rest = (int32_t) local - (incl_owner - own_total);       // rank inside the owner's words
                int which = 0;
                uint64_t word = wo[0];
#pragma unroll
                for (int i = 0; i < W - 1; ++i) {
                    const int32_t c = __popcll(wo[i]);
                    if (which == i && rest >= c) { rest -= c; which = i + 1; word = wo[i + 1]; }
                }
                const int bit = select_bit64(word, rest);
                entry = (g0 + ((int64_t) it * G + owner) * W + which) * 64 + bit;
            }
            run += step_total;
        }
        return entry;
    };

    const int64_t entry = locate(val, cnt, false);
    if (live && s < cnt) {
        const int32_t u = a.indices[entry];
        // Section 3.4: coefficient p^C_u * k / min(k, N_C(v)), weight = 1 / coefficient; p^C_u comes
        // from the table filled when the cache was drawn (u is in the cache); fp32 from here on
        const float inv_pc = a.node_inv_pc[u];
        float wgt;
        if (a.wmode == GNS_W_UNBIASED) wgt = inv_pc * ((float) m / (float) cnt);
        else                           wgt = inv_pc * ((float) cnt / (float) k);
        a.s_w[row * k + pos] = wgt;
        a.s_nbr[row * k + pos] = mark_if_new(a, (uint32_t) u);
    }

    // Section 3.3: a row with fewer than k cached neighbors fills up from its other neighbors, drawn
    // uniformly without replacement with the row's next Philox slots (cnt, cnt + 1, ...).
    int total = cnt;
    if (a.policy == GNS_CACHE_FIRST) {
        const uint32_t others = live ? (uint32_t) (end - start) - m : 0u;        // |N(v) \ C|
        const int room = k - cnt;
        const int fill = (others > (uint32_t) room) ? room : (int) others;
        if (__any(fill > 0)) {
            uint32_t fval;
            int fpos;
            floyd_in_group<G>(others > (uint32_t) room ? others : (uint32_t) room + 1u, room, k, a.st->key0,
                              a.st->key1, a.layer_number, (uint32_t) vi, s, &fval, &fpos, cnt);
            if (others <= (uint32_t) room) { fval = (uint32_t) s; fpos = s; }
            const int64_t fentry = locate(fval, fill, true);
            if (live && s < fill) {
                const int32_t u = a.indices[fentry];
                // fill neighbors: weight 1 (a node-wise sample), or the inverse inclusion probability of a
                // uniform subset of the uncached neighbors in the unbiased mode
                const float wgt = (a.wmode == GNS_W_UNBIASED) ? (float) others / (float) fill : 1.0f;
                a.s_w[row * k + cnt + fpos] = wgt;
                a.s_nbr[row * k + cnt + fpos] = mark_if_new(a, (uint32_t) u);
            }
            total = cnt + fill;
        }
    }
    if (live && s == 0) {
        a.s_cnt[row] = total;
        a.row_eligible[row] = (int32_t) m;
        a.src_nodes[row] = vi;
    }
}

// G lanes per dst row, one flag word per lane and step.  Hub rows (listed by k_plan with one
// atomic per 256 rows: an atomic per wave where nodes join the batch made the union step of a layer of 73 K new nodes 3.5 us
// longer) would keep the rest of their wave waiting, so for G < 64 the row blocks skip them
// and hub_blocks further blocks give each of them a whole wave (64 * kHubWords words per step).
// Block order: hub blocks, row blocks.
template <int G, bool kOne>
__global__ void __launch_bounds__(kBlock) k_select_rows(LayerArgs g, int hub_blocks)
{
    const GroupBlock q = group_block<kOne>(g.dealt);
    if (!kOne && q.block >= g.blocks) return;
    const SampleArgs a = bind_sample(g, q.b);
    const int wave_in_block = __builtin_amdgcn_readfirstlane((int) (threadIdx.x >> 6));
    if (q.block < hub_blocks) {
        const int32_t H = a.st->hub_count[a.layer_index];
        const int32_t nhw = hub_blocks * (kBlock / kWave);
        for (int32_t h = q.block * (kBlock / kWave) + wave_in_block; h < H; h += nhw) {
            const int lane = opaque_lane_id();
            const int32_t row = a.hub_rows[h];
            const RowExtent ext = a.row_ext[row];
            const int32_t vi = a.dst_nodes[row];
            select_row<64, kHubWords>(a, row, true, lane, ext.start, ext.end, vi);
        }
        return;
    }
    const int64_t block = (int64_t) q.block - hub_blocks;
    const int64_t nblocks = (int64_t) g.blocks - hub_blocks;
    const int32_t R = a.st->num_dst[a.layer_index];
    constexpr int kRowsPerWave = kWave / G;
    const int64_t wave_global = block * (kBlock / kWave) + wave_in_block;
    const int64_t num_waves = nblocks * (kBlock / kWave);
    for (int64_t row0 = wave_global * kRowsPerWave; row0 < R; row0 += num_waves * kRowsPerWave) {
        const int lane = opaque_lane_id();
        const int s = lane & (G - 1);
        const int64_t row = row0 + (lane / G);
        bool live = row < R;
        int32_t vi = -1;
        int64_t start = 0, end = 0;
        if (live) {
            const RowExtent ext = a.row_ext[row];
            vi = a.dst_nodes[row];
            start = ext.start;
            end = ext.end;
        }
        if (hub_blocks > 0 && is_hub_extent(start, end)) live = false;      // taken by a hub wave
        select_row<G, 1>(a, row, live, s, start, end, vi);
    }
}

// The cache pointers of the template are those of generation 0; the kernels shift them to the generation each
// batch reads.
void fill_sample_template(gns_ctx* c, int layer_index, SampleArgs* out)
{
    const Layout& L = c->lay;
    SampleArgs& a = *out;
    memset(&a, 0, sizeof(a));
    a.layer_index = layer_index;
    a.layer_number = (uint32_t) (c->config.num_layers - layer_index);
    a.fanout = c->config.fanout[layer_index];
    a.wmode = c->config.wmode;
    a.policy = c->config.policy[layer_index];
    a.indices = c->graph.indices;
    const int gen = 0;
    a.node_inv_pc = c->uses_cache && !L.slot_marks ? cache_ptr<float>(c, L.node_pc, gen) : nullptr;
    a.node_slot = L.slot_marks ? cache_ptr<CachedNode>(c, L.node_pc, gen) : nullptr;
    a.by_slot = L.slot_marks && layer_index == c->config.num_layers - 1 ? 1 : 0;
    a.cache_bitmap = cache_ptr<uint64_t>(c, L.cache_bitmap, gen);
    a.num_entries = c->graph.num_entries;
    a.max_chunks = (uint32_t) L.max_chunks;
    a.flags = c->uses_cache && c->config.flag_mode == GNS_FLAGS_PER_BATCH ? cache_ptr<uint64_t>(c, L.edge_flags, gen) : nullptr;
    a.bitmap_words = L.words;
    a.filter_groups = cache_filter(c, gen).groups;
    a.filter_mult = L.filter_mult;
    a.coarse_bitmap = L.coarse_shift ? cache_ptr<uint64_t>(c, L.coarse_bitmap, gen) : nullptr;
    a.coarse_shift = L.coarse_shift;
    const bool induced = c->uses_cache && c->config.flag_mode == GNS_FLAGS_PER_CACHE;
    a.srec = induced ? cache_ptr<ChunkRec>(c, L.srec, gen) : nullptr;
    a.s_nodes = induced ? cache_ptr<int32_t>(c, L.s_nodes, gen) : nullptr;
    a.s_count = induced ? cache_ptr<int32_t>(c, L.s_count, gen) : nullptr;
    a.s_tile_shift = L.s_tile_shift;
}

static void launch_flag_kernel(gns_ctx* c, const LayerArgs& a, int count, hipStream_t s)
{
    const size_t lds_bytes = (size_t) ((c->lay.words + 1) / 2) * 16;
    if (lds_bytes <= c->lds_bitmap_limit)
        hipLaunchKernelGGL((k_flag_chunks<1>), dim3((unsigned) c->num_cus), dim3(1024), lds_bytes, s, a, count);
    else if (c->lay.filter && kLdsBitmapBytes <= c->lds_bitmap_limit)
        hipLaunchKernelGGL((k_flag_chunks<2>), dim3((unsigned) c->num_cus), dim3(1024), kLdsBitmapBytes, s, a, count);
    else if (c->lay.coarse_shift > 0 && !getenv("GNS_NO_COARSE_L2"))
    {
        const int per_cu = getenv("GNS_FLAG_BLOCKS_PER_CU") ? atoi(getenv("GNS_FLAG_BLOCKS_PER_CU")) : 2;
        hipLaunchKernelGGL((k_flag_chunks<3>), dim3((unsigned) (c->num_cus * per_cu)), dim3(kBlock), 0, s, a, count);
    }
    else
    {
        // every wave keeps 32 x 64 bitmap reads in flight, so a few waves per CU already reach the rate the
        // memory system gives scattered reads; a grid that filled the chip would keep the kernels of other
        // streams out for the whole pass
        const int per_cu = getenv("GNS_FLAG_BLOCKS_PER_CU") ? atoi(getenv("GNS_FLAG_BLOCKS_PER_CU")) : 2;
        hipLaunchKernelGGL((k_flag_chunks<0>), dim3((unsigned) (c->num_cus * per_cu)), dim3(kBlock), 0, s, a, count);
    }
}

bool direct_layer(const gns_config& config, int layer_index)
{
    return config.policy[layer_index] == GNS_UNIFORM || config.flag_mode == GNS_FLAGS_PER_CACHE;
}

bool first_layer_enters_seeds(const gns_config& config)
{
    return direct_layer(config, 0) && config.fanout[0] <= 16;
}

// Rows per wave of the two-stage sampler: as many as leave 32 waves for every CU (all it holds) at the layer's worst-case
// number of rows, a power of two between 4 and 32.  (A mini-batch's grid ends at 16 waves for every CU, so single ones take their
// rows in more turns.)  The worst case of the call's seeds (bound_rows) is all the host knows; input layers have 0.2 (cache first) to
// 0.5 of it (fan-outs 15, 10 on 1 M nodes), so their launches have fewer waves than that.  Layers of 4 x 12,600 rows, fan-out
// 10: 25 us with 8 rows per wave, 26 with 16, 37 with 64; of 4 x 92,400 rows, fan-out 5: 36.5 us with 32, 37.5 with 64, 42
// with 16 (twice the blocks).  Captured launches go by the context's worst case: mini-batches far below it have few waves of many rows there.
static int wave_rows(const Group& g, int layer_index)
{
    const gns_ctx* c = g.ctx[0];
    const int64_t rows = g.rows[layer_index] * g.count;
    int W = 4;
    while (W < kWaveRows && (int64_t) W * c->num_cus * 32 < rows) W *= 2;
    return W;
}

int rows_per_sum(const Group& g, int layer_index)
{
    const gns_ctx* c = g.ctx[0];
    if (!direct_layer(c->config, layer_index)) return 0;
    return kBlock / kWave * (c->config.fanout[layer_index] <= 16 ? wave_rows(g, layer_index) : 1);
}

// f(kList): calls it with the kind of list a direct layer draws from as a compile-time constant.
template <typename F>
static void with_list(const gns_ctx* c, int layer_index, F&& f)
{
    const int policy = c->config.policy[layer_index];
    if (policy == GNS_UNIFORM)         f(std::integral_constant<int, kListRow>());
    else if (policy == GNS_CACHE_ONLY) f(std::integral_constant<int, kListCached>());
    else                               f(std::integral_constant<int, kListCachedFirst>());
}

// f(K): the smallest unroll length that holds the fan-out.  A Philox block gives four slots, fan-outs below 5 are not worth an
// instance of their own, and the longest is the kernel's limit (groups of four on 1 M nodes: fan-outs 8, 8, 8 take 216 us
// with 8 slots and 218 with 12; 12, 12, 5 take 275 with 12 and 277 with 16).
template <typename F>
static void with_unroll(int fanout, F&& f)
{
    if (fanout <= 8)       f(std::integral_constant<int, 8>());
    else if (fanout <= 12) f(std::integral_constant<int, 12>());
    else                   f(std::integral_constant<int, 16>());
}

hipError_t launch_first_layer(const Group& g, const BeginDyn& d, hipStream_t s)
{
    gns_ctx* c = g.ctx[0];
    LayerArgs a;
    fill_first_args(g, &a);
    const int rows_per_block = rows_per_sum(g, 0);
    const dim3 grid = group_grid(g, a, first_blocks(g, (g.rows[0] + rows_per_block - 1) / rows_per_block));
    with_unroll(a.s.fanout, [&](auto K) {
        with_list(c, 0, [&](auto kList) {
            with_one(g, [&](auto kOne) {
                hipLaunchKernelGGL((k_sample_first<decltype(K)::value, decltype(kList)::value, decltype(kOne)::value>), grid, dim3(kBlock),
                                   0, s, a, d, rows_per_block / (kBlock / kWave));
            });
        });
    });
    return hipGetLastError();
}

// The fixed argument block of a group's first launch (k_batch_begin or k_sample_first).
void fill_first_args(const Group& g, LayerArgs* out)
{
    fill_group_args(g, out);
    set_group_layer(g, 0, out);
    fill_sample_template(g.ctx[0], 0, &out->s);
    fill_finish_template(g, 0, &out->f);
}

// One layer's sampler launches for a group of mini-batches.  The previous layer's relabel rides in front
// of this layer's first kernel: both only need that layer's phase 3, and they touch disjoint memory
// (sampler scratch alternates by layer).
hipError_t launch_sample_layer(const Group& g, int layer_index, hipStream_t s)
{
    gns_ctx* c = g.ctx[0];
    LayerArgs a;
    fill_group_args(g, &a);
    set_group_layer(g, layer_index, &a);
    fill_sample_template(c, layer_index, &a.s);
    int rl = 0;
    if (layer_index > 0) {
        fill_finish_template(g, layer_index - 1, &a.f);
        rl = relabel_grid(g, layer_index - 1);
    }
    auto grid_of = [&](int64_t blocks) {
        a.blocks = (int32_t) blocks;
        return group_grid(g, a, blocks);
    };

    const int64_t rows_max = g.rows[layer_index];
    const dim3 tb(kBlock);
    const int policy = c->config.policy[layer_index];
    if (direct_layer(c->config, layer_index)) {
        StageTimer t(c, GNS_STAGE_SELECT, s, policy == GNS_CACHE_ONLY);
        const int rows_per_block = rows_per_sum(g, layer_index);
        // sized for the worst case; batches are much smaller, so from four blocks per CU on a block takes several turns
        int64_t blocks = (rows_max + rows_per_block - 1) / rows_per_block;
        const bool narrow = a.s.fanout <= 16;
        const int64_t cap = (int64_t) c->num_cus * (narrow ? 4 : 16);
        if (blocks > cap) blocks = cap;
        const dim3 grid = grid_of(blocks + rl);
        with_list(c, layer_index, [&](auto kList) {
            with_one(g, [&](auto kOne) {
                if (!narrow) {
                    hipLaunchKernelGGL((k_sample_wide<decltype(kList)::value, decltype(kOne)::value>), grid, tb, 0, s, a, rl);
                    return;
                }
                with_unroll(a.s.fanout, [&](auto K) {
                    hipLaunchKernelGGL((k_sample_rows<decltype(K)::value, decltype(kList)::value, decltype(kOne)::value>), grid, tb, 0, s,
                                       a, rows_per_block / (kBlock / kWave), rl);
                });
            });
        });
        return hipGetLastError();
    }
    const int G = a.s.fanout <= 8 ? 8 : a.s.fanout <= 16 ? 16 : 64;
    const int64_t rows_per_block = kBlock / G;
    int64_t row_blocks = (rows_max + rows_per_block - 1) / rows_per_block;
    // One step of rows per wave where that fits: rows differ a lot in cost, and with more blocks
    // than the chip holds the dispatcher hands out new rows as waves finish.
    const int64_t cap = (int64_t) c->num_cus * 64;
    if (row_blocks > cap) row_blocks = cap;
    if (row_blocks < 1) row_blocks = 1;

    // CACHE_ONLY and CACHE_FIRST without the induced subgraph: plan -> flag -> select
    {
        StageTimer t(c, GNS_STAGE_PLAN, s);
        const unsigned plan_blocks = (unsigned) ((rows_max + kPlanTile - 1) / kPlanTile);
        const dim3 grid = grid_of((int64_t) plan_blocks + rl);
        with_one(g, [&](auto kOne) { hipLaunchKernelGGL(k_plan<decltype(kOne)::value>, grid, tb, 0, s, a, rl, c->union_spins); });
    }
    {
        StageTimer t(c, GNS_STAGE_FLAG, s);
        launch_flag_kernel(c, a, g.count, s);
    }
    StageTimer t(c, GNS_STAGE_SELECT, s);
    // hub rows get dedicated waves (the count lives on the device; the waves stride over the list)
    const int hub_blocks = (G < 64) ? (int) (rows_max / (kBlock / kWave) < (int64_t) c->num_cus * 2
                                                 ? rows_max / (kBlock / kWave) + 1 : (int64_t) c->num_cus * 2) : 0;
    const dim3 rb = grid_of(row_blocks + hub_blocks);
    with_one(g, [&](auto kOne) {
        constexpr bool one = decltype(kOne)::value;
        if (G == 8)       hipLaunchKernelGGL((k_select_rows<8, one>), rb, tb, 0, s, a, hub_blocks);
        else if (G == 16) hipLaunchKernelGGL((k_select_rows<16, one>), rb, tb, 0, s, a, hub_blocks);
        else              hipLaunchKernelGGL((k_select_rows<64, one>), rb, tb, 0, s, a, hub_blocks);
    });
    return hipGetLastError();
}

}  // namespace gns
