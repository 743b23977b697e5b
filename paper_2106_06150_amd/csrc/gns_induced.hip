// The induced subgraph S of the cache (paper Section 3.3: "we construct an induced subgraph S that contains
// the nodes in the cache and their neighbor nodes.  This is done once right after we sample nodes in the
// cache.") in compact form (GNS_FLAGS_PER_CACHE):
//
//   s_nodes     the CSR entries that point into the cache (node ids), tile by tile: the entry array is cut into aligned
//               tiles of 2^s_tile_shift entries, and a tile's cached entries stand, in CSR order, from its own offset on
//               (s_nodes has the length of the entry array)
//   srec[g]     for every aligned 64-entry chunk g of the CSR entry array: its 64 membership flags and the place in
//               s_nodes of the first of them
//   s_count[t]  cached entries of tile t
//
// With P(e) = srec[e >> 6].before + popcount(srec[e >> 6].flags below bit e & 63), the cached neighbors of a row that
// lies in one tile are s_nodes[P(first) .. P(last) + flag(last)); a row that crosses tiles continues at the next tile's
// offset.  A mini-batch reads two records and the few entries it draws, never the row.  No tile depends on another, so
// one pass over the entries builds everything.
#include <stdlib.h>
#include "gns_kernels.hpp"

namespace gns {

struct InducedArgs {
    const int32_t* done;       // the draw's completing chunk, or null: below zero the cache is incomplete and there is nothing to do
    const int32_t* indices;
    int64_t num_entries;
    int64_t num_chunks;        // ceil(nnz / 64)
    int32_t tiles;
    int tile_shift;
    const uint64_t* bitmap;
    int64_t bitmap_words;
    const uint64_t* coarse;    // one bit per 2^coarse_shift ids (kCoarseLds, kCoarse)
    int64_t coarse_words;
    int coarse_shift;
    ChunkRec* srec;            // [num_chunks]
    int32_t* s_nodes;
    int32_t* s_count;          // [tiles]
};

constexpr int kSChunks = 16;                             // chunks of a wave's step: their entries stay in registers
constexpr int kSStepShift = 10;                          // entries of a step (a power of two)

// Where the membership test looks first: the exact bitmap in LDS or in global memory, its coarse companion in LDS or in
// global memory (then only entries whose group has a cached node read the exact bitmap).
enum { kExact = 0, kExactLds = 1, kCoarseLds = 2, kCoarse = 3 };

// One pass over the CSR entry array: test every entry, write the chunk records and the compacted list.  A wave walks a
// tile in steps of 1024 entries, each read once and kept in its lane's register until its place is known; the next
// step's entries are on their way meanwhile, and no wave waits for another.  Bound by the stream of entries where the
// exact bitmap fits LDS, by the rate of L2 requests (one per entry that passes the coarse bitmap) beyond.
// 40 M entries (exact bitmap in LDS): 62 us, where a flag pass, a scan of its words and a compaction that read the entries
// once more took 95; 400 M entries of a 40 M-node graph: 1.40 ms, before 1.92.
template <int kMode>
__global__ void __launch_bounds__(kMode == kExactLds || kMode == kCoarseLds ? 1024 : kBlock) k_build_induced(InducedArgs a)
{
    extern __shared__ uint4 lds_bitmap16[];
    if (a.done && *a.done < 0) return;
    if (kMode == kExactLds || kMode == kCoarseLds) {
        stage_lds(lds_bitmap16, reinterpret_cast<const uint4*>(kMode == kExactLds ? a.bitmap : a.coarse),
                  (int32_t) (((kMode == kExactLds ? a.bitmap_words : a.coarse_words) + 1) / 2));
        __syncthreads();
    }
    const uint32_t* lds32 = reinterpret_cast<const uint32_t*>(lds_bitmap16);
    const uint32_t* exact32 = reinterpret_cast<const uint32_t*>(a.bitmap);
    const uint32_t* coarse32 = reinterpret_cast<const uint32_t*>(a.coarse);
    const int waves_per_block = (int) (blockDim.x >> 6);
    const int32_t num_waves = (int32_t) gridDim.x * waves_per_block;
    // entries of the step that begins at entry e0; those past the end of the array repeat its last entry
    auto load = [&](int64_t e0, uint32_t (&dst)[kSChunks]) {
        const int32_t* src = a.indices + e0;                                                   // wave-uniform
        const int64_t left = a.num_entries - e0;
        const int lane = lane_id();
        if (left >= kSChunks * kWave) {
#pragma unroll
            for (int i = 0; i < kSChunks; ++i) dst[i] = (uint32_t) src[i * kWave + lane];
        } else if (left > 0) {
#pragma unroll
            for (int i = 0; i < kSChunks; ++i) {
                const int64_t at = i * kWave + lane;
                dst[i] = (uint32_t) src[at < left ? at : left - 1];
            }
        }
    };
    // neighboring tiles go to different blocks: a graph of fewer tiles than the chip has waves still uses every CU
    int32_t tile = __builtin_amdgcn_readfirstlane((int) (threadIdx.x >> 6)) * (int32_t) gridDim.x + (int32_t) blockIdx.x;
    if (tile >= a.tiles) return;
    const int64_t tile_entries = (int64_t) 1 << a.tile_shift;
    int64_t e0 = (int64_t) tile << a.tile_shift, tile_end = e0 + tile_entries;
    if (tile_end > a.num_entries) tile_end = a.num_entries;
    uint32_t at_tile = (uint32_t) e0;                                   // where the next cached entry goes
    uint32_t u[kSChunks];
#pragma unroll
    for (int i = 0; i < kSChunks; ++i) u[i] = 0;
    load(e0, u);
    for (;;) {
        const int lane = opaque_lane_id();
        // the step after this one: in the same tile, or the first of the wave's next tile
        int64_t e_next = e0 + ((int64_t) 1 << kSStepShift);
        const bool tile_done = e_next >= tile_end;
        if (tile_done) e_next = ((int64_t) tile + num_waves) << a.tile_shift;
        uint32_t ahead[kSChunks];
#pragma unroll
        for (int i = 0; i < kSChunks; ++i) ahead[i] = 0;
        load(e_next, ahead);
        uint32_t w[kSChunks];
#pragma unroll
        for (int i = 0; i < kSChunks; ++i) {
            if (kMode == kExactLds)       w[i] = lds32[u[i] >> 5];
            else if (kMode == kCoarseLds) w[i] = lds32[(u[i] >> a.coarse_shift) >> 5];
            else if (kMode == kCoarse)    w[i] = coarse32[(u[i] >> a.coarse_shift) >> 5];
            else                          w[i] = exact32[u[i] >> 5];
        }
        if (kMode == kCoarseLds || kMode == kCoarse) {
#pragma unroll
            for (int i = 0; i < kSChunks; ++i) {
                const bool maybe = (w[i] >> ((u[i] >> a.coarse_shift) & 31u)) & 1u;
                w[i] = maybe ? exact32[u[i] >> 5] : 0u;
            }
        }
        const int left = (int) (tile_end - e0 < (1 << kSStepShift) ? tile_end - e0 : (1 << kSStepShift));
        // lane i < kSChunks ends up with chunk i's flags
        uint64_t mine = 0;
#pragma unroll
        for (int i = 0; i < kSChunks; ++i) {
            const uint64_t f = __ballot(i * kWave + lane < left && ((w[i] >> (u[i] & 31u)) & 1u));
            if (lane == i) mine = f;
        }
        const int32_t count = __popcll(mine);
        const int32_t incl = wave_inclusive_scan(count);
        const uint32_t before = at_tile + (uint32_t) (incl - count);
        const int64_t g = (e0 >> 6) + lane;
        if (lane < kSChunks && lane * kWave < left) {
            ChunkRec r;
            r.flags = mine;
            r.before = before;
            r.pad = 0;
            a.srec[g] = r;
        }
        const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
        for (int i = 0; i < kSChunks; ++i) {
            const uint32_t lo = (uint32_t) __builtin_amdgcn_readlane((int) (uint32_t) mine, i);
            const uint32_t hi = (uint32_t) __builtin_amdgcn_readlane((int) (uint32_t) (mine >> 32), i);
            const uint64_t f = ((uint64_t) hi << 32) | lo;
            const uint32_t at = (uint32_t) __builtin_amdgcn_readlane((int) before, i);
            if ((f >> lane) & 1ull) a.s_nodes[at + (uint32_t) __popcll(f & below)] = (int32_t) u[i];
        }
        at_tile += (uint32_t) __builtin_amdgcn_readlane(incl, kWave - 1);
        if (tile_done) {
            if (lane == 0) a.s_count[tile] = (int32_t) (at_tile - (uint32_t) ((int64_t) tile << a.tile_shift));
            tile += num_waves;
            if (tile >= a.tiles) break;
            tile_end = e_next + tile_entries < a.num_entries ? e_next + tile_entries : a.num_entries;
            at_tile = (uint32_t) e_next;
        }
        e0 = e_next;
#pragma unroll
        for (int i = 0; i < kSChunks; ++i) u[i] = ahead[i];
    }
}

// Tiles of up to 16384 entries (few rows cross one), smaller ones while there would be fewer than two thousand (small
// graphs must still occupy the chip), at least one step.
int induced_tile_shift(int64_t num_entries)
{
    int shift = 14;
    while (shift > kSStepShift && (num_entries >> shift) < 2048) --shift;
    return shift;
}

hipError_t launch_build_induced(gns_ctx* c, int cache_gen, const int32_t* done, hipStream_t s)
{
    const Layout& L = c->lay;
    InducedArgs a;
    a.done = done;
    a.indices = c->graph.indices;
    a.num_entries = c->graph.num_entries;
    a.num_chunks = (c->graph.num_entries + 63) / 64;
    a.tile_shift = L.s_tile_shift;
    a.tiles = (int32_t) (((a.num_entries - 1) >> a.tile_shift) + 1);
    a.bitmap = cache_ptr<uint64_t>(c, L.cache_bitmap, cache_gen);
    a.bitmap_words = L.words;
    a.coarse = L.coarse_shift ? cache_ptr<uint64_t>(c, L.coarse_bitmap, cache_gen) : nullptr;
    a.coarse_words = L.coarse_words;
    a.coarse_shift = L.coarse_shift;
    a.srec = cache_ptr<ChunkRec>(c, L.srec, cache_gen);
    a.s_nodes = cache_ptr<int32_t>(c, L.s_nodes, cache_gen);
    a.s_count = cache_ptr<int32_t>(c, L.s_count, cache_gen);
    const size_t exact_bytes = (size_t) ((L.words + 1) / 2) * 16, coarse_bytes = (size_t) ((L.coarse_words + 1) / 2) * 16;
    const bool lds = exact_bytes <= c->lds_bitmap_limit || (L.coarse_shift > 0 && coarse_bytes <= c->lds_bitmap_limit);
    const int threads = lds ? 1024 : kBlock;
    const int32_t cap = c->num_cus * (lds ? 1 : 8);
    const dim3 grid((unsigned) (a.tiles < cap ? a.tiles : cap)), block((unsigned) threads);
    if (exact_bytes <= c->lds_bitmap_limit)
        hipLaunchKernelGGL((k_build_induced<kExactLds>), grid, block, exact_bytes, s, a);
    else if (lds)
        hipLaunchKernelGGL((k_build_induced<kCoarseLds>), grid, block, coarse_bytes, s, a);
    else if (L.coarse_shift > 0 && !getenv("GNS_NO_COARSE_L2"))
        hipLaunchKernelGGL((k_build_induced<kCoarse>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((k_build_induced<kExact>), grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace gns
