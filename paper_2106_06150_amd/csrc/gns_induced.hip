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
    CacheFilter filter;        // kFilterLds
    const uint64_t* coarse;    // one bit per 2^coarse_shift ids (kCoarse)
    int coarse_shift;
    ChunkRec* srec;            // [num_chunks]
    int32_t* s_nodes;
    int32_t* s_count;          // [tiles]
};

constexpr int kSChunks = 16;                             // chunks of a wave's step: their entries stay in registers
constexpr int kSStepShift = 10;                          // entries of a step (a power of two)

// Where the membership test looks first: the exact bitmap in LDS or in global memory, the cache filter in LDS, or a coarse
// bitmap in global memory (after these only what they leave open reads the exact bitmap).
enum { kExact = 0, kExactLds = 1, kFilterLds = 2, kCoarse = 3 };

// Inclusive scan over each row of 16 lanes.
__device__ __forceinline__ int32_t row_inclusive_scan(int32_t v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);      // row_shr:1, 2, 4, 8
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    return v;
}

// The entries of the wave's step at e0; what lies past the end of the array repeats its last entry.  No branch for that: a
// read inside one makes the compiler wait for all reads at its end.
__device__ __forceinline__ void load_step(const InducedArgs& a, int64_t e0, uint32_t (&dst)[kSChunks])
{
    const int64_t at = e0 < a.num_entries ? e0 : a.num_entries - 1, left = a.num_entries - at;
    const int32_t* src = a.indices + at;                                                   // wave-uniform
    const uint32_t last = (uint32_t) (left < kSChunks * kWave ? left : kSChunks * kWave) - 1u;
    const uint32_t lane = (uint32_t) lane_id();
#pragma unroll
    for (int i = 0; i < kSChunks; ++i) {
        const uint32_t q = (uint32_t) (i * kWave) + lane;
        dst[i] = (uint32_t) src[q < last ? q : last];
    }
}

// Membership flags of the step's chunks, the first `left` entries of it (scalars throughout); returns their number.
// kPairs: what the filter leaves open asks the list of pairs, and only what that leaves open the bitmap.
template <int kMode, bool kPairs>
__device__ __forceinline__ int32_t test_step(const InducedArgs& a, const uint32_t* lds32, const uint32_t (&u)[kSChunks], int left,
                                             uint64_t (&f)[kSChunks])
{
    const uint32_t* exact32 = reinterpret_cast<const uint32_t*>(a.bitmap);
    const uint32_t* coarse32 = reinterpret_cast<const uint32_t*>(a.coarse);
    uint32_t w[kSChunks];
#pragma unroll
    for (int i = 0; kMode != kFilterLds && i < kSChunks; ++i) {
        if (kMode == kExactLds)       w[i] = lds32[u[i] >> 5];
        else if (kMode == kCoarse)    w[i] = coarse32[(u[i] >> a.coarse_shift) >> 5];
        else                          w[i] = exact32[u[i] >> 5];
    }
    if (kMode == kFilterLds) {
        filter_test<kSChunks>(lds32, a.filter.mult, u, w);
#pragma unroll
        for (int i = 0; i < kSChunks; ++i)
            if (w[i] == 1u) w[i] = kPairs ? (uint32_t) a.filter.pairs[__umulhi(u[i], a.filter.mult)] : exact32[u[i] >> 5];
        if (kPairs) {
#pragma unroll
            for (int i = 0; i < kSChunks; ++i) {
                const uint32_t low = u[i] & kPairMask;
                const bool same = (w[i] & kPairMask) == low || ((w[i] >> kPairBits) & kPairMask) == low;
                if (w[i] + 1u > 1u) w[i] = same ? ~0u : (w[i] & kPairMore) ? 1u : 0u;           // neither ~0 nor 0: a pair
            }
#pragma unroll
            for (int i = 0; i < kSChunks; ++i)
                if (w[i] == 1u) w[i] = exact32[u[i] >> 5];
        }
    }
    if (kMode == kCoarse) {
#pragma unroll
        for (int i = 0; i < kSChunks; ++i) {
            const bool maybe = (w[i] >> ((u[i] >> a.coarse_shift) & 31u)) & 1u;
            w[i] = maybe ? exact32[u[i] >> 5] : 0u;
        }
    }
#pragma unroll
    for (int i = 0; i < kSChunks; ++i) f[i] = __ballot((w[i] >> (u[i] & 31u)) & 1u);
    if (left < kSChunks * kWave) {
#pragma unroll
        for (int i = 0; i < kSChunks; ++i) {
            const int here = left - i * kWave;
            f[i] &= here >= kWave ? ~0ull : here > 0 ? (1ull << here) - 1ull : 0ull;
        }
    }
    int32_t count = 0;
#pragma unroll
    for (int i = 0; i < kSChunks; ++i) count += __popcll(f[i]);
    return count;
}

// Writes the step's chunk records and its cached entries, the first of which goes to place `at` of s_nodes.
__device__ __forceinline__ void write_step(const InducedArgs& a, int64_t e0, const uint32_t (&u)[kSChunks], int left,
                                           const uint64_t (&f)[kSChunks], uint32_t at)
{
    const int lane = opaque_lane_id();
    uint32_t lo = 0, hi = 0;                                             // lane i < kSChunks: chunk i's flags
#pragma unroll
    for (int i = 0; i < kSChunks; ++i) {
        lo = lane == i ? (uint32_t) f[i] : lo;
        hi = lane == i ? (uint32_t) (f[i] >> 32) : hi;
    }
    const int32_t count = __popc(lo) + __popc(hi);
    ChunkRec r;
    r.flags = ((uint64_t) hi << 32) | lo;
    r.before = at + (uint32_t) (row_inclusive_scan(count) - count);
    r.pad = 0;
    if (lane < kSChunks && lane * kWave < left) a.srec[(e0 >> 6) + lane] = r;
    int32_t* dst = a.s_nodes + at;
#pragma unroll
    for (int i = 0; i < kSChunks; ++i) {
        const uint32_t below = __builtin_amdgcn_mbcnt_hi((uint32_t) (f[i] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t) f[i], 0u));
        if (__builtin_amdgcn_inverse_ballot_w64(f[i])) dst[below] = (int32_t) u[i];
        dst += __popcll(f[i]);
    }
}

// One pass over the CSR entry array: test every entry, write the chunk records and the compacted list.  A wave walks a
// tile in steps of 1024 entries, each read once and kept in its lane's register until its place is known; the next
// step's entries are on their way meanwhile, and no wave waits for another.  Bound by the stream of entries and the list where
// the exact bitmap fits LDS, by the rate of L2 requests (one per entry that the filter leaves open) beyond.  A chunk's flags
// are a scalar and an entry's place among them two instructions: with the flags in lanes, from where every chunk fetched its
// own and shifted them, the pass was bound by its instructions.
// 40 M entries (exact bitmap in LDS): 45 us, before 61 (42 with tiles shared by the waves of a block, which then wait for one
// another); 400 M entries of a 40 M-node graph, with the cache filter: 1.02 ms, before 1.38.
template <int kMode, bool kPairs = false>
__global__ void __launch_bounds__(kMode == kExactLds || kMode == kFilterLds ? 1024 : kBlock) k_build_induced(InducedArgs a)
{
    extern __shared__ uint4 lds_bitmap16[];
    if (a.done && *a.done < 0) return;
    if (kMode == kExactLds) stage_lds(lds_bitmap16, reinterpret_cast<const uint4*>(a.bitmap), (int32_t) ((a.bitmap_words + 1) / 2));
    if (kMode == kFilterLds) stage_filter(lds_bitmap16, a.filter.groups);
    if (kMode == kExactLds || kMode == kFilterLds) __syncthreads();
    const uint32_t* lds32 = reinterpret_cast<const uint32_t*>(lds_bitmap16);
    const int wave = __builtin_amdgcn_readfirstlane((int) (threadIdx.x >> 6));
    constexpr int64_t kStep = (int64_t) 1 << kSStepShift;
    uint32_t u[kSChunks], ahead[kSChunks];
    uint64_t f[kSChunks];
    const int32_t num_waves = (int32_t) gridDim.x * (int32_t) (blockDim.x >> 6);
    // neighboring tiles go to different blocks: a graph of fewer tiles than the chip has waves still uses every CU
    int32_t tile = wave * (int32_t) gridDim.x + (int32_t) blockIdx.x;
    if (tile >= a.tiles) return;
    const int64_t tile_entries = (int64_t) 1 << a.tile_shift;
    int64_t e0 = (int64_t) tile << a.tile_shift, tile_end = e0 + tile_entries;
    if (tile_end > a.num_entries) tile_end = a.num_entries;
    uint32_t at_tile = (uint32_t) e0;                                   // where the next cached entry goes
    load_step(a, e0, u);
    for (;;) {
        // the step after this one: in the same tile, or the first of the wave's next tile
        int64_t e_next = e0 + kStep;
        const bool tile_done = e_next >= tile_end;
        if (tile_done) e_next = ((int64_t) tile + num_waves) << a.tile_shift;
        load_step(a, e_next, ahead);
        const int left = (int) (tile_end - e0 < kStep ? tile_end - e0 : kStep);
        const int32_t count = test_step<kMode, kPairs>(a, lds32, u, left, f);
        write_step(a, e0, u, left, f, at_tile);
        at_tile += (uint32_t) count;
        if (tile_done) {
            if (opaque_lane_id() == 0) a.s_count[tile] = (int32_t) (at_tile - (uint32_t) ((int64_t) tile << a.tile_shift));
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
    a.filter = cache_filter(c, cache_gen);
    a.coarse_shift = L.coarse_shift;
    a.srec = cache_ptr<ChunkRec>(c, L.srec, cache_gen);
    a.s_nodes = cache_ptr<int32_t>(c, L.s_nodes, cache_gen);
    a.s_count = cache_ptr<int32_t>(c, L.s_count, cache_gen);
    const size_t exact_bytes = (size_t) ((L.words + 1) / 2) * 16;
    const bool lds = exact_bytes <= c->lds_bitmap_limit || (L.filter && kLdsBitmapBytes <= c->lds_bitmap_limit);
    const int threads = lds ? 1024 : kBlock;
    const int32_t cap = c->num_cus * (lds ? 1 : 8);
    const dim3 grid((unsigned) (a.tiles < cap ? a.tiles : cap)), block((unsigned) threads);
    if (exact_bytes <= c->lds_bitmap_limit)
        hipLaunchKernelGGL((k_build_induced<kExactLds>), grid, block, exact_bytes, s, a);
    else if (lds && a.filter.pairs)
        hipLaunchKernelGGL((k_build_induced<kFilterLds, true>), grid, block, kLdsBitmapBytes, s, a);
    else if (lds)
        hipLaunchKernelGGL((k_build_induced<kFilterLds>), grid, block, kLdsBitmapBytes, s, a);
    else if (L.coarse_shift > 0 && !getenv("GNS_NO_COARSE_L2"))
        hipLaunchKernelGGL((k_build_induced<kCoarse>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((k_build_induced<kExact>), grid, block, 0, s, a);
    return hipGetLastError();
}

}  // namespace gns
