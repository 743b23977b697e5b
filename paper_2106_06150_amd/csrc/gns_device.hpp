// Device-side building blocks shared by the GNS kernels (gfx950, wave64).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gns {

constexpr int kWave = 64;
constexpr int kBlock = 256;                 // threads per block for the scan-style kernels
constexpr int kItems = 8;                   // items per thread in a scan tile
constexpr int kTile = kBlock * kItems;      // 2048 items per scan tile
constexpr int kMarkTileMin = 64;             // frontier mark bitmap: words per tile, a power of two chosen per graph
constexpr int kMarkTileMax = 32 * kBlock;    //   so that the tiles number about a hundred (at most 32 words per thread)
constexpr int kSlotsMax = 1 << 16;           // slots of a cache whose new nodes are finished in one launch, see k_finish_cached
constexpr int kSlotTile = 16 * kBlock;       // slots of a tile of the union step beyond: so many times 1 to kSlotReads
constexpr int kSlotReads = 8;
constexpr int kMarkCap = 1024;               // marked words of a tile the union step keeps in LDS at a time

constexpr uint32_t kTagCache = 0x43414348u;     // 'CACH'
constexpr uint32_t kTagNeighbor = 0x4E424853u;  // 'NBHS'

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11).  One call yields four 32-bit words.
struct Philox4 {
    uint32_t w[4];
};

__device__ __forceinline__ Philox4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2, uint32_t c3,
                                                 uint32_t k0, uint32_t k1)
{
    constexpr uint32_t kMulA = 0xD2511F53u, kMulB = 0xCD9E8D57u;
    constexpr uint32_t kWeylA = 0x9E3779B9u, kWeylB = 0xBB67AE85u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint32_t a_hi = __umulhi(kMulA, c0), a_lo = kMulA * c0;
        const uint32_t b_hi = __umulhi(kMulB, c2), b_lo = kMulB * c2;
        c0 = b_hi ^ c1 ^ k0;
        c1 = b_lo;
        c2 = a_hi ^ c3 ^ k1;
        c3 = a_lo;
        k0 += kWeylA;
        k1 += kWeylB;
    }
    Philox4 out;
    out.w[0] = c0; out.w[1] = c1; out.w[2] = c2; out.w[3] = c3;
    return out;
}

// ---------------------------------------------------------------------------
// A group's launches: which batch a block serves, and as which of the batch's blocks.  The hardware deals blocks to the
// eight XCDs in turn, and each XCD has an L2 of its own, so a batch's blocks are given to as few XCDs as the group leaves
// it: of every eight blocks per batch an XCD takes `dealt` (the group's size) consecutive ones, in batch order.  Of four
// batches each has its node table, extents and scratch in two L2s instead of in all eight.  Groups of four, the blocks of
// a batch over all XCDs and dealt: k_sample_rows of the input layer 43 -> 42 us on 1 M nodes, 26 -> 21 with the upper layers
// cache first, 65 -> 61 on 40 M nodes (the layer above it 30 -> 24), k_relabel_last 11.6 -> 8.9, 8.7 -> 6.7 and 16.6 -> 10.9.
// dealt == 1: the batch is blockIdx.y.  kOne: the group is a single batch, of which every block is one; what a kernel reads of
// its arguments then hangs on no other argument (a mini-batch of 256 seeds, seven launches: 1.2 us).
constexpr int kXcds = 8;

struct GroupBlock {
    int b;                     // mini-batch of the group
    int32_t block;             // its block; the last few may lie past the number of blocks asked for
};

template <bool kOne>
__device__ __forceinline__ GroupBlock group_block(int dealt)
{
    const uint32_t id = blockIdx.x;
    if (kOne) return {0, (int32_t) id};
    if (dealt == 1) return {(int) blockIdx.y, (int32_t) id};
    const uint32_t turn = id / kXcds, eight = turn / (uint32_t) dealt;
    const uint32_t p = (id % kXcds) * (uint32_t) dealt + (turn - eight * (uint32_t) dealt);      // of the 8 * dealt blocks of a turn
    return {(int) (p / kXcds), (int32_t) (eight * kXcds + p % kXcds)};
}

// ---------------------------------------------------------------------------
// CSR offsets may be int32 or int64.
template <typename OffT>
__device__ __forceinline__ int64_t load_off(const void* indptr, int64_t i)
{
    return (int64_t) reinterpret_cast<const OffT*>(indptr)[i];
}

// Same with the offset width chosen at run time (kernels that touch offsets only in passing).
__device__ __forceinline__ int64_t load_off_rt(const void* indptr, int is_i64, int64_t i)
{
    return is_i64 ? load_off<int64_t>(indptr, i) : load_off<int32_t>(indptr, i);
}

// CSR extent [start, end) of one dst row's node, kept per row of the batch's node list.
struct alignas(16) RowExtent {
    int64_t start, end;
};

// First slot of a key in a table of 2^(32 - shift) slots.
__device__ __forceinline__ uint32_t hash_start(uint32_t key, uint32_t shift)
{
    return (key * 0x9E3779B1u) >> shift;    // shift = 32 - log2(capacity)
}

// ---------------------------------------------------------------------------
// Wave and block scans (wave64).
__device__ __forceinline__ int lane_id() { return (int) (threadIdx.x & (kWave - 1)); }

// Lane / thread ids the optimiser cannot prove loop-invariant.  A branch on a lane id inside
// a loop that also exchanges data between lanes (shuffles, ballots, readfirstlane, barriers)
// must use these: if the optimiser hoists such a branch out of the loop, the wave is split
// into per-lane-class copies of the loop and the cross-lane operations no longer see all of
// their lanes (observed as lanes spinning forever on a stale row index).
__device__ __forceinline__ int opaque(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}
__device__ __forceinline__ int opaque_lane_id() { return opaque(lane_id()); }

// Six steps that read other lanes' registers: through LDS (shuffles) every one is a trip there, and a block's scan of 256 numbers 0.4 us.
// One step: adds the value kCtrl selects from a lower lane (0 where there is none).  All lanes of the wave call it.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ unsigned long long dpp_add(unsigned long long v)
{
    const uint32_t lo = (uint32_t) __builtin_amdgcn_update_dpp(0, (int) (uint32_t) v, kCtrl, kRowMask, 0xf, false);
    const uint32_t hi = (uint32_t) __builtin_amdgcn_update_dpp(0, (int) (uint32_t) (v >> 32), kCtrl, kRowMask, 0xf, false);
    return v + (((unsigned long long) hi << 32) | lo);
}

__device__ __forceinline__ unsigned long long wave_inclusive_scan64(unsigned long long v)
{
    v = dpp_add<0x111, 0xf>(v);      // row_shr:1, 2, 4, 8 within the rows of 16 lanes
    v = dpp_add<0x112, 0xf>(v);
    v = dpp_add<0x114, 0xf>(v);
    v = dpp_add<0x118, 0xf>(v);
    v = dpp_add<0x142, 0xa>(v);      // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);      // row_bcast:31 into rows 2 and 3
    return v;
}

__device__ __forceinline__ int32_t wave_inclusive_scan(int32_t v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
}

__device__ __forceinline__ int32_t wave_sum(int32_t v)
{
    return __builtin_amdgcn_readlane(wave_inclusive_scan(v), kWave - 1);
}

// Exclusive scan over the kBlock threads of a block; *total receives the block
// sum in every thread.  `smem` must hold kBlock / kWave + 1 ints.
__device__ __forceinline__ int32_t block_exclusive_scan(int32_t v, int32_t* smem, int32_t* total)
{
    const int lane = opaque_lane_id();
    const int wave = opaque((int) (threadIdx.x >> 6));
    constexpr int kWaves = kBlock / kWave;
    const int32_t incl = wave_inclusive_scan(v);
    __syncthreads();                         // smem may still be read from a previous call
    if (lane == kWave - 1) smem[wave] = incl;
    __syncthreads();
    int32_t base = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const int32_t s = smem[w];
        if (w < wave) base += s;
        sum += s;
    }
    *total = sum;
    return base + incl - v;
}

__device__ __forceinline__ int32_t block_sum(int32_t v, int32_t* smem)
{
    const int lane = opaque_lane_id();
    const int wave = opaque((int) (threadIdx.x >> 6));
    constexpr int kWaves = kBlock / kWave;
    const int32_t s = wave_sum(v);
    __syncthreads();
    if (lane == 0) smem[wave] = s;
    __syncthreads();
    int32_t sum = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) sum += smem[w];
    return sum;
}

// A tile's sum travels to the blocks of later tiles of the same launch as one 64-bit word: the launch's tag above, the
// sum below, so relaxed accesses suffice and nothing is reset between launches.
__device__ __forceinline__ void publish_sum(unsigned long long* tile_sums, int32_t tile, uint32_t tag, uint32_t sum)
{
    __hip_atomic_store(&tile_sums[tile], ((unsigned long long) tag << 32) | sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum of the tiles before `tile`, by the whole block.  A sum that does not arrive within `spins` polls is taken from
// count(tile), which works it out from the tile's data, so no block ever depends on another one being scheduled.
template <typename Count>
__device__ __forceinline__ int32_t sum_before(unsigned long long* tile_sums, uint32_t tag, int32_t tile, int spins, int32_t* smem,
                                              Count&& count)
{
    uint32_t v = 0;
    for (int32_t t = (int32_t) threadIdx.x; t < tile; t += kBlock) {
        unsigned long long x = 0;
        int i = 0;
        for (;; ++i) {
            x = __hip_atomic_load(&tile_sums[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((uint32_t) (x >> 32) == tag || i >= spins) break;
            __builtin_amdgcn_s_sleep(1);
        }
        if ((uint32_t) (x >> 32) != tag) {
            const uint32_t counted = count(t);
            // the data has been read before the tag is looked at once more: had it begun to change, the tag would be out
            asm volatile("s_waitcnt vmcnt(0)" ::"v"(counted) : "memory");
            x = __hip_atomic_load(&tile_sums[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((uint32_t) (x >> 32) != tag) x = counted;
        }
        v += (uint32_t) x;
    }
    return block_sum((int32_t) v, smem);
}

// Copies n16 16-byte words into LDS by the whole block.  Four reads are in flight, in variables of their own: an array of
// them ends up in scratch memory, with which a launch that stages 125 KB took 4 us more.
__device__ __forceinline__ void stage_lds(uint4* lds, const uint4* src, int32_t n16)
{
    const int32_t stride = (int32_t) blockDim.x, last = n16 - 1;
    for (int32_t q = (int32_t) threadIdx.x; q < n16; q += 4 * stride) {
        const int32_t q1 = q + stride, q2 = q1 + stride, q3 = q2 + stride;
        const uint4 v0 = src[q], v1 = src[q1 < n16 ? q1 : last], v2 = src[q2 < n16 ? q2 : last], v3 = src[q3 < n16 ? q3 : last];
        lds[q] = v0;
        if (q1 < n16) lds[q1] = v1;
        if (q2 < n16) lds[q2] = v2;
        if (q3 < n16) lds[q3] = v3;
    }
}

// index of the n-th (0-based) set bit of a 64-bit mask that has more than n bits set
__device__ __forceinline__ int select_bit64(uint64_t mask, int n)
{
    int pos = 0;
#pragma unroll
    for (int width = 32; width >= 1; width >>= 1) {
        const uint64_t low = mask & ((1ull << width) - 1ull);
        const int c = __popcll(low);
        if (n >= c) { n -= c; mask >>= width; pos += width; }
        else        { mask = low; }
    }
    return pos;
}

// rank of node u among the set bits of a bitmap with a per-word exclusive prefix
__device__ __forceinline__ int32_t bitmap_rank(const uint64_t* bitmap, const int32_t* word_prefix, uint32_t u)
{
    const uint64_t word = bitmap[u >> 6];
    return word_prefix[u >> 6] + __popcll(word & ((1ull << (u & 63u)) - 1ull));
}

__device__ __forceinline__ bool bitmap_test(const uint64_t* bitmap, uint32_t u)
{
    const uint32_t* words32 = reinterpret_cast<const uint32_t*>(bitmap);
    return (words32[u >> 5] >> (u & 31u)) & 1u;
}

}  // namespace gns
