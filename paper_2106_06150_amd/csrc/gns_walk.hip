// Random-walk cache probability (paper Section 3.2, second approach):
//   P^0 = uniform on the training nodes,  P^l = (D_l A + I) P^(l-1),  D_l = diag(min(k_l, deg)/deg),
// kept in integer units (2^scale per training node, every step rounded down) so that the result
// is independent of the order of the additions; then its exclusive prefix sum, which takes the
// place of the CSR offsets in the cache draw (a uniform integer below the total picks the node
// whose prefix interval holds it) and in Section 3.4's p_u.
#include <stdlib.h>
#include "gns_internal.h"
#include "gns_device.hpp"

namespace gns {

constexpr unsigned long long kWalkLimit = 1ull << 62;     // sums, products and the total stay below this

// The hot nodes of a walk: node i has slot i % kHotSlots, and of the nodes that share a slot the one with the longest row
// holds it.  A copy of the table (two alternate from step to step) has the holders' current values and, as tags, i / kHotSlots;
// it is laid out to be copied into LDS as it is.
constexpr int32_t kHotSlots = 26624;                      // 6 bytes each: 156 KB of a CU's LDS
constexpr uint16_t kNoTag = 0xFFFF;
struct HotCopy {
    uint32_t value[kHotSlots];
    uint16_t tag[kHotSlots];
};
static_assert(kHotSlots % 32 == 0 && sizeof(HotCopy) == kHotSlots * 6 && sizeof(HotCopy) % 16 == 0, "copied 16 bytes at a time");

constexpr int64_t kHotNodes = (int64_t) kHotSlots * kNoTag;     // of larger graphs the tags do not tell all nodes apart
size_t walk_hot_bytes() { return 2 * sizeof(HotCopy); }

// What the walk begins with: no training node, no error, and the holders of the hot nodes' slots.  A block finds those of
// kInitSlots neighboring slots, whose rows are neighbors too, eight threads per slot: 4.2 us for 1 M nodes, where an atomic
// maximum per row took 9 us more in the launch behind.
constexpr int kInitSlots = 32, kInitParts = kBlock / kInitSlots;

template <typename OffT>
__global__ void __launch_bounds__(kBlock) k_walk_init(unsigned long long* bits, int64_t words, const void* indptr, int64_t n,
                                                      HotCopy* hot, DeviceState* st)
{
    __shared__ unsigned long long best[kBlock];
    const int64_t t = (int64_t) blockIdx.x * kBlock + threadIdx.x;
    if (t == 0) st->walk_error = 0;
    for (int64_t i = t; i < words; i += (int64_t) gridDim.x * kBlock) bits[i] = 0ull;
    if (!hot) return;
    // the longest row, of those the last; 0: no row of the slot has an entry
    const int32_t slot = (int32_t) (blockIdx.x * kInitSlots + threadIdx.x % kInitSlots);
    constexpr int64_t kStep = (int64_t) kHotSlots * kInitParts;
    unsigned long long most = 0;
    for (int64_t i0 = slot + (int64_t) (threadIdx.x / kInitSlots) * kHotSlots; i0 < n; i0 += 4 * kStep) {
        int64_t b[4], e[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t i = i0 + q * kStep < n ? i0 + q * kStep : i0;
            b[q] = load_off<OffT>(indptr, i);
            e[q] = load_off<OffT>(indptr, i + 1);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t i = i0 + q * kStep < n ? i0 + q * kStep : i0, deg = e[q] - b[q];
            const unsigned long long key = ((unsigned long long) (deg < 0xFFFFFFFFll ? deg : 0xFFFFFFFFll) << 32) | (uint32_t) i;
            if (deg > 0 && key > most) most = key;
        }
    }
    best[threadIdx.x] = most;
    __syncthreads();
    if (threadIdx.x >= kInitSlots) return;
    for (int q = 1; q < kInitParts; ++q) most = best[threadIdx.x + q * kInitSlots] > most ? best[threadIdx.x + q * kInitSlots] : most;
    hot[0].tag[slot] = hot[1].tag[slot] = most ? (uint16_t) ((uint32_t) most / kHotSlots) : kNoTag;
}

__global__ void __launch_bounds__(kBlock) k_walk_seed(const int32_t* train, int64_t num_train, int64_t n,
                                                      uint32_t* bits, DeviceState* st)
{
    const int64_t t = (int64_t) blockIdx.x * kBlock + threadIdx.x;
    if (t >= num_train) return;
    const int32_t v = train[t];
    if (v < 0 || (int64_t) v >= n) { st->walk_error = 1; return; }
    atomicOr(&bits[v >> 5], 1u << (v & 31));
}

// Addition that sticks at kWalkLimit.  Operands are at most kWalkLimit, so the plain sum fits in
// 64 bits; min(limit, a + b) is associative and commutative, so sums and scans may be taken in any
// order, are exact whenever the true result is below the limit, and equal the limit otherwise.
__device__ __forceinline__ unsigned long long sat_add(unsigned long long a, unsigned long long b)
{
    const unsigned long long s = a + b;
    return s < kWalkLimit ? s : kWalkLimit;
}

// ---------------------------------------------------------------------------
// One step: nxt[i] = cur[i] + floor(min(k, deg_i) * sum_{j in N(i)} cur[j] / deg_i).
//
// A step streams the adjacency once and reads one vector entry per CSR entry, at random.  What bounds it is the number of
// those reads that leave a CU (27.6 M a step on 1 M nodes and 40 M entries, at 173 G a second; the L2s take 266 G of nothing but such reads
// where all hit, and 171 where a third do not: here 16 % do not) and how many are in flight:
//  - Rows are short (tens of entries) and a row is a chain extent -> ids -> values, so a wave takes consecutive rows and
//    streams their entries, which are contiguous, as one list; the row sums are differences of the list's running sum,
//    which lane r picks up where row r begins.  Every lane then does one row's division.
//  - The waves' shares are cut where entries plus kRowCost per row come out even, not rows: a row can have thousands of
//    entries.
//  - The vector is kept as narrow as its values allow.  A step multiplies the largest entry by at most 1 + k, hence
//    W_l <= 2^scale * prod(1 + k_i): known on the host.
//      kBits   P^0 is zero or one unit: one bit per node, staged in LDS where it fits (n <= 1.3 M)
//      kNarrow every entry fits 32 bits: k_walk_narrow, which has the hot nodes' values in LDS
//      kWide   64 bits
//  The last step writes 64 bits (the vector the caller sees).
enum { kBits = 0, kNarrow = 1, kWide = 2 };

struct WalkStepArgs {
    const void* indptr;
    const int32_t* indices;
    int64_t n, nnz;
    int32_t k;
    unsigned long long unit;      // kBits: what a set bit stands for
    const void* cur;
    void* nxt;
    const HotCopy* hot_cur;       // kNarrow: the hot nodes' values in cur, null: no table of them
    HotCopy* hot_nxt;             // where those in nxt go if that is narrow
    DeviceState* st;
};

constexpr int64_t kRowCost = 8;

// Rows [lo, hi) of wave `wave` of num_waves: those whose first entry's number plus kRowCost per row before lies in the wave's
// equal share of all.  A search in which the 64 lanes look at 64 places at a time: four turns for a million rows.
template <typename OffT>
__device__ __forceinline__ void wave_share(const WalkStepArgs& a, int64_t wave, int64_t num_waves, int64_t* row_lo, int64_t* row_hi)
{
    const uint64_t total = (uint64_t) a.nnz + (uint64_t) a.n * kRowCost;
    const int lane = lane_id();
    int64_t below[2], at[2];                       // key(below) < target <= key(at)
    uint64_t target[2];
    for (int q = 0; q < 2; ++q) {
        target[q] = total * (uint64_t) (wave + q) / (uint64_t) num_waves;
        below[q] = -1;
        at[q] = a.n;
    }
    while (at[0] - below[0] > 1 || at[1] - below[1] > 1) {
        uint64_t key[2];
        int64_t step[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            step[q] = (at[q] - below[q] - 1 + kWave - 1) / kWave;
            int64_t p = below[q] + step[q] * (lane + 1);
            if (p > at[q]) p = at[q];
            if (p < 0) p = 0;                                  // (a search that has ended at the first row)
            key[q] = (uint64_t) load_off<OffT>(a.indptr, p) + (uint64_t) p * kRowCost;
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (at[q] - below[q] <= 1) continue;
            const uint64_t reached = __ballot(key[q] >= target[q]);
            const int first = reached ? __builtin_ctzll(reached) : kWave;
            const int64_t lo = below[q] + step[q] * first, hi = lo + step[q];
            if (hi < at[q] && first < kWave) at[q] = hi;
            below[q] = lo < at[q] ? lo : at[q] - 1;
        }
    }
    *row_lo = at[0];
    *row_hi = at[1];
}

__device__ __forceinline__ unsigned long long read_lane64(unsigned long long v, int lane)
{
    const uint32_t lo = (uint32_t) __builtin_amdgcn_readlane((int) (uint32_t) v, lane);
    const uint32_t hi = (uint32_t) __builtin_amdgcn_readlane((int) (uint32_t) (v >> 32), lane);
    return ((unsigned long long) hi << 32) | lo;
}
__device__ __forceinline__ unsigned long long last_lane64(unsigned long long v) { return read_lane64(v, kWave - 1); }

// own + floor(min(k, deg) * sum / deg); *bad if that does not stay below the limit.
__device__ __forceinline__ unsigned long long step_value(unsigned long long own, unsigned long long sum, unsigned long long deg,
                                                         int32_t k, bool* bad)
{
    unsigned long long out = own;
    if (deg > 0 && !*bad) {
        const unsigned long long kk = (unsigned long long) k < deg ? (unsigned long long) k : deg;
        if (sum < (1ull << 26) && deg < (1ull << 32)) {              // k <= 64
            out += (uint32_t) (kk * sum) / (uint32_t) deg;
        } else if (sum < (1ull << 46) && deg < (1ull << 32)) {
            // the product is an integer below 2^52: the quotient in 64-bit floating point is at most one off
            const unsigned long long x = kk * sum;
            unsigned long long q = (unsigned long long) ((double) x / (double) deg);
            const long long rest = (long long) (x - q * deg);
            if (rest < 0) --q;
            else if (rest >= (long long) deg) ++q;
            out += q;
        } else {
            const unsigned long long quo = sum / deg, rem = sum % deg;
            *bad = quo >= kWalkLimit / 64;                // kk <= 64: the product below stays under the limit
            if (!*bad) out += kk * quo + (kk * rem) / deg;
        }
    }
    *bad |= out >= kWalkLimit;
    return *bad ? 0ull : out;
}

// kBits and kWide.  1 M nodes, 40 M entries: the first step takes 54 us; 66 with shares of equal rows, windows read as far as
// they belong to a list, and none read ahead across lists.  Where the bits do not fit LDS, only entries of the list ask for
// theirs (lists of 64 rows fill half to two thirds of their windows on graphs of ten entries a row): 5 M nodes, 200 M entries 0.86 ms,
// 20 M nodes, 400 M entries 1.92, 40 M nodes 2.68, where windows asked whole took 1.02, 2.43 and 4.45.
template <typename OffT, int kIn, bool kWideOut, bool kLds>
__global__ void __launch_bounds__(kLds ? 1024 : kBlock) k_walk_step(WalkStepArgs a)
{
    static_assert(kIn != kNarrow, "k_walk_narrow");
    extern __shared__ uint4 lds_bits16[];
    const uint32_t* lds_bits = reinterpret_cast<const uint32_t*>(lds_bits16);
    constexpr int kUnroll = kIn == kBits ? 16 : 8; // 64-entry chunks whose reads are in flight together
    const uint32_t* bits = static_cast<const uint32_t*>(a.cur);
    const int waves_per_block = (int) (blockDim.x >> 6);
    const int64_t wave = (int64_t) blockIdx.x * waves_per_block + __builtin_amdgcn_readfirstlane((int) (threadIdx.x >> 6));
    int64_t row_lo, row_hi;
    wave_share<OffT>(a, wave, (int64_t) gridDim.x * waves_per_block, &row_lo, &row_hi);
    if (kLds) {
        stage_lds(lds_bits16, static_cast<const uint4*>(a.cur), (int32_t) ((a.n + 127) >> 7));
        __syncthreads();
    }
    if (row_lo >= row_hi) return;
    auto value = [&](int64_t j) -> unsigned long long {
        if (kIn == kBits) return ((kLds ? lds_bits[j >> 5] : bits[j >> 5]) >> (j & 31)) & 1u;
        return static_cast<const unsigned long long*>(a.cur)[j];
    };
    // kBits: the next window's ids are on their way while one's are tested.  Windows are read whole: what does not belong to
    // the list is left out of the ballots, and the array's last window repeats its last entry.
    constexpr int kWindow = kWave * kUnroll;
    int32_t j[kIn == kBits ? kUnroll : 1];
    auto load = [&](int64_t c0, auto& dst) {
        const int32_t* ids = a.indices + c0;
        const int lane = lane_id();
        if (c0 + kWindow <= a.nnz) {
#pragma unroll
            for (int t = 0; t < kUnroll; ++t) dst[t] = ids[t * kWave + lane];
        } else {
#pragma unroll
            for (int t = 0; t < kUnroll; ++t) dst[t] = a.indices[c0 + t * kWave + lane < a.nnz ? c0 + t * kWave + lane : a.nnz - 1];
        }
    };
    if constexpr (kIn == kBits) load(load_off<OffT>(a.indptr, row_lo) & ~(int64_t) 15, j);
    for (int64_t r0 = row_lo; r0 < row_hi; r0 += kWave) {
        const int lane = opaque_lane_id();         // see opaque(): the loop exchanges data between lanes
        const int rows = row_hi - r0 < kWave ? (int) (row_hi - r0) : kWave;
        // lane r: where row r0 + r begins (lanes past the last row: where it ends)
        const int64_t my_b = load_off<OffT>(a.indptr, r0 + (lane < rows ? lane : rows));
        const int64_t end = load_off<OffT>(a.indptr, r0 + rows);          // wave-uniform
        const int64_t first = load_off<OffT>(a.indptr, r0);
        unsigned long long carry = 0, carry_hi = 0;          // sums of the list's entries so far (kWide: and of their upper halves)
        unsigned long long at_b = 0, at_b_hi = 0;            // the same up to my_b
        const int64_t window0 = first & ~(int64_t) 15;
        if constexpr (kIn == kBits) {
            // The chunks' ballots stay in lanes 0 .. kUnroll - 1, where a row's beginning is looked up once per window.
            for (int64_t c0 = window0; c0 < end; c0 += kWindow) {
                int32_t ahead[kUnroll];
                load(c0 + kWindow < end ? c0 + kWindow : end & ~(int64_t) 15, ahead);   // this list's next window, or the next list's first
                auto rel = [&](int64_t p) { return (int) (p < c0 ? 0 : p - c0 < 2 * kWindow ? p - c0 : 2 * kWindow); };
                const int from = rel(first), to = rel(end), rel_b = rel(my_b);
                uint64_t mine = 0;
#pragma unroll
                for (int t = 0; t < kUnroll; ++t) {
                    const int q = t * kWave + lane;
                    const uint32_t w = kLds ? lds_bits[(uint32_t) j[t] >> 5] : bits[q >= from && q < to ? (uint32_t) j[t] >> 5 : 0u];
                    const uint64_t m = __ballot(q >= from && q < to && ((w >> (j[t] & 31)) & 1u));
                    if (lane == t) mine = m;
                }
                const int32_t incl = wave_inclusive_scan(__popcll(mine));
                const int at_word = rel_b >> 6 < kUnroll ? rel_b >> 6 : kUnroll;       // lane kUnroll: nothing, behind all others
                const uint32_t lo = (uint32_t) __shfl((int) (uint32_t) mine, at_word, kWave);
                const uint32_t hi = (uint32_t) __shfl((int) (uint32_t) (mine >> 32), at_word, kWave);
                const int32_t before = __shfl(incl - __popcll(mine), at_word, kWave);
                const uint64_t m = (((uint64_t) hi << 32) | lo) & ((1ull << (rel_b & 63)) - 1ull);
                if (rel_b >= 1 && rel_b <= kWindow) at_b = carry + (unsigned long long) (before + __popcll(m));
                carry += (unsigned long long) (uint32_t) __builtin_amdgcn_readlane(incl, kWave - 1);
#pragma unroll
                for (int t = 0; t < kUnroll; ++t) j[t] = ahead[t];
            }
        }
        for (int64_t c0 = window0; kIn != kBits && c0 < end; c0 += kWave * kUnroll) {
            // positions relative to c0 in 32 bits: 64-bit arithmetic per entry would cost as much as the reads
            auto rel = [&](int64_t p) { return (int) (p < c0 ? 0 : p - c0 < 2 * kWave * kUnroll ? p - c0 : 2 * kWave * kUnroll); };
            const int rel_first = rel(first), rel_end = rel(end), rel_b = rel(my_b);
            const int32_t* ids = a.indices + c0;
            int32_t j[kUnroll];
            unsigned long long v[kUnroll];
#pragma unroll
            for (int t = 0; t < kUnroll; ++t) {
                const int q = t * kWave + lane;
                j[t] = q >= rel_first && q < rel_end ? ids[q] : -1;
            }
#pragma unroll
            for (int t = 0; t < kUnroll; ++t) v[t] = j[t] >= 0 ? value(j[t]) : 0ull;
#pragma unroll
            for (int t = 0; t < kUnroll; ++t) {
                const int x = rel_b - t * kWave;                 // entries of this chunk before my_b
                const bool here = x >= 1 && x <= kWave;
                const unsigned long long incl = wave_inclusive_scan64(v[t]);
                const unsigned long long got = __shfl(incl, here ? x - 1 : 0, kWave);
                if (here) at_b = carry + got;
                carry += last_lane64(incl);
                if (kIn == kWide) {
                    const unsigned long long incl_hi = wave_inclusive_scan64(v[t] >> 32);
                    const unsigned long long got_hi = __shfl(incl_hi, here ? x - 1 : 0, kWave);
                    if (here) at_b_hi = carry_hi + got_hi;
                    carry_hi += last_lane64(incl_hi);
                }
            }
        }
        // row r ends where row r + 1 begins
        unsigned long long at_e = __shfl_down(at_b, 1, kWave), at_e_hi = kIn == kWide ? __shfl_down(at_b_hi, 1, kWave) : 0ull;
        int64_t my_e = __shfl_down(my_b, 1, kWave);
        if (lane == kWave - 1) { at_e = carry; at_e_hi = carry_hi; my_e = end; }
        if (lane < rows) {
            const int64_t i = r0 + lane;
            unsigned long long sum = at_e - at_b;                // exact modulo 2^64
            unsigned long long own = value(i);
            bool bad = false;
            if (kIn == kBits) {                                  // a count so far
                bad = sum >= kWalkLimit / a.unit;
                sum *= a.unit;
                own *= a.unit;
            }
            // fewer than 2^31 terms of at most 32 bits stay below 2^63; wider terms are judged by the sum of their upper
            // halves, below which the 64-bit sum cannot have wrapped
            if (kIn == kWide) bad = at_e_hi - at_b_hi >= (kWalkLimit >> 32);
            bad |= sum >= kWalkLimit;
            const unsigned long long out = step_value(own, sum, (unsigned long long) (my_e - my_b), a.k, &bad);
            if (kWideOut) static_cast<unsigned long long*>(a.nxt)[i] = out;
            else {
                static_cast<uint32_t*>(a.nxt)[i] = (uint32_t) out;
                const uint32_t tag = (uint32_t) i / kHotSlots, slot = (uint32_t) i - tag * kHotSlots;
                if (a.hot_nxt && a.hot_nxt->tag[slot] == tag) a.hot_nxt->value[slot] = (uint32_t) out;
            }
            if (bad) a.st->walk_error = 2;
        }
    }
}

// Four consecutive entries of a list at any 4-byte address, read at once.
struct __attribute__((packed, aligned(4))) Ids4 { int32_t id[4]; };

// kNarrow: a step that reads 32-bit values.  Every CU has the table of hot nodes in its LDS, and a read whose node holds a
// slot there leaves L2 alone: 37 % of them on a power law of 1 M nodes (gamma 2.1), 18 % at 40 M.  A lane has four consecutive
// entries of every 256, so the running sum takes one wave-wide scan per 256 entries; the next window's ids, the next rows'
// beginnings and the rows' own values are on their way while a window is summed.
// 1 M nodes, 40 M entries: 158 us a step, 168 G requests/s out of the CUs; 226 with every value from the L2s.  With the table
// and without, a step on larger graphs: 5 M nodes, 200 M entries 2.09 and 2.46 ms, 20 M nodes, 400 M entries 5.68 and 6.52, 40 M nodes
// 6.10 and 7.05.  !kHot: graphs of more than 1.7 G nodes, whose tags do not tell all nodes apart.
template <typename OffT, bool kWideOut, bool kHot>
__global__ void __launch_bounds__(kHot ? 1024 : kBlock) k_walk_narrow(WalkStepArgs a)
{
    extern __shared__ uint4 lds_hot[];
    constexpr int kSub = 2, kWindow = kSub * 4 * kWave, kWaves = (kHot ? 1024 : kBlock) / kWave;
    const uint32_t* cur = static_cast<const uint32_t*>(a.cur);
    const int64_t wave = (int64_t) blockIdx.x * kWaves + __builtin_amdgcn_readfirstlane((int) (threadIdx.x >> 6));
    int64_t row_lo, row_hi;
    wave_share<OffT>(a, wave, (int64_t) gridDim.x * kWaves, &row_lo, &row_hi);
    if (kHot) {
        constexpr int kLoads = (int) (sizeof(HotCopy) / 16), kTurns = (kLoads + 1023) / 1024;
        const uint4* src = reinterpret_cast<const uint4*>(a.hot_cur);
        uint4 v[kTurns];
#pragma unroll
        for (int i = 0; i < kTurns; ++i) {
            const int q = i * 1024 + (int) threadIdx.x;
            v[i] = src[q < kLoads ? q : kLoads - 1];
        }
#pragma unroll
        for (int i = 0; i < kTurns; ++i) {
            const int q = i * 1024 + (int) threadIdx.x;
            if (q < kLoads) lds_hot[q] = v[i];
        }
        __syncthreads();
    }
    const HotCopy* hot = reinterpret_cast<const HotCopy*>(lds_hot);
    auto load = [&](int64_t c0, int32_t (&dst)[kSub][4]) {
        const int lane = lane_id();
        if (c0 + kWindow <= a.nnz) {
            const Ids4* p = reinterpret_cast<const Ids4*>(a.indices + c0);
#pragma unroll
            for (int s = 0; s < kSub; ++s) {
                const Ids4 x = p[s * kWave + lane];
#pragma unroll
                for (int e = 0; e < 4; ++e) dst[s][e] = x.id[e];
            }
        } else {                                             // the array's last window: entries past its end repeat the last one
#pragma unroll
            for (int s = 0; s < kSub; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int64_t at = c0 + (s * kWave + lane) * 4 + e;
                    dst[s][e] = a.indices[at < a.nnz ? at : a.nnz - 1];
                }
        }
    };
    if (row_lo >= row_hi) return;
    auto begin_of = [&](int64_t r) { return load_off<OffT>(a.indptr, r < row_hi ? r : row_hi); };
    int64_t my_b = begin_of(row_lo + lane_id());
    int32_t j[kSub][4];
    load(load_off<OffT>(a.indptr, row_lo) & ~(int64_t) 15, j);
    for (int64_t r0 = row_lo; r0 < row_hi; r0 += kWave) {
        const int lane = opaque_lane_id();         // see opaque(): the loop exchanges data between lanes
        const int rows = row_hi - r0 < kWave ? (int) (row_hi - r0) : kWave;
        const int64_t next_b = begin_of(r0 + kWave + lane);
        const uint32_t own = cur[r0 + (lane < rows ? lane : 0)];
        const int64_t first = (int64_t) read_lane64((unsigned long long) my_b, 0);
        const int64_t end = (int64_t) read_lane64((unsigned long long) next_b, 0);
        unsigned long long carry = 0, at_b = 0;    // sum of the list's entries so far; the same up to my_b
        for (int64_t c0 = first & ~(int64_t) 15; c0 < end; c0 += kWindow) {
            int32_t ahead[kSub][4];
            load(c0 + kWindow < end ? c0 + kWindow : end & ~(int64_t) 15, ahead);       // this list's next window, or the next list's first
            // positions relative to c0
            const int from = first > c0 ? (int) (first - c0) : 0;
            const int to = end - c0 < kWindow ? (int) (end - c0) : kWindow;
            const int rel_b = my_b < c0 ? -1 : my_b - c0 < kWindow ? (int) (my_b - c0) : kWindow;
            uint32_t v[kSub][4], hot_v[kSub][4];
            bool in[kSub][4], hit[kSub][4];
#pragma unroll
            for (int s = 0; s < kSub; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int q = (s * kWave + lane) * 4 + e;
                    const uint32_t id = (uint32_t) j[s][e], tag = id / kHotSlots, slot = id - tag * kHotSlots;
                    in[s][e] = q >= from && q < to;
                    hit[s][e] = kHot && hot->tag[slot] == tag;
                    hot_v[s][e] = kHot ? hot->value[slot] : 0u;
                    v[s][e] = cur[in[s][e] && !hit[s][e] ? id : 0u];              // lanes with nothing to read share one line
                }
#pragma unroll
            for (int s = 0; s < kSub; ++s) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[s][e] = !in[s][e] ? 0u : hit[s][e] ? hot_v[s][e] : v[s][e];
                const unsigned long long mine = ((unsigned long long) v[s][0] + v[s][1]) + ((unsigned long long) v[s][2] + v[s][3]);
                const unsigned long long incl = wave_inclusive_scan64(mine);
                const int x = rel_b - s * 4 * kWave, from_lane = (x >> 2) & (kWave - 1);
                unsigned long long got = __shfl(incl - mine, from_lane, kWave);
                const uint32_t v0 = (uint32_t) __shfl((int) v[s][0], from_lane, kWave), v1 = (uint32_t) __shfl((int) v[s][1], from_lane, kWave),
                               v2 = (uint32_t) __shfl((int) v[s][2], from_lane, kWave);
                got += (unsigned long long) ((x & 3) > 0 ? v0 : 0u) + ((x & 3) > 1 ? v1 : 0u);
                got += (x & 3) > 2 ? v2 : 0u;
                if (x >= 0 && x < 4 * kWave) at_b = carry + got;
                carry += last_lane64(incl);
            }
#pragma unroll
            for (int s = 0; s < kSub; ++s)
#pragma unroll
                for (int e = 0; e < 4; ++e) j[s][e] = ahead[s][e];
        }
        if (my_b >= end) at_b = carry;             // lanes past the last row, rows without entries at the end
        // row r ends where row r + 1 begins
        unsigned long long at_e = __shfl_down(at_b, 1, kWave);
        int64_t my_e = __shfl_down(my_b, 1, kWave);
        if (lane == kWave - 1) { at_e = carry; my_e = end; }
        if (lane < rows) {
            const int64_t i = r0 + lane;
            const unsigned long long sum = at_e - at_b;      // fewer than 2^31 terms of at most 32 bits stay below 2^63
            bool bad = sum >= kWalkLimit;
            const unsigned long long out = step_value(own, sum, (unsigned long long) (my_e - my_b), a.k, &bad);
            if (kWideOut) static_cast<unsigned long long*>(a.nxt)[i] = out;
            else {
                static_cast<uint32_t*>(a.nxt)[i] = (uint32_t) out;
                const uint32_t tag = (uint32_t) i / kHotSlots, slot = (uint32_t) i - tag * kHotSlots;
                if (kHot && hot->tag[slot] == tag) a.hot_nxt->value[slot] = (uint32_t) out;
            }
            if (bad) a.st->walk_error = 2;
        }
        my_b = next_b;
    }
}

// Blocks of `waves` waves: as many as give every wave a couple of thousand entries, at most `most`.
static dim3 walk_grid(const WalkStepArgs& a, int waves, int64_t most)
{
    const int64_t blocks = (a.nnz + a.n * kRowCost) / (2048 * waves) + 1;
    return dim3((unsigned) (blocks < most ? blocks : most));
}

template <typename OffT>
static void launch_walk_step(const gns_ctx* c, const WalkStepArgs& a, int in, bool wide_out, hipStream_t s)
{
    const size_t bit_bytes = (size_t) ((a.n + 31) / 32) * 4;
    if (in == kNarrow && a.hot_cur) {
        const dim3 grid = walk_grid(a, 16, c->num_cus), block(1024);
        if (wide_out) hipLaunchKernelGGL((k_walk_narrow<OffT, true, true>), grid, block, sizeof(HotCopy), s, a);
        else          hipLaunchKernelGGL((k_walk_narrow<OffT, false, true>), grid, block, sizeof(HotCopy), s, a);
        return;
    }
    if (in == kBits && (bit_bytes + 15) / 16 * 16 <= c->lds_bitmap_limit) {
        const dim3 grid = walk_grid(a, 16, c->num_cus), block(1024);
        const size_t staged = (bit_bytes + 15) / 16 * 16;
        if (wide_out) hipLaunchKernelGGL((k_walk_step<OffT, kBits, true, true>), grid, block, staged, s, a);
        else          hipLaunchKernelGGL((k_walk_step<OffT, kBits, false, true>), grid, block, staged, s, a);
        return;
    }
    const dim3 grid = walk_grid(a, kBlock / kWave, (int64_t) c->num_cus * 8), block(kBlock);
    if (in == kNarrow && wide_out) hipLaunchKernelGGL((k_walk_narrow<OffT, true, false>), grid, block, 0, s, a);
    else if (in == kNarrow) hipLaunchKernelGGL((k_walk_narrow<OffT, false, false>), grid, block, 0, s, a);
    else if (in == kWide) hipLaunchKernelGGL((k_walk_step<OffT, kWide, true, false>), grid, block, 0, s, a);
    else if (wide_out) hipLaunchKernelGGL((k_walk_step<OffT, kBits, true, false>), grid, block, 0, s, a);
    else               hipLaunchKernelGGL((k_walk_step<OffT, kBits, false, false>), grid, block, 0, s, a);
}

// Exclusive prefix sum of n 64-bit values in three phases (tile sums, one block over the tile
// sums, per-tile scan) with the saturating addition above, plus the number of non-zero values.  Of up to kScanTiles tiles every
// block of the last phase adds up those before its own itself, without a launch for it (1 M nodes: 18.1 us for three phases,
// 14.3 for two; 4 M nodes 54 and 39).
constexpr int64_t kScanTiles = 2048;

__device__ __forceinline__ unsigned long long wave_inclusive_sat_scan(unsigned long long v)
{
    const int lane = opaque_lane_id();
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const unsigned long long up = __shfl_up(v, d, kWave);
        if (lane >= d) v = sat_add(v, up);
    }
    return v;
}

// exclusive scan over the block; *total = block sum.  smem: kBlock / kWave + 1 values
__device__ __forceinline__ unsigned long long block_exclusive_sat_scan(unsigned long long v, unsigned long long* smem,
                                                                        unsigned long long* total)
{
    const int lane = opaque_lane_id();
    const int wave = opaque((int) (threadIdx.x >> 6));
    constexpr int kWaves = kBlock / kWave;
    const unsigned long long incl = wave_inclusive_sat_scan(v);
    const unsigned long long before_in_wave = __shfl_up(incl, 1, kWave);
    __syncthreads();
    if (lane == kWave - 1) smem[wave] = incl;
    __syncthreads();
    unsigned long long base = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const unsigned long long s = smem[w];
        if (w < wave) base = sat_add(base, s);
        sum = sat_add(sum, s);
    }
    *total = sum;
    return lane == 0 ? base : sat_add(base, before_in_wave);
}

__global__ void __launch_bounds__(kBlock) k_walk_scan_phase1(const unsigned long long* w, int64_t n,
                                                             unsigned long long* tile_sums, int32_t* tile_nonzero)
{
    __shared__ unsigned long long smem[kBlock / kWave + 1];
    __shared__ int32_t smem32[kBlock / kWave + 1];
    const int64_t base = (int64_t) blockIdx.x * kTile + (int64_t) threadIdx.x * kItems;
    unsigned long long sum = 0;
    int32_t nz = 0;
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const unsigned long long x = (base + i < n) ? w[base + i] : 0ull;
        sum = sat_add(sum, x);
        nz += x ? 1 : 0;
    }
    unsigned long long total;
    (void) block_exclusive_sat_scan(sum, smem, &total);
    const int32_t nzt = block_sum(nz, smem32);
    if (threadIdx.x == 0) {
        tile_sums[blockIdx.x] = total;
        tile_nonzero[blockIdx.x] = nzt;
    }
}

__global__ void __launch_bounds__(kBlock) k_walk_scan_phase2(unsigned long long* tile_sums, const int32_t* tile_nonzero,
                                                             int64_t tiles, DeviceState* st)
{
    __shared__ unsigned long long smem[kBlock / kWave + 1];
    __shared__ int32_t smem32[kBlock / kWave + 1];
    unsigned long long carry = 0;
    int32_t nz = 0;
    for (int64_t base = 0; base < tiles; base += kBlock) {
        const int64_t i = base + threadIdx.x;
        const unsigned long long v = (i < tiles) ? tile_sums[i] : 0ull;
        unsigned long long total;
        const unsigned long long ex = block_exclusive_sat_scan(v, smem, &total);
        if (i < tiles) tile_sums[i] = sat_add(carry, ex);
        carry = sat_add(carry, total);
        nz += block_sum((i < tiles) ? tile_nonzero[i] : 0, smem32);
    }
    if (threadIdx.x == 0) {
        st->walk_total = carry;
        st->walk_support = nz;
        if (carry >= kWalkLimit) st->walk_error = 2;
    }
}

// kSums: `tiles` holds the tiles' sums, else what comes before each of them.
template <bool kSums>
__global__ void __launch_bounds__(kBlock) k_walk_scan_phase3(const unsigned long long* w, int64_t n,
                                                             const unsigned long long* tiles, const int32_t* tile_nonzero,
                                                             long long* prefix, DeviceState* st)
{
    __shared__ unsigned long long smem[kBlock / kWave + 1];
    __shared__ int32_t smem32[kBlock / kWave + 1];
    const bool last = blockIdx.x == gridDim.x - 1;
    const int64_t base = (int64_t) blockIdx.x * kTile + (int64_t) threadIdx.x * kItems;
    unsigned long long x[kItems];
    unsigned long long sum = 0;
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        x[i] = (base + i < n) ? w[base + i] : 0ull;
        sum = sat_add(sum, x[i]);
    }
    unsigned long long before = 0, total;
    if (kSums) {
        int32_t nz = 0;
        unsigned long long mine = 0;
        for (int32_t t = (int32_t) threadIdx.x; t < (int32_t) blockIdx.x; t += kBlock) mine = sat_add(mine, tiles[t]);
        for (int32_t t = (int32_t) threadIdx.x; last && t < (int32_t) gridDim.x; t += kBlock) nz += tile_nonzero[t];
        (void) block_exclusive_sat_scan(mine, smem, &before);
        if (last) nz = block_sum(nz, smem32);
        if (last && threadIdx.x == 0) st->walk_support = nz;
    } else {
        before = tiles[blockIdx.x];
    }
    unsigned long long off = sat_add(before, block_exclusive_sat_scan(sum, smem, &total));
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        if (base + i < n) prefix[base + i] = (long long) off;
        off = sat_add(off, x[i]);
    }
    if (!last || threadIdx.x != 0) return;
    if (kSums) {
        const unsigned long long all = sat_add(before, total);
        st->walk_total = all;
        if (all >= kWalkLimit) st->walk_error = 2;
        prefix[n] = (long long) all;
    } else {
        prefix[n] = (long long) st->walk_total;
    }
}

gns_status run_walk_probability(gns_ctx* c, const int32_t* train_nodes, int64_t num_train, int32_t scale_log2,
                                hipStream_t s)
{
    const Layout& L = c->lay;
    const int64_t n = c->graph.num_nodes;
    gns_ctx* root = c->root;
    root->prob_valid = false;
    unsigned long long* cur = ws_ptr<unsigned long long>(c, L.walk_a);
    unsigned long long* nxt = ws_ptr<unsigned long long>(c, L.walk_b);
    long long* prefix = ws_ptr<long long>(c, L.prob_prefix);
    unsigned long long* tile_sums = ws_ptr<unsigned long long>(c, L.walk_tiles);
    int32_t* tile_nz = ws_ptr<int32_t>(c, L.walk_tiles_nz);

    const bool has_hot = n <= kHotNodes && sizeof(HotCopy) <= c->lds_bitmap_limit && !getenv("GNS_WALK_NO_HOT");
    HotCopy* hot = has_hot ? ws_ptr<HotCopy>(c, L.walk_hot) : nullptr;

    // P^0 as a bitmap of the training nodes
    const int64_t words = (n + 63) / 64;
    const bool i64 = c->graph.indptr_is_i64 != 0;
    const dim3 init(kHotSlots / kInitSlots);
    if (i64) hipLaunchKernelGGL((k_walk_init<int64_t>), init, dim3(kBlock), 0, s, cur, words, c->graph.indptr, n, hot, c->d_state);
    else     hipLaunchKernelGGL((k_walk_init<int32_t>), init, dim3(kBlock), 0, s, cur, words, c->graph.indptr, n, hot, c->d_state);
    hipLaunchKernelGGL(k_walk_seed, dim3((unsigned) ((num_train + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, train_nodes,
                       num_train, n, reinterpret_cast<uint32_t*>(cur), c->d_state);
    unsigned long long bound = 1ull << scale_log2;       // no entry of the current vector exceeds it
    for (int l = 0; l < c->config.num_layers; ++l) {
        WalkStepArgs a;
        a.indptr = c->graph.indptr;
        a.indices = c->graph.indices;
        a.n = n;
        a.nnz = c->graph.num_entries;
        a.k = c->config.fanout[l];
        a.unit = 1ull << scale_log2;
        a.cur = cur;
        a.nxt = nxt;
        a.hot_cur = hot ? &hot[l & 1] : nullptr;
        a.hot_nxt = hot ? &hot[(l + 1) & 1] : nullptr;
        a.st = c->d_state;
        const int in = l == 0 ? kBits : (bound >> 32) == 0 ? kNarrow : kWide;
        bound = bound >= kWalkLimit / 128 ? kWalkLimit : bound * (unsigned long long) (1 + a.k);
        const bool wide_out = l == c->config.num_layers - 1 || (bound >> 32) != 0;
        if (i64) launch_walk_step<int64_t>(c, a, in, wide_out, s);
        else     launch_walk_step<int32_t>(c, a, in, wide_out, s);
        unsigned long long* t = cur; cur = nxt; nxt = t;
    }
    const int64_t tiles = (n + kTile - 1) / kTile;
    hipLaunchKernelGGL(k_walk_scan_phase1, dim3((unsigned) tiles), dim3(kBlock), 0, s, cur, n, tile_sums, tile_nz);
    if (tiles <= kScanTiles) {
        hipLaunchKernelGGL(k_walk_scan_phase3<true>, dim3((unsigned) tiles), dim3(kBlock), 0, s, cur, n, tile_sums, tile_nz, prefix, c->d_state);
    } else {
        hipLaunchKernelGGL(k_walk_scan_phase2, dim3(1), dim3(kBlock), 0, s, tile_sums, tile_nz, tiles, c->d_state);
        hipLaunchKernelGGL(k_walk_scan_phase3<false>, dim3((unsigned) tiles), dim3(kBlock), 0, s, cur, n, tile_sums, tile_nz, prefix, c->d_state);
    }
    hipError_t e = hipGetLastError();
    // only the walk's own fields (walk_total, walk_support, walk_error): a draw in flight leaves its outcome beside them
    if (e == hipSuccess)
        e = hipMemcpyAsync(&c->h_draw->walk_total, &c->d_state->walk_total,
                           offsetof(DeviceState, walk_error) + sizeof(int32_t) - offsetof(DeviceState, walk_total),
                           hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return ctx_fail(c, GNS_EHIP, "walk probability", e);
    if (c->h_draw->walk_error == 1) return ctx_fail(c, GNS_EINVAL, "a training node id lies outside [0, num_nodes)");
    if (c->h_draw->walk_error) return ctx_fail(c, GNS_ECAPACITY, "the walk probability does not fit in 62 bits: lower scale_log2");
    if (c->h_draw->walk_total == 0) return ctx_fail(c, GNS_EINVAL, "the walk probability is zero everywhere");
    root->prob_weights = cur;
    root->prob_total = c->h_draw->walk_total;
    root->prob_support = c->h_draw->walk_support;
    root->prob_valid = true;
    return GNS_OK;
}

}  // namespace gns
