// Random-walk cache probability (paper Section 3.2, second approach):
//   P^0 = uniform on the training nodes,  P^l = (D_l A + I) P^(l-1),  D_l = diag(min(k_l, deg)/deg),
// kept in integer units (2^scale per training node, every step rounded down) so that the result
// is independent of the order of the additions; then its exclusive prefix sum, which takes the
// place of the CSR offsets in the cache draw (a uniform integer below the total picks the node
// whose prefix interval holds it) and in Section 3.4's p_u.
#include "gns_internal.h"
#include "gns_device.hpp"

namespace gns {

constexpr unsigned long long kWalkLimit = 1ull << 62;     // sums, products and the total stay below this

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
// A step streams the adjacency once and reads one vector entry per CSR entry, at random.  Two things bound it:
//  - how many of those reads are in flight.  Rows are short (tens of entries) and a row is a chain extent -> ids ->
//    values, so a wave takes a run of consecutive rows and streams their entries, which are contiguous, as one list,
//    kUnroll * 64 at a time; the row sums are differences of the list's running sum, which lane r picks up where row r
//    begins.  Every lane then does one row's division.
//  - how much of the vector the 4 MB L2 of an XCD holds.  So the vector is kept as narrow as its values allow.  A step
//    multiplies the largest entry by at most 1 + k, hence W_l <= 2^scale * prod(1 + k_i): known on the host.
//      kBits   P^0 is zero or one unit: one bit per node, staged in LDS where it fits (n <= 1.3 M)
//      kNarrow every entry fits 32 bits
//      kWide   64 bits
// The last step writes 64 bits (the vector the caller sees).
// 1 M nodes, 40 M entries, scale 24, fan-outs 15/10/5: 68 + 229 + 227 us for the three steps (the two narrow ones at
// 177 G requests/s, what the L2s take of scattered ones: 92 % of them hit); one row per 16 lanes on 64-bit vectors took
// 3 x 490 us, the first step with its rows' sums taken chunk by chunk and no reads ahead 78.
enum { kBits = 0, kNarrow = 1, kWide = 2 };

struct WalkStepArgs {
    const void* indptr;
    const int32_t* indices;
    int64_t n;
    int32_t k;
    int32_t rows_per_wave;        // 1 .. 64
    unsigned long long unit;      // kBits: what a set bit stands for
    const void* cur;
    void* nxt;
    DeviceState* st;
};

// One DPP step of a wave-wide inclusive scan: adds the value kCtrl selects from a lower lane (0 where there is none).
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

__device__ __forceinline__ unsigned long long last_lane64(unsigned long long v)
{
    const uint32_t lo = (uint32_t) __builtin_amdgcn_readlane((int) (uint32_t) v, kWave - 1);
    const uint32_t hi = (uint32_t) __builtin_amdgcn_readlane((int) (uint32_t) (v >> 32), kWave - 1);
    return ((unsigned long long) hi << 32) | lo;
}

template <typename OffT, int kIn, bool kWideOut, bool kLds>
__global__ void __launch_bounds__(kLds ? 1024 : kBlock) k_walk_step(WalkStepArgs a)
{
    extern __shared__ uint32_t lds_bits[];
    constexpr int kUnroll = kIn == kBits ? 16 : 8; // 64-entry chunks whose reads are in flight together
    const uint32_t* bits = static_cast<const uint32_t*>(a.cur);
    if (kLds) {
        const int64_t words = (a.n + 31) >> 5;
        for (int64_t w = threadIdx.x; w < words; w += blockDim.x) lds_bits[w] = bits[w];
        __syncthreads();
    }
    auto value = [&](int64_t j) -> unsigned long long {
        if (kIn == kBits) return ((kLds ? lds_bits[j >> 5] : bits[j >> 5]) >> (j & 31)) & 1u;
        if (kIn == kNarrow) return static_cast<const uint32_t*>(a.cur)[j];
        return static_cast<const unsigned long long*>(a.cur)[j];
    };
    const int waves_per_block = (int) (blockDim.x >> 6);
    const int64_t wave = (int64_t) blockIdx.x * waves_per_block + __builtin_amdgcn_readfirstlane((int) (threadIdx.x >> 6));
    const int64_t num_waves = (int64_t) gridDim.x * waves_per_block;
    const int R = a.rows_per_wave;
    for (int64_t r0 = wave * R; r0 < a.n; r0 += num_waves * R) {
        const int lane = opaque_lane_id();         // see opaque(): the loop exchanges data between lanes
        const int rows = a.n - r0 < R ? (int) (a.n - r0) : R;
        // lane r: where row r0 + r begins (lanes past the last row: where it ends)
        const int64_t my_b = load_off<OffT>(a.indptr, r0 + (lane < rows ? lane : rows));
        const int64_t end = load_off<OffT>(a.indptr, r0 + rows);          // wave-uniform
        const int64_t first = load_off<OffT>(a.indptr, r0);
        unsigned long long carry = 0, carry_hi = 0;          // sums of the list's entries so far (kWide: and of their upper halves)
        unsigned long long at_b = 0, at_b_hi = 0;            // the same up to my_b
        const int64_t window0 = first & ~(int64_t) 15;
        if constexpr (kIn == kBits) {
            // The next window's ids are on their way while this one's are tested.  The chunks' ballots stay in lanes
            // 0 .. kUnroll - 1, where a row's beginning is looked up once per window.
            constexpr int kWindow = kWave * kUnroll;
            auto rel_to = [&](int64_t c0, int64_t p) { return (int) (p < c0 ? 0 : p - c0 < 2 * kWindow ? p - c0 : 2 * kWindow); };
            auto load = [&](int64_t c0, int32_t (&dst)[kUnroll]) {
                const int32_t* ids = a.indices + c0;
                const int from = rel_to(c0, first), to = rel_to(c0, end);
                if (from == 0 && to >= kWindow) {
#pragma unroll
                    for (int t = 0; t < kUnroll; ++t) dst[t] = ids[t * kWave + lane];
                } else {
#pragma unroll
                    for (int t = 0; t < kUnroll; ++t) {      // (a run of empty rows has from == to: the entry before them)
                        const int q = t * kWave + lane, at = q < from ? from : q;
                        dst[t] = ids[at < to ? at : to - 1];
                    }
                }
            };
            int32_t j[kUnroll], ahead[kUnroll];
#pragma unroll
            for (int t = 0; t < kUnroll; ++t) j[t] = ahead[t] = 0;
            if (window0 < end) load(window0, j);
            for (int64_t c0 = window0; c0 < end; c0 += kWindow) {
                if (c0 + kWindow < end) load(c0 + kWindow, ahead);
                const int from = rel_to(c0, first), to = rel_to(c0, end), rel_b = rel_to(c0, my_b);
                uint64_t mine = 0;
#pragma unroll
                for (int t = 0; t < kUnroll; ++t) {
                    const int q = t * kWave + lane;
                    const uint32_t w = kLds ? lds_bits[(uint32_t) j[t] >> 5] : bits[(uint32_t) j[t] >> 5];
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
            const unsigned long long deg = (unsigned long long) (my_e - my_b);
            unsigned long long out = value(i);
            bool bad = false;
            if (kIn == kBits) {                                  // a count so far
                bad = sum >= kWalkLimit / a.unit;
                sum *= a.unit;
                out *= a.unit;
            }
            // fewer than 2^31 terms of at most 32 bits stay below 2^63; wider terms are judged by the sum of their upper
            // halves, below which the 64-bit sum cannot have wrapped
            if (kIn == kWide) bad = at_e_hi - at_b_hi >= (kWalkLimit >> 32);
            bad |= sum >= kWalkLimit;
            if (deg > 0 && !bad) {
                const unsigned long long kk = (unsigned long long) a.k < deg ? (unsigned long long) a.k : deg;
                if (kk * sum < (1ull << 32) && sum < (1ull << 32) && deg < (1ull << 32)) {
                    out += (uint32_t) (kk * sum) / (uint32_t) deg;
                } else {
                    const unsigned long long quo = sum / deg, rem = sum % deg;
                    bad = quo >= kWalkLimit / 64;                // kk <= 64: the product below stays under the limit
                    if (!bad) out += kk * quo + (kk * rem) / deg;
                }
            }
            bad |= out >= kWalkLimit;
            if (kWideOut) static_cast<unsigned long long*>(a.nxt)[i] = bad ? 0ull : out;
            else          static_cast<uint32_t*>(a.nxt)[i] = bad ? 0u : (uint32_t) out;
            if (bad) a.st->walk_error = 2;
        }
    }
}

template <typename OffT>
static void launch_walk_step(const gns_ctx* c, WalkStepArgs a, int in, bool wide_out, hipStream_t s)
{
    // runs of rows: long enough to keep a wave streaming, short enough that every wave the chip holds gets two
    const int64_t per = a.n / ((int64_t) c->num_cus * 64);
    a.rows_per_wave = (int) (per < 1 ? 1 : per > kWave ? kWave : per);
    const int64_t waves = (a.n + a.rows_per_wave - 1) / a.rows_per_wave;
    const size_t bit_bytes = (size_t) ((a.n + 31) / 32) * 4;
    if (in == kBits && bit_bytes <= c->lds_bitmap_limit) {
        const int64_t blocks = (waves + 15) / 16;
        const dim3 grid((unsigned) (blocks < c->num_cus ? blocks : c->num_cus)), block(1024);
        if (wide_out) hipLaunchKernelGGL((k_walk_step<OffT, kBits, true, true>), grid, block, bit_bytes, s, a);
        else          hipLaunchKernelGGL((k_walk_step<OffT, kBits, false, true>), grid, block, bit_bytes, s, a);
        return;
    }
    int64_t blocks = (waves + kBlock / kWave - 1) / (kBlock / kWave);
    const int64_t cap = (int64_t) c->num_cus * 64;
    if (blocks > cap) blocks = cap;
    const dim3 grid((unsigned) blocks), block(kBlock);
    switch (in * 2 + (wide_out ? 1 : 0)) {
        case kBits * 2:       hipLaunchKernelGGL((k_walk_step<OffT, kBits, false, false>), grid, block, 0, s, a); break;
        case kBits * 2 + 1:   hipLaunchKernelGGL((k_walk_step<OffT, kBits, true, false>), grid, block, 0, s, a); break;
        case kNarrow * 2:     hipLaunchKernelGGL((k_walk_step<OffT, kNarrow, false, false>), grid, block, 0, s, a); break;
        case kNarrow * 2 + 1: hipLaunchKernelGGL((k_walk_step<OffT, kNarrow, true, false>), grid, block, 0, s, a); break;
        default:              hipLaunchKernelGGL((k_walk_step<OffT, kWide, true, false>), grid, block, 0, s, a); break;
    }
}

// Exclusive prefix sum of n 64-bit values in three phases (tile sums, one block over the tile
// sums, per-tile scan) with the saturating addition above, plus the number of non-zero values.
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

__global__ void __launch_bounds__(kBlock) k_walk_scan_phase3(const unsigned long long* w, int64_t n,
                                                             const unsigned long long* tile_offsets,
                                                             long long* prefix, const DeviceState* st)
{
    __shared__ unsigned long long smem[kBlock / kWave + 1];
    const int64_t base = (int64_t) blockIdx.x * kTile + (int64_t) threadIdx.x * kItems;
    unsigned long long x[kItems];
    unsigned long long sum = 0;
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        x[i] = (base + i < n) ? w[base + i] : 0ull;
        sum = sat_add(sum, x[i]);
    }
    unsigned long long total;
    unsigned long long off = sat_add(tile_offsets[blockIdx.x], block_exclusive_sat_scan(sum, smem, &total));
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        if (base + i < n) prefix[base + i] = (long long) off;
        off = sat_add(off, x[i]);
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) prefix[n] = (long long) st->walk_total;
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

    // P^0 as a bitmap of the training nodes
    hipError_t e = launch_fill_u64(cur, (size_t) (n + 63) / 64, 0ull, s);
    if (e == hipSuccess) e = launch_fill_u32(reinterpret_cast<uint32_t*>(&c->d_state->walk_error), 1, 0u, s);
    if (e != hipSuccess) return ctx_fail(c, GNS_EHIP, "walk init", e);
    hipLaunchKernelGGL(k_walk_seed, dim3((unsigned) ((num_train + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, train_nodes,
                       num_train, n, reinterpret_cast<uint32_t*>(cur), c->d_state);
    unsigned long long bound = 1ull << scale_log2;       // no entry of the current vector exceeds it
    for (int l = 0; l < c->config.num_layers; ++l) {
        WalkStepArgs a;
        a.indptr = c->graph.indptr;
        a.indices = c->graph.indices;
        a.n = n;
        a.k = c->config.fanout[l];
        a.unit = 1ull << scale_log2;
        a.cur = cur;
        a.nxt = nxt;
        a.st = c->d_state;
        const int in = l == 0 ? kBits : (bound >> 32) == 0 ? kNarrow : kWide;
        bound = bound >= kWalkLimit / 128 ? kWalkLimit : bound * (unsigned long long) (1 + a.k);
        const bool wide_out = l == c->config.num_layers - 1 || (bound >> 32) != 0;
        if (c->graph.indptr_is_i64) launch_walk_step<int64_t>(c, a, in, wide_out, s);
        else                        launch_walk_step<int32_t>(c, a, in, wide_out, s);
        unsigned long long* t = cur; cur = nxt; nxt = t;
    }
    const int64_t tiles = (n + kTile - 1) / kTile;
    hipLaunchKernelGGL(k_walk_scan_phase1, dim3((unsigned) tiles), dim3(kBlock), 0, s, cur, n, tile_sums, tile_nz);
    hipLaunchKernelGGL(k_walk_scan_phase2, dim3(1), dim3(kBlock), 0, s, tile_sums, tile_nz, tiles, c->d_state);
    hipLaunchKernelGGL(k_walk_scan_phase3, dim3((unsigned) tiles), dim3(kBlock), 0, s, cur, n, tile_sums, prefix, c->d_state);
    e = hipGetLastError();
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
