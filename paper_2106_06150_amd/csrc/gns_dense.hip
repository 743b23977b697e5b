// The update step of one layer (paper Algorithm 1, h_u = g(W . (h_u, h_N(u))), GraphSAGE form of
// Section 2.1), forward only:  out = g([h_self | h_neigh] . W + bias).  This is the one dense
// contraction of the path, so it runs on the matrix cores, with the precision of fp32 products and fp32 sums.
//
// Three kernels: k_sage_rows keeps a slab of the weights in LDS and streams rows past it (from a few thousand rows on);
// k_sage_terms does the same with the factors in bf16 terms on the faster matrix cores (large products), no less exactly;
// k_sage_split cuts k into four for everything the others have no rows or no LDS for.
#include "gns_internal.h"
#include "gns_device.hpp"

namespace gns {

typedef float floatx16 __attribute__((ext_vector_type(16)));

struct DenseArgs {
    const float* a1;
    const float* a2;
    const float* w;
    const float* bias;
    float* out;
    int32_t f1, f2, hdim, relu;
    int32_t rows;
    int32_t m_blocks, n_blocks;
    const int32_t* rows_dev;                  // if not null the row count is read here (rows is then the worst case)
};

template <int NT> struct alignas(4 * NT) FloatN { float v[NT]; };

typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kRowsBlock = 512;               // eight waves: two per SIMD
constexpr int kRowsTile = 16;

// k_sage_rows: one block per CU holds a slab of kSlab columns of W in LDS (all K rows of it) and its waves walk tiles of
// 16 rows, so W is read once per CU and not once per tile, and nothing but the rows themselves crosses L2 in the loop.
// 16x16x4 products: a step is 16 k; lane l reads one float4 of row l % 16 of the activations, columns 4 * (l / 16) .. + 3
// of the step (64-byte pieces), and for product i the weights of k-row 4 * (l / 16) + i from LDS, kVec consecutive
// columns in one read that feeds kVec products: column c of column group h is 64 * h + kVec * (l % 16) + c of the slab.
// Tiles of 16 rows rather than 32, because the time of the launch is that of the SIMD with the most tiles: 85,000 rows
// x 256 columns are 5.2 tiles of 32 x 128 per SIMD (six rounds) but 10.4 of 16 x 128 (eleven, half as long each).  Two
// waves per SIMD: one's first reads and its stores run under the other's products.
// 85,000 rows, K = 256, 256 columns: 106 us = 105 TFLOP/s of the 137 that the fp32 products reach at the 2.1 GHz the chip
// runs them at (128 x 128 tiles staged through LDS with two barriers per step: 128 us); what is left is the last round
// and the slab's way into LDS.
template <int kSlab>
__global__ void __launch_bounds__(kRowsBlock) k_sage_rows(DenseArgs a)
{
    constexpr int kVec = kSlab >= 64 ? 4 : kSlab / 16;
    constexpr int kGroups = kSlab / (16 * kVec);
    constexpr int kDepth = 4;                     // steps of activations in flight
    typedef FloatN<kVec> BVec;
    extern __shared__ float4 s_w16[];
    float* s_w = reinterpret_cast<float*>(s_w16);
    const int32_t K = a.f1 + a.f2, steps = K / 16;
    const int32_t rows_k = (K + 15) / 16 * 16;
    // block b runs on XCD b % 8: the slabs of one set of rows stay together there
    const int32_t q = (int32_t) blockIdx.x / 8, xcd = (int32_t) blockIdx.x % 8;
    const int32_t n0 = q % a.n_blocks * kSlab;
    const int32_t strip = q / a.n_blocks * 8 + xcd;
    const int32_t rows = a.rows_dev ? *a.rows_dev : a.rows;
    constexpr int kRow4 = kSlab / 4;
    constexpr int kFill = 8;                      // reads in flight per thread while the slab comes in
    for (int32_t i0 = (int32_t) threadIdx.x; i0 < rows_k * kRow4; i0 += kRowsBlock * kFill) {
        float4 v[kFill];
#pragma unroll
        for (int u = 0; u < kFill; ++u) {
            const int32_t i = i0 + u * kRowsBlock, k = i / kRow4, col = n0 + i % kRow4 * 4;
            v[u] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (k < K && col < a.hdim) v[u] = *reinterpret_cast<const float4*>(a.w + (int64_t) k * a.hdim + col);
        }
#pragma unroll
        for (int u = 0; u < kFill; ++u) {
            const int32_t i = i0 + u * kRowsBlock;
            if (i < rows_k * kRow4) s_w16[i] = v[u];
        }
    }
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane((int) (threadIdx.x >> 6));
    const int lane = (int) threadIdx.x & 63, g = lane >> 4, l16 = lane & 15;
    float bias[kGroups][kVec];
#pragma unroll
    for (int h = 0; h < kGroups; ++h)
#pragma unroll
        for (int c = 0; c < kVec; ++c) {
            const int32_t col = n0 + h * 64 + kVec * l16 + c;
            bias[h][c] = a.bias && col < a.hdim ? a.bias[col] : 0.f;
        }
    const float* my_w = s_w + (4 * g) * kSlab + kVec * l16;
    const int32_t tiles = (rows + kRowsTile - 1) / kRowsTile;
    // the strips' first waves take the first tiles: a remainder spreads over all CUs, one tile per SIMD
    for (int32_t tile = wave * a.m_blocks + strip; tile < tiles; tile += a.m_blocks * (kRowsBlock / kWave)) {
        const int64_t r0 = (int64_t) tile * kRowsTile;
        const int64_t r = r0 + l16 < rows ? r0 + l16 : rows - 1;          // read, never stored
        const float* row1 = a.a1 + r * a.f1;
        const float* row2 = a.a2 + r * a.f2 - a.f1;
        float4 x[kDepth];
        auto fetch = [&](int d, int32_t step) {
            const int32_t k = step * 16 + 4 * g;
            x[d] = *reinterpret_cast<const float4*>((k < a.f1 ? row1 : row2) + k);
        };
        floatx4 acc[kGroups][kVec];
#pragma unroll
        for (int h = 0; h < kGroups; ++h)
#pragma unroll
            for (int c = 0; c < kVec; ++c) acc[h][c] = floatx4{0.f, 0.f, 0.f, 0.f};
        BVec w[2][kGroups];
        auto read_w = [&](int p, int32_t step, int i) {
#pragma unroll
            for (int h = 0; h < kGroups; ++h)
                w[p][h] = *reinterpret_cast<const BVec*>(my_w + (step * 16 + i) * kSlab + h * 64);
        };
        auto multiply = [&](const float4& v, int32_t step, int32_t next) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                read_w((i + 1) & 1, i < 3 ? step : next, (i + 1) & 3);
                const float e = i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w;
                __builtin_amdgcn_sched_barrier(0);                        // the read of the next weights stays ahead of these products
#pragma unroll
                for (int h = 0; h < kGroups; ++h)
#pragma unroll
                    for (int c = 0; c < kVec; ++c)
                        acc[h][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(e, w[i & 1][h].v[c], acc[h][c], 0, 0, 0);
            }
        };
        read_w(0, 0, 0);
        // steps past the last re-read it (and the weights' first row), so that no read of the loop sits in a branch
        auto clamped = [&](int32_t step) { return step < steps ? step : steps - 1; };
        int32_t s = 0;
        if (steps > 0) {
#pragma unroll
            for (int d = 0; d < kDepth; ++d) fetch(d, clamped(d));
            for (; s + kDepth <= steps; s += kDepth) {
#pragma unroll
                for (int d = 0; d < kDepth; ++d) {
                    multiply(x[d], s + d, (s + d + 1) * 16 < rows_k ? s + d + 1 : 0);
                    fetch(d, clamped(s + d + kDepth));
                }
            }
#pragma unroll
            for (int d = 0; d < kDepth; ++d)
                if (s + d < steps) multiply(x[d], s + d, (s + d + 1) * 16 < rows_k ? s + d + 1 : 0);
        }
        if (K % 16) {                                                     // lanes past K multiply zeros (and W's padding rows are zero)
            const bool none = steps * 16 + 4 * g >= K;
            const int32_t k = none ? 0 : steps * 16 + 4 * g;
            float4 v = *reinterpret_cast<const float4*>((k < a.f1 ? row1 : row2) + k);
            if (none) v = make_float4(0.f, 0.f, 0.f, 0.f);
            multiply(v, steps, 0);
        }
#pragma unroll
        for (int h = 0; h < kGroups; ++h) {
            const int32_t col = n0 + h * 64 + kVec * l16;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                BVec o;
#pragma unroll
                for (int c = 0; c < kVec; ++c) {
                    float y = acc[h][c][v] + bias[h][c];
                    if (a.relu) y = fmaxf(y, 0.f);
                    o.v[c] = y;
                }
                const int64_t row = r0 + 4 * g + v;
                if (row < rows && col < a.hdim) *reinterpret_cast<BVec*>(a.out + row * a.hdim + col) = o;
            }
        }
    }
}

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

// Both factors are multiplied by 2^24 before they are split, and the result by 2^-48: every term of every fp32 value, the
// subnormal ones too, is then a normal bf16 or zero.  A factor of 2^104 and more, or a sum of 2^80 and more, overflows
// instead; such results are not finite and are computed once more.
constexpr float kTermScale = 0x1p24f;

// Eight consecutive k of one row or column as three bf16 terms each, every term what is left rounded to nearest:
// x = hi + mid + lo exactly (for x in [2^e, 2^(e+1)) |mid| <= 2^(e-8) and |lo| <= 2^(e-17), a multiple of 2^(e-23)).
struct SplitFrag { uint32_t term[3][4]; };

// Stage q of the splitting of values 2 * i and 2 * i + 1 (r: the values, then what is left of them).
__device__ __forceinline__ void split_stage(SplitFrag& f, float (&r)[8], int q, int i)
{
    if (q == 0) { r[2 * i] *= kTermScale; r[2 * i + 1] *= kTermScale; }
    const uint32_t t = __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{r[2 * i], r[2 * i + 1]}, bf16x2));
    f.term[q][i] = t;
    if (q < 2) {
        r[2 * i] -= __uint_as_float(t << 16);
        r[2 * i + 1] -= __uint_as_float(t & 0xFFFF0000u);
    }
}

__device__ __forceinline__ SplitFrag split8(const float4& x0, const float4& x1)
{
    float r[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
    SplitFrag f;
#pragma unroll
    for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) split_stage(f, r, q, i);
    return f;
}

__device__ __forceinline__ bf16x8 as_bf16(const uint32_t (&t)[4])
{
    const uint4 v = make_uint4(t[0], t[1], t[2], t[3]);
    return __builtin_bit_cast(bf16x8, v);
}

constexpr int terms_block(int slab) { return slab == 64 ? 768 : 1024; }        // three or four waves per SIMD
constexpr int kTermsTile = 32;
constexpr int kTermsMinK = 64;
// the slab in terms, a step's rows of every wave, the slab's bias
constexpr size_t terms_lds(int32_t K, int slab)
{
    return (size_t) ((K + 15) / 16 * 16) * slab * 6 + (size_t) (terms_block(slab) / kWave) * kTermsTile * 64 + (size_t) slab * 4;
}

// k_sage_terms: the products on the bf16 matrix cores, at no less than the precision of k_sage_rows.  Both factors are split
// into three bf16 terms, which hold every bit of an fp32 value of any size; of the nine products of terms seven are taken.
// The two left out (mid of a row's value times lo of the weight, lo times lo) are at most 2^-25 + 2^-34 of |a||w|, less than
// the rounding of one fp32 product.  The products of the leading terms and the rest have an accumulator each, so the large
// sum is rounded once per 16 k, not with every k, and the rest, at 2^-8 of its size, adds next to nothing.
// Error against 64 bits (2-norm), here and of k_sage_rows: normal inputs 4.9e-8 and 1.4e-7 at K = 64, 8.9e-8 and 2.9e-7 at
// K = 256, 1.3e-7 and 4.1e-7 at K = 512; all factors of one bit pattern that cuts badly (3F808040, 3F807EC0) 3.9e-8 to 4.4e-8
// and 6.4e-8 to 7.2e-8 at K = 64; log-normal ones of sigma 3 9.4e-8 and 9.7e-8; inputs of 1e-36 as of 1.  Where all rows
// and all weights are of one magnitude each and the product of the two is nearly an fp32 value, a chain has less to round and
// is the closer one; the terms stay below 5.4e-8 there, one rounding of the result.  Below K = 64 a
// fp32 chain is too short to lose to (log-normal, K = 32: 7.4e-8 and 6.7e-8).  With six products (mid times lo left out both
// ways) the bad patterns give 6.9e-8 to 7.5e-8; with eight every figure is that of seven but for those patterns (3.5e-8), and
// the launch takes 8 % longer.
// One block per CU holds a slab of kSlab columns of W in LDS, in terms, and its waves walk tiles of 32 rows, splitting the
// rows as they come in.  32x32x16 products: lane l holds k 8 * (l / 32) .. + 7 of the step, of row l % 32 and of column
// l % 32 of a group; a fragment of W is one 16-byte read of LDS.
// The matrix cores' power bounds it: with inputs of zeros, which switch nothing, a launch takes 63 us for 79.  So what counts
// is that they never wait: the splitting of the next step stands between the products of this one, rows are read four steps
// ahead and across tiles, and come in as whole 64-byte pieces.
// 85,000 rows, K = 256, 256 columns: 77 us (k_sage_rows 95); 12,600 rows, K = 512: 35.6 us (39.2); 200,000 rows, K = 128:
// 105 us (125); in a forward pass 79 and 37 us for the first two (100 and 40).
// A result that is not finite (an infinity or NaN among its inputs, or an overflow) is computed once more with plain fp32
// products: the terms of an infinity do not add up to it.
// kWhole: f1 and f2 are multiples of 16, so that a step's columns are all of one input.
template <int kSlab, bool kWhole>
__global__ void __launch_bounds__(terms_block(kSlab)) k_sage_terms(DenseArgs a)
{
    constexpr int kGroups = kSlab / 32, kTermsBlock = terms_block(kSlab);
    extern __shared__ uint4 s_terms[];            // [step][term][half of the step][column]: eight k each
    const int32_t K = a.f1 + a.f2, steps = (K + 15) / 16;
    const int32_t q = (int32_t) blockIdx.x / 8, xcd = (int32_t) blockIdx.x % 8;      // as in k_sage_rows
    const int32_t n0 = q % a.n_blocks * kSlab;
    const int32_t strip = q / a.n_blocks * 8 + xcd;
    const int32_t rows = a.rows_dev ? *a.rows_dev : a.rows;
    // what a thread alone does for an element
    auto plain = [&](int64_t row, int32_t col) {
        float z = 0.f;
        for (int32_t k = 0; k < K; ++k)
            z = fmaf(k < a.f1 ? a.a1[row * a.f1 + k] : a.a2[row * a.f2 + k - a.f1], a.w[(int64_t) k * a.hdim + col], z);
        if (a.bias) z += a.bias[col];
        a.out[row * a.hdim + col] = a.relu ? fmaxf(z, 0.f) : z;
    };
    if (rows < kTermsTile) {                                                             // a count from the device may be this small
        for (int32_t i = (int32_t) threadIdx.x; strip == 0 && i < rows * kSlab; i += kTermsBlock)
            if (n0 + i % kSlab < a.hdim) plain(i / kSlab, n0 + i % kSlab);
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane((int) (threadIdx.x >> 6));
    const int lane = (int) threadIdx.x & 63, kh = lane >> 5, l32 = lane & 31;
    const int32_t tiles = (rows + kTermsTile - 1) / kTermsTile;
    const int32_t stride = a.m_blocks * (kTermsBlock / kWave);
    // The last tile ends with the last row and begins as far above (its first rows are another tile's too, who stores them),
    // so that every tile is read alike.
    auto first_row = [&](int32_t tile) { return tile * kTermsTile < rows - kTermsTile ? tile * kTermsTile : rows - kTermsTile; };
    const int32_t chunk = (lane & 3) ^ ((lane >> 3) & 3);
    const uint32_t off1 = (uint32_t) ((lane >> 2) * a.f1 + 4 * chunk), off2 = (uint32_t) ((lane >> 2) * a.f2 + 4 * chunk);
    // Rows are one stream of steps through the wave's tiles, read up to four steps ahead (K is at least four steps long): those
    // of the next tile are on their way while this one's results are stored.
    int32_t tile = wave * a.m_blocks + strip;
    const float *base1, *base2, *next1, *next2;                                          // wave-uniform
    auto bases = [&](int32_t t, const float** b1, const float** b2) {
        const int64_t r = first_row(t < tiles ? t : tiles - 1);
        *b1 = a.a1 + r * a.f1;
        *b2 = a.a2 + r * a.f2 - a.f1;
    };
    bases(tile, &base1, &base2);
    bases(tile + stride, &next1, &next2);
    float4 x[2][2];                               // step s is read into x[s % 2]
    auto fetch = [&](int d, int32_t step) {
        const bool ahead = step >= steps;
        const float* b1 = ahead ? next1 : base1;
        const float* b2 = ahead ? next2 : base2;
        const int32_t k0 = (ahead ? step - steps : step) * 16;
        if (kWhole) {
            const bool self = k0 < a.f1;                                                 // wave-uniform
            const float* p = (self ? b1 : b2) + k0;
#pragma unroll
            for (int j = 0; j < 2; ++j) x[d][j] = *reinterpret_cast<const float4*>(p + j * 16 * (self ? a.f1 : a.f2) + (self ? off1 : off2));
        } else {
            // k of the step past K read the row's last ones again; their weights in LDS are zero, so only a row with a value
            // that is not finite notices, and that one is computed once more
            const int32_t past = k0 + 4 * chunk + 4 - K, k = past > 0 ? k0 - past : k0;
            const bool self = k + 4 * chunk < a.f1;
            const float* p = (self ? b1 : b2) + k;
#pragma unroll
            for (int j = 0; j < 2; ++j) x[d][j] = *reinterpret_cast<const float4*>(p + ((self ? off1 : off2) + (uint32_t) (j * 16 * (self ? a.f1 : a.f2))));
        }
    };
    fetch(0, 0);
    fetch(1, 1);
    constexpr int kFill = 2;                      // groups of eight weights in flight per thread while the slab comes in
    for (int32_t i0 = (int32_t) threadIdx.x; i0 < steps * 2 * kSlab; i0 += kTermsBlock * kFill) {
        float v[kFill][8];
#pragma unroll
        for (int p = 0; p < kFill; ++p) {
            const int32_t i = i0 + p * kTermsBlock, k0 = i / kSlab * 8, col = n0 + i % kSlab;
#pragma unroll
            for (int u = 0; u < 8; ++u) v[p][u] = k0 + u < K && col < a.hdim ? a.w[(int64_t) (k0 + u) * a.hdim + col] : 0.f;
        }
#pragma unroll
        for (int p = 0; p < kFill; ++p) {
            const int32_t i = i0 + p * kTermsBlock, k0 = i / kSlab * 8, c = i % kSlab;
            const SplitFrag f = split8(make_float4(v[p][0], v[p][1], v[p][2], v[p][3]), make_float4(v[p][4], v[p][5], v[p][6], v[p][7]));
            if (i < steps * 2 * kSlab) {
#pragma unroll
                for (int t = 0; t < 3; ++t)
                    s_terms[(((k0 >> 4) * 3 + t) * 2 + ((k0 >> 3) & 1)) * kSlab + c] = make_uint4(f.term[t][0], f.term[t][1], f.term[t][2], f.term[t][3]);
            }
        }
    }
    float* s_bias = reinterpret_cast<float*>(s_terms + steps * 6 * kSlab) + (kTermsBlock / kWave) * (kTermsTile * 16);
    if (threadIdx.x < kSlab) s_bias[threadIdx.x] = a.bias && n0 + (int32_t) threadIdx.x < a.hdim ? a.bias[n0 + threadIdx.x] : 0.f;
    // A step's rows come in as pieces of 64 bytes (a lane's own row would be 32 bytes of 32 lines: the L1 looks every one of
    // them up) and are turned through a piece of LDS of the wave's own, where chunk c of row r lies at c ^ (r / 2 % 4) of the
    // row, so that reads of 16 bytes of eight rows spread over all banks.
    float4* stage = reinterpret_cast<float4*>(s_terms + steps * 6 * kSlab) + wave * (kTermsTile * 4);
    auto put = [&](int d) {
#pragma unroll
        for (int j = 0; j < 2; ++j) stage[j * kWave + lane] = x[d][j];
    };
    const float4* staged = stage + l32 * 4;
    const int32_t at0 = (2 * kh) ^ ((l32 >> 1) & 3);
    put(0);
    __builtin_amdgcn_wave_barrier();
    SplitFrag frag = split8(staged[at0], staged[at0 ^ 1]);
    __builtin_amdgcn_wave_barrier();
    fetch(0, 2);
    put(1);
    fetch(1, 3);
    __syncthreads();
    for (; tile < tiles; tile += stride) {
        floatx16 acc[kGroups], rest[kGroups];
#pragma unroll
        for (int h = 0; h < kGroups; ++h)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[h][v] = rest[h][v] = 0.f;
        // The products of one step, and between them the splitting of the next one, whose rows are staged; those of the step
        // after it (in x[d]) are staged then, and x[d] is read anew.  In this order: the compiler's own has the splitting in
        // front of all products.
        auto multiply = [&](const SplitFrag& f, int32_t step, int d) -> SplitFrag {
            const bf16x8 t[3] = {as_bf16(f.term[0]), as_bf16(f.term[1]), as_bf16(f.term[2])};
            bf16x8 w[kGroups][3];
            auto read_w = [&](int j) {
#pragma unroll
                for (int h = 0; h < kGroups; ++h)
                    w[h][j] = __builtin_bit_cast(bf16x8, s_terms[(step * 6 + 2 * j + kh) * kSlab + h * 32 + l32]);
            };
            read_w(0);
            read_w(1);
            const float4 raw0 = staged[at0], raw1 = staged[at0 ^ 1];
            float r[8] = {raw0.x, raw0.y, raw0.z, raw0.w, raw1.x, raw1.y, raw1.z, raw1.w};
            SplitFrag next;
            // terms of the row and of the weight: the weight's first terms are done with first (the last ones take their place)
            constexpr int kPairs = 7, kA[kPairs] = {2, 0, 1, 0, 1, 2, 0}, kB[kPairs] = {0, 0, 0, 1, 1, 1, 2};
            constexpr int kProducts = kPairs * kGroups, kStages = 12;
#pragma unroll
            for (int m = 0; m < kProducts; ++m) {
                const int i = kA[m / kGroups], j = kB[m / kGroups], h = m % kGroups;
                floatx16& to = m / kGroups == 1 ? acc[h] : rest[h];
                to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(t[i], w[h][j], to, 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (m == 3 * kGroups - 1) read_w(2);
#pragma unroll
                for (int c = kStages * m / (kProducts - 1); c < kStages * (m + 1) / (kProducts - 1); ++c) {
                    split_stage(next, r, c / 4, c % 4);
                    asm volatile("" : "+v"(next.term[c / 4][c % 4]), "+v"(r[c % 4 * 2]), "+v"(r[c % 4 * 2 + 1]));
                    if (c == 3) { put(d); fetch(d, step + 4); }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            return next;
        };
        int32_t s = 0;
        SplitFrag odd;
        for (; s + 2 <= steps; s += 2) {
            odd = multiply(frag, s, 0);
            frag = multiply(odd, s + 1, 1);
        }
        if (s < steps) {
            frag = multiply(frag, s, 0);
            // the next tile's steps count from 0 again
#pragma unroll
            for (int j = 0; j < 2; ++j) { const float4 y = x[0][j]; x[0][j] = x[1][j]; x[1][j] = y; }
        }
        const int32_t r0 = first_row(tile), own = tile * kTermsTile - r0;                // rows of the tile from `own` on are its own
        base1 = next1;
        base2 = next2;
        bases(tile + 2 * stride, &next1, &next2);
        // (from a lane id the compiler cannot see through: what it would keep of this from tile to tile costs the products registers)
        const int e_lane = opaque_lane_id(), row0 = 4 * (e_lane >> 5);
        float* out = a.out + (int64_t) r0 * a.hdim;                                      // wave-uniform
#pragma unroll
        for (int h = 0; h < kGroups; ++h) {
            const int32_t col = n0 + h * 32 + (e_lane & 31);
            const float bias = s_bias[h * 32 + (e_lane & 31)];
            float y[16];
            float any = 0.f;                                                             // NaN if a sum is not finite
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float sum = acc[h][v] + rest[h][v];
                any = fmaf(sum, 0.f, any);
                y[v] = fmaf(sum, 1.f / (kTermScale * kTermScale), bias);
                if (a.relu) y[v] = fmaxf(y[v], 0.f);
            }
            if (col >= a.hdim) continue;
            const uint32_t off = (uint32_t) (row0 * a.hdim + col);
            if (own == 0) {
#pragma unroll
                for (int v = 0; v < 16; ++v) (out + (int64_t) (8 * (v >> 2) + (v & 3)) * a.hdim)[off] = y[v];
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (8 * (v >> 2) + row0 + (v & 3) >= own) (out + (int64_t) (8 * (v >> 2) + (v & 3)) * a.hdim)[off] = y[v];
            }
            if (any == 0.f) continue;
            uint32_t again = 0;
#pragma unroll
            for (int v = 0; v < 16; ++v)
                if (!(fabsf(acc[h][v] + rest[h][v]) < __builtin_inff())) again |= 1u << v;
            for (; again; again &= again - 1) {
                const int v = __builtin_ctz(again), row = 8 * (v >> 2) + row0 + (v & 3);
                if (row >= own) plain((int64_t) r0 + row, col);
            }
        }
    }
}

// k_sage_split: a block of four waves owns 32 rows x 32 * NT columns and cuts k in four (the waves' sums meet in LDS), so
// that a thousand rows still occupy every CU and no wave's chain of products is long.  32x32x2 products, k in steps of
// 32: A comes in as whole 128-byte lines (eight lanes per row) and is turned through a piece of LDS of the wave's own;
// lane l multiplies row l % 32, columns 16 * (l / 32) .. + 15 of the step, with the NT consecutive weights of columns
// NT * (l % 32) .. of the same k-rows, which come straight from L2.  No barrier stands between the reads and the products.
// 1024 rows, K = 512, 256 columns: 8 us (128 x 128 tiles: 49 us on 16 of the CUs).
// Element v of lane l of an accumulator is row 8*(v/4) + 4*(l/32) + v%4.
template <int NT>
__global__ void __launch_bounds__(kBlock) k_sage_split(DenseArgs a)
{
    constexpr int WK = kBlock / kWave;
    typedef FloatN<NT> BVec;
    __shared__ float s_a[WK][32][36];         // rows of 32, padded: 16-byte reads of eight rows spread over all banks
    __shared__ float s_part[WK][NT * 16][kWave];
    const int32_t q = (int32_t) blockIdx.x / 8, xcd = (int32_t) blockIdx.x % 8;      // as in k_sage_rows
    const int32_t mb = q / a.n_blocks * 8 + xcd, nb = q % a.n_blocks;
    const int32_t rows = a.rows_dev ? *a.rows_dev : a.rows;
    const int wave = __builtin_amdgcn_readfirstlane((int) (threadIdx.x >> 6));
    const int lane = (int) threadIdx.x & 63, kh = lane >> 5, l32 = lane & 31;
    const int64_t m0 = (int64_t) mb * 32;
    if (m0 >= rows) return;
    const int32_t col = nb * (NT * 32) + NT * l32;                     // first of this lane's NT columns
    const int32_t colc = col < a.hdim ? col : 0;
    const int32_t K = a.f1 + a.f2;
    const float* base1 = a.a1 + m0 * a.f1;
    const float* base2 = a.a2 + m0 * a.f2;
    const int32_t last_row = (int32_t) (rows - 1 - m0 < 31 ? rows - 1 - m0 : 31);
    const int32_t steps = K >> 5;
    const int32_t s0 = steps * wave / WK, s1 = steps * (wave + 1) / WK;

    float4 ga[4], ra[4];
    BVec rb[4][4];
    auto a_at = [&](int32_t row, int32_t k) -> float4 {
        const int32_t r = row < last_row ? row : last_row;              // read, never stored
        const bool self = k < a.f1;
        return *reinterpret_cast<const float4*>((self ? base1 : base2 - a.f1) + ((int64_t) r * (self ? a.f1 : a.f2) + k));
    };
    auto fetch_a = [&](int32_t step) {
#pragma unroll
        for (int j = 0; j < 4; ++j) ga[j] = a_at(j * 8 + (lane >> 3), step * 32 + (lane & 7) * 4);
    };
    auto stage_a = [&]() {
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<float4*>(&s_a[wave][j * 8 + (lane >> 3)][(lane & 7) * 4]) = ga[j];
    };
    auto fetch_b = [&](int c, int32_t k) {
        const float* w = a.w + (int64_t) k * a.hdim + colc;
#pragma unroll
        for (int i = 0; i < 4; ++i) rb[c][i] = *reinterpret_cast<const BVec*>(w + (int64_t) i * a.hdim);
    };
    floatx16 acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[nt][v] = 0.f;
    auto multiply = [&](const float4& x4, int c) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float x = i == 0 ? x4.x : i == 1 ? x4.y : i == 2 ? x4.z : x4.w;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
                acc[nt] = __builtin_amdgcn_mfma_f32_32x32x2f32(x, rb[c][i].v[nt], acc[nt], 0, 0, 0);
        }
    };
    if (s0 < s1) {
        fetch_a(s0);
#pragma unroll
        for (int c = 0; c < 4; ++c) fetch_b(c, s0 * 32 + kh * 16 + c * 4);
        stage_a();
        for (int32_t s = s0; s < s1; ++s) {
            // steps past the last re-read it, so that no read of the loop sits in a branch
            const int32_t next = s + 1 < s1 ? s + 1 : s1 - 1;
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int c = 0; c < 4; ++c) ra[c] = *reinterpret_cast<const float4*>(&s_a[wave][l32][kh * 16 + c * 4]);
            fetch_a(next);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                multiply(ra[c], c);
                fetch_b(c, next * 32 + kh * 16 + c * 4);
                __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_wave_barrier();
            stage_a();
        }
    }
    if (wave == WK - 1) {
        // what K leaves beyond a multiple of 32: eight k at a time, then four with lanes 32-63 at zero
        for (int32_t k = steps * 32; k < K; k += 8) {
            const bool none = k + kh * 4 >= K;
            const int32_t kc = none ? k : k + kh * 4;
            ra[0] = a_at(l32, kc);
            fetch_b(0, kc);
            if (none) {
                ra[0] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int t = 0; t < NT; ++t) rb[0][i].v[t] = 0.f;
            }
            multiply(ra[0], 0);
        }
    }
    // the four sums of an element meet in LDS; every wave finishes a quarter of the elements
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int v = 0; v < 16; ++v) s_part[wave][v * NT + nt][lane] = acc[nt][v];
    __syncthreads();
    float bias[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) bias[nt] = a.bias ? a.bias[colc + nt] : 0.f;
#pragma unroll
    for (int e0 = 0; e0 < 16 / WK; ++e0) {
        const int v = wave * (16 / WK) + e0;
        BVec o;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            float x = 0.f;
#pragma unroll
            for (int p = 0; p < WK; ++p) x += s_part[p][v * NT + nt][lane];
            x += bias[nt];
            if (a.relu) x = fmaxf(x, 0.f);
            o.v[nt] = x;
        }
        const int64_t row = m0 + 8 * (v >> 2) + 4 * kh + (v & 3);
        if (row < rows && col < a.hdim) *reinterpret_cast<BVec*>(a.out + row * a.hdim + col) = o;
    }
}

template <int kSlab>
static void launch_rows(const gns_ctx* c, DenseArgs a, hipStream_t s)
{
    a.n_blocks = (a.hdim + kSlab - 1) / kSlab;
    a.m_blocks = c->num_cus / 8 / a.n_blocks * 8;              // strips of rows
    const size_t lds = (size_t) ((a.f1 + a.f2 + 15) / 16 * 16) * kSlab * 4;
    hipLaunchKernelGGL(k_sage_rows<kSlab>, dim3((unsigned) (a.m_blocks * a.n_blocks)), dim3(kRowsBlock), lds, s, a);
}

template <int kSlab, bool kWhole>
static void launch_terms(const gns_ctx* c, DenseArgs a, hipStream_t s)
{
    a.n_blocks = (a.hdim + kSlab - 1) / kSlab;
    a.m_blocks = c->num_cus / 8 / a.n_blocks * 8;              // strips of rows
    hipLaunchKernelGGL((k_sage_terms<kSlab, kWhole>), dim3((unsigned) (a.m_blocks * a.n_blocks)), dim3(terms_block(kSlab)),
                       terms_lds(a.f1 + a.f2, kSlab), s, a);
}

template <int NT>
static void launch_split(DenseArgs a, hipStream_t s)
{
    a.m_blocks = (a.rows + 31) / 32;
    a.n_blocks = (a.hdim + NT * 32 - 1) / (NT * 32);
    hipLaunchKernelGGL(k_sage_split<NT>, dim3((unsigned) ((a.m_blocks + 7) / 8 * 8 * a.n_blocks)), dim3(kBlock), 0, s, a);
}

hipError_t launch_sage_dense(gns_ctx* c, const float* h_self, int32_t f1, const float* h_neigh, int32_t f2,
                             const float* w, const float* bias, int32_t hdim, int32_t relu, float* out,
                             int32_t num_rows, hipStream_t s)
{
    if (num_rows == 0) return hipSuccess;
    DenseArgs a;
    a.a1 = h_self; a.a2 = h_neigh; a.w = w; a.bias = bias; a.out = out;
    a.f1 = f1; a.f2 = f2; a.hdim = hdim; a.relu = relu;
    a.rows_dev = nullptr;
    int32_t rows = num_rows;
    if (rows < 0) {                 // GNS_DEVICE_COUNTS(layer): rows counted on the device
        const int layer = -1 - rows;
        a.rows_dev = &c->d_state->num_dst[layer];
        rows = (int32_t) c->lay.rows[layer];
    }
    a.rows = rows;
    // The widest slab whose K rows fit LDS (no wider than the output needs).  k_sage_rows has one tile per SIMD at
    // num_cus * 4 tiles; below three quarters of that, and where no slab fits, the split kernel is ahead (256 columns,
    // K = 512: 13.0 against 8.2 us at 1024 rows, 14.4 against 15.8 us at 4000).
    const int32_t K = f1 + f2;
    // k_sage_terms from twelve tiles of 32 x 32 per CU on where its slab of 64 or 32 columns fits LDS (K up to 352 and 672); with
    // fewer, and for narrow outputs, which leave its splitting of the rows little to be spread over, the fp32 products are as
    // fast or faster.  256 columns, here and k_sage_rows: 4096 rows, K = 256, 15.5 and 10.5 us, 8192 rows 13.8 and 15.0, 16,384
    // rows 23.9 and 23.9, 36,000 rows 41 and 47; 12,600 rows, K = 128, 12.7 and 14.8 us; 85,000 rows, K = 640, 207 and 267; 64
    // columns (50,000 rows) 25.7 and 23.3.  Widths that are not multiples of 16 cost it the choice of the input for every lane
    // and step: from 32 tiles per CU on and with 64 columns only (K = 200, 256 columns: 24,576 rows 29.8 and 27.6 us, 50,000 rows
    // 48.7 and 53.2, 85,000 rows 72 and 81; K = 504, 85,000 rows, 190 and 183).
    const int64_t tiles32 = ((int64_t) rows + 31) / 32 * ((hdim + 31) / 32);
    const bool whole = f1 % 16 == 0 && f2 % 16 == 0;
    int32_t terms = 64;
    while (terms >= (whole ? 32 : 64) && terms_lds(K, terms) > c->lds_bitmap_limit) terms /= 2;
    if (K >= kTermsMinK && hdim > 64 && terms >= (whole ? 32 : 64) && (hdim + terms - 1) / terms <= c->num_cus / 8 &&
        tiles32 >= (int64_t) c->num_cus * (whole ? 12 : 32)) {
        if (!whole)           launch_terms<64, false>(c, a, s);
        else if (terms == 64) launch_terms<64, true>(c, a, s);
        else                  launch_terms<32, true>(c, a, s);
        return hipGetLastError();
    }
    const size_t k_bytes = (size_t) ((K + 15) / 16 * 16) * 4;
    const int32_t want = hdim > 64 ? 128 : hdim > 32 ? 64 : 32;
    int32_t slab = want;
    while (slab >= 32 && k_bytes * slab > c->lds_bitmap_limit) slab /= 2;
    const int64_t tiles = slab >= 32 ? ((int64_t) (rows + kRowsTile - 1) / kRowsTile) * ((hdim + slab - 1) / slab) : 0;
    if (tiles >= (int64_t) c->num_cus * 3 && (hdim + slab - 1) / slab <= c->num_cus / 8) {
        if (slab == 128)     launch_rows<128>(c, a, s);
        else if (slab == 64) launch_rows<64>(c, a, s);
        else                 launch_rows<32>(c, a, s);
    } else {
        if (hdim <= 32) launch_split<1>(a, s);
        else            launch_split<2>(a, s);
    }
    return hipGetLastError();
}

}  // namespace gns
