// Small decode batches (B = 1..8 rows per step) through one DIP / DIP-CA layer.
//
// The paper is strictly batch 1 (every product is a matrix-vector product, Sec. 1); a batch
// here is B independent batch-1 results that share the weight reads: each row keeps its own
// top-K masks (Alg. 1 step 2 per row), a stored column is read once if any row selected it
// (the union of the row masks) and is accumulated only into the rows that did select it
// (their multiplier is the row's activation, the others' is zero), and the cache sees one
// update per step with the union mask (Alg. 1 step 3).
//
// Kernels in this file:
//   union_kernel     union of the B row masks -> ascending index list, its length, and the
//                    B multipliers of every listed column (lists padded by 16 entries)
//   bgemv_kernel     column-gathered product for all B rows at once, partial sums per
//                    row share; the number of listed columns is read from device memory
//   bgemv_q4_mfma_kernel  the same product for int4 weights and three or more rows, as a
//                    dense contraction on the matrix cores
//   breduce_kernel   adds the partial sums of the shares and applies the epilogue
//                    (SwiGLU for the bundled up/gate matrix, Sec. 3 Eq. 2)

#include <algorithm>

#include "dip_internal.h"
#include "dip_select_device.h"

namespace dip {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------------------
// union of the row masks
// ---------------------------------------------------------------------------------------
constexpr int kUnionThreads = 512;
constexpr int kUnionWordsPerWg = kUnionThreads / 32;   // one lane per feature of 16 mask words

// Every workgroup scans the popcounts of all union words (two words per thread, at most 1024
// words), which gives each word the number of listed indices before it; it then lists the
// features of its own 16 words, one lane per feature, so the reads of x are coalesced.
// Everything a lane will need -- the words it counts, the word of its own feature in every
// row and the feature's activations -- is requested before anything is waited for: the kernel
// is one memory round trip, a scan and the stores.
__global__ __launch_bounds__(kUnionThreads) void union_kernel(UnionParams p) {
    const int layer = blockIdx.y;
    p.masks += layer * p.masks_layer_stride;
    p.x += layer * p.x_layer_stride;
    p.union_words += layer * p.union_layer_stride;
    p.uidx += layer * p.list_layer_stride;
    p.uval += layer * p.list_layer_stride * p.batch;
    p.count_out += layer;
    __shared__ uint32_t s_base[2 * kUnionThreads];
    __shared__ uint32_t s_wave[kUnionThreads / 64];
    constexpr int kMaxBatch = 8;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int B = p.batch;
    const int nwords = (p.n + 31) >> 5;
    const int w0 = 2 * tid, w1 = 2 * tid + 1;
    const int w = blockIdx.x * kUnionWordsPerWg + (tid >> 5), bit = tid & 31;
    // (reads past the end are redirected to the last word / feature and dropped)
    const int w0c = min(w0, nwords - 1), w1c = min(w1, nwords - 1), wc = min(w, nwords - 1);
    const int i = w * 32 + bit, ic = min(i, p.n - 1);
    uint32_t a0[kMaxBatch], a1[kMaxBatch], mw[kMaxBatch];
    float xv[kMaxBatch];
#pragma unroll
    for (int b = 0; b < kMaxBatch; ++b) {
        a0[b] = 0u; a1[b] = 0u; mw[b] = 0u; xv[b] = 0.f;
        if (b < B) {    // (uniform)
            const uint32_t* mrow = p.masks + (size_t)b * p.words_stride;
            a0[b] = mrow[w0c];
            a1[b] = mrow[w1c];
            mw[b] = mrow[wc];
            xv[b] = p.x[(size_t)b * p.x_stride + ic];
        }
    }
    uint32_t u0 = 0u, u1 = 0u;
#pragma unroll
    for (int b = 0; b < kMaxBatch; ++b) {
        u0 |= a0[b];
        u1 |= a1[b];
    }
    if (w0 >= nwords) u0 = 0u;
    if (w1 >= nwords) u1 = 0u;
    const uint32_t c0 = (uint32_t)__popc(u0), c1 = (uint32_t)__popc(u1);
    const uint32_t inc = sel::wave_incl_scan(c0 + c1);
    if (lane == 63) s_wave[wave] = inc;
    __syncthreads();
    uint32_t before = 0, total = 0;
#pragma unroll
    for (int ww = 0; ww < kUnionThreads / 64; ++ww) {
        const uint32_t t = s_wave[ww];
        if (ww < wave) before += t;
        total += t;
    }
    const uint32_t excl = before + inc - (c0 + c1);
    s_base[w0] = excl;
    s_base[w1] = excl + c0;
    if (blockIdx.x == 0) {
        if (w0 < nwords) p.union_words[w0] = u0;
        if (w1 < nwords) p.union_words[w1] = u1;
        if (tid == 0) p.count_out[0] = total;
    }
    __syncthreads();

    if (w >= nwords) return;
    uint32_t rows = 0, uw = 0;    // bit b of rows: row b selected this feature
#pragma unroll
    for (int b = 0; b < kMaxBatch; ++b) {
        uw |= mw[b];
        rows |= ((mw[b] >> bit) & 1u) << b;
    }
    if (!rows) return;
    const uint32_t pos = s_base[w] + (uint32_t)__popc(uw & ((1u << bit) - 1u));
    p.uidx[pos] = i;
    float m[kMaxBatch];
#pragma unroll
    for (int b = 0; b < kMaxBatch; ++b) m[b] = ((rows >> b) & 1u) ? xv[b] : 0.f;
    float* dst = p.uval + (size_t)pos * B;
    if (p.row_major) {
#pragma unroll
        for (int b = 0; b < kMaxBatch; ++b)
            if (b < B) p.uval[b * p.list_layer_stride + pos] = m[b];
    } else if (B == 8) {
        reinterpret_cast<float4*>(dst)[0] = make_float4(m[0], m[1], m[2], m[3]);
        reinterpret_cast<float4*>(dst)[1] = make_float4(m[4], m[5], m[6], m[7]);
    } else if (B == 4) {
        reinterpret_cast<float4*>(dst)[0] = make_float4(m[0], m[1], m[2], m[3]);
    } else {
#pragma unroll
        for (int b = 0; b < kMaxBatch; ++b)
            if (b < B) dst[b] = m[b];
    }
}

// ---------------------------------------------------------------------------------------
// batched gathered product
// ---------------------------------------------------------------------------------------
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <int DT>
struct BElem;
template <>
struct BElem<DIP_F32> {   // 16-byte load, 4 values
    static constexpr int kElems = 4, kBits = 32, kLanes = 16;
    static constexpr bool kScaled = false;
    typedef u32x4 raw_t;
    __device__ static __forceinline__ raw_t load(const char* p) {
        return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    }
    __device__ static __forceinline__ void widen(const raw_t& q, float (&f)[4]) {
        f[0] = __uint_as_float(q.x); f[1] = __uint_as_float(q.y);
        f[2] = __uint_as_float(q.z); f[3] = __uint_as_float(q.w);
    }
};
template <>
struct BElem<DIP_BF16> {  // 16-byte load, 8 values
    static constexpr int kElems = 8, kBits = 16, kLanes = 16;
    static constexpr bool kScaled = false;
    typedef u32x4 raw_t;
    __device__ static __forceinline__ raw_t load(const char* p) {
        return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    }
    __device__ static __forceinline__ void widen(const raw_t& q, float (&f)[8]) {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __uint_as_float(w[i] << 16);
            f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
};
template <>
struct BElem<DIP_INT4_G128> {
    // 8-byte load, 16 codes: a batch multiplies every code B times, so fewer codes per lane
    // keep the B x 16 accumulators in registers.  Flipping bit 3 of every nibble turns the
    // two's-complement code q into q + 8 in [0, 15]; even and odd nibbles, masked apart, are
    // bytes that convert to float in one instruction each.  The caller removes the offset:
    // sum (q + 8) m - 8 sum m.
    static constexpr int kElems = 16, kBits = 4, kLanes = 32;
    static constexpr bool kScaled = true;
    typedef u32x2 raw_t;
    __device__ static __forceinline__ raw_t load(const char* p) {
        return __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(p));
    }
    __device__ static __forceinline__ void widen(const raw_t& q, float (&f)[16]) {
        const uint32_t w[2] = {q.x, q.y};
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t o = w[i] ^ 0x88888888u;
            uint32_t ev = o & 0x0f0f0f0fu, od = (o >> 4) & 0x0f0f0f0fu;
            // keeps the byte extracts below from being narrowed into bit-field extracts
            asm volatile("" : "+v"(ev), "+v"(od));
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                f[i * 8 + 2 * b] = (float)((ev >> (8 * b)) & 0xffu);
                f[i * 8 + 2 * b + 1] = (float)((od >> (8 * b)) & 0xffu);
            }
        }
    }
};

struct BElemQ4Narrow {
    // 4-byte load, 8 codes, all 64 lanes on one stored row: for the larger batches, whose
    // B x 16 accumulators would not leave registers for anything else
    static constexpr int kElems = 8, kBits = 4, kLanes = 64;
    static constexpr bool kScaled = true;
    typedef uint32_t raw_t;
    __device__ static __forceinline__ raw_t load(const char* p) {
        return __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(p));
    }
    __device__ static __forceinline__ void widen(const raw_t& q, float (&f)[8]) {
        const uint32_t o = q ^ 0x88888888u;
        uint32_t ev = o & 0x0f0f0f0fu, od = (o >> 4) & 0x0f0f0f0fu;
        asm volatile("" : "+v"(ev), "+v"(od));
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            f[2 * b] = (float)((ev >> (8 * b)) & 0xffu);
            f[2 * b + 1] = (float)((od >> (8 * b)) & 0xffu);
        }
    }
};

template <int DT, int B>
struct BPick { using type = BElem<DT>; };
template <> struct BPick<DIP_INT4_G128, 5> { using type = BElemQ4Narrow; };
template <> struct BPick<DIP_INT4_G128, 6> { using type = BElemQ4Narrow; };
template <> struct BPick<DIP_INT4_G128, 7> { using type = BElemQ4Narrow; };
template <> struct BPick<DIP_INT4_G128, 8> { using type = BElemQ4Narrow; };

// B consecutive multipliers of one listed column
template <int B>
__device__ __forceinline__ void load_mult(const float* p, float (&m)[B]) {
    if constexpr (B % 4 == 0) {
#pragma unroll
        for (int b = 0; b < B; b += 4) {
            const float4 v = *reinterpret_cast<const float4*>(p + b);
            m[b] = v.x; m[b + 1] = v.y; m[b + 2] = v.z; m[b + 3] = v.w;
        }
    } else if constexpr (B % 2 == 0) {
#pragma unroll
        for (int b = 0; b < B; b += 2) {
            const float2 v = *reinterpret_cast<const float2*>(p + b);
            m[b] = v.x; m[b + 1] = v.y;
        }
    } else {
#pragma unroll
        for (int b = 0; b < B; ++b) m[b] = p[b];
    }
}

constexpr int kBWaves = 4;
constexpr int kBUnroll = 4;   // listed columns in flight per lane group

template <int DT, int B, int LAYERS>
__global__ __launch_bounds__(kBWaves * 64) void bgemv_kernel(BatchedGemvParamsT<LAYERS> p) {
    using E = typename BPick<DT, B>::type;
    constexpr int EPL = E::kElems;
    constexpr int LPR = E::kLanes;
    constexpr int RPW = 64 / LPR;
    constexpr int SC = LPR * EPL;
    constexpr int NG = kBWaves * RPW;
    constexpr int U = kBUnroll;
    __shared__ float red[B][SC];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sub = lane / LPR, l = lane % LPR;
    const int strip = blockIdx.x, g = blockIdx.y, G = gridDim.y;
    const int col_raw = strip * SC + l * EPL;
    // lanes past the right edge of a ragged last strip re-read its last piece; they own no output
    const int col = col_raw < p.n_out ? col_raw : p.n_out - EPL;

    const int layer = LAYERS == 1 ? 0 : blockIdx.z;
    // (the parameters stay untouched: a table in them indexed by the layer is read from where it
    //  is only as long as nothing writes to them)
    const int32_t* uidx = p.uidx + layer * p.list_layer_stride;
    const float* uval = p.uval + layer * p.list_layer_stride * B;
    const uint16_t* scales = p.layer[layer].scales;
    const int k = min((int)p.k_dev[layer], p.k_max);
    const int share = ((k + G - 1) / G + U - 1) / U * U;
    const int kb = min(k, g * share), ke = min(k, kb + share);

    float acc[B][EPL];
    float msum[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
        msum[b] = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[b][e] = 0.f;
    }

    const char* wbase = static_cast<const char*>(p.layer[layer].w) + (size_t)col * E::kBits / 8;
    const int sgroup = col >> 7;
    // a lane group takes U consecutive listed columns per step; the lists are padded so that
    // whole vectors can be read past position k, and what lies past the share is dropped
    for (int t0 = kb + (wave * RPW + sub) * U; t0 < ke; t0 += NG * U) {
        const int4 r4 = *reinterpret_cast<const int4*>(uidx + t0);
        const int r[U] = {r4.x, r4.y, r4.z, r4.w};
        typename E::raw_t q[U];
        float scale[U];
        bool live[U];
        float m[U][B];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            live[u] = t0 + u < ke && (unsigned)r[u] < (unsigned)p.n_in;
            const int rr = live[u] ? r[u] : 0;
            q[u] = E::load(wbase + (size_t)rr * (size_t)p.row_stride);
            scale[u] = 1.f;
            if constexpr (E::kScaled) {
                _Float16 hs;
                const uint16_t raw = scales[(size_t)rr * p.scale_stride + sgroup];
                __builtin_memcpy(&hs, &raw, 2);
                scale[u] = (float)hs;
            }
            load_mult<B>(uval + (size_t)(t0 + u) * B, m[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float f[EPL];
            E::widen(q[u], f);
#pragma unroll
            for (int b = 0; b < B; ++b) {
                // entries past the share hold whatever the list memory held: select, never multiply
                const float mb = live[u] ? m[u][b] * scale[u] : 0.f;
                if constexpr (E::kScaled) msum[b] += mb;
#pragma unroll
                for (int e = 0; e < EPL; ++e) acc[b][e] = fmaf(f[e], mb, acc[b][e]);
            }
        }
    }
    if constexpr (E::kScaled) {
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[b][e] = fmaf(-8.0f, msum[b], acc[b][e]);
    }
    // lane groups of one wavefront, then wavefronts through LDS, both in a fixed order
#pragma unroll
    for (int off = LPR; off < 64; off <<= 1)
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[b][e] += __shfl_xor(acc[b][e], off);
    // (one wavefront after the other adds its sums into the same LDS strip)
    for (int w = 0; w < kBWaves; ++w) {
        if (wave == w && sub == 0) {
#pragma unroll
            for (int b = 0; b < B; ++b)
#pragma unroll
                for (int e = 0; e < EPL; ++e) {
                    float* dst = &red[b][l * EPL + e];
                    *dst = w == 0 ? acc[b][e] : *dst + acc[b][e];
                }
        }
        __syncthreads();
    }
    for (int o = tid; o < B * SC; o += kBWaves * 64) {
        const int b = o / SC, c = o % SC;
        const int gcol = strip * SC + c;
        if (gcol >= p.n_out) continue;
        p.partial[layer * p.partial_layer_stride + ((size_t)g * B + b) * (size_t)p.n_out + gcol] = red[b][c];
    }
}

// ---------------------------------------------------------------------------------------
// int4-g128 weights, kMfmaMinBatch rows and more: the product on the matrix cores.
//
// With B rows the union columns times the row multipliers is a dense contraction
//     P[b][j] = sum_u  m[b][u] * scale[u][j / 128] * q[u][j],
// B x K_union x n_out, and on the vector ALU every 4-bit code costs B multiply-adds plus its
// unpacking.  v_mfma_f32_16x16x32_f16 takes it instead: K = 32 listed columns, N = 16 stored
// columns.  The scale belongs to (u, 128-column group), so it goes into the left operand next to
// the multiplier, and m * scale enters as the sum of two fp16 numbers: its significand cut to
// 11 bits, and the rest times 2^10.  A batch has at most 8 rows and the operand has 16: rows
// 0-7 hold the (negated) first terms, rows 8-15 the second ones, so one product takes both.
// fp16 has a fixed range, and the re-weighting of Sec. 5.2 normalises by ||x||_inf precisely so
// that the dynamic range of the activations does not matter: every batch row is therefore
// multiplied by the power of two that brings its largest |activation| into [8, 16) before the
// split -- exact in fp32 -- and the partial sums are multiplied by the inverse power when they
// are stored, also exact.  The product then depends on the weights only: with |m| < 16 it stays
// inside the fp16 range for group scales up to 4094, and the two terms carry m * scale to 2^-21
// of its value (to 2^-25 absolute where it lies below the fp16 normal range).
//
// The right operand holds the codes themselves, exact in fp16.  Lane l of a wavefront, k-block
// r = l / 16, c = l % 16, loads 8 bytes = 16 codes of each of its 8 stored rows (listed columns
// 8r .. 8r+7 of the 32) at byte 8c of the 128-byte piece of two groups: whole cache lines, read
// past the caches.  Lanes 0-7 then hold group 0 and lanes 8-15 group 1; one rotation of the row of
// 16 lanes per dword gives lanes 8-15 the second dwords of lanes 0-7 and the other way round, after
// which both registers hold one group each, 8 codes per lane.  A byte permute joins the halves of
// two rows' dwords; two nibbles 16 bits apart, masked and completed in place by one three-operand
// logic instruction, are the fp16 numbers 1024 + (q + 8) (bits 0-3) or 1024 + 16 (q + 8) (bits 4-7),
// and a packed add leaves q or 16 q: 20 instructions for 16 codes of product t (0..7) = code t of
// the rows, where a conversion per code took 40.  (The masked nibbles alone, as fp16 denormals,
// save the add, but the matrix cores align the terms of a sum by the exponent field, and small
// terms beside large ones lose as many bits as the denormals have leading zeros: errors of 3e-5
// instead of 3e-7 where every column is listed.)  Product t yields the stored columns 16c + t
// (c < 8) and 16(c - 8) + 8 + t of its group; the factor 16 leaves at the end; sums are fp32.
//
// Row indices, multipliers ([batch row][listed column]) and scales ([group][listed column]) of up
// to kMChunk listed columns are staged in LDS, so that a step is six 16-byte LDS reads and eight
// loads of codes, and the codes of the next kMAhead sets are in flight while one is multiplied.  A
// wavefront covers two groups (256 stored columns, 128 bytes of a row) and the four of a workgroup
// lie side by side (KW == 1: 512 bytes of a row, every wavefront takes all sets of 32 listed
// columns and no sum crosses wavefronts) or, where that gives too few workgroups, take the sets of
// one strip in turn (KW == 4).
//
// Bound: HBM and instruction issue side by side.  40 layers of the Phi-3-Medium shape, 8 rows, up /
// gate product: 2.1 GB of codes in 436 us, where the loads alone take 359 us and the arithmetic
// alone about as long (330 vector and 16 matrix instructions per 32 x 256 codes); down product
// 333 us.  The conversion-per-code form with K = 16 and a matrix product per term took 781 and
// 516 us; three workgroups per compute unit with one set ahead 519 and 351 us.
// ---------------------------------------------------------------------------------------
typedef _Float16 h8_t __attribute__((ext_vector_type(8)));
typedef float f4_t __attribute__((ext_vector_type(4)));

constexpr int kMfmaMinBatch = 3;
constexpr int kMWaves = 4;
constexpr int kMGroups = 2;                    // groups of 128 stored columns per wavefront
constexpr int kMWaveCols = 128 * kMGroups;
constexpr int kMRowSet = 32;                   // listed columns per step of a wavefront
constexpr int kMChunk = 512;                   // listed columns staged at a time
constexpr int kMAhead = 2;                     // sets requested ahead of the one that is multiplied
constexpr int kMaxRows = 8;

// The power of two that brings a row's largest |activation| (given as its bit pattern) into
// [8, 16); 1 for an all-zero row.  Denormal and near-overflow maxima are clamped to factors
// fp32 can hold; such rows only lose the part of the range fp16 could not carry anyway.
__device__ __forceinline__ float row_scale_up(uint32_t max_bits) {
    const int e = (int)((max_bits >> 23) & 0xffu);       // biased exponent of the maximum
    if (max_bits == 0u) return 1.0f;
    int up = 127 + 3 - (e - 127);                        // biased exponent of 2^(3 - unbiased e)
    up = up < 1 ? 1 : (up > 254 ? 254 : up);
    return __uint_as_float((uint32_t)up << 23);
}

// Two fp16 numbers 1024 + (q + 8) 16^e, given as bits, and what takes them to q 16^e (exactly)
typedef _Float16 h2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t signed_codes(uint32_t bits, float offset) {
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(h2_t, bits) + h2_t{(_Float16)offset, (_Float16)offset});
}

template <int KW>
struct MfmaShared {
    static constexpr int kGroups = kMGroups * (kMWaves / KW);   // groups of a workgroup
    struct Stage {
        int32_t row[kMChunk];                          // stored row ...
        uint32_t off[kMChunk];                         // ... and its byte offset
        float m[kMaxRows][kMChunk + 4];                // multipliers times their row's power of two (0 past the share)
        uint16_t sc[kGroups][kMChunk + 8];             // fp16 scales
    };
    union {
        Stage st;
        float red[KW > 1 ? KW : 1][kMaxRows][KW > 1 ? kGroups * 128 : 1];   // sums of the wavefronts
    };
};

template <int KW, int LAYERS>
__global__ __launch_bounds__(kMWaves * 64, 2) void bgemv_q4_mfma_kernel(BatchedGemvParamsT<LAYERS> p) {
    typedef MfmaShared<KW> SH;
    constexpr int CW = kMWaves / KW, STRIP = kMWaveCols * CW;
    __shared__ __align__(16) SH sh;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane >> 4, c = lane & 15;
    const int strip = blockIdx.x, g = blockIdx.y, G = gridDim.y;
    const int B = p.batch;
    const int ngroups = p.n_out >> 7;

    const int layer = LAYERS == 1 ? 0 : blockIdx.z;
    const int32_t* uidx = p.uidx + layer * p.list_layer_stride;
    const float* uval = p.uval + layer * p.list_layer_stride * B;
    const uint32_t* rowmax = p.rowmax + 8 * layer;
    const uint16_t* scales = p.layer[layer].scales;
    const char* wbytes = static_cast<const char*>(p.layer[layer].w);
    const uint32_t row_stride = (uint32_t)p.row_stride;
    const int k = min((int)p.k_dev[layer], p.k_max);
    // (asked for together with k: left to itself the compiler puts them into a round trip of their own)
    uint32_t row_max[kMaxRows];
#pragma unroll
    for (int b = 0; b < kMaxRows; ++b) row_max[b] = rowmax[b];
#pragma unroll
    for (int b = 0; b < kMaxRows; ++b) asm volatile("" : : "s"(row_max[b]));
    const int share = ((k + G - 1) / G + kMRowSet - 1) / kMRowSet * kMRowSet;
    const int kb = min(k, g * share), ke = min(k, kb + share);

    f4_t acc[kMGroups][8];
#pragma unroll
    for (int gg = 0; gg < kMGroups; ++gg)
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[gg][t] = f4_t{0.f, 0.f, 0.f, 0.f};

    // the wavefront's groups (past the right edge: the last one again, dropped at the end)
    const int cw = wave % CW, kw = wave / CW;                // place along the columns, along the list
    const int gslot = cw * kMGroups;                         // ... within the workgroup
    const int g0 = strip * SH::kGroups + gslot;
    const uint32_t wcol = (uint32_t)(min(g0 + (c >> 3), ngroups - 1) * 64 + 8 * (c & 7));
    // this lane's row of the left operand: batch row c % 8, first term (c < 8) or 2^10 * second
    const int b_lane = min(c & 7, B - 1);
    const bool second = c >= 8;
    const float m_scale = second ? 1024.0f : 1.0f;
    const float whole = second ? 1.0f : 0.0f;
    struct Codes { u32x2 q[8]; };
    auto request = [&](int t, Codes& x) {
        const uint4 o0 = *reinterpret_cast<const uint4*>(&sh.st.off[t + 8 * r]);
        const uint4 o1 = *reinterpret_cast<const uint4*>(&sh.st.off[t + 8 * r + 4]);
        const uint32_t off[8] = {o0.x, o0.y, o0.z, o0.w, o1.x, o1.y, o1.z, o1.w};
#pragma unroll
        for (int i = 0; i < 8; ++i)
            x.q[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(wbytes + (off[i] + wcol)));
    };
    auto multiply = [&](int t, const Codes& x) {
        const float4 m0 = *reinterpret_cast<const float4*>(&sh.st.m[b_lane][t + 8 * r]);
        const float4 m1 = *reinterpret_cast<const float4*>(&sh.st.m[b_lane][t + 8 * r + 4]);
        const float m[8] = {m0.x, m0.y, m0.z, m0.w, m1.x, m1.y, m1.z, m1.w};
        float ms[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) ms[i] = m[i] * m_scale;
#pragma unroll
        for (int gg = 0; gg < kMGroups; ++gg) {
            const h8_t sc = *reinterpret_cast<const h8_t*>(&sh.st.sc[gslot + gg][t + 8 * r]);
            h8_t a;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float v = fmaf(ms[i], (float)sc[i], 0.0f);     // (one v_fma_mix_f32)
                const float top = __uint_as_float(__float_as_uint(v) & 0xffffe000u);
                a[i] = (_Float16)fmaf(v, whole, -top);      // -top, or v - top
            }
            // the group's dwords of the 8 rows (see above)
            uint32_t q[8];
#pragma unroll
            for (int i = 0; i < 8; ++i)
                q[i] = (uint32_t)(gg == 0 ? __builtin_amdgcn_update_dpp((int)x.q[i].x, (int)x.q[i].y, 0x128, 0xf, 0xc, false)
                                          : __builtin_amdgcn_update_dpp((int)x.q[i].y, (int)x.q[i].x, 0x128, 0xf, 0x3, false));
            // pair (2i, 2i+1) of rows: the low (codes 0-3) or the high (codes 4-7) halves of their dwords
#pragma unroll
            for (int half = 0; half < 2; ++half) {
                u32x4 b[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t v = __builtin_amdgcn_perm(q[2 * i + 1], q[2 * i], half ? 0x07060302u : 0x05040100u);
                    const uint32_t v8 = v >> 8;
                    b[0][i] = signed_codes((v & 0x000f000fu) ^ 0x64086408u, -1032.0f);
                    b[1][i] = signed_codes((v & 0x00f000f0u) ^ 0x64806480u, -1152.0f);
                    b[2][i] = signed_codes((v8 & 0x000f000fu) ^ 0x64086408u, -1032.0f);
                    b[3][i] = signed_codes((v8 & 0x00f000f0u) ^ 0x64806480u, -1152.0f);
                }
#pragma unroll
                for (int tt = 0; tt < 4; ++tt)
                    acc[gg][4 * half + tt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(
                        a, __builtin_bit_cast(h8_t, b[tt]), acc[gg][4 * half + tt], 0, 0, 0);
            }
        }
    };

    for (int c0 = kb; c0 < ke; c0 += kMChunk) {
        // Stage the chunk, filled up with row 0 and zero multipliers.  Every thread requests all it
        // stages before it waits for any of it (reads past the end are redirected and dropped).
        constexpr int kThreads = kMWaves * 64;
        const int n = min(ke - c0, kMChunk), n32 = (n + kMRowSet - 1) / kMRowSet * kMRowSet;
        if (c0 > kb) __syncthreads();
        {
            constexpr int R = kMChunk / kThreads;
            int row[R];
            float m[R][kMaxRows];
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int t = min(j * kThreads + tid, n - 1);
                row[j] = uidx[c0 + t];
#pragma unroll
                for (int b = 0; b < kMaxRows; ++b) m[j][b] = uval[min(b, B - 1) * p.list_layer_stride + c0 + t];
            }
            // The rows' powers of two, on their own (below maxima of 2^-114 they have no room for the 2^10) and
            // not before the loads above are on their way, which is what the asm is for.  Rows past the
            // batch are staged, with whatever factor, and not read.
            float up[kMaxRows];
#pragma unroll
            for (int b = 0; b < kMaxRows; ++b) {
                uint32_t bits = row_max[b];
                asm volatile("" : "+s"(bits));
                up[b] = row_scale_up(bits);
            }
#pragma unroll
            for (int j = 0; j < R; ++j) {
                const int t = j * kThreads + tid;
                const bool live = t < n && (unsigned)row[j] < (unsigned)p.n_in;
                sh.st.row[t] = live ? row[j] : 0;
                sh.st.off[t] = live ? (uint32_t)row[j] * row_stride : 0u;
#pragma unroll
                for (int b = 0; b < kMaxRows; ++b) sh.st.m[b][t] = live ? m[j][b] * up[b] : 0.f;
            }
        }
        __syncthreads();
        {
            constexpr int E = kMChunk * SH::kGroups / kThreads, EB = E < 8 ? E : 8;
            const int gs = tid % SH::kGroups, col = min(strip * SH::kGroups + gs, ngroups - 1);
#pragma unroll
            for (int e0 = 0; e0 < E; e0 += EB) {
                uint16_t sc[EB];
#pragma unroll
                for (int j = 0; j < EB; ++j) {
                    const int t = (tid + (e0 + j) * kThreads) / SH::kGroups;
                    sc[j] = scales[(size_t)sh.st.row[t] * p.scale_stride + col];
                }
#pragma unroll
                for (int j = 0; j < EB; ++j) sh.st.sc[gs][(tid + (e0 + j) * kThreads) / SH::kGroups] = sc[j];
            }
        }
        __syncthreads();
        // The codes of the next kMAhead sets are in flight while one is multiplied.  No request is
        // under a branch -- past the end the last set is requested again and dropped -- since the
        // wait behind a branch would be for all of them.
        constexpr int STEP = KW * kMRowSet, RING = kMAhead + 1;
        const int last = n32 - kMRowSet;
        int t = kw * kMRowSet;
        Codes x[RING];
#pragma unroll
        for (int s = 0; s < kMAhead; ++s) request(min(t + s * STEP, last), x[s]);
        for (; t + kMAhead * STEP < n32; t += RING * STEP) {
#pragma unroll
            for (int s = 0; s < RING; ++s) {
                request(min(t + (s + kMAhead) * STEP, last), x[(s + kMAhead) % RING]);
                multiply(t + s * STEP, x[s]);
            }
        }
#pragma unroll
        for (int s = 0; s < kMAhead; ++s)
            if (t + s * STEP < n32) multiply(t + s * STEP, x[s]);
    }

    // Result register i of lane l is operand row 4 * (l / 16) + i, lane column l % 16: lanes 0-31
    // hold the first terms of the 8 batch rows, lanes 32-63 the second ones.
    if (KW > 1) __syncthreads();
    const int col = c < 8 ? 16 * c : 16 * (c - 8) + 8;      // first of the lane's 8 columns of a group
    auto join = [&](float v) { return __shfl_xor(v, 32) * (1.0f / 1024.0f) - v; };   // (for lanes 0-31)
#pragma unroll
    for (int gg = 0; gg < kMGroups; ++gg) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int b = 4 * r + i;                                   // (lanes 0-31)
            float o[8];
#pragma unroll
            for (int t = 0; t < 8; ++t)
                o[t] = join(acc[gg][t][i]) * ((t & 1) ? 0.0625f : 1.0f);
            if (lane < 32 && b < B) {
                if constexpr (KW > 1) {
                    float4* dst = reinterpret_cast<float4*>(&sh.red[kw][b][(gslot + gg) * 128 + col]);
                    dst[0] = make_float4(o[0], o[1], o[2], o[3]);
                    dst[1] = make_float4(o[4], o[5], o[6], o[7]);
                } else if (g0 + gg < ngroups) {
                    const float down = 1.0f / row_scale_up(rowmax[b]);     // a power of two: exact
                    float4* dst = reinterpret_cast<float4*>(p.partial + layer * p.partial_layer_stride +
                                                            ((size_t)g * B + b) * (size_t)p.n_out + (g0 + gg) * 128 + col);
                    dst[0] = make_float4(o[0] * down, o[1] * down, o[2] * down, o[3] * down);
                    dst[1] = make_float4(o[4] * down, o[5] * down, o[6] * down, o[7] * down);
                }
            }
        }
    }
    if constexpr (KW > 1) {
        // the wavefronts' sums, added in order
        __syncthreads();
        for (int o = tid; o < B * STRIP; o += kMWaves * 64) {
            const int b = o / STRIP, cc = o % STRIP;
            const int gcol = strip * STRIP + cc;
            if (gcol >= p.n_out) continue;
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < KW; ++w) s += sh.red[w][b][cc];
            p.partial[layer * p.partial_layer_stride + ((size_t)g * B + b) * (size_t)p.n_out + gcol] =
                s * (1.0f / row_scale_up(rowmax[b]));
        }
    }
}

// out[b][j] = sum over shares of partial[g][b][j]   (glu == 0), or
// out[b][j] = up * SiLU(gate), up = sum partial[g][b][j], gate = sum partial[g][b][half + j];
// V outputs per lane, up to FLIGHT shares in flight at a time, added in pairs.  Bound: the
// reads of the sums; their number per lane is that of the shares (a fixed 20 in flight, the spare
// ones re-reading the last share, took 49 us for two shares of 40 layers of the Phi-3-Medium
// shape at 8 rows, where two in flight and 16 bytes per lane take 19 us).
template <bool GLU, int V, int FLIGHT>
__global__ __launch_bounds__(256) void breduce_kernel(BatchedReduceParams p) {
    typedef float vec __attribute__((ext_vector_type(V)));
    const int j = (blockIdx.x * 256 + threadIdx.x) * V;
    const int b = blockIdx.y;
    const int width = GLU ? p.n_out / 2 : p.n_out;
    if (j >= width) return;
    const size_t gstride = (size_t)p.batch * (size_t)p.n_out;
    const float* src = p.partial + blockIdx.z * p.partial_layer_stride + (size_t)b * (size_t)p.n_out + j;
    vec s = vec(0.f), gate = vec(0.f);
    for (int g0 = 0; g0 < p.shares; g0 += FLIGHT) {
        vec a[FLIGHT], b[FLIGHT];
        // (loads past the last share re-read it and are dropped: a load under a branch would be
        //  waited for where the branch ends, one round trip each)
#pragma unroll
        for (int i = 0; i < FLIGHT; ++i) {
            const float* q = src + (size_t)min(g0 + i, p.shares - 1) * gstride;
            a[i] = *reinterpret_cast<const vec*>(q);
            if constexpr (GLU) b[i] = *reinterpret_cast<const vec*>(q + width);
        }
        // in pairs (a sum in share order would be the longest chain of additions of the whole product)
#pragma unroll
        for (int i = 1; i < FLIGHT; ++i)
            if (g0 + i >= p.shares) {
                a[i] = vec(0.f);
                if constexpr (GLU) b[i] = vec(0.f);
            }
#pragma unroll
        for (int n = FLIGHT; n > 1; n = (n + 1) / 2)
#pragma unroll
            for (int i = 0; i < n / 2; ++i) {
                a[i] += a[n - 1 - i];
                if constexpr (GLU) b[i] += b[n - 1 - i];
            }
        s += a[0];
        if constexpr (GLU) gate += b[0];
    }
    if constexpr (GLU) {
#pragma unroll
        for (int v = 0; v < V; ++v) s[v] = s[v] * (gate[v] / (1.0f + expf(-gate[v])));
    }
    *reinterpret_cast<vec*>(p.out + blockIdx.z * p.out_layer_stride + (size_t)b * p.out_stride + j) = s;
}

template <int DT, int LAYERS>
hipError_t launch_dt(const BatchedGemvParamsT<LAYERS>& p, dim3 grid, hipStream_t stream, int pk) {
    const dim3 block(kBWaves * 64);
    switch (p.batch) {
        case 1: return launch_timed(bgemv_kernel<DT, 1, LAYERS>, grid, block, stream, pk, p);
        case 2: return launch_timed(bgemv_kernel<DT, 2, LAYERS>, grid, block, stream, pk, p);
        case 3: return launch_timed(bgemv_kernel<DT, 3, LAYERS>, grid, block, stream, pk, p);
        case 4: return launch_timed(bgemv_kernel<DT, 4, LAYERS>, grid, block, stream, pk, p);
        case 5: return launch_timed(bgemv_kernel<DT, 5, LAYERS>, grid, block, stream, pk, p);
        case 6: return launch_timed(bgemv_kernel<DT, 6, LAYERS>, grid, block, stream, pk, p);
        case 7: return launch_timed(bgemv_kernel<DT, 7, LAYERS>, grid, block, stream, pk, p);
        case 8: return launch_timed(bgemv_kernel<DT, 8, LAYERS>, grid, block, stream, pk, p);
    }
    return hipErrorInvalidValue;
}

template <int LAYERS>
hipError_t launch_product(const BatchedGemvParamsT<LAYERS>& p, bool mc, int kw, dim3 grid, hipStream_t stream, int pk) {
    if (mc) {
        if (!p.rowmax || p.dtype != DIP_INT4_G128 || (int64_t)p.n_in * p.row_stride >= ((int64_t)1 << 32))
            return hipErrorInvalidValue;
        const dim3 block(kMWaves * 64);
        if (kw == 1) return launch_timed(bgemv_q4_mfma_kernel<1, LAYERS>, grid, block, stream, pk, p);
        return launch_timed(bgemv_q4_mfma_kernel<kMWaves, LAYERS>, grid, block, stream, pk, p);
    }
    if (p.dtype == DIP_F32) return launch_dt<DIP_F32>(p, grid, stream, pk);
    if (p.dtype == DIP_BF16) return launch_dt<DIP_BF16>(p, grid, stream, pk);
    if (p.dtype == DIP_INT4_G128) return launch_dt<DIP_INT4_G128>(p, grid, stream, pk);
    return hipErrorInvalidValue;
}

}  // namespace

bool batched_on_matrix_cores(int dtype, int batch, int64_t n_in, int64_t row_stride) {
    // the matrix-core kernel addresses the stored matrix with 32-bit byte offsets
    return dtype == DIP_INT4_G128 && batch >= kMfmaMinBatch && n_in * row_stride < ((int64_t)1 << 32);
}

// Launch shape of the product: strip width, wavefronts of a workgroup along the list (matrix-core
// product) and shares of the list.
struct BatchedShape { int strip, kw, shares; };
static BatchedShape batched_shape(int dtype, int n_out, int k_max, int k_row, bool mc, int layers) {
    if (!mc) {
        // Vector-ALU product: about 1024 workgroups, at least 32 listed columns each; every share's sums are
        // written and read.  bf16 does with 768 (one layer, 1024 against 768: 5120 x 17920 at 8 rows 163
        // against 148 us) unless a batch row itself selects so many columns that the longer chains
        // show (from more than kRows on: error 1.03 times at 5120 x 17920, 55 % of the columns); fp32 rows, in
        // strips of 64 columns, do not (3072 x 8192 at 2 rows: 236 against 241).  Over several layers
        // there are workgroups enough: shares of at most kLong listed columns keep the last round short.
        // int4 takes the shares of a layer on its own at any number of layers (the kernel of the
        // stacks has the small batches, the matrix cores the others: what is left are matrices beyond
        // 4 GiB): the offset of the codes grows with the share (768 workgroups for one layer: 2 % less
        // time, 1.1 times the error).
        constexpr int kLong = 512, kRows = 640;
        const int sc = dtype == DIP_F32 ? 16 * 4 : (dtype == DIP_BF16 ? 16 * 8 : 32 * 16);
        if (dtype == DIP_INT4_G128) layers = 1;
        const int strips = (n_out + sc - 1) / sc * layers;
        int g = (768 + strips - 1) / strips;
        if (dtype != DIP_BF16 || (layers == 1 && k_row > kRows * g)) g = (1024 + strips - 1) / strips;
        if (layers > 1 && g < (k_max + kLong - 1) / kLong) g = (k_max + kLong - 1) / kLong;
        return {sc, 1, std::max(1, std::min(g, k_max / 32))};
    }
    // Matrix-core product, two workgroups to a compute unit.  Wavefronts side by side stage the
    // list once for 1024 stored columns and add nothing across wavefronts; taken where five rounds
    // of such workgroups have a chunk of the list each or more.  Sums of more shares than that only
    // cost: written between the reads of the codes, 230 MB of them (five shares at the
    // Phi-3-Medium shape, 40 layers, 8 rows) take 85 of 444 us.
    constexpr int kWide = kMWaves * kMWaveCols;
    const int wide = (n_out + kWide - 1) / kWide * layers;
    int g = std::max(1, std::min((5 * 512 + wide - 1) / wide, k_max / kMChunk));
    if ((int64_t)wide * g >= 1024) return {kWide, 1, g};
    // One round of workgroups whose wavefronts take the sets of a narrow strip in turn, at least
    // one set of 32 per wavefront.
    const int strips = (n_out + kMWaveCols - 1) / kMWaveCols * layers;
    g = std::max(1, std::min(512 / strips, k_max / (kMWaves * kMRowSet)));
    return {kMWaveCols, kMWaves, g};
}

int batched_shares(int dtype, int n_out, int k_max, int k_row, bool mc, int layers) {
    return batched_shape(dtype, n_out, k_max, k_row, mc, layers).shares;
}

hipError_t launch_union(const UnionParams& p, int layers, hipStream_t stream) {
    const int nwords = (p.n + 31) >> 5;
    hipLaunchKernelGGL(union_kernel, dim3((nwords + kUnionWordsPerWg - 1) / kUnionWordsPerWg, layers),
                       dim3(kUnionThreads), 0, stream, p);
    return hipGetLastError();
}

hipError_t launch_batched_gemv(const BatchedGemvParams& p, int shares, bool mc, int layers, hipStream_t stream,
                               int pk) {
    const BatchedShape shape = batched_shape(p.dtype, p.n_out, p.k_max, p.k_max, mc, layers);   // (strip and kw)
    dim3 grid((p.n_out + shape.strip - 1) / shape.strip, shares, layers);
    if (layers < 1 || layers > kStackLayers) return hipErrorInvalidValue;
    if (layers == 1) return launch_product(one_layer(p), mc, shape.kw, grid, stream, pk);
    return launch_product(p, mc, shape.kw, grid, stream, pk);
}

template <bool GLU, int V>
static hipError_t launch_reduce(const BatchedReduceParams& p, int layers, hipStream_t stream) {
    const int width = GLU ? p.n_out / 2 : p.n_out;
    const dim3 grid((width + 256 * V - 1) / (256 * V), p.batch, layers), block(256);
    constexpr int kMost = GLU && V > 1 ? 12 : 20;      // (96 and 40 or 80 registers)
    if (p.shares <= 2) hipLaunchKernelGGL((breduce_kernel<GLU, V, 2>), grid, block, 0, stream, p);
    else if (p.shares <= 6) hipLaunchKernelGGL((breduce_kernel<GLU, V, 6>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((breduce_kernel<GLU, V, kMost>), grid, block, 0, stream, p);
    return hipGetLastError();
}

hipError_t launch_batched_reduce(const BatchedReduceParams& p, int layers, hipStream_t stream) {
    // 16 bytes per lane where every row of sums and outputs starts on 16 bytes and that still makes
    // a workgroup for every second compute unit; a single layer wants the lanes instead
    const int width = p.glu ? p.n_out / 2 : p.n_out;
    const bool vec = width % 4 == 0 && p.n_out % 4 == 0 && p.partial_layer_stride % 4 == 0 && p.out_stride % 4 == 0 &&
                     p.out_layer_stride % 4 == 0 &&
                     ((reinterpret_cast<uintptr_t>(p.partial) | reinterpret_cast<uintptr_t>(p.out)) & 15) == 0 &&
                     (int64_t)width * p.batch * layers >= 128 * 1024;
    if (p.glu) return vec ? launch_reduce<true, 4>(p, layers, stream) : launch_reduce<true, 1>(p, layers, stream);
    return vec ? launch_reduce<false, 4>(p, layers, stream) : launch_reduce<false, 1>(p, layers, stream);
}

}  // namespace dip
