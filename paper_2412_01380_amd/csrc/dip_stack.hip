// Gathered products of a whole stack of layers in one launch.
//
// The layers of a stack call are independent (the caller hands over every layer's x), so each
// phase of a step -- selection, product, reduction -- runs once for all of them.  A product of
// one layer is a 10 us launch on its own: the ramp, the selection in front of it and the
// reduction behind it leave the memory idle for half of that time.  Over a stack the same
// phases cost one ramp and one tail per call and the row loop streams in between.
//
// Bound: HBM for fp32 and bf16 rows.  The kernel is therefore only the row loop, arranged so
// that it issues little besides loads and multiply-adds.  A wavefront reads 64 consecutive
// pieces of one stored row: the row index and its multiplier are the same for all lanes, so
// they come through scalar loads, the row address is scalar arithmetic and the multiply-add
// takes its multiplier from a scalar register.  Blocks of kBlock consecutive selected rows are
// in flight while the previous block is multiplied (two register sets).  The wavefronts of a
// workgroup take the blocks of the workgroup's share in turn and add their sums through LDS.
// Up and gate halves of a bundled row are just more columns here; the reduction launch behind
// the product adds the shares and applies SwiGLU.
//
// Rounding: sums of short spans of rows are added to the totals, wavefronts and shares in pairs.  In
// one chain per wavefront the error against 64 bits was up to 3 times that of a layer on its own
// (40 layers of the Phi-3-Medium shape: bf16 1.2, at 8 rows 1.6, int4 2.1, at 2 rows 3.1 times); in
// spans it is 0.75 to 1.0 times, for 1 to 7 % more time with int4 rows and none with the others.
//
// A small batch reads the union of its rows' lists with one multiplier per batch row, which stay
// scalar; the row of weights is widened once for all of them.
//
// int4 rows are a quarter of the bytes and bound by vector instructions: see Q4.
#include <algorithm>
#include <type_traits>

#include "dip_internal.h"

namespace dip {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

template <typename T, T V>
using Const = std::integral_constant<T, V>;

#define DIP_CONSTANT __attribute__((address_space(4)))

struct F32 {
    typedef u32x4 raw_t;
    static constexpr int kElems = 4, kBits = 32;
    static constexpr bool kScaled = false;
    template <int B>
    __device__ static __forceinline__ void fma(const raw_t& q, const float (&m)[B], float (&acc)[B][4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int b = 0; b < B; ++b) acc[b][i] = fmaf(__uint_as_float(q[i]), m[b], acc[b][i]);
    }
};
struct Bf16 {  // the upper half of an fp32 pattern
    typedef u32x4 raw_t;
    static constexpr int kElems = 8, kBits = 16;
    static constexpr bool kScaled = false;
    template <int B>
    __device__ static __forceinline__ void fma(const raw_t& q, const float (&m)[B], float (&acc)[B][8]) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int b = 0; b < B; ++b) {
                acc[b][2 * i] = fmaf(__uint_as_float(q[i] << 16), m[b], acc[b][2 * i]);
                acc[b][2 * i + 1] = fmaf(__uint_as_float(q[i] & 0xffff0000u), m[b], acc[b][2 * i + 1]);
            }
    }
};
struct Q4 {
    // 16 codes per 8-byte load, low nibble = even element.  Flipping bit 3 of every nibble turns
    // the code q into q + 8 in [0, 15].  Two nibbles 16 bits apart, masked in place, are the bit
    // patterns of two fp16 denormals, (q + 8) * 2^-24 (bits 0-3) or (q + 8) * 2^-20 (bits 4-7),
    // which v_fma_mix_f32 widens exactly while it multiplies and adds in fp32: 6 instructions
    // unpack 8 codes, where a byte conversion per code takes 12.  The factor leaves through the
    // multiplier (times `up`) and the sums (times 2^24 / up), both exact; the offset as -8 * sum
    // of multipliers.
    typedef u32x2 raw_t;
    static constexpr int kElems = 16, kBits = 4;
    static constexpr bool kScaled = true;
    // `up` for a batch row whose largest |activation| has these bits.  Multipliers and sums move away
    // from where the caller's numbers lie by 2^12 each, which a row beyond 2^64 (or below 2^-64) has
    // no room for: 2^0 leaves its multipliers alone and moves the sums down, 2^24 the other way round.
    __device__ static __forceinline__ float up(uint32_t max_bits) {
        const int e = (int)(max_bits >> 23) - 127;
        return e >= 64 ? 1.0f : (e < -64 ? 16777216.0f : 4096.0f);
    }
    __device__ static __forceinline__ float lo(uint32_t v) {
        const uint16_t b = (uint16_t)v;
        return (float)__builtin_bit_cast(_Float16, b);
    }
    __device__ static __forceinline__ float hi(uint32_t v) {
        const uint16_t b = (uint16_t)(v >> 16);
        return (float)__builtin_bit_cast(_Float16, b);
    }
    // (odd codes are read 16 times as large as even ones, and their sums stay so until a span ends)
    template <int B>
    __device__ static __forceinline__ void fma(const raw_t& q, const float (&m)[B], float (&acc)[B][16]) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t o = q[i] ^ 0x88888888u, o8 = o >> 8;
            const uint32_t c04 = o & 0x000f000fu, c15 = o & 0x00f000f0u;
            const uint32_t c26 = o8 & 0x000f000fu, c37 = o8 & 0x00f000f0u;
#pragma unroll
            for (int b = 0; b < B; ++b) {
                float* a = acc[b] + 8 * i;
                a[0] = fmaf(lo(c04), m[b], a[0]);
                a[4] = fmaf(hi(c04), m[b], a[4]);
                a[1] = fmaf(lo(c15), m[b], a[1]);
                a[5] = fmaf(hi(c15), m[b], a[5]);
                a[2] = fmaf(lo(c26), m[b], a[2]);
                a[6] = fmaf(hi(c26), m[b], a[6]);
                a[3] = fmaf(lo(c37), m[b], a[3]);
                a[7] = fmaf(hi(c37), m[b], a[7]);
            }
        }
    }
};

// Wavefronts per workgroup and, for each, rows in flight per register set.  With one batch row
// eight of both; with more, whose sums and multipliers fill registers, four of both (eight
// wavefronts: up to 1.12 times as long, 40 layers of 3072 x 8192 at 8 rows of bf16 1048 against 1013 us).
template <int B>
struct Shape { static constexpr int kWaves = B == 1 ? 8 : 4, kBlock = B == 1 ? 8 : 4; };

// Rows per span.  The sums of a span are added up on their own before they join the totals: rounding
// errors grow with the length of the chains, and a span followed by their number is two short
// chains in the place of a long one.  The offset of int4 codes makes the sums within a span larger
// than what they come to: shorter spans.
template <typename E, int B>
constexpr int kSpan = E::kScaled ? 4 : (B == 1 ? 8 : 16);

template <typename E, int B>
__global__ __launch_bounds__(Shape<B>::kWaves * 64) void stack_product_kernel(StackProductParams p) {
    constexpr int EPL = E::kElems, SC = 64 * EPL;
    constexpr int kWaves = Shape<B>::kWaves, kBlock = Shape<B>::kBlock, SPAN = kSpan<E, B>;
    __shared__ float red[kWaves][SC];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int strip = blockIdx.x, g = blockIdx.y, G = gridDim.y, layer = blockIdx.z;
    const int k = p.k_dev ? min((int)p.k_dev[layer], p.k_max) : p.layer[layer].k;
    const int share = ((k + G - 1) / G + kBlock - 1) / kBlock * kBlock;
    const int kb = min(k, g * share), ke = min(k, kb + share);

    // lanes past the right edge of a ragged last strip re-read the row's last piece; they own no output
    const int col = min(strip * SC + lane * EPL, p.n_out - EPL);
    const uint32_t voff = (uint32_t)col * E::kBits / 8;
    const char* w = static_cast<const char*>(p.layer[layer].w);
    const uint16_t* scales = p.layer[layer].scales;
    const uint32_t sgroup = (uint32_t)col >> 7;
    // uniform addresses in the constant address space: scalar loads
    const DIP_CONSTANT int32_t* idx = (const DIP_CONSTANT int32_t*)(uintptr_t)(p.idx + layer * p.list_layer_stride);
    const DIP_CONSTANT float* val = (const DIP_CONSTANT float*)(uintptr_t)(p.val + layer * p.list_layer_stride * B);

    float acc[B][EPL], tot[B][EPL];
#pragma unroll
    for (int b = 0; b < B; ++b)
#pragma unroll
        for (int e = 0; e < EPL; ++e) tot[b][e] = 0.f;

    float up[B];
    if constexpr (E::kScaled) {
        const DIP_CONSTANT uint32_t* rowmax = (const DIP_CONSTANT uint32_t*)(uintptr_t)(p.rowmax + 8 * layer);
#pragma unroll
        for (int b = 0; b < B; ++b) up[b] = E::up(rowmax[b]);
    }

    struct Pairs { int r[kBlock]; float m[kBlock][B]; };
    struct Rows { typename E::raw_t q[kBlock]; uint16_t sc[kBlock]; };
    auto fetch = [&](int t, Pairs& b) {
#pragma unroll
        for (int u = 0; u < kBlock; ++u) {
            b.r[u] = idx[t + u];
#pragma unroll
            for (int i = 0; i < B; ++i) b.m[u][i] = val[(t + u) * B + i];
        }
    };
    auto request = [&](const Pairs& b, Rows& x) {
#pragma unroll
        for (int u = 0; u < kBlock; ++u) {
            // (an entry outside the matrix -- non-finite inputs -- reads row 0)
            const uint32_t r = (uint32_t)b.r[u] < (uint32_t)p.n_in ? (uint32_t)b.r[u] : 0u;
            x.q[u] = __builtin_nontemporal_load(
                reinterpret_cast<const typename E::raw_t*>(w + (size_t)r * (size_t)p.row_stride + voff));
            if constexpr (E::kScaled) x.sc[u] = (scales + (size_t)r * (size_t)p.scale_stride)[sgroup];
        }
    };
    // Rows times multipliers, N of them from row FIRST of a block.  OPEN: they are the first of a span.
    // int4 sums start at the offset of the span's codes.
    auto rows = [&](auto OPEN, auto FIRST, auto N, const auto& m, const auto& x) {
        static_assert(OPEN || !E::kScaled, "the offset is that of the rows at hand");
        float mult[N][B];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            float sum = 0.f;
#pragma unroll
            for (int u = 0; u < N; ++u) {
                mult[u][b] = m[FIRST + u][b];
                if constexpr (E::kScaled) {
                    mult[u][b] = fmaf(mult[u][b] * up[b], (float)__builtin_bit_cast(_Float16, x.sc[FIRST + u]), 0.0f);
                    sum += mult[u][b];
                }
            }
            if constexpr (OPEN) {
                const float first = E::kScaled ? sum * (-8.0f / 16777216.0f) : 0.f;
#pragma unroll
                for (int e = 0; e < EPL; ++e) acc[b][e] = E::kScaled && (e & 1) ? 16.0f * first : first;
            }
        }
#pragma unroll
        for (int u = 0; u < N; ++u) E::template fma<B>(x.q[FIRST + u], mult[u], acc);
    };
    // ... and ends in the totals
    auto close = [&] {
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int e = 0; e < EPL; ++e)
                tot[b][e] = E::kScaled && (e & 1) ? fmaf(acc[b][e], 0.0625f, tot[b][e]) : tot[b][e] + acc[b][e];
    };
    // block number POS after the start of a span
    auto multiply = [&](auto POS, const Pairs& b, const Rows& x) {
        constexpr int R = SPAN < kBlock ? SPAN : kBlock;
        static_assert(kBlock <= 2 * R);
        Const<bool, POS * kBlock % SPAN == 0> opens;
        rows(opens, Const<int, 0>(), Const<int, R>(), b.m, x);
        if constexpr ((POS * kBlock + R) % SPAN == 0) close();
        if constexpr (R < kBlock) {
            rows(Const<bool, true>(), Const<int, R>(), Const<int, R>(), b.m, x);
            close();
        }
    };

    // full blocks t = kb + (wave + i * kWaves) * kBlock
    const int n_blocks = (ke - kb) / kBlock;
    int left = n_blocks > wave ? (n_blocks - wave - 1) / kWaves + 1 : 0;
    constexpr int STEP = kWaves * kBlock;
    int t = kb + wave * kBlock;
    if (left > 0) {
        Pairs pa, pb;
        Rows xa, xb;
        fetch(t, pa);
        request(pa, xa);
        if constexpr (B == 1) {
            // (every wavefront has a handful of blocks: none is requested twice)
            static_assert(SPAN <= kBlock);
            while (true) {
                if (left == 1) {
                    multiply(Const<int, 0>(), pa, xa);
                    break;
                }
                t += STEP;
                fetch(t, pb);
                request(pb, xb);
                multiply(Const<int, 0>(), pa, xa);
                if (left == 2) {
                    multiply(Const<int, 0>(), pb, xb);
                    break;
                }
                t += STEP;
                fetch(t, pa);
                request(pa, xa);
                multiply(Const<int, 0>(), pb, xb);
                left -= 2;
            }
        } else {
            // (past the end the last block is requested again and dropped: loads under a branch would
            // all be waited for where it ends)
            const int last = t + (left - 1) * STEP;
            auto next = [&](Pairs& p, Rows& x) {
                t = min(t + STEP, last);
                fetch(t, p);
                request(p, x);
                __builtin_amdgcn_sched_barrier(0);     // the loads stay ahead of the products they run beside
            };
            constexpr int BLOCKS = SPAN / kBlock;
            static_assert(BLOCKS == 1 || BLOCKS == 4);
            constexpr int UNROLL = BLOCKS == 1 ? 2 : BLOCKS;
            for (; left >= UNROLL; left -= UNROLL) {
                next(pb, xb);
                multiply(Const<int, 0>(), pa, xa);
                next(pa, xa);
                multiply(Const<int, 1>(), pb, xb);
                if constexpr (BLOCKS == 4) {
                    next(pb, xb);
                    multiply(Const<int, 2>(), pa, xa);
                    next(pa, xa);
                    multiply(Const<int, 3>(), pb, xb);
                }
            }
            if (left > 0) {
                if (BLOCKS > 1 && left > 1) next(pb, xb);
                multiply(Const<int, 0>(), pa, xa);
                if (BLOCKS == 4 && left > 1) {
                    if (left > 2) next(pa, xa);
                    multiply(Const<int, 1>(), pb, xb);
                    if (left > 2) multiply(Const<int, 2>(), pa, xa);
                }
                if (BLOCKS > 1) close();
            }
        }
    }
    // what is left of the share, fewer than kBlock rows: one wavefront each
    const int rest = kb + n_blocks * kBlock + wave;
    if (rest < ke) {
        const int r0 = idx[rest];
        struct { typename E::raw_t q[1]; uint16_t sc[1]; } x;
        float m[1][B];
#pragma unroll
        for (int i = 0; i < B; ++i) m[0][i] = val[rest * B + i];
        const uint32_t r = (uint32_t)r0 < (uint32_t)p.n_in ? (uint32_t)r0 : 0u;
        x.q[0] = __builtin_nontemporal_load(
            reinterpret_cast<const typename E::raw_t*>(w + (size_t)r * (size_t)p.row_stride + voff));
        if constexpr (E::kScaled) x.sc[0] = (scales + (size_t)r * (size_t)p.scale_stride)[sgroup];
        rows(Const<bool, true>(), Const<int, 0>(), Const<int, 1>(), m, x);
        close();
    }
    static_assert(kBlock <= kWaves, "one leftover row per wavefront");
    // wavefronts through LDS, added in pairs
#pragma unroll
    for (int b = 0; b < B; ++b) {
        if constexpr (E::kScaled) {
#pragma unroll
            for (int e = 0; e < EPL; ++e) tot[b][e] *= 16777216.0f / up[b];
        }
        if (b > 0) __syncthreads();
#pragma unroll
        for (int e = 0; e < EPL; e += 4)
            *reinterpret_cast<float4*>(&red[wave][lane * EPL + e]) =
                make_float4(tot[b][e], tot[b][e + 1], tot[b][e + 2], tot[b][e + 3]);
        __syncthreads();
        float* out = p.out + layer * p.out_layer_stride + ((int64_t)g * B + b) * p.n_out;
#pragma unroll
        for (int c0 = 0; c0 < SC; c0 += kWaves * 64) {
            const int c = c0 + tid;
            const int gcol = strip * SC + c;
            if (c < SC && gcol < p.n_out) {
                float s[kWaves];
#pragma unroll
                for (int i = 0; i < kWaves; ++i) s[i] = red[i][c];
#pragma unroll
                for (int h = kWaves / 2; h > 0; h /= 2)
#pragma unroll
                    for (int i = 0; i < h; ++i) s[i] += s[i + h];
                out[gcol] = s[0];
            }
        }
    }
}

// (int4 batches of three and more run on the matrix cores)
template <typename E>
hipError_t launch_rows(const StackProductParams& p, dim3 grid, dim3 block, hipStream_t stream, int pk) {
    if (p.rows == 1) return launch_timed(stack_product_kernel<E, 1>, grid, block, stream, pk, p);
    if (p.rows == 2) return launch_timed(stack_product_kernel<E, 2>, grid, block, stream, pk, p);
    if constexpr (!E::kScaled) switch (p.rows) {
        case 3: return launch_timed(stack_product_kernel<E, 3>, grid, block, stream, pk, p);
        case 4: return launch_timed(stack_product_kernel<E, 4>, grid, block, stream, pk, p);
        case 5: return launch_timed(stack_product_kernel<E, 5>, grid, block, stream, pk, p);
        case 6: return launch_timed(stack_product_kernel<E, 6>, grid, block, stream, pk, p);
        case 7: return launch_timed(stack_product_kernel<E, 7>, grid, block, stream, pk, p);
        case 8: return launch_timed(stack_product_kernel<E, 8>, grid, block, stream, pk, p);
    }
    return hipErrorInvalidValue;
}

}  // namespace

static int stack_strips(int dtype, int n_out) {
    const int sc = 64 * (dtype == DIP_F32 ? 4 : (dtype == DIP_BF16 ? 8 : 16));
    return (n_out + sc - 1) / sc;
}

bool stack_pays(int dtype, int n_out, int k_max, int layers, int rows) {
    // fp32 and bf16: one round of workgroups, four to a compute unit, with 512 listed columns each.
    // Below that the narrower strips of bgemv_kernel fill the chip better (bf16 at 3 rows, 4 layers of
    // 2048 x 7168: 70 against 79 us), from twice as many on they are never ahead (bf16 at 8 rows, 40 layers
    // of 2048 x 7168: 774 against 637 us); in between the two are within 7 % of each other.
    // int4: bgemv_kernel adds up its codes with their offset in one chain; its error fits the short
    // shares of a single layer only.
    if (dtype == DIP_INT4_G128) return layers >= 2 && rows <= 2;
    return layers >= 4 && (int64_t)stack_strips(dtype, n_out) * layers * ((k_max + 511) / 512) >= 1024;
}

int stack_shares(int dtype, int n_out, int k_max, int layers, int rows) {
    const int wgs = stack_strips(dtype, n_out) * layers;
    // Shares of at most kLong columns, which bounds the rounding error as well, and for few layers as many
    // as make `target` workgroups of at least `least` columns.  The sums of a share are written and read
    // once per batch row: longer shares for more rows.  Half or twice any of these moves the mean over
    // sizes of 512 to 5120 and 4 to 40 layers by 0 to 2 % (`least`: int4 at one row 3.5 % at 32, 6.6 % at 256, at
    // two rows 2.5 and 12 %).
    constexpr int least = 64;
    const int kLong = rows == 1 ? 384 : 1536, target = rows == 1 ? 1024 : 2048;
    return std::max((k_max + kLong - 1) / kLong, std::min((target + wgs - 1) / wgs, k_max / least));
}

hipError_t launch_stack_product(const StackProductParams& p, int dtype, int shares, int layers, hipStream_t stream,
                                int pk) {
    if (!p.idx || !p.val || !p.out || (dtype == DIP_INT4_G128 && !p.rowmax) || layers < 1 || layers > kStackLayers || shares < 1) return hipErrorInvalidValue;
    const dim3 grid(stack_strips(dtype, p.n_out), shares, layers),
        block(64 * (p.rows == 1 ? Shape<1>::kWaves : Shape<2>::kWaves));
    if (dtype == DIP_F32) return launch_rows<F32>(p, grid, block, stream, pk);
    if (dtype == DIP_BF16) return launch_rows<Bf16>(p, grid, block, stream, pk);
    if (dtype == DIP_INT4_G128) return launch_rows<Q4>(p, grid, block, stream, pk);
    return hipErrorInvalidValue;
}

}  // namespace dip
