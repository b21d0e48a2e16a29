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
// int4 rows are a quarter of the bytes and bound by vector instructions: see Q4.
#include "dip_internal.h"

namespace dip {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

#define DIP_CONSTANT __attribute__((address_space(4)))

struct F32 {
    typedef u32x4 raw_t;
    static constexpr int kElems = 4, kBits = 32;
    static constexpr bool kScaled = false;
    __device__ static __forceinline__ void fma(const raw_t& q, float m, float (&acc)[4]) {
        acc[0] = fmaf(__uint_as_float(q.x), m, acc[0]);
        acc[1] = fmaf(__uint_as_float(q.y), m, acc[1]);
        acc[2] = fmaf(__uint_as_float(q.z), m, acc[2]);
        acc[3] = fmaf(__uint_as_float(q.w), m, acc[3]);
    }
};
struct Bf16 {  // the upper half of an fp32 pattern
    typedef u32x4 raw_t;
    static constexpr int kElems = 8, kBits = 16;
    static constexpr bool kScaled = false;
    __device__ static __forceinline__ void fma(const raw_t& q, float m, float (&acc)[8]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            acc[2 * i] = fmaf(__uint_as_float(q[i] << 16), m, acc[2 * i]);
            acc[2 * i + 1] = fmaf(__uint_as_float(q[i] & 0xffff0000u), m, acc[2 * i + 1]);
        }
    }
};
struct Q4 {
    // 16 codes per 8-byte load, low nibble = even element.  Flipping bit 3 of every nibble turns
    // the code q into q + 8 in [0, 15].  Two nibbles 16 bits apart, masked in place, are the bit
    // patterns of two fp16 denormals, (q + 8) * 2^-24 (bits 0-3) or (q + 8) * 2^-20 (bits 4-7),
    // which v_fma_mix_f32 widens exactly while it multiplies and adds in fp32: 6 instructions
    // unpack 8 codes, where a byte conversion per code takes 12.  The factor leaves through the
    // multiplier (2^12, exact) and the sums (2^12); the offset as -8 * sum of multipliers.
    typedef u32x2 raw_t;
    static constexpr int kElems = 16, kBits = 4;
    static constexpr bool kScaled = true;
    static constexpr float kUp = 4096.0f;      // 2^12 on the multiplier and on the sums
    __device__ static __forceinline__ float lo(uint32_t v) {
        const uint16_t b = (uint16_t)v;
        return (float)__builtin_bit_cast(_Float16, b);
    }
    __device__ static __forceinline__ float hi(uint32_t v) {
        const uint16_t b = (uint16_t)(v >> 16);
        return (float)__builtin_bit_cast(_Float16, b);
    }
    // m24 = multiplier * 2^12 for codes in bits 0-3 of a half, m20 = multiplier * 2^8 for bits 4-7
    __device__ static __forceinline__ void fma(const raw_t& q, float m24, float m20, float (&acc)[16]) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t o = q[i] ^ 0x88888888u, o8 = o >> 8;
            const uint32_t c04 = o & 0x000f000fu, c15 = o & 0x00f000f0u;
            const uint32_t c26 = o8 & 0x000f000fu, c37 = o8 & 0x00f000f0u;
            float* a = acc + 8 * i;
            a[0] = fmaf(lo(c04), m24, a[0]);
            a[4] = fmaf(hi(c04), m24, a[4]);
            a[1] = fmaf(lo(c15), m20, a[1]);
            a[5] = fmaf(hi(c15), m20, a[5]);
            a[2] = fmaf(lo(c26), m24, a[2]);
            a[6] = fmaf(hi(c26), m24, a[6]);
            a[3] = fmaf(lo(c37), m20, a[3]);
            a[7] = fmaf(hi(c37), m20, a[7]);
        }
    }
};

constexpr int kWaves = 8;     // wavefronts per workgroup
constexpr int kBlock = 8;     // selected rows in flight per wavefront and register set

template <typename E>
__global__ __launch_bounds__(kWaves * 64) void stack_product_kernel(StackProductParams p) {
    constexpr int EPL = E::kElems, SC = 64 * EPL;
    __shared__ float red[kWaves][SC];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int strip = blockIdx.x, g = blockIdx.y, G = gridDim.y, layer = blockIdx.z;
    const int k = p.layer[layer].k;
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
    const DIP_CONSTANT float* val = (const DIP_CONSTANT float*)(uintptr_t)(p.val + layer * p.list_layer_stride);

    float acc[EPL], msum = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = 0.f;

    struct Pairs { int r[kBlock]; float m[kBlock]; };
    struct Rows { typename E::raw_t q[kBlock]; uint16_t sc[kBlock]; };
    auto fetch = [&](int t, Pairs& b) {
#pragma unroll
        for (int u = 0; u < kBlock; ++u) {
            b.r[u] = idx[t + u];
            b.m[u] = val[t + u];
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
    auto multiply = [&](const Pairs& b, const Rows& x) {
#pragma unroll
        for (int u = 0; u < kBlock; ++u) {
            if constexpr (E::kScaled) {
                const float mult = b.m[u] * (float)__builtin_bit_cast(_Float16, x.sc[u]);
                msum += mult;
                E::fma(x.q[u], mult * E::kUp, mult * (E::kUp / 16.0f), acc);
            } else {
                E::fma(x.q[u], b.m[u], acc);
            }
        }
    };

    // full blocks t = kb + (wave + i * kWaves) * kBlock
    const int n_blocks = (ke - kb) / kBlock;
    const int mine = n_blocks > wave ? (n_blocks - wave - 1) / kWaves + 1 : 0;
    constexpr int STEP = kWaves * kBlock;
    int t = kb + wave * kBlock;
    if (mine > 0) {
        Pairs pa, pb;
        Rows xa, xb;
        fetch(t, pa);
        request(pa, xa);
        int left = mine;
        while (true) {
            if (left == 1) { multiply(pa, xa); break; }
            t += STEP;
            fetch(t, pb);
            request(pb, xb);
            multiply(pa, xa);
            if (left == 2) { multiply(pb, xb); break; }
            t += STEP;
            fetch(t, pa);
            request(pa, xa);
            multiply(pb, xb);
            left -= 2;
        }
    }
    // what is left of the share, fewer than kBlock rows: one wavefront each
    const int rest = kb + n_blocks * kBlock + wave;
    if (rest < ke) {
        const int r0 = idx[rest];
        const float m = val[rest];
        const uint32_t r = (uint32_t)r0 < (uint32_t)p.n_in ? (uint32_t)r0 : 0u;
        const typename E::raw_t q = __builtin_nontemporal_load(
            reinterpret_cast<const typename E::raw_t*>(w + (size_t)r * (size_t)p.row_stride + voff));
        if constexpr (E::kScaled) {
            const float mult = m * (float)__builtin_bit_cast(_Float16, (scales + (size_t)r * (size_t)p.scale_stride)[sgroup]);
            msum += mult;
            E::fma(q, mult * E::kUp, mult * (E::kUp / 16.0f), acc);
        } else {
            E::fma(q, m, acc);
        }
    }
    static_assert(kBlock <= kWaves, "one leftover row per wavefront");
    if constexpr (E::kScaled) {
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] = fmaf(-8.0f, msum, acc[e] * E::kUp);
    }

    // wavefronts through LDS, added in order
#pragma unroll
    for (int e = 0; e < EPL; e += 4)
        *reinterpret_cast<float4*>(&red[wave][lane * EPL + e]) = make_float4(acc[e], acc[e + 1], acc[e + 2], acc[e + 3]);
    __syncthreads();
    float* out = p.out + layer * p.out_layer_stride + (int64_t)g * p.n_out;
#pragma unroll
    for (int c0 = 0; c0 < SC; c0 += kWaves * 64) {
        const int c = c0 + tid;
        const int gcol = strip * SC + c;
        if (c < SC && gcol < p.n_out) {
            float s = 0.f;
#pragma unroll
            for (int i = 0; i < kWaves; ++i) s += red[i][c];
            out[gcol] = s;
        }
    }
}

}  // namespace

int stack_shares(int dtype, int n_out, int k_max, int layers) {
    const int sc = 64 * (dtype == DIP_F32 ? 4 : (dtype == DIP_BF16 ? 8 : 16));
    const int strips = (n_out + sc - 1) / sc;
    const int wgs = strips * layers;
    int g = (k_max + 383) / 384;
    while (wgs * g < 1024 && k_max / (g + 1) >= kWaves * kBlock) ++g;
    return g < 1 ? 1 : g;
}

hipError_t launch_stack_product(const StackProductParams& p, int dtype, int shares, int layers, hipStream_t stream,
                                int pk) {
    if (!p.idx || !p.val || !p.out || layers < 1 || layers > kStackLayers || shares < 1) return hipErrorInvalidValue;
    const int sc = 64 * (dtype == DIP_F32 ? 4 : (dtype == DIP_BF16 ? 8 : 16));
    const dim3 grid((p.n_out + sc - 1) / sc, shares, layers), block(kWaves * 64);
    if (dtype == DIP_F32) return launch_timed(stack_product_kernel<F32>, grid, block, stream, pk, p);
    if (dtype == DIP_BF16) return launch_timed(stack_product_kernel<Bf16>, grid, block, stream, pk, p);
    if (dtype == DIP_INT4_G128) return launch_timed(stack_product_kernel<Q4>, grid, block, stream, pk, p);
    return hipErrorInvalidValue;
}

}  // namespace dip
