// Selections of several vectors in one launch, one workgroup each: the rows of a small batch and
// the layers of a stack call.  Every workgroup runs the selection of dip_head_device.h on its
// vector and leaves the mask words and, as asked, the index list with its multipliers (what
// the products of a stack read) and the bit pattern of max |v| (what the matrix-core product
// scales a row by).
//
// One compute unit per vector: a single vector leaves the rest of the chip idle (5 us over
// d_model = 5120, 9 us over d_ff = 17920 of the Phi-3-Medium shape), a stack of 40 layers takes
// as long as one, which is why a stack call selects for all of its layers at once.
#include "dip_head_device.h"

namespace dip {
namespace {

using namespace sel;

struct RowsShared {
    HeadShared head;
    uint32_t mwords[kMaxWords];
    uint32_t wave_cnt[kWaves];
};

// The index list and the multipliers of the selection, slot by slot (a template recursion: the
// lane numbers are constants).  Lane j of `before` / `eq_seen` belongs to the wavefront's tile in
// slot j: selected keys (fast) or keys above the threshold (otherwise) before the tile, and
// ties before it.
template <int J, int ITEMS>
struct EmitList {
    __device__ static __forceinline__ void run(const uint32_t (&key)[ITEMS], const float (&v)[ITEMS], uint32_t K_lo,
                                               uint32_t K_hi, bool fast, uint32_t take, uint32_t before,
                                               uint32_t eq_seen, uint32_t k, int32_t* idx_out, float* val_out) {
        uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)before, J);
        bool mine = key[J] >= K_lo;
        if (!fast) {
            const uint32_t eq_before = (uint32_t)__builtin_amdgcn_readlane((int)eq_seen, J);
            const bool above = key[J] >= K_hi;
            const bool tie = mine && !above;
            const uint64_t be = __ballot(tie);
            mine = above || (tie && eq_before + lanes_below(be) < take);
            first += min(eq_before, take);
        }
        const uint64_t bs = __ballot(mine);
        const uint32_t pos = first + lanes_below(bs);
        // pos < k always holds; the test keeps a logic slip from writing out of bounds (and the
        // mask tells the compiler that a 32-bit offset is enough)
        if (mine && pos < k) {
            idx_out[pos & (DIP_MAX_N - 1)] = J * kSelThreads + (int)threadIdx.x;
            val_out[pos & (DIP_MAX_N - 1)] = v[J];
        }
        if constexpr (J + 1 < ITEMS)
            EmitList<J + 1, ITEMS>::run(key, v, K_lo, K_hi, fast, take, before, eq_seen, k, idx_out, val_out);
    }
};

template <int ITEMS, bool LISTS, int LAYERS>
__global__ __launch_bounds__(kSelThreads) void rows_select_kernel(RowsSelectParamsT<LAYERS> p) {
    __shared__ __align__(16) RowsShared sh;
    HeadShared& hs = sh.head;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nwords = (p.n + 31) >> 5;
    const int row = blockIdx.x, layer = LAYERS == 1 ? 0 : blockIdx.y;
    const uint32_t k = (uint32_t)p.layer[layer].k;
    int phase = 0;

    float v[ITEMS];
    uint32_t key[ITEMS];
    float M;
    uint32_t K_lo, K_hi;
    head_threshold<ITEMS>(p.v + layer * p.v_layer_stride + row * p.v_row_stride, p.n, k, p.layer[layer].score_bits,
                          p.gamma, hs, phase, v, key, M, K_lo, K_hi);
    if (p.rowmax_out && tid == 0) p.rowmax_out[layer * p.rowmax_layer_stride + row] = __float_as_uint(M);

    // how many keys reach K_lo: exactly k means no tie is split at the threshold
    uint32_t n_ge, before = 0u, eq_seen = 0u, take = 0u;
    if constexpr (LISTS) {
        int cnt = 0;
        TileCount<0, ITEMS>::ge(key, K_lo, cnt);
        before = tile_scan<ITEMS>((uint32_t)cnt, hs, phase, n_ge);
    } else {
        uint32_t n_wave = 0u;
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) n_wave += (uint32_t)__popcll(__ballot(key[j] >= K_lo));
        if (lane == 0) sh.wave_cnt[wave] = n_wave;
        __syncthreads();
        n_ge = 0u;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) n_ge += sh.wave_cnt[w];
    }
    const bool fast = n_ge == k;
    if (!fast) {
        uint32_t totals;
        const uint32_t pre = tile_prefix_window<ITEMS>(key, K_lo, K_hi, hs, phase, totals);
        take = k > (totals >> 16) ? k - (totals >> 16) : 0u;
        eq_seen = pre & 0xffffu;
        before = pre >> 16;
    }
    if constexpr (LISTS)
        EmitList<0, ITEMS>::run(key, v, K_lo, K_hi, fast, take, before, eq_seen, k,
                                p.idx_out + layer * p.list_layer_stride, p.val_out + layer * p.list_layer_stride);
    if (p.mask_out) {
        int my_word = 0;
        MaskWords<0, ITEMS>::run(key, K_lo, K_hi, fast, take, eq_seen, 0, 1, my_word);
        if (lane < 2 * ITEMS)
            sh.mwords[((lane >> 1) * (kSelThreads / 32) + wave * 2 + (lane & 1)) & (kMaxWords - 1)] = (uint32_t)my_word;
        __syncthreads();
        if (tid < nwords) p.mask_out[layer * p.mask_layer_stride + row * p.mask_row_stride + tid] = sh.mwords[tid];
    }
}

template <int ITEMS>
hipError_t launch_items(const RowsSelectParams& p, int layers, hipStream_t stream, int pk) {
    const dim3 grid(p.rows, layers), block(kSelThreads);
    if (p.idx_out) return launch_timed(rows_select_kernel<ITEMS, true, kStackLayers>, grid, block, stream, pk, p);
    if (layers == 1) return launch_timed(rows_select_kernel<ITEMS, false, 1>, grid, block, stream, pk, one_layer(p));
    return launch_timed(rows_select_kernel<ITEMS, false, kStackLayers>, grid, block, stream, pk, p);
}

}  // namespace

hipError_t launch_select_rows(const RowsSelectParams& p, int layers, hipStream_t stream, int pk) {
    if (!p.v || !(p.mask_out || p.idx_out) || p.rows < 1 || layers < 1 || layers > kStackLayers || p.n < 1 ||
        p.n > DIP_MAX_N || (p.idx_out && (p.rows != 1 || !p.val_out)))
        return hipErrorInvalidValue;
    for (int l = 0; l < layers; ++l)
        if (p.layer[l].k < 1 || p.layer[l].k > p.n) return hipErrorInvalidValue;
    const int items = (p.n + kSelThreads - 1) / kSelThreads;
    if (items <= 2) return launch_items<2>(p, layers, stream, pk);
    if (items <= 4) return launch_items<4>(p, layers, stream, pk);
    if (items <= 6) return launch_items<6>(p, layers, stream, pk);
    if (items <= 8) return launch_items<8>(p, layers, stream, pk);
    if (items <= 11) return launch_items<11>(p, layers, stream, pk);
    if (items <= 14) return launch_items<14>(p, layers, stream, pk);
    if (items <= 18) return launch_items<18>(p, layers, stream, pk);
    if (items <= 24) return launch_items<24>(p, layers, stream, pk);
    return launch_items<32>(p, layers, stream, pk);
}

}  // namespace dip
