// The selection of a pruning point (Alg. 1 steps 1-2) as every workgroup of 1024 lanes runs it:
// at the head of the gathered products (dip_fused.hip) and, one workgroup per input vector,
// for the rows of a batch and the layers of a stack (dip_rows.hip).
//
// Cache-aware scores without a division per key.  Eq. 10 of Sec. 5.2 is s = fl(p / M) with
// p = |v| for resident columns, fl(|v| * gamma) otherwise, and M = ||v||_inf.  q -> fl(q / M)
// is monotone, so the k-th largest score is T_s = fl(T_p / M) with T_p the k-th largest p, and
//     { s > T_s }  = { p >= P_hi },  P_hi = the smallest float with fl(P_hi / M) >  T_s
//     { s == T_s } = { P_lo <= p < P_hi },  P_lo = the smallest float with fl(P_lo / M) >= T_s.
// The selection therefore runs on the bit patterns of p, and only P_lo and P_hi need
// divisions: 64 candidates around T_p, one per lane, settle them in one step (a bisection
// over all floats covers the case that the window is too small, e.g. denormal scores).  The
// selected set is then exactly the top-K of the rounded scores with lowest-index ties -- the
// set the stand-alone selection kernel and the oracle produce from the emitted s.
#ifndef DIP_HEAD_DEVICE_H_
#define DIP_HEAD_DEVICE_H_

#include "dip_select_device.h"

namespace dip {
namespace sel {

struct HeadShared {
    uint32_t hist[kBinsA + kBinsB + kBinsC];
    uint32_t cw[kMaxWords];          // residency words used for scoring
    uint32_t tile[2][kMaxTiles];
    uint32_t wave_tot[2][kWaves];
    float wave_max[kWaves];
    uint32_t bcast[4];
    uint32_t cand[kNearCand];        // keys of the threshold bin
    uint32_t ncand;
};
constexpr int kHeadHistWords = kBinsA + kBinsB + kBinsC;

// Exclusive running sums of the per-tile counts over the tiles in index order: lane j of each
// wavefront passes the count of the wavefront's tile in slot j and gets the sum over the tiles
// before it; `total` is the sum over all tiles.
template <int ITEMS>
__device__ __forceinline__ uint32_t tile_scan(uint32_t cnt, HeadShared& sh, int& phase, uint32_t& total) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int ntiles = ITEMS * kWaves;
    if (lane < ITEMS) sh.tile[0][lane * kWaves + wave] = cnt;
    __syncthreads();
    const uint32_t t = tid < ntiles ? sh.tile[0][tid] : 0u;
    const uint32_t ex = block_excl_scan(t, sh, phase);
    if (tid < ntiles) sh.tile[0][tid] = ex;
    if (tid == ntiles - 1) sh.bcast[3] = ex + t;
    __syncthreads();
    total = sh.bcast[3];
    return lane < ITEMS ? sh.tile[0][lane * kWaves + wave] : 0u;
}

// Smallest float bit pattern c in [lo, hi] with pred(fl(c / M)) true, where pred is monotone
// (false ... false true ... true) and true at hi.  Every lane runs the same bisection.
template <bool STRICT>
__device__ __forceinline__ uint32_t bisect_quotient(uint32_t lo, uint32_t hi, float M, float Ts) {
    while (lo < hi) {
        const uint32_t mid = lo + ((hi - lo) >> 1);
        const float q = __fdiv_rn(__uint_as_float(mid), M);
        const bool ok = STRICT ? (q > Ts) : (q >= Ts);
        if (ok) hi = mid; else lo = mid + 1u;
    }
    return lo;
}

// The keys that tie with the k-th largest score, and those above it (Eq. 10 without a division
// per key, see the head of this file): Tk is the k-th largest key (bits(p) << 1), M = ||v||_inf.
// Leaves K_lo, K_hi alone when M is 0 (all scores are 0).
__device__ __forceinline__ void score_window(uint32_t Tk, float M, int lane, uint32_t& K_lo, uint32_t& K_hi) {
    if (!(M > 0.f)) return;
    const uint32_t Tb = Tk >> 1;
    const float Ts = __fdiv_rn(__uint_as_float(Tb), M);
    constexpr uint32_t kInf = 0x7f800000u;
    const int64_t cand = (int64_t)Tb + lane - 31;
    const uint32_t cb = cand < 0 ? 0u : (cand > (int64_t)kInf ? kInf : (uint32_t)cand);
    const float qc = __fdiv_rn(__uint_as_float(cb), M);
    const uint64_t ge = __ballot(qc >= Ts), gt = __ballot(qc > Ts);   // lane 31 is T_p: in ge
    const uint32_t c0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)cb);
    uint32_t Plo, Phi;
    if ((ge & 1ull) && c0 > 0u) {
        Plo = bisect_quotient<false>(0u, c0, M, Ts);
    } else {
        // (ge is never empty for finite inputs: lane 31 holds T_p itself)
        Plo = ge ? (uint32_t)__builtin_amdgcn_readlane((int)cb, __builtin_ctzll(ge)) : Tb;
    }
    if (gt == 0ull) {
        Phi = bisect_quotient<true>(Tb + 1u, kInf, M, Ts);
    } else {
        Phi = (uint32_t)__builtin_amdgcn_readlane((int)cb, __builtin_ctzll(gt));
    }
    K_lo = Plo << 1;
    K_hi = Phi << 1;
}

// Per-tile counts of the keys in [K_lo, K_hi) (low 16 bits) and >= K_hi (high 16 bits), their
// exclusive prefix over the tiles in index order (lane j of each wavefront returns the prefix
// of the wavefront's tile in slot j), and the totals.
template <int ITEMS>
__device__ __forceinline__ uint32_t tile_prefix_window(const uint32_t (&key)[ITEMS], uint32_t K_lo, uint32_t K_hi,
                                                       HeadShared& sh, int& phase, uint32_t& totals) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int ntiles = ITEMS * kWaves;
    uint32_t mine = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const uint32_t ce = (uint32_t)__popcll(__ballot(key[j] >= K_lo && key[j] < K_hi));
        const uint32_t cg = (uint32_t)__popcll(__ballot(key[j] >= K_hi));
        mine = lane == j ? (ce | (cg << 16)) : mine;
    }
    __syncthreads();       // (the table may still be read by a slower wavefront)
    if (lane < ITEMS) sh.tile[0][lane * kWaves + wave] = mine;
    __syncthreads();
    const uint32_t t = tid < ntiles ? sh.tile[0][tid] : 0u;
    const uint32_t ex = block_excl_scan(t, sh, phase);
    if (tid < ntiles) sh.tile[0][tid] = ex;
    if (tid == kSelThreads - 1) sh.bcast[3] = ex + t;
    __syncthreads();
    totals = sh.bcast[3];
    return lane < ITEMS ? sh.tile[0][lane * kWaves + wave] : 0u;
}

// Keys of one vector and its selection threshold: v and key hold the lane's features tid,
// tid + 1024, ... (0 past the end), M = ||v||_inf, and afterwards the keys in [K_lo, K_hi) tie
// at the k-th largest score while the keys >= K_hi lie above it.  score_bits: residency words
// for the cache-aware scores, or null for the plain DIP key |v|.
template <int ITEMS>
__device__ __forceinline__ void head_threshold(const float* vec, int n, uint32_t k, const uint32_t* score_bits,
                                               float gamma, HeadShared& hs, int& phase, float (&v)[ITEMS],
                                               uint32_t (&key)[ITEMS], float& M, uint32_t& K_lo, uint32_t& K_hi) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nwords = (n + 31) >> 5;
    {
        const float* vp = vec + tid;
        const int full = n >> 10;       // slots that lie inside the vector entirely (wave-uniform)
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            if (j < full) {
                v[j] = vp[j * kSelThreads];
            } else {
                const uint32_t i = (uint32_t)(j * kSelThreads + tid);
                v[j] = 0.f;
                if (i < (uint32_t)n) v[j] = vec[i & (DIP_MAX_N - 1)];
            }
        }
    }
    static_assert(kHeadHistWords % (2 * kSelThreads) == 0, "the histograms are cleared in 8-byte pieces");
#pragma unroll
    for (int b = 0; b < kHeadHistWords / (2 * kSelThreads); ++b)
        reinterpret_cast<uint2*>(hs.hist)[b * kSelThreads + tid] = make_uint2(0u, 0u);
    hs.cw[tid] = (score_bits && tid < nwords) ? score_bits[tid] : 0u;
    {
        // ||v||_inf: the denominator of Eq. 10, and the anchor of the selection's histogram
        float vmax = 0.f;
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) vmax = fmaxf(vmax, fabsf(v[j]));
        // (fmaxf drops a NaN operand: non-finite inputs leave M finite or infinite, never NaN)
        vmax = wave_max_nonneg(vmax);
        if (lane == 0) hs.wave_max[wave] = vmax;
    }
    __syncthreads();
    static_assert(kWaves == 16, "one wavefront maximum per lane of a 16-lane row");
    M = row_max_nonneg(hs.wave_max[lane & (kWaves - 1)]);

    // p = |v| for resident columns, fl(|v| * gamma) for the others (plain DIP: p = |v|); p <= M
    if (score_bits) {
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const float a = fabsf(v[j]);
            const uint32_t c = (hs.cw[j * (kSelThreads / 32) + (tid >> 5)] >> (tid & 31)) & 1u;
            key[j] = __float_as_uint(c ? a : __fmul_rn(a, gamma)) << 1;
        }
    } else {
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) key[j] = __float_as_uint(fabsf(v[j])) << 1;
    }
    uint32_t Tk, need;
    block_select_largest_near_max<ITEMS>(key, __float_as_uint(M) << 1, k, hs, phase, Tk, need);
    K_lo = Tk;
    K_hi = Tk + 1u;
    if (score_bits) score_window(Tk, M, lane, K_lo, K_hi);
}

// Mask words of the selection, slot by slot (a template recursion: the lane numbers are constants).
template <int J, int ITEMS>
struct MaskWords {
    __device__ static __forceinline__ void run(const uint32_t (&key)[ITEMS], uint32_t K_lo, uint32_t K_hi, bool fast,
                                               uint32_t take, uint32_t eq_seen, int next, int G, int& my_word) {
        // `next`: the next slot of this workgroup (g, g + G, ...; uniform, and no division)
        if (J == next) {
            slot(key, K_lo, K_hi, fast, take, eq_seen, my_word);
            next += G;
        }
        if constexpr (J + 1 < ITEMS) MaskWords<J + 1, ITEMS>::run(key, K_lo, K_hi, fast, take, eq_seen, next, G, my_word);
    }
    __device__ static __forceinline__ void slot(const uint32_t (&key)[ITEMS], uint32_t K_lo, uint32_t K_hi, bool fast,
                                                uint32_t take, uint32_t eq_seen, int& my_word) {
        bool mine;
        if (fast) {
            mine = key[J] >= K_lo;
        } else {
            // ties at the threshold: the `take` lowest indices among them are selected
            mine = key[J] >= K_hi;
            const bool tie = key[J] >= K_lo && !mine;
            const uint64_t be = __ballot(tie);
            const uint32_t eq_before = (uint32_t)__builtin_amdgcn_readlane((int)eq_seen, J) & 0xffffu;
            mine = mine || (tie && eq_before + lanes_below(be) < take);
        }
        const uint64_t bs = __ballot(mine);
        write_lane<(2 * J) & 63>(my_word, (uint32_t)bs);
        write_lane<(2 * J + 1) & 63>(my_word, (uint32_t)(bs >> 32));
    }
};

}  // namespace sel
}  // namespace dip

#endif  // DIP_HEAD_DEVICE_H_
