// Column-gathered GEMV (Alg. 1 step 4 applied to x; Sec. 4 for the bundled up/gate case):
//     y[j] = sum_{t<k} W[j, idx[t]] * x[idx[t]]
// over a feature-major matrix, so each selected column is one contiguous row in HBM.
//
// Decode at batch 1 reads every selected weight exactly once and does two flops per
// element: the kernel is bound by HBM bandwidth, not arithmetic, so there are no matrix
// cores here -- only wide coalesced loads, many of them in flight, and fp32 FMAs.
//
// Work split.  The outputs are cut into strips of LPR*EPL columns (EPL = elements per
// 16-byte load).  A workgroup owns one strip (both the up and the gate strip when the
// matrix is the bundled pair) and a contiguous share of the k selected rows; inside it
// every wavefront handles 64/LPR rows per step, LPR lanes side by side on one row, each
// lane loading 16 bytes.  Sums are combined in a fixed order: lane groups inside a
// wavefront (xor butterfly), wavefronts through LDS in index order, workgroups of one
// strip through a partial buffer that the last workgroup to arrive adds in index order.
// The result is bit-repeatable for a given launch shape.

#include <time.h>
#include <unistd.h>

#include <atomic>

#include "dip_gemv_device.h"

namespace dip {

GemvShape g_gemv_override = {0, 0, 0, 0};
constexpr int kComputeUnits = 256;   // MI355X

namespace {

using namespace gemv;

template <typename WT, int LPR, int WAVES, int UNROLL, int NSEG>
__global__ __launch_bounds__(WAVES * 64) void gemv_kernel(GemvParams p) {
    typedef Tile<WT, LPR, WAVES, UNROLL, NSEG> T;
    __shared__ float red[WAVES][NSEG][T::SC];
    __shared__ int s_last;
    const int strip = blockIdx.x;
    const int g = blockIdx.y, G = gridDim.y;
    // this workgroup's share of the selected rows
    const int kb = min(p.k, g * p.rows_per_split);   // rows_per_split is a multiple of 8
    const int ke = min(p.k, kb + p.rows_per_split);
    float acc[NSEG][T::EPL];
    accumulate<WT, LPR, WAVES, UNROLL, NSEG>(p, p.idx, p.val, 0, kb, ke, strip, acc);
    finish<WT, LPR, WAVES, UNROLL, NSEG>(p, acc, strip, g, G, red, s_last);
}

// The same in the default shape for a caller's own index list: the workgroup takes its share of the
// list and the activations at it into LDS, where the row loop reads aligned vectors whatever the
// caller's alignment.  (A launch in front that copied the list and gathered the activations took
// as long as a third of the product: 2.4 us and the gap behind it, 4100 x 1229 in fp32.)
constexpr int kGatherLpr = 16, kGatherWaves = 8, kGatherUnroll = 4;
constexpr int kGatherCap = 2048;     // rows of a share: 16 KB of LDS
template <typename WT>
__global__ __launch_bounds__(kGatherWaves * 64) void gemv_gather_kernel(GemvParams p, const float* x) {
    typedef Tile<WT, kGatherLpr, kGatherWaves, kGatherUnroll, 1> T;
    __shared__ __align__(16) int32_t l_idx[kGatherCap];
    __shared__ __align__(16) float l_val[kGatherCap];
    __shared__ float red[kGatherWaves][1][T::SC];
    __shared__ int s_last;
    const int strip = blockIdx.x;
    const int g = blockIdx.y, G = gridDim.y;
    const int kb = min(p.k, g * p.rows_per_split);   // rows_per_split is a multiple of 8, <= kGatherCap
    const int ke = min(p.k, kb + p.rows_per_split);
    for (int t = threadIdx.x; t < ke - kb; t += kGatherWaves * 64) {
        const int r = p.idx[kb + t];
        l_idx[t] = r;
        l_val[t] = (unsigned)r < (unsigned)p.n_in ? x[r] : 0.f;
    }
    __syncthreads();
    float acc[1][T::EPL];
    accumulate<WT, kGatherLpr, kGatherWaves, kGatherUnroll, 1>(p, l_idx, l_val, kb, kb, ke, strip, acc);
    finish<WT, kGatherLpr, kGatherWaves, kGatherUnroll, 1>(p, acc, strip, g, G, red, s_last);
}

// ---------------------------------------------------------------------------------------
// Row-gathered dot products (Sec. 3.2, Gate / Up pruning): the matrix whose rows a mask
// removes is stored neuron-major, so the selected neuron j is one contiguous row and
//     out[t] = W[idx[t], :] . x
// streams k whole rows.  One wavefront takes one row at a time, 16 bytes per lane.  A row is
// cut into chunks of P loads per lane (one chunk when the row fits); the loads of the next
// chunk are issued into a second set of registers before the current chunk is multiplied,
// so a wavefront always has one to two chunks outstanding.  The steady-state step has no
// lane-dependent branch -- columns past the end of a row are re-read from its last 16
// bytes and dropped by a select -- which lets the compiler wait for exactly the older
// chunk.  x sits in LDS, laid out in planes of 64 x 16 bytes so that the lanes of a
// wavefront read consecutive 16-byte pieces.  The sum runs over this lane's elements in
// column order, then across lanes in a fixed butterfly: bit-repeatable.
// ---------------------------------------------------------------------------------------
constexpr int kRowdotWaves = 4;

template <typename WT, int P, bool SINGLE>
__global__ __launch_bounds__(kRowdotWaves * 64) void rowdot_kernel(RowdotParams p, int rows_per_wg, int nchunks) {
    extern __shared__ __align__(16) float xs[];
    constexpr int EPL = Elem<WT>::kPerLoad;
    constexpr int PLANES = EPL / 4;          // 16-byte pieces of x per weight load
    constexpr int STEP = 64 * EPL;
    constexpr int CHUNK = P * STEP;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t_begin = blockIdx.x * rows_per_wg;
    const int t_end = min(p.k, t_begin + rows_per_wg);

    // element j of x: load group g = j / EPL (one lane's 16 bytes of weights), piece h of it
    for (int j = tid * 4; j < p.n_cols; j += kRowdotWaves * 64 * 4) {
        const int g = j / EPL, h = (j % EPL) / 4;
        *reinterpret_cast<float4*>(xs + ((g >> 6) * PLANES + h) * 256 + (g & 63) * 4) =
            *reinterpret_cast<const float4*>(p.x + j);
    }
    __syncthreads();

    // This wavefront's rows: list positions t0, t0 + 4, ... (at most 64 of them: lane i holds
    // the index and the partial activation of the i-th, fetched once, handed out with
    // readlane so that everything that steers the loop sits in scalar registers).
    // A unit is one chunk of one row.
    const int t0 = t_begin + wave;
    if (t0 >= t_end) return;
    const int n_rows_w = (t_end - t0 + kRowdotWaves - 1) / kRowdotWaves;
    const int n_units = SINGLE ? n_rows_w : n_rows_w * nchunks;
    const int last_col = p.n_cols - EPL;
    int my_r = 0;
    float my_av = 0.f;
    bool my_ok = false;
    if (lane < n_rows_w) {
        my_r = p.idx[t0 + kRowdotWaves * lane];
        my_ok = (unsigned)my_r < (unsigned)p.n_rows;   // a row outside the matrix contributes nothing
        if (!my_ok) my_r = 0;
        if (p.a) my_av = p.a[my_r];
    }
    const uint64_t ok_rows = __ballot(my_ok);

    struct Buf {
        u32x4 q[P];
        uint16_t sc[P];
    };
    auto issue = [&](int u, Buf& b) {
        const int i = SINGLE ? u : u / nchunks;
        const int c0 = SINGLE ? 0 : (u - i * nchunks) * CHUNK;
        const int r = __builtin_amdgcn_readlane(my_r, i);
        const char* row = static_cast<const char*>(p.w) + (size_t)r * (size_t)p.row_stride;
#pragma unroll
        for (int v = 0; v < P; ++v) {
            const int c = min(c0 + v * STEP + lane * EPL, last_col);
            b.q[v] = load16(row + (size_t)c * Elem<WT>::kBits / 8);
            b.sc[v] = 0;
            if constexpr (Elem<WT>::kScaled) b.sc[v] = p.scales[(size_t)r * p.scale_stride + (c >> 7)];
        }
    };
    float dot = 0.f;
    auto consume = [&](int u, const Buf& b) {
        const int i = SINGLE ? u : u / nchunks;
        const int cc = SINGLE ? 0 : u - i * nchunks;
        const int c0 = cc * CHUNK;
        float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int v = 0; v < P; ++v) {
            const int craw = c0 + v * STEP + lane * EPL;
            const int c = min(craw, last_col);
            const int g = c / EPL;
            const float* xp = xs + (g >> 6) * (PLANES * 256) + (g & 63) * 4;
            float f[EPL];
            Elem<WT>::widen(b.q[v], f);
            float part[4] = {0.f, 0.f, 0.f, 0.f}, xsum = 0.f;
#pragma unroll
            for (int h = 0; h < PLANES; ++h) {
                const float4 xv = *reinterpret_cast<const float4*>(xp + h * 256);
                part[0] = fmaf(f[4 * h], xv.x, part[0]);
                part[1] = fmaf(f[4 * h + 1], xv.y, part[1]);
                part[2] = fmaf(f[4 * h + 2], xv.z, part[2]);
                part[3] = fmaf(f[4 * h + 3], xv.w, part[3]);
                if constexpr (Elem<WT>::kScaled) xsum += (xv.x + xv.y) + (xv.z + xv.w);
            }
            const bool live = craw < p.n_cols;
            if constexpr (Elem<WT>::kScaled) {
                // codes arrive offset by 8 (see Elem<q4_t>)
                const float sv = half_bits_to_float(b.sc[v]);
                const float val = ((part[0] + part[1]) + (part[2] + part[3])) - 8.0f * xsum;
                acc[v & 3] += live ? sv * val : 0.f;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[e] += live ? part[e] : 0.f;
            }
        }
        dot += (acc[0] + acc[1]) + (acc[2] + acc[3]);
        if (!SINGLE && cc != nchunks - 1) return;
        // the last chunk of row i has been added
        float total = dot;
        dot = 0.f;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) total += __shfl_xor(total, off);
        const float av = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(my_av), i));
        float o = total;
        if (p.mode == 1) o = total * av;
        if (p.mode == 2) o = av * silu(total);
        if (!((ok_rows >> i) & 1ull)) o = 0.f;
        if (lane == 0) p.out[t0 + kRowdotWaves * i] = o;
    };

    Buf A, B;
    issue(0, A);
    int u = 0;
    while (true) {
        if (u + 1 == n_units) { consume(u, A); break; }
        issue(u + 1, B);
        consume(u, A);
        ++u;
        if (u + 1 == n_units) { consume(u, B); break; }
        issue(u + 1, A);
        consume(u, B);
        ++u;
    }
}

template <typename WT, int P, bool SINGLE>
hipError_t launch_rowdot_p(const RowdotParams& p, int nchunks, hipStream_t stream, int pk) {
    // one resident generation of workgroups (two per compute unit), whole rows per wavefront
    int rows_per_wg = (p.k + 511) / 512;
    rows_per_wg = (rows_per_wg + kRowdotWaves - 1) / kRowdotWaves * kRowdotWaves;
    if (rows_per_wg > 64 * kRowdotWaves) rows_per_wg = 64 * kRowdotWaves;   // one row per lane of a wavefront at most
    const int grid = (p.k + rows_per_wg - 1) / rows_per_wg;
    constexpr int STEP = 64 * Elem<WT>::kPerLoad;
    const size_t lds = sizeof(float) * (size_t)((p.n_cols + STEP - 1) / STEP) * STEP;
    auto kernel = rowdot_kernel<WT, P, SINGLE>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    hipEvent_t e0, e1;
    if (pk >= 0 && prof_next(pk, &e0, &e1)) {
        hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(kRowdotWaves * 64), lds, stream, e0, e1, 0, p,
                              rows_per_wg, nchunks);
    } else {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kRowdotWaves * 64), lds, stream, p, rows_per_wg, nchunks);
    }
    return hipGetLastError();
}

template <typename WT>
hipError_t launch_rowdot_t(const RowdotParams& p, hipStream_t stream, int pk) {
    const int step = 64 * Elem<WT>::kPerLoad;
    const int passes = (p.n_cols + step - 1) / step;
    // whole row in flight, twice (x then stays in registers) ...
    if (passes <= 2) return launch_rowdot_p<WT, 2, true>(p, 1, stream, pk);
    if (passes <= 4) return launch_rowdot_p<WT, 4, true>(p, 1, stream, pk);
    if (passes <= 6) return launch_rowdot_p<WT, 6, true>(p, 1, stream, pk);
    if (passes <= 8) return launch_rowdot_p<WT, 8, true>(p, 1, stream, pk);
    // ... or in two or more chunks when that would not fit the register file
    if (passes <= 10) return launch_rowdot_p<WT, 5, false>(p, 2, stream, pk);
    if (passes <= 12) return launch_rowdot_p<WT, 6, false>(p, 2, stream, pk);
    return launch_rowdot_p<WT, 8, false>(p, (passes + 7) / 8, stream, pk);
}

template <typename WT, int LPR, int WAVES, int UNROLL>
hipError_t launch_nseg(const GemvParams& p, const GemvShape& s, hipStream_t stream, int pk) {
    constexpr int SC = LPR * Elem<WT>::kPerLoad;
    const int strips = (p.n_out + SC - 1) / SC;
    dim3 grid(strips, s.ksplit), block(WAVES * 64);
    if (p.nseg == 2) {
        if constexpr (2 * SC <= WAVES * 64) {
            return launch_timed(gemv_kernel<WT, LPR, WAVES, UNROLL, 2>, grid, block, stream, pk, p);
        } else {
            return hipErrorInvalidConfiguration;
        }
    } else {
        if constexpr (SC <= WAVES * 64) {
            return launch_timed(gemv_kernel<WT, LPR, WAVES, UNROLL, 1>, grid, block, stream, pk, p);
        } else {
            return hipErrorInvalidConfiguration;
        }
    }
}

template <typename WT, int LPR, int WAVES>
hipError_t launch_unroll(const GemvParams& p, const GemvShape& s, hipStream_t stream, int pk) {
    switch (s.unroll) {
        case 1: return launch_nseg<WT, LPR, WAVES, 1>(p, s, stream, pk);
        case 2: return launch_nseg<WT, LPR, WAVES, 2>(p, s, stream, pk);
        case 4: return launch_nseg<WT, LPR, WAVES, 4>(p, s, stream, pk);
        case 8: return launch_nseg<WT, LPR, WAVES, 8>(p, s, stream, pk);
    }
    return hipErrorInvalidConfiguration;
}

template <typename WT, int LPR>
hipError_t launch_waves(const GemvParams& p, const GemvShape& s, hipStream_t stream, int pk) {
    switch (s.waves) {
        case 2: return launch_unroll<WT, LPR, 2>(p, s, stream, pk);
        case 4: return launch_unroll<WT, LPR, 4>(p, s, stream, pk);
        case 8: return launch_unroll<WT, LPR, 8>(p, s, stream, pk);
        case 16: return launch_unroll<WT, LPR, 16>(p, s, stream, pk);
    }
    return hipErrorInvalidConfiguration;
}

template <typename WT>
hipError_t launch_lpr(const GemvParams& p, const GemvShape& s, hipStream_t stream, int pk) {
    switch (s.lpr) {
        case 8: return launch_waves<WT, 8>(p, s, stream, pk);
        case 16: return launch_waves<WT, 16>(p, s, stream, pk);
        case 32: return launch_waves<WT, 32>(p, s, stream, pk);
        case 64: return launch_waves<WT, 64>(p, s, stream, pk);
    }
    return hipErrorInvalidConfiguration;
}

}  // namespace

static int elems_per_load(int dtype) { return dtype == DIP_F32 ? 4 : (dtype == DIP_BF16 ? 8 : 16); }

int gemv_strips(const GemvShape& s, int dtype, int n_out) {
    const int epl = elems_per_load(dtype);
    const int sc = s.lpr * epl;
    return (n_out + sc - 1) / sc;
}

GemvShape choose_gemv_shape(int dtype, int n_out, int nseg, int k) {
    // Defaults from launch-shape sweeps and same-box comparisons on MI355X (Phi-3-Mini,
    // Llama-3-8B and Phi-3-Medium shaped layers): 8 wavefronts, 4 rows in flight per lane
    // group, 16 lanes per row (32 for the bundled up/gate matrix when that gives whole
    // rounds), and row shares of a few hundred rows -- long enough to amortise a workgroup's
    // prologue and reduction, short enough to fill 256 compute units.
    GemvShape s;
    const bool q4 = dtype == DIP_INT4_G128;
    const int epl = elems_per_load(dtype);
    s.lpr = g_gemv_override.lpr ? g_gemv_override.lpr : 16;
    s.waves = g_gemv_override.waves ? g_gemv_override.waves : 8;
    s.unroll = g_gemv_override.unroll ? g_gemv_override.unroll : 4;
    int ks = 0;
    // Whole rounds of workgroups: with strips * ksplit just below one or two times the 256
    // compute units no unit is left with an extra workgroup while the others idle (280
    // workgroups take as long as 512).  Take the fewest rounds whose row shares fall into
    // the given range.
    auto whole_rounds = [&](int lpr, int min_share, int max_share) {
        const int strips = (n_out + lpr * epl - 1) / (lpr * epl);
        for (int m = 1; m <= 2; ++m) {
            const int cand = kComputeUnits * m / strips;
            if (cand < 1) continue;
            const int share = (k + cand - 1) / cand;
            if (share >= min_share && share <= max_share) return cand;
        }
        return 0;
    };
    if (!g_gemv_override.lpr && !g_gemv_override.ksplit) {
        if (q4) {
            // 4-bit rows are a quarter of the bytes while a workgroup's fixed costs (prologue,
            // 32 or 64 accumulators through the cross-lane reduction, the ticket protocol) are
            // the same: longer shares
            ks = whole_rounds(16, 256, 640);
        } else if (nseg == 2) {
            // bundled up/gate: the widest strip whose shares come out between 200 and 400 rows
            const int lprs[2] = {32, 16};
            for (int li = 0; li < 2 && !ks; ++li) {
                ks = whole_rounds(lprs[li], 200, 400);
                if (ks) s.lpr = lprs[li];
            }
        } else {
            // single matrix (down): whole rounds when the shares come out at 420-700 rows
            ks = whole_rounds(16, 420, 700);
        }
    }
    // a bundled strip needs 2*SC lanes for its epilogue
    while (nseg * s.lpr * epl > s.waves * 64 && s.waves < 16) s.waves *= 2;
    if (g_gemv_override.ksplit) {
        s.ksplit = g_gemv_override.ksplit;
    } else {
        if (!ks) {
            const int strips = gemv_strips(s, dtype, n_out);
            // (int4 rows are a quarter of the bytes and the reduction costs the same: longer shares)
            const int rows_per_wg = q4 ? (nseg == 2 ? 768 : 640) : (nseg == 2 ? 384 : 512);
            ks = (k + rows_per_wg / 2) / rows_per_wg;
            if (ks < 1) ks = 1;
            const int min_wgs = q4 ? 128 : 192;
            if (strips * ks < min_wgs) ks = (min_wgs + strips - 1) / strips;
        }
        // but keep at least one full iteration of rows per workgroup
        const int rows_per_iter = s.waves * (64 / s.lpr) * s.unroll;
        while (ks > 1 && k / ks < rows_per_iter) --ks;
        s.ksplit = ks;
    }
    if (s.ksplit > k) s.ksplit = k;
    if (s.ksplit < 1) s.ksplit = 1;
    return s;
}

int g_fusion = 1;

// Launch shape of a product that runs its own selection: 16 wavefronts per workgroup, one
// workgroup per compute unit (every workgroup repeats the selection, so a second round would
// pay it twice), hence strips * ksplit as close to the 256 compute units as the strip widths
// allow, every share at least one full iteration of rows and at most the LDS list.
bool fused_shape(int dtype, int n_sel, int n_out, int nseg, int k, GemvShape* shape) {
    if (!g_fusion) return false;
    if (n_sel > DIP_MAX_N || (nseg == 2 && n_sel > kFusedMaxIn)) return false;
    const int epl = elems_per_load(dtype);
    GemvShape best = {0, 16, 0, 4};
    int best_wgs = 0;
    // Same-box comparisons: 512-byte pieces (32 lanes per row) do as well as 1024-byte ones with
    // fewer partial sums; 4-bit rows, a quarter of the bytes, do best with the narrowest strip
    // (longest shares).  The first width that fills 200 of the 256 compute units is taken.
    const bool q4 = dtype == DIP_INT4_G128;
    const int lprs[3] = {q4 ? 16 : 32, q4 ? 32 : 64, q4 ? 64 : 16};
    for (int li = 0; li < 3 && best_wgs < 200; ++li) {
        const int lpr = lprs[li];
        if (g_gemv_override.lpr && g_gemv_override.lpr != lpr) continue;
        if (nseg * lpr * epl > kSelThreads) continue;        // a strip's outputs, one lane each
        const int strips = (n_out + lpr * epl - 1) / (lpr * epl);
        const int rows_per_iter = 4 * 16 * (64 / lpr);
        int ks = kComputeUnits / strips;
        if (ks > k / rows_per_iter) ks = k / rows_per_iter;
        if (ks < 1) ks = 1;
        if (g_gemv_override.ksplit) ks = g_gemv_override.ksplit;
        if (ks > k) ks = k;
        const int share = ((k + ks - 1) / ks + 7) / 8 * 8;
        if (share > kFusedListCap) continue;
        int wgs = strips * ks;
        if (wgs > kComputeUnits) wgs = kComputeUnits - 1;    // more than one round: last choice
        if (wgs > best_wgs) {
            best_wgs = wgs;
            best.lpr = lpr;
            best.ksplit = ks;
        }
    }
    if (!best_wgs) return false;
    *shape = best;
    return true;
}

hipError_t launch_fused(const FusedParams& p0, const GemvShape& s, hipStream_t stream, int pk) {
    FusedParams p = p0;
    p.g.epoch = next_epoch();
    p.g.rows_per_split = ((p.g.k + s.ksplit - 1) / s.ksplit + 7) / 8 * 8;
    if (p.g.rows_per_split > kFusedListCap || s.waves != 16 || s.unroll != 4) return hipErrorInvalidConfiguration;
    if (p.s.n < 1 || p.s.n > DIP_MAX_N || p.g.k < 1 || p.g.k > p.s.n || p.s.n != p.g.n_in) return hipErrorInvalidValue;
    p.g.idx = nullptr;
    p.g.val = nullptr;
    p.g.w_alt = nullptr;
    p.g.n_alt = 0;
    if (p.g.nseg == 2) {
        if (p.g.dtype == DIP_F32) return launch_fused_2_0(p, s, stream, pk);
        if (p.g.dtype == DIP_BF16) return launch_fused_2_1(p, s, stream, pk);
        if (p.g.dtype == DIP_INT4_G128) return launch_fused_2_2(p, s, stream, pk);
    } else {
        if (p.g.dtype == DIP_F32) return launch_fused_1_0(p, s, stream, pk);
        if (p.g.dtype == DIP_BF16) return launch_fused_1_1(p, s, stream, pk);
        if (p.g.dtype == DIP_INT4_G128) return launch_fused_1_2(p, s, stream, pk);
    }
    return hipErrorInvalidValue;
}

// The tags start at a point that differs from process to process (time and process, mixed by the
// finaliser of splitmix64), so that words left in memory by another one do not match either.
uint64_t next_epoch() {
    static std::atomic<uint64_t> next{[] {
        struct timespec t = {0, 0};
        clock_gettime(CLOCK_REALTIME, &t);
        uint64_t z = (uint64_t)t.tv_sec * 1000000000ull + (uint64_t)t.tv_nsec + ((uint64_t)getpid() << 40);
        z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
        z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
        return z ^ (z >> 31);
    }()};
    return next.fetch_add(1, std::memory_order_relaxed) << 16;
}

hipError_t launch_gemv(const GemvParams& p0, const GemvShape& s, hipStream_t stream, int pk) {
    GemvParams p = p0;
    if (!p.epoch) p.epoch = next_epoch();
    p.rows_per_split = ((p.k + s.ksplit - 1) / s.ksplit + 7) / 8 * 8;   // keeps vector index loads aligned
    if (p.dtype == DIP_F32) return launch_lpr<float>(p, s, stream, pk);
    if (p.dtype == DIP_BF16) return launch_lpr<uint16_t>(p, s, stream, pk);
    if (p.dtype == DIP_INT4_G128) return launch_lpr<q4n_t>(p, s, stream, pk);
    return hipErrorInvalidValue;
}

bool gather_in_gemv(const GemvShape& s, int k) {
    return s.lpr == kGatherLpr && s.waves == kGatherWaves && s.unroll == kGatherUnroll &&
           ((k + s.ksplit - 1) / s.ksplit + 7) / 8 * 8 <= kGatherCap;
}

hipError_t launch_gemv_gather(const GemvParams& p0, const float* x, const GemvShape& s, hipStream_t stream, int pk) {
    if (!gather_in_gemv(s, p0.k) || p0.nseg != 1 || p0.w_alt) return hipErrorInvalidValue;
    GemvParams p = p0;
    p.epoch = next_epoch();
    p.rows_per_split = ((p.k + s.ksplit - 1) / s.ksplit + 7) / 8 * 8;
    const dim3 grid(gemv_strips(s, p.dtype, p.n_out), s.ksplit), block(kGatherWaves * 64);
    auto go = [&](auto kernel) {
        hipEvent_t e0, e1;
        if (pk >= 0 && prof_next(pk, &e0, &e1)) hipExtLaunchKernelGGL(kernel, grid, block, 0, stream, e0, e1, 0, p, x);
        else hipLaunchKernelGGL(kernel, grid, block, 0, stream, p, x);
        return hipGetLastError();
    };
    if (p.dtype == DIP_F32) return go(gemv_gather_kernel<float>);
    if (p.dtype == DIP_BF16) return go(gemv_gather_kernel<uint16_t>);
    if (p.dtype == DIP_INT4_G128) return go(gemv_gather_kernel<q4n_t>);
    return hipErrorInvalidValue;
}

__global__ void gather_kernel(const float* x, const int32_t* idx, int k, int n, float* val, int32_t* idx_copy) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= k) return;
    const int r = idx[t];
    idx_copy[t] = r;
    val[t] = (unsigned)r < (unsigned)n ? x[r] : 0.f;
}

hipError_t launch_gather(const float* x, const int32_t* idx, int k, int n, float* val, int32_t* idx_copy,
                         hipStream_t stream) {
    hipLaunchKernelGGL(gather_kernel, dim3((k + 255) / 256), dim3(256), 0, stream, x, idx, k, n, val, idx_copy);
    return hipGetLastError();
}

// A plain streaming read of `bytes` bytes (whole 16-byte pieces), for benchmarks: what the
// memory system delivers to a kernel that does nothing but load, in the same run and on the
// same box as the gathered products it is compared with.
__global__ __launch_bounds__(256) void stream_read_kernel(const u32x4* src, size_t n16, uint32_t* sink) {
    const size_t stride = (size_t)gridDim.x * 256;
    size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    u32x4 acc = {0u, 0u, 0u, 0u};
    for (; i + 7 * stride < n16; i += 8 * stride) {
        u32x4 q[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) q[u] = __builtin_nontemporal_load(src + i + u * stride);
#pragma unroll
        for (int u = 0; u < 8; ++u) acc ^= q[u];
    }
    for (; i < n16; i += stride) acc ^= __builtin_nontemporal_load(src + i);
    // (never true for the buffers benchmarks use; keeps the loads alive)
    if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9e3779b9u) sink[0] = acc.x;
}

hipError_t launch_stream_read(const void* src, size_t bytes, uint32_t* sink, hipStream_t stream, int prof_kind) {
    const size_t n16 = bytes / 16;
    struct Args { const u32x4* src; size_t n16; uint32_t* sink; };
    hipEvent_t e0, e1;
    const dim3 grid(kComputeUnits * 16), block(256);
    if (prof_kind >= 0 && prof_next(prof_kind, &e0, &e1)) {
        hipExtLaunchKernelGGL(stream_read_kernel, grid, block, 0, stream, e0, e1, 0,
                              static_cast<const u32x4*>(src), n16, sink);
    } else {
        hipLaunchKernelGGL(stream_read_kernel, grid, block, 0, stream, static_cast<const u32x4*>(src), n16, sink);
    }
    return hipGetLastError();
}

hipError_t launch_rowdot(const RowdotParams& p, hipStream_t stream, int prof_kind) {
    if (p.k <= 0) return hipSuccess;
    if (p.dtype == DIP_F32) return launch_rowdot_t<float>(p, stream, prof_kind);
    if (p.dtype == DIP_BF16) return launch_rowdot_t<uint16_t>(p, stream, prof_kind);
    if (p.dtype == DIP_INT4_G128) return launch_rowdot_t<q4_t>(p, stream, prof_kind);
    return hipErrorInvalidValue;
}

}  // namespace dip
