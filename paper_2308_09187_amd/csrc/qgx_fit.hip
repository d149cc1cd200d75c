// Adaptive levels (Section 3.3): the weighted empirical CDF of eq. (QAda) as a histogram of the
// normalised coordinates, and the one-level-at-a-time solver on it.
//
// Histogram: persistent workgroups walk the (worker, bucket) pairs with a fixed stride; per bucket the
// data is read once into registers (same row layout as the encoder), the norm is reduced, every
// coordinate bumps an integer LDS counter of its bin, and the counters are folded into per-workgroup
// binary64 sums weighted by the squared norm.  Workgroup sums go to scratch and are added in a fixed
// order, so the histogram is reproducible bit for bit.
//
// Bins follow the binary32 grid: 64 equal-width bins per octave over n_bins/64 octaves below 1 (bin 0
// also takes everything smaller, u = 1 goes to the last bin), so the bin of u is an integer function
// of its bits and the resolution follows the heavy concentration of u near zero.
#include "qgx_device.h"

namespace qgx {

__device__ __forceinline__ uint32_t bin_of(float u, uint32_t n_bins)
{
    const int key = (int)(__float_as_uint(u) >> 17) - (127 * 64 - (int)n_bins);
    return (uint32_t)min(max(key, 0), (int)n_bins - 1);
}

__device__ __forceinline__ double bin_edge(uint32_t b, uint32_t n_bins)
{
    if (b == 0) return 0.0;
    if (b >= n_bins) return 1.0;
    return (double)__uint_as_float((uint32_t)((int)b + (127 * 64 - (int)n_bins)) << 17);
}

// A workgroup walks its buckets one after the other, each in two phases divided by barriers: norm, then count and fold (a
// wave that has folded a bucket's counters meets the others again before anyone counts the next).  A compute unit holds one
// workgroup of sixteen waves (registers) or three of four (LDS), so nothing but the workgroup itself hides a phase's latency:
// a row's registers are free once it is counted, and the next bucket's row is asked for there and then.
// 16 x 2^26 coordinates in buckets of 65536 take 0.64 ms (6.7 TB/s; 0.85 with the loads at a bucket's start), 8 x 2^24 in
// buckets of 16384 0.123 (0.151 with a second set of registers for the next bucket's rows, two workgroups to a unit).
// The barriers between the rows are for the scheduler, which else forms all rows' bins first and spills.
template <int MAXW>
__global__ __launch_bounds__(MAXW * kWave) void k_histogram(Layout lay, const float* __restrict__ V, int norm_kind,
                                                            uint32_t n_bins, double* __restrict__ partial, Scalars* sc)
{
    extern __shared__ __align__(16) unsigned char s_raw[];
    double* s_acc = reinterpret_cast<double*>(s_raw);                    // [n_bins]
    uint32_t* s_cnt = reinterpret_cast<uint32_t*>(s_acc + n_bins);       // [n_bins]
    __shared__ double s_red[kMaxWaves];

    const int tid = (int)threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(wave_id());
    const int nwaves = (int)(blockDim.x >> 6);
    for (uint32_t i = (uint32_t)tid; i < n_bins; i += blockDim.x) { s_acc[i] = 0.0; s_cnt[i] = 0; }

    const uint32_t n_work = lay.K * lay.NB;
    // this wave's chunk of unit t (bucket t / K of worker t % K); none past the bucket's end or the last unit
    struct Piece { const float* first; uint32_t len; };
    auto piece_of = [&](uint32_t t) {
        if (t >= n_work) return Piece{V, 0u};
        const uint32_t b = t / lay.K, k = t - b * lay.K;
        const uint32_t lo = scalar_load(lay.bucket_start + b), hi = scalar_load(lay.bucket_start + b + 1);
        const uint32_t clo = lo + (uint32_t)w * kChunk;
        const uint32_t left = clo < hi ? hi - clo : 0u;
        return Piece{V + (size_t)k * lay.d + clo, left < (uint32_t)kChunk ? left : (uint32_t)kChunk};
    };
    float4 v[kRows];
    Piece cur = piece_of(blockIdx.x);
    load_rows(v, chunk_rows(cur.first, cur.len), lane);
    for (uint32_t t = blockIdx.x; t < n_work; t += gridDim.x) {
        const Piece next = piece_of(t + gridDim.x);
        const __amdgpu_buffer_rsrc_t next_rows = chunk_rows(next.first, next.len);
        load_rest(v, cur.first, cur.len, lane);
        // a non-finite coordinate shows in the sum of squares (which no finite ones overflow) and in the maximum
        double red;
        if (norm_kind == QGX_NORM_L2) {
            double acc = 0.0;
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                acc = fma((double)v[r].x, (double)v[r].x, acc);
                acc = fma((double)v[r].y, (double)v[r].y, acc);
                acc = fma((double)v[r].z, (double)v[r].z, acc);
                acc = fma((double)v[r].w, (double)v[r].w, acc);
                __builtin_amdgcn_sched_barrier(0);
            }
            red = wave_sum(acc);
        } else {
            float mx = 0.0f;
#pragma unroll
            for (int r = 0; r < kRows; ++r) mx = largest_of(v[r], mx);
            red = (double)__uint_as_float(wave_max_u32(__float_as_uint(mx)));
        }
        if (lane == 0) s_red[w] = red;
        __syncthreads();
        double tot = 0.0;
        bool finite = true;
        for (int i = 0; i < nwaves; ++i) {
            if (norm_kind == QGX_NORM_L2) tot += s_red[i];
            else tot = fmax(tot, s_red[i]);
            finite = finite && fabs(s_red[i]) <= 1.7976931348623157e308;
        }
        float n = (norm_kind == QGX_NORM_L2) ? (float)sqrt(tot) : (float)tot;
        if (norm_kind != QGX_NORM_L2 && norm_kind != QGX_NORM_LINF && finite && tot > 0.0) {
            // general q: (sum |v_i|^q)^(1/q) relative to the largest magnitude, as in the encoder
            const double inv_m = 1.0 / tot;
            double sum = 0.0;
#pragma unroll 1
            for (uint32_t i = (uint32_t)lane; i < cur.len; i += kWave)                   // rolled, from memory
                sum += pow_int(fabs((double)cur.first[i]) * inv_m, (uint32_t)norm_kind);
            sum = wave_sum(sum);
            __syncthreads();                         // everyone has read the first set of partial results
            if (lane == 0) s_red[w] = sum;
            __syncthreads();
            double all = 0.0;
            for (int i = 0; i < nwaves; ++i) all += s_red[i];
            n = (float)(tot * root_int(all, (uint32_t)norm_kind));
        }
        const bool usable = finite && (n > 0.0f) && (n <= 3.402823466e+38f);
        if (!finite && tid == 0) raise_error(sc, QGX_EBIT_NONFINITE);
        const float rinv = usable ? 1.0f / n : 0.0f;
        const uint32_t len = usable ? cur.len : 0u;
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const float e[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
            // (u above 1, by a rounding, ends in the last bin with the clamp of the bin number alone)
            if ((uint32_t)r * 256u + 256u <= len) {
#pragma unroll
                for (int q = 0; q < 4; ++q) atomicAdd(&s_cnt[bin_of(fabsf(e[q]) * rinv, n_bins)], 1u);
            } else if ((uint32_t)r * 256u < len) {               // the short last row
                const uint32_t i0 = (uint32_t)r * 256u + (uint32_t)lane * 4u;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (i0 + (uint32_t)q < len) atomicAdd(&s_cnt[bin_of(fabsf(e[q]) * rinv, n_bins)], 1u);
            }
            v[r] = load_row(next_rows, r, lane);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
        if (usable) {
            const double wgt = (double)n * (double)n;           // lambda of Section 3.3, unnormalised
            for (uint32_t i = (uint32_t)tid; i < n_bins; i += blockDim.x) {
                const uint32_t cnt = s_cnt[i];
                if (cnt) { s_acc[i] += (double)cnt * wgt; s_cnt[i] = 0; }
            }
        }
        cur = next;
    }
    for (uint32_t i = (uint32_t)tid; i < n_bins; i += blockDim.x)        // (a thread's own bins)
        partial[(size_t)blockIdx.x * n_bins + i] = s_acc[i];
}

// Buckets of 256..2048 coordinates (one to eight rows of 256): a workgroup of one wave per bucket
// would leave the chip nearly empty and spend its time folding 4096 counters per bucket.  Here a
// workgroup is four waves with a bucket each.  A wave counts into 16-bit counters of its own (two to
// a word; a count is at most 2048), and the lane that takes a counter from zero remembers it: after
// the count exactly those lanes fold their counters into the workgroup's binary64 sums, weighted by
// the squared norm, and clear them, so a fold costs what the bucket touched, not the whole table.
// The waves fold one after the other, in wave order, so every sum still receives its terms in a
// fixed order and the histogram is reproducible bit for bit.
template <int RPB>
__global__ __launch_bounds__(256) void k_histogram_small(Layout lay, const float* __restrict__ V, int norm_kind,
                                                         uint32_t n_bins, double* __restrict__ partial, Scalars* sc)
{
    extern __shared__ __align__(16) unsigned char s_raw[];
    constexpr int kW = 4;
    const int tid = (int)threadIdx.x, lane = lane_id(), w = wave_id();
    double* s_acc = reinterpret_cast<double*>(s_raw);                                   // [n_bins]
    uint32_t* s_cnt = reinterpret_cast<uint32_t*>(s_acc + n_bins) + (size_t)w * (n_bins / 2);   // [n_bins / 2] per wave
    for (uint32_t i = (uint32_t)tid; i < n_bins; i += kW * kWave) s_acc[i] = 0.0;
    for (uint32_t i = (uint32_t)lane; i < n_bins / 2; i += kWave) s_cnt[i] = 0u;
    __syncthreads();

    const uint32_t n_work = lay.K * lay.NB;
    for (uint32_t t0 = (uint32_t)blockIdx.x * kW; t0 < n_work; t0 += gridDim.x * kW) {
        const uint32_t t = t0 + (uint32_t)w;
        const bool have = t < n_work;                     // wave-uniform
        const uint32_t b = have ? t / lay.K : 0u, k = have ? t - b * lay.K : 0u;
        const uint32_t lo = lay.bucket_start[b], hi = have ? lay.bucket_start[b + 1] : lo;
        const size_t kbase = (size_t)k * lay.d;
        const bool vec_ok = (kbase & 3u) == 0;
        const float* __restrict__ Vk = V + kbase;
        float4 v[RPB];
#pragma unroll
        for (int r = 0; r < RPB; ++r) {
            const uint32_t i0 = lo + (uint32_t)r * 256u + (uint32_t)lane * 4u;
            float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
            if (i0 + 4u <= hi) {
                if (vec_ok) x = nt_load4(Vk + i0);                // (read once)
                else x = make_float4(Vk[i0], Vk[i0 + 1], Vk[i0 + 2], Vk[i0 + 3]);
            } else if (i0 < hi) {
                x.x = Vk[i0];
                if (i0 + 1 < hi) x.y = Vk[i0 + 1];
                if (i0 + 2 < hi) x.z = Vk[i0 + 2];
            }
            v[r] = x;
        }
        // the norm, with the arithmetic of k_histogram for a bucket of one wave
        double acc = 0.0;
        float mx = 0.0f;
        uint32_t bad = 0;
#pragma unroll
        for (int r = 0; r < RPB; ++r) {
            const float e[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float ax = fabsf(e[q]);
                bad |= !(ax <= 3.402823466e+38f);
                if (norm_kind == QGX_NORM_L2) acc = fma((double)e[q], (double)e[q], acc);
                else mx = fmaxf(mx, ax);
            }
        }
        double tot = (norm_kind == QGX_NORM_L2) ? wave_sum(acc) : (double)wave_max(mx);
        bad = wave_or(bad);
        float n = (norm_kind == QGX_NORM_L2) ? (float)sqrt(tot) : (float)tot;
        if (norm_kind != QGX_NORM_L2 && norm_kind != QGX_NORM_LINF && bad == 0 && tot > 0.0) {
            const double inv_m = 1.0 / tot;
            double sum = 0.0;
#pragma unroll 1
            for (uint32_t i = lo + (uint32_t)lane; i < hi; i += kWave)
                sum += pow_int(fabs((double)Vk[i]) * inv_m, (uint32_t)norm_kind);
            n = (float)(tot * root_int(wave_sum(sum), (uint32_t)norm_kind));
        }
        const bool usable = have && (bad == 0) && (n > 0.0f) && (n <= 3.402823466e+38f);
        if (have && bad != 0 && lane == 0) raise_error(sc, QGX_EBIT_NONFINITE);

        uint32_t bins[4 * RPB];
        uint32_t mine = 0;                                // slots whose counter this lane took from zero
        if (usable) {
            const float rinv = 1.0f / n;
#pragma unroll
            for (int r = 0; r < RPB; ++r) {
                const uint32_t i0 = lo + (uint32_t)r * 256u + (uint32_t)lane * 4u;
                const float e[4] = {v[r].x, v[r].y, v[r].z, v[r].w};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    bins[4 * r + q] = 0;
                    if (i0 + (uint32_t)q < hi) {
                        const float u = fminf(fabsf(e[q]) * rinv, 1.0f);
                        const uint32_t bin = bin_of(u, n_bins), sh = (bin & 1u) * 16u;
                        bins[4 * r + q] = bin;
                        const uint32_t old = atomicAdd(&s_cnt[bin >> 1], 1u << sh);
                        if (((old >> sh) & 0xFFFFu) == 0u) mine |= 1u << (4 * r + q);
                    }
                }
            }
        }
        const double wgt = (double)n * (double)n;         // lambda of Section 3.3, unnormalised
        wave_lds_fence();                                 // the counts a lane folds hold other lanes' additions
        for (int turn = 0; turn < kW; ++turn) {
            if (turn == w && usable) {
#pragma unroll
                for (int s = 0; s < 4 * RPB; ++s) {
                    if (mine & (1u << s)) {
                        const uint32_t bin = bins[s], sh = (bin & 1u) * 16u;
                        const uint32_t cnt = (s_cnt[bin >> 1] >> sh) & 0xFFFFu;
                        s_acc[bin] += (double)cnt * wgt;
                        atomicAnd(&s_cnt[bin >> 1], ~(0xFFFFu << sh));
                    }
                }
            }
            __syncthreads();
        }
    }
    for (uint32_t i = (uint32_t)tid; i < n_bins; i += kW * kWave)
        partial[(size_t)blockIdx.x * n_bins + i] = s_acc[i];
}

// Workgroup sums -> histogram, in an order that does not depend on timing: the workgroups' values of a
// bin are cut into kRedSegs runs of consecutive workgroups, a thread adds one run, then the runs of a bin
// are added in order.  16 bins to a workgroup: 256 workgroups for the largest histogram, a row of 16 lanes
// reads 128 consecutive bytes of one workgroup's sums.
constexpr uint32_t kRedBins = 16;
constexpr uint32_t kRedSegs = 16;

__global__ __launch_bounds__(kRedBins * kRedSegs) void k_hist_reduce(uint32_t n_bins, uint32_t n_partial,
                                                                     const double* __restrict__ partial,
                                                                     double* __restrict__ hist, double* __restrict__ copy)
{
    __shared__ double s_run[kRedSegs][kRedBins];
    const uint32_t bl = threadIdx.x & (kRedBins - 1u), seg = threadIdx.x / kRedBins;
    const uint32_t i = blockIdx.x * kRedBins + bl;
    const uint32_t run = (n_partial + kRedSegs - 1u) / kRedSegs;
    const uint32_t lo = min(seg * run, n_partial), hi = min(lo + run, n_partial);
    double acc = 0.0;
    if (i < n_bins) {
        uint32_t g = lo;
        for (; g + 4u <= hi; g += 4u) {                   // four loads on their way, added in order
            const double v0 = partial[(size_t)g * n_bins + i], v1 = partial[(size_t)(g + 1u) * n_bins + i];
            const double v2 = partial[(size_t)(g + 2u) * n_bins + i], v3 = partial[(size_t)(g + 3u) * n_bins + i];
            acc += v0; acc += v1; acc += v2; acc += v3;
        }
        for (; g < hi; ++g) acc += partial[(size_t)g * n_bins + i];
    }
    s_run[seg][bl] = acc;
    __syncthreads();
    if (seg == 0 && i < n_bins) {
        double tot = 0.0;
        for (uint32_t q = 0; q < kRedSegs; ++q) tot += s_run[q][bl];
        hist[i] = tot;
        if (copy) copy[i] = tot;
    }
}

uint32_t histogram_groups(const Layout& lay)
{
    // as many as the compute units hold at once: three each (LDS with 4096 bins) of up to four waves, two of up to eight,
    // one of up to sixteen (registers); shared chunks: two
    const uint32_t n_work = lay.K * lay.NB;
    const uint32_t groups = lay.shared_chunks ? 512u : lay.waves_per_bucket <= 4u ? 768u : lay.waves_per_bucket <= 8u ? 512u : 256u;
    return n_work < groups ? n_work : groups;
}

hipError_t launch_histogram(const Layout& lay, const float* V, int norm_kind, uint32_t n_bins, double* partial,
                            uint32_t n_partial, double* hist, double* copy, Scalars* sc, hipStream_t st)
{
    if (lay.shared_chunks) {                              // buckets of 256 << s coordinates, s = 0..3
        const size_t lds = (size_t)n_bins * (sizeof(double) + 4 * sizeof(uint16_t));
        switch (lay.bucket_shift) {
            case 8: hipLaunchKernelGGL(k_histogram_small<1>, dim3(n_partial), dim3(256), lds, st, lay, V, norm_kind, n_bins, partial, sc); break;
            case 9: hipLaunchKernelGGL(k_histogram_small<2>, dim3(n_partial), dim3(256), lds, st, lay, V, norm_kind, n_bins, partial, sc); break;
            case 10: hipLaunchKernelGGL(k_histogram_small<4>, dim3(n_partial), dim3(256), lds, st, lay, V, norm_kind, n_bins, partial, sc); break;
            default: hipLaunchKernelGGL(k_histogram_small<8>, dim3(n_partial), dim3(256), lds, st, lay, V, norm_kind, n_bins, partial, sc); break;
        }
    } else {
        const size_t lds = (size_t)n_bins * (sizeof(double) + sizeof(uint32_t));
        if (lay.waves_per_bucket <= 4u)
            hipLaunchKernelGGL(k_histogram<4>, dim3(n_partial), dim3(lay.waves_per_bucket * kWave), lds, st, lay, V, norm_kind,
                               n_bins, partial, sc);
        else
            hipLaunchKernelGGL(k_histogram<kMaxWaves>, dim3(n_partial), dim3(lay.waves_per_bucket * kWave), lds, st, lay, V,
                               norm_kind, n_bins, partial, sc);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_hist_reduce, dim3((n_bins + kRedBins - 1u) / kRedBins), dim3(kRedBins * kRedSegs), 0, st, n_bins, n_partial,
                       partial, hist, copy);
    return hipGetLastError();
}

// ---- solver ---------------------------------------------------------------------------------------
// With F~ piecewise uniform inside bins, the stationarity condition of (QAda) in l_j = x between its
// neighbours a = l_{j-1}, c = l_{j+1},
//     G(x) = int_a^x (u - a) dF~ - int_x^c (c - u) dF~ = 0 ,
// has dG/dx = (c - a) * density(x), so G(x) = (c - a) * mass(a, x) - int_a^c (c - u) dF~: the level goes
// where the mass between a and x reaches  t = int_a^c (c - u) dF~ / (c - a).  Where that holds on a
// whole interval (no mass there) the smallest such x is taken; with no mass at all between the
// neighbours that is a.  Levels stay in binary64 between the sweeps and are rounded to the table's
// binary32 once, at the end.
//
// Everything is summed from a onwards, non-negative terms only (a difference of cumulative sums taken
// from 0 would lose a sliver of mass next to a level against the total).  Nodes of 64 bins keep that short: they hold
// their mass and their moment about their own right
// edge, rho = sum H_b (edge - mid_b), so that int (c - u) dF~ over a node is (c - edge) * mass + rho.
// The whole bins between a and c are then at most 63 bins up to a multiple of 64, at most 64 nodes, and at most 63 bins.
// One update is the work of a wave, a lane per item of each of the three runs: the integral is one sum across the wave, and
// the place where the mass reaches t is found with a prefix sum across it per run, then inside the node that holds it.
// Updates depend on each other, so a step's latency is all that counts: what is the same in all lanes is kept in scalar
// registers (branches, the place found), sums and broadcasts stay in vector registers, and divisions by the width of a bin,
// a power of two, are exact multiplications.  (A row of 16 lanes per update over a tree of nodes of 16 and 256 bins, four
// updates to a wave whose lanes went through each other's branches: a fit of 2^17 coordinates with 33 levels and 10 sweeps 116 us, now
// 99; 17 levels 89, now 71; 65 levels 159, now 126; 127 levels 226, now 218.  Without a form of its own for short intervals
// 127 levels took 250.)

// In LDS, one array of doubles: the bins' masses, then the nodes' masses, then their moments.
constexpr uint32_t kNodes = QGX_MAX_BINS / kWave;
constexpr uint32_t kTreeDoubles = 2u * kNodes;      // beside the bins
struct Tree {
    const double* H;      // [n_bins], [kNodes], [kNodes]
    uint32_t n_bins;
};

// The bin whose half-open interval [edge, next edge) holds x >= 0: the bins are 64 to an octave, so the bin
// number is the exponent and the top six fraction bits, which a binary64 number shows as its bits 46 and up.
__device__ __forceinline__ uint32_t bin_containing(uint32_t n_bins, double x)
{
    const int key = (int)((unsigned long long)__double_as_longlong(x) >> 46) - (1023 * 64 - (int)n_bins);
    return (uint32_t)min(max(key, 0), (int)n_bins - 1);
}

// y / (width of bin b), exactly: a power of two but for the first bin, which goes down to zero.
__device__ __forceinline__ double by_bin_width(double y, uint32_t b, uint32_t n_bins)
{
    if (b == 0u) return y / bin_edge(1u, n_bins);
    const int octave = (int)((b + (127u * 64u - n_bins)) >> 6) - 127;          // the bin lies in [2^octave, 2^(octave + 1))
    return __builtin_amdgcn_ldexp(y, 6 - octave);
}

// inclusive prefix sum over the lanes of the wave, as wave_incl_scan
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or_zero(double x)
{
    if constexpr (ROWS == 0xf)       // (lanes without a source read 0)
        return __hiloint2double(__builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true),
                                __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true));
    else
        return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, ROWS, 0xf, false),
                                __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ double wave_prefix(double x)
{
    x += dpp_or_zero<0x111, 0xf>(x);
    x += dpp_or_zero<0x112, 0xf>(x);
    x += dpp_or_zero<0x114, 0xf>(x);
    x += dpp_or_zero<0x118, 0xf>(x);
    x += dpp_or_zero<0x142, 0xa>(x);
    x += dpp_or_zero<0x143, 0xc>(x);
    return x;
}

__device__ __forceinline__ double lane_value(double x, uint32_t lane)           // (lane the same in all lanes)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), (int)lane), __builtin_amdgcn_readlane(__double2loint(x), (int)lane));
}

__device__ __forceinline__ bool same_in_all(bool b) { return __builtin_amdgcn_ballot_w64(b) != 0ull; }
__device__ __forceinline__ uint32_t same_in_all(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }

// Right edge of the last bin with mass in [first, last_plus_1), or `fallback` if none has any.
__device__ double last_mass_edge(const Tree& T, uint32_t first, uint32_t last_plus_1, double fallback)
{
    for (uint32_t b = last_plus_1; b > first; --b)
        if (T.H[b - 1u] > 0.0) return bin_edge(b, T.n_bins);
    return fallback;
}

// The middle of bin b > 0: a binary32 number as its edges are.
__device__ __forceinline__ double bin_middle(uint32_t b, uint32_t n_bins)
{
    return (double)__uint_as_float(((b + (127u * 64u - n_bins)) << 17) | 0x10000u);
}

// The level between its neighbours a < c, which lie in bins ba and bc.  SHORT: all the whole bins between them are in the first run.
template <bool SHORT>
__device__ __forceinline__ double stationary_between(const Tree& T, double a, double c, uint32_t ba, uint32_t bc)
{
    const uint32_t nb = T.n_bins, lane = (uint32_t)lane_id();
    // the whole bins P .. Q - 1 between those that hold a and c: bins [P, P1), nodes [p1, q1), bins [Q1, Q)
    const uint32_t P = ba + 1u, Q = bc > P ? bc : P;
    const uint32_t up = (P + (kWave - 1u)) & ~(kWave - 1u), dn = Q & ~(kWave - 1u);
    const uint32_t P1 = Q < up ? Q : up, Q1 = dn > P1 ? dn : P1;
    const uint32_t p1 = P1 / kWave, q1 = Q1 / kWave;           // equal when no whole node lies between
    const bool in1 = P + lane < P1, in2 = !SHORT && p1 + lane < q1, in3 = !SHORT && Q1 + lane < Q;
    const uint32_t b1 = in1 ? P + lane : P, node = in2 ? p1 + lane : 0u, b3 = in3 ? Q1 + lane : P;
    const double H_a = T.H[ba], H_c = T.H[bc];
    // (P may be one past the last bin: the first node's mass, which is left out like every other item outside its run)
    double m1 = T.H[b1], m2 = 0.0, rest = 0.0, m3 = 0.0;
    if constexpr (!SHORT) { m2 = T.H[nb + node]; rest = T.H[nb + kNodes + node]; m3 = T.H[b3]; }
    m1 = in1 ? m1 : 0.0;
    if constexpr (!SHORT) { m2 = in2 ? m2 : 0.0; rest = in2 ? rest : 0.0; m3 = in3 ? m3 : 0.0; }
    // the pieces of the bins that hold a and c
    const double a_e1 = bin_edge(ba + 1u, nb);
    const double a_hi = c < a_e1 ? c : a_e1;
    const double m_a = by_bin_width(H_a * (a_hi - a), ba, nb);
    double m_c = 0.0, c_e0 = c;
    if (bc > ba) {
        c_e0 = bin_edge(bc, nb);
        m_c = by_bin_width(H_c * (c - c_e0), bc, nb);
    }
    // the runs' prefix sums, then each run's mass on top of the runs before it (before they are known to be needed: beside the
    // integral and the division they take no time)
    double cum1 = wave_prefix(m1), cum2 = 0.0, cum3 = 0.0;
    const double base2 = m_a + lane_value(cum1, kWave - 1u);
    double base3 = base2, all = base2;
    cum1 += m_a;
    if constexpr (!SHORT) {
        cum2 = wave_prefix(m2);
        cum3 = wave_prefix(m3);
        base3 = base2 + lane_value(cum2, kWave - 1u);
        all = base3 + lane_value(cum3, kWave - 1u);
        cum2 += base2;
        cum3 += base3;
    }
    // int_a^c (c - u) dF~: an item's mass times the distance of its middle (a bin) or right edge (a node, and its moment about that)
    double part = (c - bin_middle(b1, nb)) * m1;
    if constexpr (!SHORT) part += ((c - bin_edge((node + 1u) * kWave, nb)) * m2 + rest) + (c - bin_middle(b3, nb)) * m3;
    const double right_all = m_a * (c - 0.5 * (a + a_hi)) + wave_sum(part) + m_c * (c - 0.5 * (c_e0 + c));
    if (!same_in_all(right_all > 0.0)) return a;                       // no mass between the neighbours
    const double t = right_all / (c - a);
    // the smallest x with mass(a, x) >= t: x = from + share / of * span in the bin or piece that holds it
    double from = a, share = t, of = m_a, span = a_hi - a;
    if (!same_in_all(m_a >= t)) {
        uint32_t bin = Q;
        // the first place in the first run in which the mass reaches t
        const unsigned long long there1 = __ballot(in1 && cum1 >= t), there2 = __ballot(in2 && cum2 >= t), there3 = __ballot(in3 && cum3 >= t);
        if ((there1 | there2 | there3) == 0ull) {
            // in the piece of c's bin
            from = c_e0; share = t - all; of = m_c; span = c - c_e0;
        } else {
            const unsigned long long there = there1 != 0ull ? there1 : there2 != 0ull ? there2 : there3;
            uint32_t first = (uint32_t)__ffsll((long long)there) - 1u;
            const double cum = there1 != 0ull ? cum1 : there2 != 0ull ? cum2 : cum3;
            const double base = there1 != 0ull ? m_a : there2 != 0ull ? base2 : base3;
            double prev = first > 0u ? lane_value(cum, first - 1u) : base;
            bin = there1 != 0ull ? P + first : Q1 + first;
            if (there1 == 0ull && there2 != 0ull) {                    // into the node that holds it
                const uint32_t b0 = (p1 + first) * kWave;
                const double below = prev + wave_prefix(T.H[b0 + lane]);
                const unsigned long long reached = __ballot(below >= t);
                if (reached == 0ull)       // the node's mass reached t and the sum of its parts, rounded otherwise, did not
                    return fmin(fmax(last_mass_edge(T, P, b0 + kWave, same_in_all(m_a > 0.0) ? a_hi : a), a), c);
                first = (uint32_t)__ffsll((long long)reached) - 1u;
                prev = first > 0u ? lane_value(below, first - 1u) : prev;
                bin = b0 + first;
            }
            from = bin_edge(bin, nb);
            share = t - prev; of = T.H[bin]; span = bin_edge(bin + 1u, nb) - from;
        }
        // The sums of neighbouring lanes are rounded apart, so t can be reached in a bin without mass, or past all the mass, by a
        // rounding (or be behind that place already): then the answer is where the mass before it ends.
        if (!same_in_all(of > 0.0 && share > 0.0))
            return fmin(fmax(last_mass_edge(T, P, bin, same_in_all(m_a > 0.0) ? a_hi : a), a), c);
    }
    const double x = fmin(from + share / of * span, from + span);        // (a little mass may be less than t's rounding)
    return fmin(fmax(x, a), c);
}

// All lanes of a wave call this with the same a and c and get the same x.
__device__ __forceinline__ double stationary_point(const Tree& T, double a, double c)
{
    if (!same_in_all(c > a)) return a;
    const uint32_t ba = same_in_all(bin_containing(T.n_bins, a)), bc = same_in_all(bin_containing(T.n_bins, c));
    return bc <= ((ba + kWave) & ~(kWave - 1u)) ? stationary_between<true>(T, a, c, ba, bc) : stationary_between<false>(T, a, c, ba, bc);
}

// The sweeps update level j from the new l_{j-1} and the old l_{j+1}, one level after the other.
// Update (sweep s, level j) therefore only waits for (s, j-1) and (s-1, j+1), and all updates with
// the same 2s + j can run together: wave s of the workgroup carries sweep s, two
// levels behind wave s-1, and takes its upper neighbour from what that wave left in LDS one step ago.
// Same updates in the same order as the plain double loop, in 2 sweeps + n_sym steps instead of
// sweeps * n_sym.
constexpr uint32_t kFitWaves = 16;
__global__ __launch_bounds__(kFitWaves * kWave) void k_fit(Tables* tab, const double* __restrict__ hist, uint32_t n_bins,
                                                           uint32_t sweeps)
{
    extern __shared__ __align__(16) unsigned char s_raw[];
    double* H = reinterpret_cast<double*>(s_raw);                // [n_bins + kTreeDoubles]
    __shared__ double s_lev[kSymMax + 1];                         // the table between passes
    __shared__ double s_moved[2][kFitWaves];                      // what each wave moved in the last two steps

    const uint32_t tid = threadIdx.x, nthreads = blockDim.x;
    for (uint32_t b = tid; b < n_bins; b += nthreads) H[b] = hist[b];
    __syncthreads();
    // the nodes, a wave each (n_bins is a multiple of 64)
    const uint32_t wave = same_in_all(tid / kWave), waves = nthreads / kWave, lane = tid % kWave;
    for (uint32_t i = wave; i < n_bins / kWave; i += waves) {
        const uint32_t b = i * kWave + lane;
        const double edge = bin_edge((i + 1u) * kWave, n_bins), mid = 0.5 * (bin_edge(b, n_bins) + bin_edge(b + 1u, n_bins));
        const double m = wave_sum(H[b]), r = wave_sum(H[b] * (edge - mid));
        if (lane == 0u) { H[n_bins + i] = m; H[n_bins + kNodes + i] = r; }
    }
    const uint32_t n_sym = tab->n_sym;
    if (tid < n_sym) s_lev[tid] = (double)tab->levels[tid];
    __syncthreads();
    // is there any mass at all?
    const double total = wave_sum(lane < n_bins / kWave ? H[n_bins + lane] : 0.0);

    const Tree T = {H, n_bins};
    const uint32_t top = n_sym - 1u;
    if (same_in_all(total > 0.0) && n_sym > 2u) {
        for (uint32_t first = 0; first < sweeps; first += waves) {
            const uint32_t ns = min(waves, sweeps - first);              // sweeps of this pass, one per wave
            double mine = 0.0;                      // the level this wave moved in its last step
            const uint32_t steps = 2u * (ns - 1u) + (top - 1u);
            for (uint32_t t = 1; t <= steps; ++t) {
                const int j = (int)t - 2 * (int)wave;
                if (wave < ns && j >= 1 && j < (int)top) {
                    // the wave before moved level j + 1 one step ago; the first wave reads the table of the last pass
                    double above = wave == 0u ? s_lev[j + 1] : s_moved[(t - 1u) & 1u][wave - 1u];
                    if (j + 1 == (int)top) above = 1.0;
                    const double below = j == 1 ? 0.0 : mine;
                    mine = stationary_point(T, below, above);
                    if ((tid & (kWave - 1u)) == 0u) {
                        s_moved[t & 1u][wave] = mine;
                        if (wave == ns - 1u) s_lev[j] = mine;
                    }
                }
                __syncthreads();
            }
        }
    }
    // strictly increasing with gaps of at least 2^-24: up from l_0 = 0, then down from l_s = 1; one
    // lane, in LDS (in the table itself each step waits for global memory: 0.25 us a level)
    __shared__ float s_out[kSymMax];
    __syncthreads();
    if (tid == 0) {
        float below = 0.0f;
#pragma unroll 4
        for (uint32_t j = 1; j < top; ++j) {
            const float x = (float)s_lev[j];
            const float floor_ = below + 0x1p-24f;
            below = x < floor_ ? floor_ : x;
            s_out[j] = below;
        }
        float above = 1.0f;
#pragma unroll 4
        for (uint32_t j = top - 1u; j >= 1u; --j) {
            const float ceil_ = above - 0x1p-24f, x = s_out[j];
            above = x > ceil_ ? ceil_ : x;
            s_out[j] = above;
        }
        s_out[0] = 0.0f;
        s_out[top] = 1.0f;
    }
    __syncthreads();
    if (tid < n_sym) tab->levels[tid] = s_out[tid];
}

hipError_t launch_fit(Tables* tab, const double* hist, uint32_t n_bins, uint32_t sweeps, hipStream_t st)
{
    const size_t lds = ((size_t)n_bins + kTreeDoubles) * sizeof(double);
    const uint32_t waves = min(max(sweeps, 8u), kFitWaves);        // (eight for the nodes)
    hipLaunchKernelGGL(k_fit, dim3(1), dim3(waves * kWave), lds, st, tab, hist, n_bins, sweeps);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_build_tables(tab, st);
}

// ---- Psi from estimated symbol probabilities (Proposition 1; Appendix J, Huffman coding) ---------------
// p_j: the mass F~ sends to level j through the random rounding: the gap below it sends it the rising part of its
// hat function, the gap above the falling part.  A piece of a bin contributes its mass times the rounding
// probability at its midpoint, which is exact for the piecewise-uniform density.
//
// The code: optimal prefix code for the weights round(p 2^32) (at least 1) with no word longer than
// max_len, by package-merge (Larmore and Hirschberg 1990); with a slack limit that is Huffman's code.
// Every level offers each symbol one coin at the symbol's weight; from the deepest level up, the
// sorted list of a level is paired into packages that are merged into the next level's coins; the
// cheapest 2 (n - 1) entries of the top list are bought, a package standing for its two entries one
// level down.  A symbol's length is the number of its coins bought.  Equal weights: coin before
// package, lower index first.  Words are numbered canonically by (length, index), first bit first.
constexpr uint32_t kFitCodeThreads = 1024;
// pieces of 64 bins: 64 for all the bins, and one more for every gap (its first piece starts anywhere, its last ends anywhere)
constexpr uint32_t kFitPieces = QGX_MAX_BINS / 64 + 2 * kSymMax;
__global__ __launch_bounds__(kFitCodeThreads) void k_fit_code(Tables* tab, const double* __restrict__ hist, uint32_t n_bins,
                                                  uint32_t max_len, FitCodeResult* __restrict__ result)
{
    extern __shared__ __align__(16) unsigned char s_raw[];
    double* H = reinterpret_cast<double*>(s_raw);                      // [n_bins]
    __shared__ double s_part[kFitCodeThreads / kWave];
    __shared__ double s_lev[kSymMax];
    __shared__ unsigned long long s_w[kSymMax], s_sw[kSymMax], s_cur[2 * kSymMax], s_nxt[2 * kSymMax];
    __shared__ uint8_t s_pkg[kMaxCode][2 * kSymMax];
    __shared__ uint32_t s_count[kMaxCode];
    __shared__ uint8_t s_order[kSymMax], s_len[kSymMax];

    const uint32_t tid = threadIdx.x, n = tab->n_sym;
    double part = 0.0;
    for (uint32_t b = tid; b < n_bins; b += kFitCodeThreads) { const double h = hist[b]; H[b] = h; part += h; }
    const uint32_t lane = tid % kWave, wave = tid / kWave;
    part = wave_sum(part);
    if (lane == 0u) s_part[wave] = part;
    if (tid < n) s_lev[tid] = (double)tab->levels[tid];
    __syncthreads();
    const double total = wave_sum(lane < kFitCodeThreads / kWave ? s_part[lane] : 0.0);

    // p_j.  The bins under a gap [l_j, l_{j+1}], a piece of 64 of them per wave and turn, a bin per lane: what the
    // piece sends up to l_{j+1} and down to l_j, summed across the wave; then a wave per level adds up the pieces of the
    // gap below it and of the gap above.  Nothing here fills the chip, so what counts is the number of dependent
    // accesses to LDS: which gap a piece belongs to is looked up for all pieces at once, counts are scanned across a wave,
    // and loops over all symbols have their loads ahead.  (33 symbols: a row of lanes per level 91 us, pieces found and added
    // up one after the other by half as many waves 35, now 28.)
    __shared__ uint32_t s_b0[kSymMax], s_first[kSymMax + 1];
    __shared__ uint8_t s_gap[kFitPieces];
    __shared__ double s_up[kFitPieces], s_down[kFitPieces];
    static_assert(kSymMax == 2 * kWave && kFitPieces <= kFitCodeThreads, "two gaps a lane, a thread per piece");
    if (wave == 0u) {
        uint32_t count[2];
#pragma unroll
        for (uint32_t h = 0; h < 2u; ++h) {                                      // gaps 2 lane and 2 lane + 1
            const uint32_t j = 2u * lane + h;
            count[h] = 0u;
            if (j + 1u < n) {
                uint32_t b = bin_of((float)s_lev[j], n_bins);
                while (b > 0 && bin_edge(b, n_bins) > s_lev[j]) --b;
                const uint32_t b_end = bin_of((float)s_lev[j + 1u], n_bins) + 1u;    // one past the last bin the gap may reach
                s_b0[j] = b;
                count[h] = b_end > b ? (b_end - b + (kWave - 1u)) / kWave : 0u;
            }
        }
        const uint32_t both = count[0] + count[1], before = wave_incl_scan(both) - both;
        s_first[2u * lane] = before;                                             // first piece of a gap; past the last gap: all of them
        s_first[2u * lane + 1u] = before + count[0];
    }
    __syncthreads();
    const uint32_t pieces = s_first[n - 1u];
    if (tid < pieces) {
        uint32_t lo_j = 0, hi_j = n - 2u;                                        // the last gap that starts at or before the piece
        while (lo_j < hi_j) {
            const uint32_t mid = (lo_j + hi_j + 1u) >> 1;
            if (s_first[mid] <= tid) lo_j = mid; else hi_j = mid - 1u;
        }
        s_gap[tid] = (uint8_t)lo_j;
    }
    __syncthreads();
    for (uint32_t q = wave; q < pieces; q += kFitCodeThreads / kWave) {
        const uint32_t j = s_gap[q];
        const double a = s_lev[j], c = s_lev[j + 1u];
        const uint32_t b = s_b0[j] + (q - s_first[j]) * kWave + lane;
        double rise = 0.0, fall = 0.0;
        if (b < n_bins) {
            const double e0 = bin_edge(b, n_bins), e1 = bin_edge(b + 1, n_bins);
            const double lo = a > e0 ? a : e0, hi = c < e1 ? c : e1;
            if (hi > lo) {
                const double mass = H[b] * (hi - lo) / (e1 - e0);
                const double up = (0.5 * (lo + hi) - a) / (c - a);
                rise = mass * up;
                fall = mass * (1.0 - up);
            }
        }
        rise = wave_sum(rise);
        fall = wave_sum(fall);
        if (lane == 0u) { s_up[q] = rise; s_down[q] = fall; }
    }
    __syncthreads();
    for (uint32_t j = wave; j < n; j += kFitCodeThreads / kWave) {
        double acc = 0.0;
        if (j > 0u) for (uint32_t q = s_first[j - 1u] + lane; q < s_first[j]; q += kWave) acc += s_up[q];
        if (j + 1u < n) for (uint32_t q = s_first[j] + lane; q < s_first[j + 1u]; q += kWave) acc += s_down[q];
        acc = total > 0.0 ? wave_sum(acc) / total : 0.0;
        if (lane != 0u) continue;
        result->p[j] = acc;
        const double x = floor(acc * 4294967296.0 + 0.5);
        s_w[j] = x >= 1.0 ? (unsigned long long)x : 1ull;
    }
    __syncthreads();

    // Symbols by weight, then index: a symbol's place is the number of symbols that come before it.
    if (tid < n) {
        const unsigned long long wi = s_w[tid];
        uint32_t rank = 0;
#pragma unroll 8
        for (uint32_t k = 0; k < n; ++k) {
            const unsigned long long wk = s_w[k];
            rank += (wk < wi || (wk == wi && k < tid)) ? 1u : 0u;
        }
        s_order[rank] = (uint8_t)tid;
    }
    __syncthreads();
    if (tid < n) s_sw[tid] = s_w[s_order[tid]];
    __syncthreads();
    // Package-merge, a level per round: the list of a level is the merge of the n single symbols with the
    // packages (pairs, in order) of the level above; at equal weight the single comes first.  Both lists are
    // sorted, so an item's place is its own index plus the number of items of the other list before it
    // (a binary search): a thread per item.
    unsigned long long* cur = s_cur;
    unsigned long long* nxt = s_nxt;
    uint32_t m = n;
    if (tid < n) { cur[tid] = s_sw[tid]; s_pkg[max_len - 1][tid] = 0; }
    if (tid == 0) s_count[max_len - 1] = m;
    __syncthreads();
    for (int l = (int)max_len - 2; l >= 0; --l) {
        const uint32_t n_pk = m >> 1;
        if (tid < n) {                                   // single tid: after the packages that weigh less
            const unsigned long long wa = s_sw[tid];
            uint32_t lo = 0, hi = n_pk;                  // first package with weight >= wa
            while (lo < hi) {
                const uint32_t mid = (lo + hi) >> 1;
                if (cur[2 * mid] + cur[2 * mid + 1] < wa) lo = mid + 1; else hi = mid;
            }
            nxt[tid + lo] = wa;
            s_pkg[l][tid + lo] = 0;
        } else if (tid - n < n_pk) {                     // package tid - n: after the singles that weigh no more
            const uint32_t ib = tid - n;
            const unsigned long long wb = cur[2 * ib] + cur[2 * ib + 1];
            uint32_t lo = 0, hi = n;                     // first single with weight > wb
            while (lo < hi) {
                const uint32_t mid = (lo + hi) >> 1;
                if (s_sw[mid] <= wb) lo = mid + 1; else hi = mid;
            }
            nxt[ib + lo] = wb;
            s_pkg[l][ib + lo] = 1;
        }
        m = n + n_pk;
        if (tid == 0) s_count[l] = m;
        __syncthreads();
        unsigned long long* t = cur; cur = nxt; nxt = t;
    }
    // The 2 (n - 1) lightest items of the lowest level are taken; every single among the items taken at a
    // level adds a bit to its symbol (the singles are the lightest symbols in order), every package sends
    // its two parts of the level above.
    if (tid < n) s_len[tid] = 0;
    __syncthreads();
    uint32_t take = 2u * (n - 1u);
    for (uint32_t l = 0; l < max_len; ++l) {                           // (take falls to 0 and stays there)
        take = min(take, s_count[l]);
        const uint32_t packages = (uint32_t)__syncthreads_count(tid < take && s_pkg[l][tid] != 0);
        const uint32_t singles = take - packages;
        if (tid < singles) s_len[s_order[tid]] += 1;
        take = 2u * packages;
    }
    __syncthreads();
    // canonical words: the symbols in the order (length, index), each word the count of the words before it at
    // its own length's scale; the table wants the first-written bit in bit 0
    if (tid < n) {
        const uint32_t L = s_len[tid];
        uint32_t code = 0;
#pragma unroll 8
        for (uint32_t k = 0; k < n; ++k) {
            const uint32_t lk = s_len[k];
            if (lk < L || (lk == L && k < tid)) code += 1u << (L - lk);
        }
        const uint32_t word = (__brev(code) >> (32u - L)) | (L << 16);
        tab->code[tid] = word;
        result->code[tid] = word;
    }
}

hipError_t launch_fit_code(Tables* tab, const double* hist, uint32_t n_bins, uint32_t max_len, FitCodeResult* result,
                           hipStream_t st)
{
    hipLaunchKernelGGL(k_fit_code, dim3(1), dim3(kFitCodeThreads), (size_t)n_bins * sizeof(double), st, tab, hist, n_bins, max_len, result);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_build_tables(tab, st);
}

}  // namespace qgx
