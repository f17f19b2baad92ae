// ss_sample_drop: the input sampling block (section 3.3, Eq. 1-2 of the paper).
//
// For a set of sampled inputs it counts, for every threshold of a ladder at
// once, how many of them could be dropped: those with at least alpha lookups
// that reach a stale hot row.  The paper evaluates one threshold per pass over
// the sampled rows; here the drift of every hot row is computed once (by
// ss_detect_stale, which can write it out) and this kernel only looks drifts
// up, so a pass costs 8 bytes per lookup whatever the row length, and up to 32
// thresholds share that pass.
//
// The thresholds are sorted on the host, so a lookup's drift falls into one class: the
// first threshold it does not exceed.  An input can be dropped from the alpha-th smallest
// class of its lookups on, so one number per input replaces a count per threshold.
//
// A workgroup takes 64 inputs, one per lane, and its wavefronts split the T * L lookups of
// an input between them (fewer inputs, and several lanes for each, where a sample is small and
// its inputs are long).  A lookup maps its row to a hot slot by a branch-free lower-bound
// search in the ascending hot_ids of its table; a lane runs up to four such searches
// interleaved, since each step is one dependent load that only latency bounds.  All lanes
// of a wavefront search the same table: its popular rows and the first steps of every
// search are the same few cache lines, and the lines that the loads bring to the compute
// unit are what bounds the kernel (with neighbouring lanes in different tables, nearly as
// many lines as lanes: 51.4 us for 65536 inputs of 26 lookups, 5000 hot rows per table and
// 32 thresholds, 24.6 now; 84 and 40 with the hot rows scattered over the table).  Classes are
// counted per input in LDS, inputs per class in LDS, and each workgroup adds its share to the
// counts at the end.
#include <math.h>

#include "ss_common.h"

namespace ss {

// Thresholds in ascending order as the kernel compares them: widened to fp64 on the host, -1
// where no row may be stale (threshold 0), since a drift is never below 0, and +inf in unused
// slots at the end; and which of the caller's thresholds each one is.
struct Ladder {
    double thr[SS_MAX_THRESHOLDS];
    uint8_t slot[SS_MAX_THRESHOLDS];
};

constexpr int kBatch = 4;        // searches a lane keeps in flight
constexpr int kMaxWaves = 8;
// More workgroups only add more to the few words of the counts (us for 65536 inputs of 26
// lookups / 44414 of 12 / 190000 of 2, at 256, 512, 1024 and 2048 workgroups: 31.8 / 17.3 / 17.8,
// 24.8 / 15.6 / 16.5, 25.0 / 15.8 / 18.8, 25.0 / 16.3 / 18.8).
constexpr int64_t kMaxGroups = 512;

typedef int32_t i4 __attribute__((ext_vector_type(4), aligned(4)));

// Drifts of N lookups of input s: q0, q0 + step, ... of its TL (a lookup at TL or beyond: that of
// q0).  found[i]: the row is hot; d[i] means nothing otherwise.
template <int N>
__device__ __forceinline__ void lookup_drifts(
    const int32_t *const *__restrict__ hot_ids, int H, const double *const *__restrict__ drift,
    const int32_t *__restrict__ sidx, int S, uint32_t L, uint32_t TL, int s, uint32_t q0,
    uint32_t step, double (&d)[N], bool (&found)[N])
{
    int32_t row[N];
    int base[N];
    gptr<const int32_t> ids[N];
    gptr<const double> dr[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const uint32_t q = q0 + i * step < TL ? q0 + i * step : q0;    // TL < 2^31
        const uint32_t t = q / L, l = q - t * L;
        row[i] = sidx[((int64_t)t * S + s) * L + l];
        ids[i] = as_global(hot_ids[t]);
        dr[i] = as_global(drift[t]);
        base[i] = 0;
    }
    // lower bound: the last slot whose id is <= row (slot 0 if none is), down to four
    // candidates, which one load fetches
    for (int n = H; n > 4;) {
        const int half = n >> 1;
#pragma unroll
        for (int i = 0; i < N; ++i)
            if (ids[i][base[i] + half] <= row[i]) base[i] += half;
        n -= half;
    }
    if (H >= 4) {
        i4 four[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            base[i] = base[i] <= H - 4 ? base[i] : H - 4;
            four[i] = *(gptr<const i4>)(ids[i] + base[i]);
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
            found[i] = four[i].x == row[i] || four[i].y == row[i] || four[i].z == row[i] ||
                       four[i].w == row[i];
            base[i] += four[i].w <= row[i] ? 3 : four[i].z <= row[i] ? 2
                       : four[i].y <= row[i] ? 1 : 0;
        }
    } else {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            for (int h = 1; h < H; ++h)
                if (ids[i][h] <= row[i]) base[i] = h;
            found[i] = ids[i][base[i]] == row[i];
        }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) d[i] = dr[i][base[i]];
}

// Classes of those lookups (at TL or beyond: none).  The class of a lookup is the first threshold
// its row's drift does not exceed, K where there is none or the row is not hot.
template <int N>
__device__ __forceinline__ void lookup_classes(
    const int32_t *const *__restrict__ hot_ids, int H, const double *const *__restrict__ drift,
    const int32_t *__restrict__ sidx, int S, uint32_t L, uint32_t TL, int s, uint32_t q0,
    uint32_t step, const double *s_thr, int (&cls)[N])
{
    constexpr int K = SS_MAX_THRESHOLDS;
    static_assert(K == 32, "the class search takes five steps");
    double d[N];
    bool found[N];
    lookup_drifts(hot_ids, H, drift, sidx, S, L, TL, s, q0, step, d, found);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        // same verdict as ss_detect_stale; a NaN drift exceeds all thresholds
        int k = 0;
#pragma unroll
        for (int half = K / 2; half > 0; half >>= 1) k += d[i] <= s_thr[k + half - 1] ? 0 : half;
        cls[i] = q0 + i * step < TL && found[i] && d[i] <= s_thr[k] ? k : K;
    }
}

// Adds the workgroup's inputs per class to the counts: threshold k drops those of classes 0 .. k.
// Few workgroups: all of them add to the same few words of memory, one after the other.
__device__ __forceinline__ void add_counts(const uint32_t *s_inputs, const Ladder &ladder,
                                           int n_thr, uint32_t *__restrict__ counts)
{
    const int tid = threadIdx.x;
    if (tid < n_thr) {
        uint32_t c = 0;
        for (int k = 0; k <= tid; ++k) c += s_inputs[k];
        if (c) atomicAdd(&counts[ladder.slot[tid]], c);
    }
}

// I inputs per workgroup and round, 64 / I lanes of each wavefront for one.
template <int I>
__global__ __launch_bounds__(64 * kMaxWaves) void sample_drop_kernel(
    const int32_t *const *__restrict__ hot_ids, int H,
    const double *const *__restrict__ drift, const int32_t *__restrict__ sidx, int S,
    int L, int TL, int alpha, Ladder ladder, int n_thr, uint32_t *__restrict__ counts)
{
    constexpr int K = SS_MAX_THRESHOLDS;
    __shared__ double s_thr[K];
    __shared__ uint32_t s_cnt[K][I];            // lookups per class and input
    __shared__ uint32_t s_inputs[K];            // inputs that can be dropped from class k on
    const int tid = threadIdx.x, in = tid & (I - 1);
    // lookups q0, q0 + step, ... of its input are this lane's
    const uint32_t first_q = I == 64 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid / I;
    const uint32_t step = blockDim.x / I;
    if (tid < K) {
        s_thr[tid] = ladder.thr[tid];
        s_inputs[tid] = 0;
    }
    for (int64_t s0 = (int64_t)blockIdx.x * I; s0 < S; s0 += (int64_t)gridDim.x * I) {
        const int s = s0 + in < S ? (int)s0 + in : S - 1;       // lanes past the last: not counted
        for (int i = tid; i < K * I; i += blockDim.x) (&s_cnt[0][0])[i] = 0;
        __syncthreads();
        for (uint32_t q0 = first_q; q0 < (uint32_t)TL && H > 0; q0 += step * kBatch) {
            int cls[kBatch];
            lookup_classes(hot_ids, H, drift, sidx, S, L, TL, s, q0, step, s_thr, cls);
#pragma unroll
            for (int i = 0; i < kBatch; ++i)
                if (cls[i] < K) atomicAdd(&s_cnt[cls[i]][in], 1u);
        }
        __syncthreads();
        if (tid < I && s0 + tid < S) {
            int64_t below = 0;
            int first = K;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                below += s_cnt[k][tid];
                first = first == K && below >= alpha ? k : first;
            }
            if (first < K) atomicAdd(&s_inputs[first], 1u);
        }
        __syncthreads();
    }
    add_counts(s_inputs, ladder, n_thr, counts);
}

// Inputs of at most N lookups: an input is one lane's alone, its classes stay in
// registers, and the alpha-th smallest is the least class that alpha of them do not exceed.
// (The kernel above clears and reads back 32 counters per input, more than a short input's
// searches cost: a threshold search over 190000 inputs of 2 lookups took 328 us, 245 now.)
template <int N>
__global__ __launch_bounds__(256) void sample_drop_few_kernel(
    const int32_t *const *__restrict__ hot_ids, int H,
    const double *const *__restrict__ drift, const int32_t *__restrict__ sidx, int S,
    int L, int TL, int alpha, Ladder ladder, int n_thr, uint32_t *__restrict__ counts)
{
    constexpr int K = SS_MAX_THRESHOLDS;
    __shared__ double s_thr[K];
    __shared__ uint32_t s_inputs[K];
    const int tid = threadIdx.x;
    if (tid < K) {
        s_thr[tid] = ladder.thr[tid];
        s_inputs[tid] = 0;
    }
    __syncthreads();
    for (int64_t s = (int64_t)blockIdx.x * blockDim.x + tid; s < S;
         s += (int64_t)gridDim.x * blockDim.x) {
        int first = alpha <= 0 ? 0 : K;
        if (alpha > 0 && H > 0) {
            int cls[N];
            lookup_classes(hot_ids, H, drift, sidx, S, L, TL, (int)s, 0, 1, s_thr, cls);
#pragma unroll
            for (int i = 0; i < N; ++i) {
                int below = 0;
#pragma unroll
                for (int j = 0; j < N; ++j) below += cls[j] < K && cls[j] <= cls[i];
                if (below >= alpha && cls[i] < first) first = cls[i];
            }
        }
        if (first < K) atomicAdd(&s_inputs[first], 1u);
    }
    __syncthreads();
    add_counts(s_inputs, ladder, n_thr, counts);
}

// ---- one level per input -------------------------------------------------
// With alpha = T * L an input can be dropped from the largest drift of its lookups on, whatever the
// thresholds are: a search over several ladders maps rows to hot slots once and then counts levels.
// (A threshold search over 65536 inputs of 26 lookups, 5000 hot rows: three passes of the kernel
// above 75 us; levels 20 us and 7 per count.)  A level is kept as the least float that is not
// below it: a threshold is a float, and reaches the one where it reaches the other.  NaN: a lookup
// that is never stale.
__device__ __forceinline__ float float_not_below(double x)
{
    float f = (float)x;
    if ((double)f < x) {                 // (x >= 0: the next float up has the next bits)
        f = __uint_as_float(__float_as_uint(f) + 1u);
    }
    return f;
}
// N searches of a lane side by side: as many as an input has lookups, four at most.
template <int I, int N>
__global__ __launch_bounds__(64 * kMaxWaves) void sample_level_kernel(
    const int32_t *const *__restrict__ hot_ids, int H,
    const double *const *__restrict__ drift, const int32_t *__restrict__ sidx, int S,
    int L, int TL, float *__restrict__ levels)
{
    __shared__ double s_level[64 * kMaxWaves];
    const int tid = threadIdx.x, in = tid & (I - 1);
    const uint32_t first_q = I == 64 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid / I;
    const uint32_t step = blockDim.x / I;
    const int64_t s0 = (int64_t)blockIdx.x * I;
    const int s = s0 + in < S ? (int)(s0 + in) : S - 1;
    double level = H > 0 ? 0.0 : __builtin_nan("");       // (a drift is never below 0)
    for (uint32_t q0 = first_q; q0 < (uint32_t)TL && H > 0; q0 += step * N) {
        double d[N];
        bool found[N];
        lookup_drifts(hot_ids, H, drift, sidx, S, L, TL, s, q0, step, d, found);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const double x = found[i] ? d[i] : __builtin_nan("");
            level = level >= x || level != level ? level : x;
        }
    }
    s_level[tid] = level;
    __syncthreads();
    if (tid < I && s0 + tid < S) {
        for (uint32_t k = 1; k < step; ++k) {
            const double x = s_level[k * I + tid];
            level = level >= x || level != level ? level : x;
        }
        levels[s0 + tid] = float_not_below(level);
    }
}

// Threshold k = blockIdx.x: how many of the `part` levels from blockIdx.y * part on it reaches.  What
// bounds it is the rate at which one compute unit reads: up to 65536 levels a workgroup takes
// all of them, 32 at a time per thread, and counts need neither clearing nor adding up (65536
// levels: 6.7 us; 9.9 as doubles).  More are shared out to 512 workgroups, two per compute unit, but
// no fewer than 16384 to each (a search over 190000 levels 85 us, 96 with 131072 to each; over
// 400000 98 and 104, over a million 138 and 141; 159 with 16384).
struct LevelLadder {
    float thr[SS_MAX_LEVEL_THRESHOLDS];
};
constexpr int kLevelThreads = 1024;
constexpr int kLevelsAlone = 1 << 16, kLevelsLeast = 1 << 14, kLevelGroups = 512;
__global__ __launch_bounds__(kLevelThreads) void level_count_kernel(
    const float *__restrict__ levels, int S, int part, LevelLadder ladder,
    uint32_t *__restrict__ counts)
{
    __shared__ uint32_t s_sum[kLevelThreads / 64];
    const int tid = threadIdx.x;
    const float thr = ladder.thr[blockIdx.x];
    const int64_t p0 = (int64_t)blockIdx.y * part;
    const int64_t p1 = p0 + part < S ? p0 + part : S;
    uint32_t n = 0;
    constexpr int U = 32;
    for (int64_t i0 = p0 + tid; i0 < p1; i0 += U * kLevelThreads) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = i0 + u * kLevelThreads;
            v[u] = levels[i < p1 ? i : i0];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) n += i0 + u * kLevelThreads < p1 && v[u] <= thr ? 1u : 0u;
    }
    for (int off = 32; off; off >>= 1) n += __shfl_xor(n, off);
    if ((tid & 63) == 0) s_sum[tid >> 6] = n;
    __syncthreads();
    if (tid == 0) {
        uint32_t all = 0;
        for (int w = 0; w < kLevelThreads / 64; ++w) all += s_sum[w];
        if (gridDim.y == 1) counts[blockIdx.x] = all;
        else if (all) atomicAdd(&counts[blockIdx.x], all);
    }
}

// Inputs per workgroup of the general kernels, 64 / I lanes of each wavefront for one.
static int inputs_per_group(int S, int TL)
{
    // With 64 inputs each there are S / 64 workgroups, and a lane of eight wavefronts has
    // TL / 32 rounds of searches before it.  Where both leave the chip waiting an input
    // gets 4 or 16 lanes of every wavefront.  us with 64 / 16 / 4 inputs per workgroup, and
    // with a group of lanes per input and no regard to tables as it once was, 5000 hot rows
    // next to each other and Zipf lookups; the same scattered and uniform:
    //    2000 inputs of 1280   208 / 63 / 32, 42        275 / 89 / 76, 102
    //    9000 of 1280          227 / 152 / 122, 135     277 / 325 / 306, 408
    //    4096 of 520           76 / 28 / 31, 41         116 / 58 / 68, 98
    //    9000 of 520           88 / 64 / 63, 77         125 / 137 / 144, 200
    //   12000 of 520           94 / 65 / 81, 99         131 / 158 / 190, 261
    //   16000 of 520           95 / 80 / 102, 125       144 / 207 / 249, 347
    //    5950 of 104           23 / 14 / 19, 22         32 / 24 / 27, 37
    int I = 64;
    if (TL > kMaxWaves * kBatch && S <= 12288) I = 16;
    if ((TL > kMaxWaves * kBatch * 4 && S <= 4096) || (TL > 1024 && S <= 16384)) I = 4;
    return I;
}

int32_t launch_sample_levels(int T, int32_t *const *hot_ids, int H, double *const *drift,
                             const int32_t *sidx, int S, int L, float *levels, hipStream_t s)
{
    if (S > 0) {
        const int TL = T * L, I = inputs_per_group(S, TL), N = TL < 3 ? TL : kBatch,
                  per_wave = N * (64 / I);
        int waves = (TL + per_wave - 1) / per_wave;
        if (waves > kMaxWaves) waves = kMaxWaves;
        const unsigned grid = (unsigned)(((int64_t)S + I - 1) / I);
        ProfScope prof("sample_level_kernel", s);
#define SS_LEVEL(I_, N_)                                                                    \
    launch(sample_level_kernel<I_, N_>, dim3(grid), dim3(64 * waves), s,                         \
           (const int32_t *const *)hot_ids, H, (const double *const *)drift, sidx, S, L, TL, levels)
        if (TL == 1) SS_LEVEL(64, 1);
        else if (TL == 2) SS_LEVEL(64, 2);
        else if (I == 64) SS_LEVEL(64, kBatch);
        else if (I == 16) SS_LEVEL(16, kBatch);
        else SS_LEVEL(4, kBatch);
#undef SS_LEVEL
    }
    return check_launch("ss_sample_levels");
}

int32_t launch_level_counts(const float *levels, int S, const float *thresholds, int n_thr,
                            uint32_t *counts, hipStream_t s)
{
    LevelLadder ladder = {};
    for (int k = 0; k < n_thr; ++k)
        ladder.thr[k] = thresholds[k] > 0.0f ? thresholds[k] : -1.0f;
    const int64_t share = (int64_t)S * n_thr / kLevelGroups;
    const int part = S <= kLevelsAlone ? kLevelsAlone
                                       : (int)(share < kLevelsLeast ? kLevelsLeast : share);
    const int64_t parts = S > 0 ? ((int64_t)S + part - 1) / part : 1;
    if (parts > 1) launch_zero_u32(counts, n_thr, s);
    ProfScope prof("level_count_kernel", s);
    launch(level_count_kernel, dim3(n_thr, (unsigned)parts), dim3(kLevelThreads), s, levels, S,
           part, ladder, counts);
    return check_launch("ss_level_counts");
}

int32_t launch_sample_drop(int T, int32_t *const *hot_ids, int H, double *const *drift,
                           const int32_t *sidx, int S, int L, int alpha,
                           const float *thresholds, int n_thr, uint32_t *counts,
                           hipStream_t s)
{
    launch_zero_u32(counts, n_thr, s);
    if (S > 0) {
        Ladder ladder;
        for (int k = 0; k < SS_MAX_THRESHOLDS; ++k) {
            ladder.thr[k] = INFINITY;
            ladder.slot[k] = 0;
        }
        for (int k = 0; k < n_thr; ++k) {         // insertion sort
            const double thr = thresholds[k] > 0.0f ? (double)thresholds[k] : -1.0;
            int i = k;
            for (; i > 0 && ladder.thr[i - 1] > thr; --i) {
                ladder.thr[i] = ladder.thr[i - 1];
                ladder.slot[i] = ladder.slot[i - 1];
            }
            ladder.thr[i] = thr;
            ladder.slot[i] = (uint8_t)k;
        }
        const int TL = T * L;
        ProfScope prof("sample_drop_kernel", s);
#define SS_SAMPLE(kernel_, grid_, threads_)                                                 \
    launch(kernel_, dim3(grid_), dim3(threads_), s, (const int32_t *const *)hot_ids, H,      \
           (const double *const *)drift, sidx, S, L, TL, alpha, ladder, n_thr, counts)
        // Five to eight lookups: where the workgroups of the general kernel, 64 inputs each, would
        // go round more than once (us, general kernel and this one, 5 and 8 lookups, 100 hot rows:
        // 65536 inputs 14.7 / 10.8 and 15.2 / 11.4, 28000 10.5 / 9.9 and 10.7 / 10.5; 5000 hot rows:
        // 65536 19.9 / 17.7 and 24.1 / 22.3, 28000 12.8 / 14.4 and 14.9 / 16.9).
        if (TL <= kBatch || (TL <= 2 * kBatch && S > 64 * kMaxGroups)) {
            const int64_t groups = ((int64_t)S + 255) / 256;
            const unsigned grid = (unsigned)(groups < kMaxGroups ? groups : kMaxGroups);
            if (TL <= kBatch) SS_SAMPLE(sample_drop_few_kernel<kBatch>, grid, 256);
            else SS_SAMPLE(sample_drop_few_kernel<2 * kBatch>, grid, 256);
        } else {
            const int I = inputs_per_group(S, TL);
            const int per_wave = kBatch * (64 / I);
            int waves = (TL + per_wave - 1) / per_wave;
            if (waves > kMaxWaves) waves = kMaxWaves;
            const int64_t groups = ((int64_t)S + I - 1) / I;
            const unsigned grid = (unsigned)(groups < kMaxGroups ? groups : kMaxGroups);
            if (I == 64) SS_SAMPLE(sample_drop_kernel<64>, grid, 64 * waves);
            else if (I == 16) SS_SAMPLE(sample_drop_kernel<16>, grid, 64 * waves);
            else SS_SAMPLE(sample_drop_kernel<4>, grid, 64 * waves);
        }
#undef SS_SAMPLE
    }
    return check_launch("ss_sample_drop");
}

}  // namespace ss
