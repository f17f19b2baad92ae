// Hot-set identification (section 3.1 of the paper and the preprocessing loop of
// Algorithm 1): per-row access counters over the sampled inputs, then the set of
// hot rows of every table, either by the paper's share rule (C_r / total >=
// lambda) or as the H most accessed rows (ties to the lower row id), written as
// an ascending id list and as a bitmap.
//
// Counting.  Accesses are Zipf-like, so a few rows of a table take most of its
// lookups; sent to memory as they come, those would be thousands of atomics on
// one address.  Each workgroup therefore counts its chunk of lookups in a small
// LDS table first (open slot per row, claimed with a compare-and-swap on the
// tag; a lookup that finds its slot taken by another row goes to memory
// directly) and adds the table to the global counters at the end.  Integer
// adds commute, so the counters do not depend on the order of anything.
//
// Selecting.  Both rules reduce to "count > c, or count == c and fewer than e
// such rows came before": for the share rule c = (smallest passing count) - 1
// and e = 0, computed on the host; for top-H, c is the H-th largest count and e
// what is left of H after the rows above c.  The counters are the only large
// thing here (104 MB for 26 x 1 M rows), so what counts is how often they are
// read: twice.  One pass builds a histogram whose bins tell counts below 1024
// apart, as nearly all are, and larger ones to an eighth of an octave; its last
// workgroup per table picks the bin that holds the H-th largest count.  Where
// that bin holds several counts, up to three further passes split it by ten bits
// each (they are always launched and leave at once where nothing is left to
// split).  A second pass over the counters writes two bitmaps, "above c" and
// "equal to c", and their bits per 4096 rows; the last step works on these
// bitmaps, a sixteenth of the counters: every workgroup adds up what lies
// before its 32768 rows, ranks its bits, and writes ids in ascending order and
// the bitmap.  26 x 1 M rows: histogram 28 us (and 3 x 1.2), bitmaps 18, ids 5, instead of
// four histogram passes of 34 us with 5 us each to pick a digit, 25 to count, 54 to write;
// one table of 200 M rows 0.39 instead of 3.2 ms.
#include "ss_common.h"

namespace ss {
namespace {

constexpr int kBlockRows = 4096;         // selection: rows per workgroup of the bitmap pass
constexpr int kBlockWords = kBlockRows / 32;
constexpr int kSuper = 64;               // ... blocks whose totals are also summed up,
constexpr int kManyBlocks = 2048;        // ... in tables of more blocks than this
constexpr int kWriteBlocks = 8;          // ... blocks per workgroup of the last step
constexpr uint32_t kFewIds = 40;         // ... ids of 128 rows that a thread writes by itself
constexpr int kHistThreads = 512;        // histogram passes: threads per workgroup
constexpr int kHistStep = kHistThreads * 4;   // ... rows of a step of a workgroup
constexpr uint32_t kExact = 1024;        // counts below this have a bin each
constexpr int kExactBits = 10;
constexpr int kSubBits = 3;              // larger ones: 2^3 bins per octave
constexpr int kBins = (int)kExact + ((32 - kExactBits) << kSubBits);
constexpr int kRefine = 3;               // passes that split a bin, kExactBits each

// NT threads with ITEMS lookups each, all requested before the first is counted.  What
// bounds it is the rate of adds to memory (about 30 per nanosecond, far fewer to rows next to
// each other): fewer, the more lookups share an LDS table; but few lookups want many short
// workgroups, each of which is one chain of trips to memory (row ids, LDS slots, counters).
template <int NT, int ITEMS, int SLOTS>
__global__ __launch_bounds__(NT) void count_kernel(
    const int32_t *__restrict__ idx, int Bcap, int L, const int32_t *__restrict__ n_valid,
    uint32_t *const *__restrict__ counts, int chunks_per_table)
{
    __shared__ uint32_t s_tag[SLOTS];
    __shared__ uint32_t s_cnt[SLOTS];
    const int t = blockIdx.x / chunks_per_table;
    const int chunk = blockIdx.x - t * chunks_per_table;
    const int64_t cap = (int64_t)Bcap * L;
    const int64_t first = (int64_t)chunk * (ITEMS * NT) + threadIdx.x;
    const int32_t *__restrict__ ip = idx + (int64_t)t * cap;
    uint32_t row[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)      // (requested before the number of valid ones is known)
        row[i] = (uint32_t)ip[first + i * NT < cap ? first + i * NT : 0];
    const int64_t n = (int64_t)clamp_valid(n_valid, Bcap) * L;     // lookups of this table
    for (int i = threadIdx.x; i < SLOTS; i += NT) {
        s_tag[i] = kNoRow;
        s_cnt[i] = 0;
    }
    __syncthreads();
    uint32_t *cg = counts[t];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
        if (first + i * NT >= n) continue;
        const uint32_t r = row[i];
        const uint32_t slot = (r * 2654435761u) / (uint32_t)(0x100000000ull / SLOTS);
        const uint32_t seen = atomicCAS(&s_tag[slot], kNoRow, r);
        if (seen == kNoRow || seen == r)
            atomicAdd(&s_cnt[slot], 1u);
        else
            atomicAdd(&cg[r], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < SLOTS; i += NT) {
        const uint32_t r = s_tag[i];
        if (r != kNoRow) atomicAdd(&cg[r], s_cnt[i]);
    }
}

// ---- selection ---------------------------------------------------------
// state[t]: while the histogram passes run, the H-th largest count is known to lie in
// [c, c + 2^width), and e of the rows in that range (by count, then by id) are still to be
// taken.  In the end width = 0: rows with count > c are taken, and the first e rows (by row
// id) with count == c.
struct SelState {
    uint32_t c, e;
    int32_t width;
    uint32_t pad;
};

// Four neighbouring counters; a table's counters are only 4-byte aligned.
typedef uint32_t u4 __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ void load4(gptr<const uint32_t> cg, int64_t r, int64_t R,
                                      uint32_t (&c)[4], bool (&in)[4])
{
    if (r + 4 <= R) {
        const u4 v = *(gptr<const u4>)(cg + r);
        c[0] = v.x, c[1] = v.y, c[2] = v.z, c[3] = v.w;
        in[0] = in[1] = in[2] = in[3] = true;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            in[j] = r + j < R;
            c[j] = in[j] ? cg[r + j] : 0u;
        }
    }
}

__global__ void sel_init_kernel(SelState *state, int T, uint32_t c, uint32_t e, int width,
                                uint32_t *__restrict__ zero, int64_t n_zero)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < T) state[i] = SelState{c, e, width, 0u};
    if (i < n_zero) zero[i] = 0u;
}

// Bin of a count in the first pass, and back: the bin's smallest count and the logarithm of
// how many counts it holds.
__device__ __forceinline__ uint32_t first_bin(uint32_t v)
{
    if (v < kExact) return v;
    const int o = 31 - __clz((int)v);
    return kExact + ((uint32_t)(o - kExactBits) << kSubBits) +
           ((v >> (o - kSubBits)) & ((1u << kSubBits) - 1u));
}
__device__ __forceinline__ void first_bin_range(uint32_t bin, uint32_t &lo, int &width)
{
    lo = bin;
    width = 0;
    if (bin >= kExact) {
        const uint32_t k = bin - kExact;
        const int o = kExactBits + (int)(k >> kSubBits);
        width = o - kSubBits;
        lo = ((1u << kSubBits) + (k & ((1u << kSubBits) - 1u))) << width;
    }
}

// One histogram pass.  FIRST: all counts, the bins above; else the counts of the range that
// the passes before have left, by the next ten bits.  The last workgroup of a table to add
// its bins picks the one with  #(rows in bins above) < e <= #(rows in it or above)  and
// clears the histogram for the next pass.  A table has few workgroups: all of them add to
// the bins of the smallest counts, and memory takes adds to one address one after the other
// (0.14 us each).
template <bool FIRST>
__device__ __forceinline__ void sel_hist_pass(gptr<const uint32_t> cg, int64_t R, SelState &st,
                                              uint32_t *__restrict__ ht,
                                              uint32_t *__restrict__ done, uint32_t *s_hist)
{
    constexpr int NT = kHistThreads, NB = FIRST ? kBins : (int)kExact, PER = (NB + NT - 1) / NT;
    __shared__ uint32_t s_part[NT / 64];
    __shared__ bool s_last;
    __shared__ SelState s_state;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int shift = st.width > kExactBits ? st.width - kExactBits : 0;
    for (int i = tid; i < NB; i += NT) s_hist[i] = 0;
    __syncthreads();
    // most counters are 0 or 1: those are counted in registers
    uint32_t few[2] = {0, 0};
    const int64_t stride = (int64_t)gridDim.x * kHistStep;
    for (int64_t r0 = (int64_t)blockIdx.x * kHistStep + tid * 4; r0 < R; r0 += 4 * stride) {
        uint32_t c[4][4];
        bool in[4][4];
#pragma unroll
        for (int k = 0; k < 4; ++k) load4(cg, r0 + k * stride, R, c[k], in[k]);
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t v = c[k][j];
                if (FIRST) {
                    few[0] += in[k][j] && v == 0u;
                    few[1] += v == 1u;
                    if (v > 1u) atomicAdd(&s_hist[first_bin(v)], 1u);
                } else if (in[k][j] && ((v - st.c) >> st.width) == 0u) {
                    atomicAdd(&s_hist[(v - st.c) >> shift], 1u);
                }
            }
    }
    if (FIRST) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            for (int off = 32; off; off >>= 1) few[q] += __shfl_xor(few[q], off);
            if (lane == 0 && few[q]) atomicAdd(&s_hist[q], few[q]);
        }
    }
    __syncthreads();
    if (gridDim.x > 1) {
        for (int i = tid; i < NB; i += NT)
            if (s_hist[i]) atomicAdd(&ht[i], s_hist[i]);
        // This workgroup's adds are done before it says so.  (They are device-scope and leave
        // nothing behind in a cache; a fence would write the XCD's L2 back, once per wavefront:
        // 181 instead of 32 us for the whole kernel at 26 x 1 M rows.)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (tid == 0) s_last = atomicAdd(done, 1u) == gridDim.x - 1;
        __syncthreads();
        if (!s_last) return;
    }

    // thread i owns bins [i * PER, (i + 1) * PER); rows above them from a suffix sum
    uint32_t h[PER], sum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const int bin = tid * PER + q;
        h[q] = bin >= NB ? 0u
               : gridDim.x > 1
                   ? __hip_atomic_load(&ht[bin], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                   : s_hist[bin];
        sum += h[q];
    }
    if (gridDim.x > 1)
#pragma unroll
        for (int q = 0; q < PER; ++q)
            if (tid * PER + q < NB) ht[tid * PER + q] = 0u;
    uint32_t incl = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t up = __shfl_down(incl, off);
        if (lane + off < 64) incl += up;
    }
    if (lane == 0) s_part[wave] = incl;
    __syncthreads();
    uint32_t above = incl - sum;
    for (int w = wave + 1; w < NT / 64; ++w) above += s_part[w];
    // e >= 1 and the rows still in the race number at least e, so exactly one bin qualifies
#pragma unroll
    for (int q = PER - 1; q >= 0; --q) {
        if (above < st.e && st.e <= above + h[q]) {
            const uint32_t bin = (uint32_t)(tid * PER + q);
            uint32_t lo = st.c + (bin << shift);
            int width = shift;
            if (FIRST) first_bin_range(bin, lo, width);
            s_state = SelState{lo, st.e - above, width, 0u};
        }
        above += h[q];
    }
    __syncthreads();
    st = s_state;
}

__global__ __launch_bounds__(kHistThreads) void sel_hist_kernel(
    uint32_t *const *__restrict__ counts, int64_t R, SelState *__restrict__ state,
    uint32_t *__restrict__ hist, uint32_t *__restrict__ done, int pass)
{
    __shared__ uint32_t s_hist[kBins];
    const int t = blockIdx.y;
    SelState st = state[t];
    if (st.width == 0) return;
    const auto cg = as_global((const uint32_t *)counts[t]);
    const int width = st.width;
    if (pass == 0)
        sel_hist_pass<true>(cg, R, st, hist + (int64_t)t * kBins, done + t * (kRefine + 1), s_hist);
    else
        sel_hist_pass<false>(cg, R, st, hist + (int64_t)t * kBins,
                             done + t * (kRefine + 1) + pass, s_hist);
    if (gridDim.x == 1)                    // a table of one workgroup needs no launch per pass
        while (st.width > 0) {
            __syncthreads();
            sel_hist_pass<false>(cg, R, st, nullptr, nullptr, s_hist);
        }
    if (st.width < width && threadIdx.x == 0) state[t] = st;       // the workgroup that picked
}

// Bitmaps of "count > c" and "count == c" over 4096 rows, and how many bits each has there.
__global__ __launch_bounds__(kWG) void sel_mark_kernel(
    uint32_t *const *__restrict__ counts, int64_t R, const SelState *__restrict__ state,
    uint32_t *__restrict__ gt_bits, uint32_t *__restrict__ eq_bits, int nb,
    uint2 *__restrict__ block_totals)
{
    __shared__ uint32_t s_gt[kWG / 64], s_eq[kWG / 64];
    const int t = blockIdx.y, blk = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const SelState st = state[t];
    const auto cg = as_global((const uint32_t *)counts[t]);
    constexpr int K = kBlockRows / (kWG * 4);
    uint32_t c[K][4];
    bool in[K][4];
#pragma unroll
    for (int k = 0; k < K; ++k)
        load4(cg, (int64_t)blk * kBlockRows + (k * kWG + tid) * 4, R, c[k], in[k]);
    const int64_t w0 = ((int64_t)t * nb + blk) * kBlockWords;
    uint32_t n_gt = 0, n_eq = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        uint32_t gt = 0, eq = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            gt |= (in[k][j] && c[k][j] > st.c ? 1u : 0u) << j;
            eq |= (in[k][j] && c[k][j] == st.c ? 1u : 0u) << j;
        }
        n_gt += __popc(gt);
        n_eq += __popc(eq);
        // eight lanes hold the 32 rows of a word
        gt <<= 4 * (lane & 7);
        eq <<= 4 * (lane & 7);
#pragma unroll
        for (int off = 1; off < 8; off <<= 1) {
            gt |= __shfl_xor(gt, off);
            eq |= __shfl_xor(eq, off);
        }
        if ((lane & 7) == 0) {
            gt_bits[w0 + (k * kWG + tid) / 8] = gt;
            eq_bits[w0 + (k * kWG + tid) / 8] = eq;
        }
    }
    for (int off = 32; off; off >>= 1) {
        n_gt += __shfl_xor(n_gt, off);
        n_eq += __shfl_xor(n_eq, off);
    }
    if (lane == 0) {
        s_gt[wave] = n_gt;
        s_eq[wave] = n_eq;
    }
    __syncthreads();
    if (tid == 0) {
        n_gt = n_eq = 0;
        for (int w = 0; w < kWG / 64; ++w) {
            n_gt += s_gt[w];
            n_eq += s_eq[w];
        }
        block_totals[(int64_t)t * nb + blk] = make_uint2(n_gt, n_eq);
    }
}

// Totals of kSuper blocks each, for tables of so many blocks that the last step's workgroups
// should not each add up all blocks before theirs.
__global__ __launch_bounds__(64) void sel_super_kernel(const uint2 *__restrict__ block_totals,
                                                       int nb, uint2 *__restrict__ super_totals,
                                                       int ns)
{
    const int t = blockIdx.y, b = blockIdx.x * kSuper + threadIdx.x;
    uint2 v = make_uint2(0u, 0u);
    if (b < nb) v = block_totals[(int64_t)t * nb + b];
    for (int off = 32; off; off >>= 1) {
        v.x += __shfl_xor(v.x, off);
        v.y += __shfl_xor(v.y, off);
    }
    if (threadIdx.x == 0) super_totals[(int64_t)t * ns + blockIdx.x] = v;
}

// Sum over all threads of the workgroup, for every thread.
__device__ __forceinline__ uint2 wg_sum(uint2 v, uint32_t (&s_x)[kWG / 64],
                                        uint32_t (&s_y)[kWG / 64])
{
    for (int off = 32; off; off >>= 1) {
        v.x += __shfl_xor(v.x, off);
        v.y += __shfl_xor(v.y, off);
    }
    __syncthreads();
    if ((threadIdx.x & 63) == 0) {
        s_x[threadIdx.x >> 6] = v.x;
        s_y[threadIdx.x >> 6] = v.y;
    }
    __syncthreads();
    v = make_uint2(0u, 0u);
    for (int w = 0; w < kWG / 64; ++w) {
        v.x += s_x[w];
        v.y += s_y[w];
    }
    return v;
}

// Ids and bitmap of kWriteBlocks blocks, four bitmap words per thread.  Where hot rows are few,
// a thread writes its ids by itself; where a thread of the wavefront has more than kFewIds, its
// lanes take a row each and the ids leave in whole lines (26 x 1 M rows, all of them hot: the share
// rule takes 90 us, 196 with a thread at a time and 136 with three passes over the counters; the
// half of them 125, 174 and 280; 1 x 1000 rows, 100 hot: 50 us either way).
__global__ __launch_bounds__(kWG) void sel_write_kernel(
    const SelState *__restrict__ state, int64_t R, const uint32_t *__restrict__ gt_bits,
    const uint32_t *__restrict__ eq_bits, int nb, const uint2 *__restrict__ block_totals,
    const uint2 *__restrict__ super_totals, int ns, int32_t *const *__restrict__ hot_ids,
    int cap, uint32_t *const *__restrict__ hot_bits, uint32_t *__restrict__ n_hot)
{
    static_assert(kWriteBlocks * kBlockWords == kWG * 4 && kSuper % kWriteBlocks == 0, "");
    __shared__ uint32_t s_x[kWG / 64], s_y[kWG / 64];
    const int t = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int blk0 = blockIdx.x * kWriteBlocks;          // first block of this workgroup
    const int word0 = blk0 * kBlockWords + tid * 4;      // first word of this thread
    uint4 gt = make_uint4(0, 0, 0, 0), eq = gt;
    if (word0 < nb * kBlockWords) {
        const int64_t w = (int64_t)t * nb * kBlockWords + word0;
        gt = *reinterpret_cast<const uint4 *>(gt_bits + w);
        eq = *reinterpret_cast<const uint4 *>(eq_bits + w);
    }
    const uint32_t e = state[t].e;
    // bits before this workgroup's: whole groups of blocks where there are such totals, and
    // blocks
    const uint2 *__restrict__ st = super_totals + (int64_t)t * ns;
    const uint2 *__restrict__ bt = block_totals + (int64_t)t * nb;
    const int sup = ns ? blk0 / kSuper : 0;
    uint2 v = make_uint2(0u, 0u);
    for (int i = tid; i < sup; i += kWG) {
        v.x += st[i].x;
        v.y += st[i].y;
    }
    for (int i = sup * kSuper + tid; i < blk0; i += kWG) {
        v.x += bt[i].x;
        v.y += bt[i].y;
    }
    const uint2 before = wg_sum(v, s_x, s_y);
    if (n_hot && blockIdx.x == 0) {
        v = make_uint2(0u, 0u);
        for (int i = tid; i < (ns ? ns : nb); i += kWG) {
            const uint2 x = ns ? st[i] : bt[i];
            v.x += x.x;
            v.y += x.y;
        }
        v = wg_sum(v, s_x, s_y);
        if (tid == 0) n_hot[t] = v.x + (v.y < e ? v.y : e);
    }
    // ... then those of the threads before this one
    uint32_t g[4] = {gt.x, gt.y, gt.z, gt.w}, q[4] = {eq.x, eq.y, eq.z, eq.w};
    uint32_t n_gt = 0, n_eq = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        n_gt += __popc(g[k]);
        n_eq += __popc(q[k]);
    }
    uint32_t inc_gt = n_gt, inc_eq = n_eq;
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t a = __shfl_up(inc_gt, off), b = __shfl_up(inc_eq, off);
        if (lane >= off) {
            inc_gt += a;
            inc_eq += b;
        }
    }
    __syncthreads();
    if (lane == 63) {
        s_x[wave] = inc_gt;
        s_y[wave] = inc_eq;
    }
    __syncthreads();
    uint32_t gb = before.x + inc_gt - n_gt, qb = before.y + inc_eq - n_eq;
    for (int w = 0; w < wave; ++w) {
        gb += s_x[w];
        qb += s_y[w];
    }
    int32_t *ids = hot_ids ? hot_ids[t] : nullptr;
    uint32_t *bits = hot_bits ? hot_bits[t] : nullptr;
    const int64_t words = (R + 31) >> 5;
    uint32_t take[4], pos[4], n_take = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        // the equal rows that are taken: all of the word's, none, or (in one word of a table)
        // its first few
        const uint32_t left = qb < e ? e - qb : 0u;
        uint32_t not_taken = 0;
        if (left < (uint32_t)__popc(q[k])) {
            not_taken = q[k];
            for (uint32_t i = 0; i < left; ++i) not_taken &= not_taken - 1u;
        }
        take[k] = g[k] | (q[k] ^ not_taken);
        pos[k] = gb + (qb < e ? qb : e);
        n_take += __popc(take[k]);
        if (bits && word0 + k < words) bits[word0 + k] = take[k];
        gb += __popc(g[k]);
        qb += __popc(q[k]);
    }
    if (!ids) return;
    if (!__any(n_take > kFewIds)) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint32_t p = pos[k];
            for (uint32_t todo = take[k]; todo && p < (uint32_t)cap; todo &= todo - 1u)
                ids[p++] = (word0 + k) * 32 + __ffs((int)todo) - 1;
        }
        return;
    }
    // Many: the wavefront writes two words' ids at a time, one lane per row.
    const uint32_t wave_row0 = (uint32_t)(word0 - lane * 4) * 32u;
    const uint32_t below = lane & 31 ? ~0u >> (32 - (lane & 31)) : 0u;
    for (int j0 = 0; j0 < 64; j0 += 4) {
        if (__builtin_amdgcn_readlane(pos[0], j0) >= (uint32_t)cap) return;     // as all that follow
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int j = j0 + i / 2, k = (i & 1) * 2;
            const uint32_t lo = __builtin_amdgcn_readlane(take[k], j);
            const uint32_t hi = __builtin_amdgcn_readlane(take[k + 1], j);
            const uint32_t p0 = __builtin_amdgcn_readlane(pos[k], j);
            const uint32_t mine = lane < 32 ? lo : hi;
            const uint32_t p = p0 + (lane < 32 ? 0u : (uint32_t)__popc(lo)) + __popc(mine & below);
            if ((mine >> (lane & 31)) & 1u && p < (uint32_t)cap)
                ids[p] = (int32_t)(wave_row0 + (j * 4 + k) * 32 + lane);
        }
    }
}

struct SelLayout {
    int nb, ns;
    int64_t n_zero;          // words at the start that begin as zeros
    size_t hist, done, supers, state, block_totals, gt_bits, eq_bits, total;
};

SelLayout make_sel_layout(int T, int64_t R)
{
    SelLayout y;
    y.nb = (int)((R + kBlockRows - 1) / kBlockRows);
    y.ns = y.nb > kManyBlocks ? (y.nb + kSuper - 1) / kSuper : 0;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off += align_up(bytes, 256);
        return o;
    };
    y.done = take((size_t)T * (kRefine + 1) * sizeof(uint32_t));
    y.hist = take((size_t)T * kBins * sizeof(uint32_t));
    y.n_zero = (int64_t)(off / sizeof(uint32_t));
    y.state = take((size_t)T * sizeof(SelState));
    y.supers = take((size_t)T * y.ns * sizeof(uint2));
    y.block_totals = take((size_t)T * y.nb * sizeof(uint2));
    y.gt_bits = take((size_t)T * y.nb * kBlockWords * sizeof(uint32_t));
    y.eq_bits = take((size_t)T * y.nb * kBlockWords * sizeof(uint32_t));
    y.total = off;
    return y;
}

}  // namespace

int32_t launch_count_accesses(int T, const int32_t *idx, int Bcap, int L,
                              const int32_t *n_valid, uint32_t *const *counts,
                              hipStream_t s)
{
    const int64_t nnz = (int64_t)Bcap * L;
    if (nnz == 0) return SS_OK;
    const auto chunks = [&](int per) { return (nnz + per - 1) / per; };
    if (chunks(2048) * T > 0x7fffffffLL)
        return fail(SS_ERR_UNSUPPORTED, "ss_count_accesses: grid too large");
    ProfScope prof("count_kernel", s);
#define SS_COUNT(NT_, I_, SLOTS_)                                                            \
    launch(count_kernel<NT_, I_, SLOTS_>, dim3((unsigned)(chunks(NT_ * I_) * T)), dim3(NT_), s, \
           idx, Bcap, L, n_valid, counts, (int)chunks(NT_ * I_))
    // Rule (us; 1024 x 2 and 1024 x 8 lookups per workgroup, popular rows next to each other / scattered
    // over the table, and 2048 lookups by 256 threads as it once was): 8 tables x 81920 36.0 / 17.1
    // and 21.8 / 15.7, 36.9 / 18.3; 40 x 16384 19.0 / 13.5 and 14.5 / 13.3, 20.0 / 14.5; 26 x 16384
    // 13.5 / 11.8 and 12.6 / 12.1, 13.7 / 12.2; 26 x 8192 8.7 / 6.7 and 10.2 / 10.0, 9.5 / 8.3;
    // 1 x 65536 12.5 / 4.6 and 10.2 / 10.2, 14.2 / 6.3.  (Smaller workgroups send the same popular
    // rows to memory more often: 512 lookups each take 29.8 / 4.9 at 1 x 65536.)
    if (nnz * T >= 64 * 8192) SS_COUNT(1024, 8, 8192);
    else SS_COUNT(1024, 2, 4096);
#undef SS_COUNT
    return check_launch("ss_count_accesses");
}

size_t select_hot_ws_bytes(int T, int64_t R) { return make_sel_layout(T, R).total; }

int32_t launch_select_hot(int T, int64_t R, uint32_t *const *counts, bool top, uint32_t c,
                          uint32_t e, int32_t *const *hot_ids, int cap,
                          uint32_t *const *hot_bits, uint32_t *n_hot, void *ws, hipStream_t s)
{
    const SelLayout y = make_sel_layout(T, R);
    char *w8 = static_cast<char *>(ws);
    SelState *state = reinterpret_cast<SelState *>(w8 + y.state);
    uint32_t *hist = reinterpret_cast<uint32_t *>(w8 + y.hist);
    uint32_t *done = reinterpret_cast<uint32_t *>(w8 + y.done);
    uint32_t *gt = reinterpret_cast<uint32_t *>(w8 + y.gt_bits);
    uint32_t *eq = reinterpret_cast<uint32_t *>(w8 + y.eq_bits);
    uint2 *blocks = reinterpret_cast<uint2 *>(w8 + y.block_totals);
    uint2 *supers = reinterpret_cast<uint2 *>(w8 + y.supers);
    const int64_t n_init = y.n_zero > T ? y.n_zero : T;
    // top-H starts from "nothing decided, e = H still to find"
    launch(sel_init_kernel, dim3((unsigned)((n_init + 255) / 256)), dim3(256), s, state, T, c, e,
           top ? 32 : 0, reinterpret_cast<uint32_t *>(w8), y.n_zero);
    if (top && e > 0) {
        int64_t per_table = (R + 4 * kHistStep - 1) / (4 * kHistStep), most = 1024 / T;
        most = most < 1 ? 1 : most > 256 ? 256 : most;
        if (per_table > most) per_table = most;
        const dim3 grid((unsigned)per_table, T);
        ProfScope prof("sel_hist_kernel", s);
        for (int pass = 0; pass <= (per_table > 1 ? kRefine : 0); ++pass)
            launch(sel_hist_kernel, grid, dim3(kHistThreads), s, counts, R, state, hist, done, pass);
    }
    {
        ProfScope prof("sel_mark_kernel", s);
        launch(sel_mark_kernel, dim3(y.nb, T), dim3(kWG), s, counts, R, (const SelState *)state,
               gt, eq, y.nb, blocks);
    }
    if (y.ns)
        launch(sel_super_kernel, dim3(y.ns, T), dim3(64), s, (const uint2 *)blocks, y.nb, supers,
               y.ns);
    ProfScope prof("sel_write_kernel", s);
    launch(sel_write_kernel, dim3((y.nb + kWriteBlocks - 1) / kWriteBlocks, T), dim3(kWG), s,
           (const SelState *)state, R, (const uint32_t *)gt, (const uint32_t *)eq, y.nb,
           (const uint2 *)blocks, (const uint2 *)supers, y.ns, hot_ids, cap, hot_bits, n_hot);
    return check_launch("ss_select_hot");
}

}  // namespace ss
