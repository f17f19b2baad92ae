// Pooled lookup as device functions: one-hot bags (a kernel of its own, or one role of the
// fused forward + grouping launch) and multi-hot bags (the lookup kernel, and the
// normalization that pools its vectors on the fly).
#pragma once
#include "ss_common.h"

namespace ss {

// block index b -> (table, tile)
__device__ __forceinline__ void block_to_table_tile(int b, int tiles_per_table, int &t,
                                                    int &tile)
{
    t = b / tiles_per_table;
    tile = b - t * tiles_per_table;
}

constexpr int kOneHotBags = 8;     // bags per lane group in the one-hot kernel

// L = 1: a group of G lanes takes kOneHotBags bags, fetches their indices, then issues
// the 8 row loads back to back before the first store.
template <int G, int THREADS>
__device__ __forceinline__ void forward_onehot_body(
    int b, const float *const *__restrict__ weights, const int32_t *__restrict__ idx,
    int Bcap, const int32_t *__restrict__ n_valid, float *__restrict__ out, int D4,
    int tiles_per_table)
{
    constexpr int GROUPS = THREADS / G, BPG = kOneHotBags;
    int t, tile;
    block_to_table_tile(b, tiles_per_table, t, tile);
    const int g = threadIdx.x / G, c = threadIdx.x % G;
    const int j0 = tile * GROUPS * BPG + g;      // bags j0 + k * GROUPS
    if (j0 >= Bcap) return;
    const auto W = as_global(reinterpret_cast<const f4 *>(weights[t]));
    const int32_t *__restrict__ ip = idx + (int64_t)t * Bcap;
    f4 *__restrict__ o = reinterpret_cast<f4 *>(out) + (int64_t)t * Bcap * D4;

    // The index words are requested before the number of valid bags is looked at (it
    // sits in device memory, one more round trip away): every position below Bcap can
    // be read, and what lies past n_valid is replaced by bag j0's index before it is
    // used as a row number.  Those bags store nothing.
    int32_t r[BPG];
#pragma unroll
    for (int k = 0; k < BPG; ++k) {
        const int j = j0 + k * GROUPS;
        r[k] = ip[j < Bcap ? j : j0];
    }
    const int n = clamp_valid(n_valid, Bcap);
    if (j0 >= n) return;
#pragma unroll
    for (int k = 0; k < BPG; ++k)
        if (j0 + k * GROUPS >= n) r[k] = r[0];
    for (int col = c; col < D4; col += G) {
        f4 v[BPG];
#pragma unroll
        for (int k = 0; k < BPG; ++k) v[k] = W[(int64_t)r[k] * D4 + col];
        // The pooled vectors are as many bytes as the rows just read and are not read
        // again on this path: streamed past the caches they leave the gradients and
        // the hot rows of the update that follows in place (26 tables x 8192 bags x 64:
        // the lookup takes 0.5 us longer, the update 1.2 us less).
#pragma unroll
        for (int k = 0; k < BPG; ++k)
            if (j0 + k * GROUPS < n)
                __builtin_nontemporal_store(v[k], &o[(int64_t)(j0 + k * GROUPS) * D4 + col]);
    }
}

// Pieces of a multi-hot bag.  All lanes of a workgroup see the same bag length, so a bag is
// cut into pieces of 16, 8, 4, 2 and 1 lookups by scalar branches on the bits of the length:
// every piece is straight-line code with a known number of row loads.  FULL (a row fills its
// group of lanes exactly) turns the row address into shifts.
template <int N>
__device__ __forceinline__ void fetch_ids(int32_t (&r)[N], const int32_t *__restrict__ ip)
{
#pragma unroll
    for (int k = 0; k < N; ++k) r[k] = ip[k];
}

template <int N, int G, bool FULL, typename P>
__device__ __forceinline__ void fetch_rows(f4 (&v)[N], const int32_t (&r)[N],
                                           P lane_base, uint32_t d4)
{
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = *row_ptr<G, FULL>(lane_base, (uint32_t)r[k], d4);
}

template <int N> __device__ __forceinline__ void unset_rows(f4 (&v)[N])
{
#pragma unroll
    for (int k = 0; k < N; ++k) v[k] = unset_f4();
}

template <int N> __device__ __forceinline__ void add_rows(f4 &acc, const f4 (&v)[N])
{
#pragma unroll
    for (int k = 0; k < N; ++k) acc = acc + v[k];
}

// Makes the compiler wait for a piece's row numbers, and so for all loads before them, and
// compute nothing from them earlier.
template <int N> __device__ __forceinline__ void arrived(int32_t (&r)[N])
{
    if constexpr (N >= 8) {
#pragma unroll
        for (int k = 0; k < N; k += 8)
            asm volatile("" : "+v"(r[k]), "+v"(r[k + 1]), "+v"(r[k + 2]), "+v"(r[k + 3]),
                              "+v"(r[k + 4]), "+v"(r[k + 5]), "+v"(r[k + 6]), "+v"(r[k + 7]));
    } else if constexpr (N == 4) {
        asm volatile("" : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]));
    } else if constexpr (N == 2) {
        asm volatile("" : "+v"(r[0]), "+v"(r[1]));
    } else {
        asm volatile("" : "+v"(r[0]));
    }
}

constexpr int kRounds = 5;

// Sums of the rows of V bags of m lookups each, this lane's f4 of them, in bag order; q[0]
// is a valid bag, q[v] the row numbers of bag v (of bag 0 again where there is none).  BITS:
// m < 2^BITS, or any m >= 8 with BITS = kRounds.  A wavefront's registers are sized for the
// longest bag its kernel may meet: with those of the lookup of long bags (164 to 168: three
// wavefronts per SIMD) a bag of three keeps three loads in flight where there is room for 31,
// so short bags have kernels of their own (the lookup kernel at 2 tables x 32157 bags of 2 x 64
// floats 6.2 instead of 10.0 us, 5 x 29847 of 4 x 208 56 instead of 90), and in large launches
// of the lookup two bags per lane group.
// kRounds: rounds of 8 rows, so more wavefronts beside each other (82 registers; 130 with rounds
// of 16).  The normalization wants that (us of its forward and its backward pass with rounds of
// 16, of 8, and with four rows of one bag at a time as it once had them: 8 tables x 8192 bags of
// 17 x 88 floats 40.7 / 26.9 / 36.5 and 49.1 / 36.8 / 55.4, of 40 x 64 32.6 / 30.2 / 42.2 and
// 39.5 / 38.7 / 90.8), also for bags of 8 to 15 (against all of a bag's rows at once and four at a
// time: 2 x 59010 of 12 x 128 37.4 / 45.1 / 44.3 forward, of 15 x 200 129 / 143 / 141 backward; at
// 8 x 1024 up to 0.6 us slower in the kernel, no slower in a stream); the lookup of long bags does
// not where rows come from memory (rounds of 16: 8 x 4096 bags of 20, 128 floats, 10 M rows: 93 us
// per step, 88 with its own kernel).
template <int G, bool FULL, int BITS, int V, typename P>
__device__ __forceinline__ void pool_bags(P Wc, const int32_t *__restrict__ const (&q0)[V], int m,
                                          uint32_t d4, f4 (&acc)[V])
{
    static_assert(BITS < 4 || V == 1, "long bags are taken one at a time");
    const int32_t *__restrict__ q[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        acc[v] = f4{0.f, 0.f, 0.f, 0.f};
        q[v] = q0[v] + (BITS == kRounds ? m & ~7 : 0);
    }
    // loads come back in the order they were issued: all row numbers first,
    // so that no wait for a row number also waits for rows
    int32_t ra[8] = {}, rb[V][8] = {}, rd[V][4] = {}, re[V][2] = {}, rf[V][1] = {};
    if (BITS == kRounds) fetch_ids(ra, q0[0]);
#define SS_PIECES(DO_)                                                             \
    if (BITS == 4 && (m & 8)) { DO_(rb, b, 8) }                                    \
    if (BITS >= 3 && (m & 4)) { DO_(rd, d, 4) }                                    \
    if (m & 2) { DO_(re, e, 2) }                                                   \
    if (m & 1) { DO_(rf, f, 1) }
#define SS_FETCH_IDS(r_, x_, n_)                                                   \
    _Pragma("unroll") for (int v = 0; v < V; ++v) { fetch_ids(r_[v], q[v]); q[v] += n_; }
#define SS_FETCH_ROWS(r_, x_, n_)                                                  \
    _Pragma("unroll") for (int v = 0; v < V; ++v) fetch_rows<n_, G, FULL>(x_[v], r_[v], Wc, d4);
#define SS_ADD_ROWS(r_, x_, n_)                                                    \
    _Pragma("unroll") for (int v = 0; v < V; ++v) add_rows(acc[v], x_[v]);
    SS_PIECES(SS_FETCH_IDS)
    // All row numbers are waited for here.  Left to the compiler, which does not know which
    // pieces were requested, the wait for a later piece's row numbers covers the rows of the
    // earlier ones.
    if constexpr (BITS == kRounds) arrived(ra);
#pragma unroll
    for (int v = 0; v < V; ++v) {
        if constexpr (BITS == 4) arrived(rb[v]);
        if constexpr (BITS >= 3) arrived(rd[v]);
        arrived(re[v]);
        arrived(rf[v]);
    }
    if constexpr (BITS == kRounds) {
        const int32_t *__restrict__ qa = q0[0];
        for (int left = m >> 3; left > 0; --left) {
            f4 a[8];
            fetch_rows<8, G, FULL>(a, ra, Wc, d4);
            qa += 8;
            if (left > 1) fetch_ids(ra, qa);
            add_rows(acc[0], a);
        }
    }
    f4 b[V][8], d[V][4], e[V][2], f[V][1];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        unset_rows(b[v]); unset_rows(d[v]); unset_rows(e[v]); unset_rows(f[v]);
    }
    SS_PIECES(SS_FETCH_ROWS)
    SS_PIECES(SS_ADD_ROWS)
#undef SS_PIECES
#undef SS_FETCH_IDS
#undef SS_FETCH_ROWS
#undef SS_ADD_ROWS
}

// The normalization's kernel for bags of L lookups: BITS of pool_bags.
#define SS_DISPATCH_LN_BAG(L, ...)                              \
    if ((L) < 4) { constexpr int BITS = 2; __VA_ARGS__; }       \
    else if ((L) < 8) { constexpr int BITS = 3; __VA_ARGS__; }  \
    else { constexpr int BITS = kRounds; __VA_ARGS__; }

}  // namespace ss
