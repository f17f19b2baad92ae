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

// Multi-hot bags.  All lanes of a workgroup see the same bag length, so the bag
// is cut into pieces of 16, 8, 4, 2 and 1 lookups by scalar branches on the bits
// of the length: every piece is straight-line code with a known number of row
// loads, all pieces are requested before the first add (up to 31 loads in
// flight per lane), and the rows are added in bag order.  Bags of 32 lookups or
// more first run full rounds of 16.  FULL (a row fills its group of lanes
// exactly) turns the row address into shifts.
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

// Sum of the rows of a bag of m lookups at q, this lane's f4 of them, in bag order.
template <int G, bool FULL, typename P>
__device__ __forceinline__ f4 pool_bag(P Wc, const int32_t *__restrict__ q, int m, uint32_t d4)
{
    f4 acc = f4{0.f, 0.f, 0.f, 0.f};
    for (; m >= 32; m -= 16, q += 16) {
        int32_t r[16];
        f4 a[16];
        fetch_ids(r, q);
        fetch_rows<16, G, FULL>(a, r, Wc, d4);
        add_rows(acc, a);
    }
    // loads come back in the order they were issued: all row numbers first,
    // so that no wait for a row number also waits for rows
    int32_t ra[16] = {}, rb[8] = {}, rd[4] = {}, re[2] = {}, rf[1] = {};
    if (m & 16) { fetch_ids(ra, q); q += 16; }
    if (m & 8) { fetch_ids(rb, q); q += 8; }
    if (m & 4) { fetch_ids(rd, q); q += 4; }
    if (m & 2) { fetch_ids(re, q); q += 2; }
    if (m & 1) { fetch_ids(rf, q); }
    f4 a[16], b[8], d[4], e[2], f[1];
    unset_rows(a); unset_rows(b); unset_rows(d); unset_rows(e); unset_rows(f);
    if (m & 16) fetch_rows<16, G, FULL>(a, ra, Wc, d4);
    if (m & 8) fetch_rows<8, G, FULL>(b, rb, Wc, d4);
    if (m & 4) fetch_rows<4, G, FULL>(d, rd, Wc, d4);
    if (m & 2) fetch_rows<2, G, FULL>(e, re, Wc, d4);
    if (m & 1) fetch_rows<1, G, FULL>(f, rf, Wc, d4);
    if (m & 16) add_rows(acc, a);
    if (m & 8) add_rows(acc, b);
    if (m & 4) add_rows(acc, d);
    if (m & 2) add_rows(acc, e);
    if (m & 1) add_rows(acc, f);
    return acc;
}

}  // namespace ss
