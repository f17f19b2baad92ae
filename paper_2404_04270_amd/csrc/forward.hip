// ss_embbag_forward: sum-pooled gather (section 2.1 of the paper: one pooled
// vector per table and sample).
//
// Bound by HBM: every looked-up row is read once (duplicates hit L2 / MALL),
// every pooled row written once, no arithmetic for L = 1.  A group of G lanes
// owns a bag; each lane carries one f4 of the row, so a wavefront reads
// 64/G rows per load instruction with 16-byte accesses that cover whole rows.
// What limits a gather is the number of independent loads in flight, so
//   - one-hot bags (L = 1): a group takes 8 bags, fetches their 8 indices, then
//     issues the 8 row loads back to back before the first store;
//   - multi-hot bags: the row numbers of up to 31 lookups of the bag are fetched
//     first and their row loads issued together (see forward_kernel below).
// All workgroups of a table run on one XCD in the multi-hot kernel, so that its
// hot rows live in one L2 instead of eight: 64 instead of 89 MB fetched from HBM
// per launch at 8 tables x 10M rows x 128, at the same duration (26-27 us).
#include "forward_body.h"
#include "ss_common.h"

namespace ss {

template <int G, typename TS>
__global__ __launch_bounds__(kWG) void forward_onehot_kernel(
    const float *const *__restrict__ weights, const int32_t *__restrict__ idx,
    int Bcap, const int32_t *__restrict__ n_valid, float *__restrict__ out,
    int D4, int tiles_per_table, int pinned_blocks, TS ts)
{
    const unsigned long long trace_t0 = trace_begin<TS>();
    // a table's hot rows are wanted by all its tiles: keep them in one L2
    int t, tile;
    block_to_table_pinned(blockIdx.x, tiles_per_table, pinned_blocks, t, tile);
    forward_onehot_body<G, kWG>(t * tiles_per_table + tile, weights, idx, Bcap, n_valid, out, D4,
                                tiles_per_table);
    trace_end(ts, trace_t0);
}

constexpr int kLongBag = 16;

// Bags of kLongBag lookups and more: all pieces are requested before the first add (up to 31 loads
// in flight per lane), and the rows are added in bag order.  Bags of 32 or more first run full
// rounds of 16.  (The loop body stays in the kernel: as a function of its own the same text
// compiles to piece-by-piece waits where rows leave lanes idle, 20.1 instead of 15.9 us at 14
// tables x 5131 bags of 16 x 40 floats, 41.1 instead of 29.3 at 8 x 8192 of 20 x 88, and 16.2
// and 33.6 with the row numbers waited for all at once.)
template <int G, bool FULL, typename TS>
__global__ __launch_bounds__(kWG) void forward_kernel(
    const float *const *__restrict__ weights, const int32_t *__restrict__ idx,
    int Bcap, int L, const int32_t *__restrict__ n_valid,
    float *__restrict__ out, int D4, int tiles_per_table, int pinned_blocks, TS ts)
{
    constexpr int BAGS = kWG / G;
    const unsigned long long trace_t0 = trace_begin<TS>();
    int t, tile;
    block_to_table_pinned(blockIdx.x, tiles_per_table, pinned_blocks, t, tile);
    const int n = clamp_valid(n_valid, Bcap);
    const int j = tile * BAGS + (int)threadIdx.x / G;
    if (j >= n) return;
    const int c = threadIdx.x % G;
    const uint32_t d4 = FULL ? (uint32_t)G : (uint32_t)D4;
    const auto W = as_global(reinterpret_cast<const f4 *>(weights[t]));
    const int32_t *__restrict__ ip = idx + ((int64_t)t * Bcap + j) * L;
    f4 *__restrict__ o = reinterpret_cast<f4 *>(out) + ((int64_t)t * Bcap + j) * d4;

    for (int col = c; FULL ? col == c : col < D4; col += G) {
        const auto Wc = W + col;            // this lane's f4 of row 0
        f4 acc = f4{0.f, 0.f, 0.f, 0.f};
        const int32_t *__restrict__ q = ip;
        int m = L;
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
        o[col] = acc;
    }
    trace_end(ts, trace_t0);
}

// Bags of fewer than 2^BITS lookups (BITS = 2, 3, 4), V per lane group.
template <int G, bool FULL, int BITS, int V, typename TS>
__global__ __launch_bounds__(kWG) void forward_short_kernel(
    const float *const *__restrict__ weights, const int32_t *__restrict__ idx,
    int Bcap, int L, const int32_t *__restrict__ n_valid,
    float *__restrict__ out, int D4, int tiles_per_table, int pinned_blocks, TS ts)
{
    constexpr int GROUPS = kWG / G;
    const unsigned long long trace_t0 = trace_begin<TS>();
    int t, tile;
    block_to_table_pinned(blockIdx.x, tiles_per_table, pinned_blocks, t, tile);
    const int n = clamp_valid(n_valid, Bcap);
    const int j0 = tile * GROUPS * V + (int)threadIdx.x / G;       // bags j0 + v * GROUPS
    if (j0 >= n) return;
    const int c = threadIdx.x % G;
    const uint32_t d4 = FULL ? (uint32_t)G : (uint32_t)D4;
    const auto W = as_global(reinterpret_cast<const f4 *>(weights[t]));
    const int32_t *__restrict__ ip[V];
#pragma unroll
    for (int v = 0; v < V; ++v) {
        const int j = j0 + v * GROUPS;
        ip[v] = idx + ((int64_t)t * Bcap + (v == 0 || j < n ? j : j0)) * L;
    }
    f4 *__restrict__ o = reinterpret_cast<f4 *>(out) + ((int64_t)t * Bcap + j0) * d4;

    for (int col = c; FULL ? col == c : col < D4; col += G) {
        const auto Wc = W + col;            // this lane's f4 of row 0
        f4 acc[V];
        pool_bags<G, FULL, BITS, V>(Wc, ip, L, d4, acc);
#pragma unroll
        for (int v = 0; v < V; ++v)
            if (v == 0 || j0 + v * GROUPS < n) o[(int64_t)v * GROUPS * d4 + col] = acc[v];
    }
    trace_end(ts, trace_t0);
}

int32_t launch_forward(const ss_tables *tb, const int32_t *idx, int Bcap, int L,
                       const int32_t *n_valid, float *out, hipStream_t s)
{
    const int D4 = tb->dim / 4;
    const int g = lanes_per_row(tb->dim);
    const int groups = kWG / g;
    // Bags of a lane group.  Two of fewer than 8 lookups where that leaves four workgroups per
    // compute unit (us of the kernel with one, two and four per group, bags of 2 or 3, and before
    // the kernels for short bags: 26 tables x 2000 x 36 floats 6.3 / 5.7 / 6.1, then 8.7; 5 x 20000
    // x 208 31.8 / 28.2 / 29.4, 54; but 5 x 777 x 36 4.2 / 4.1 / 4.2, 4.1; 1 x 777 x 1024 4.7 / 5.2
    // / 6.7, 4.6; 1 x 6000 x 208 4.6 / 4.9 / 4.8, 4.5).
    const bool two = L > 1 && L < 8 &&
                     (int64_t)tb->num_tables * ((Bcap + groups - 1) / groups) >= 2048;
    const int bags = groups * (L == 1 ? kOneHotBags : two ? 2 : 1);
    const int tiles = (Bcap + bags - 1) / bags;
    const int64_t blocks = (int64_t)tiles * tb->num_tables;
    if (blocks > 0x7fffffffLL)
        return fail(SS_ERR_UNSUPPORTED, "ss_embbag_forward: grid too large");
    ProfScope prof("forward_kernel", s);
    if (L == 1) {
        SS_DISPATCH_G(g, launch(SS_BOTH(forward_onehot_kernel, G),
                                            dim3((unsigned)blocks), dim3(kWG), s,
                                            tb->weights, idx, Bcap, n_valid, out,
                                            D4, tiles, (tb->num_tables / 8) * 8 * tiles));
    } else {
#define SS_FWD1(K_, ...)                                                               \
    launch(SS_BOTH(K_, G, __VA_ARGS__), dim3((unsigned)blocks), dim3(kWG), s, tb->weights, \
           idx, Bcap, L, n_valid, out, D4, tiles, (tb->num_tables / 8) * 8 * tiles)
#define SS_FWD(F_)                                                                     \
    SS_DISPATCH_G(g, if (L >= kLongBag) { SS_FWD1(forward_kernel, F_); }                \
                     else if (L >= 8) { SS_FWD1(forward_short_kernel, F_, 4, 1); }      \
                     else if (L >= 4 && two) { SS_FWD1(forward_short_kernel, F_, 3, 2); } \
                     else if (L >= 4) { SS_FWD1(forward_short_kernel, F_, 3, 1); }      \
                     else if (two) { SS_FWD1(forward_short_kernel, F_, 2, 2); }         \
                     else { SS_FWD1(forward_short_kernel, F_, 2, 1); })
        if (D4 == g) { SS_FWD(true); } else { SS_FWD(false); }
#undef SS_FWD
#undef SS_FWD1
    }
    return check_launch("ss_embbag_forward");
}

}  // namespace ss
