// Feature normalization of the pooled vectors (section 3.5 of the paper: a
// LayerNorm layer brings every sparse vector to zero mean and unit variance),
// forward and backward.
//
// Both directions are bound by HBM: the forward pass reads x and writes y, the
// backward pass reads dy and x and writes dx (12 bytes per element; the
// statistics and the parameters are noise).  What keeps them from its rate is the
// number of independent loads in flight, so a group asks for several vectors at
// once.  A group of G lanes owns a vector
// and keeps it in registers (one f4 per lane for dim <= 256, up to four for
// dim = 1024), so every element is read once; means are reduced with wavefront
// shuffles, the variance from the centred values (two passes over registers,
// not the E[x^2] - mu^2 form).  The backward pass recomputes x-hat from x, mean
// and rstd instead of storing it.  The parameter gradients are sums over the
// batch: each workgroup adds up its vectors column by column in a fixed order
// and writes one partial row; a second kernel adds the partial rows in index
// order, so dgamma and dbeta do not depend on scheduling.
//
// Both kernels also come in a form that pools the vector from the tables on the
// fly (the sum of the bag's rows, in bag order, exactly as ss_embbag_forward
// forms it) instead of reading it from memory: the pooled tensor is then never
// written nor read, which at 26 x 8192 x 64 takes 109 MB out of the 273 MB the
// two passes move.  One-hot bags have a form of their own (one load of the row
// number and one of the row per vector, those of 4 or 2 vectors together, where
// the bag loop asked for four rows of one bag and then waited): 21.1 instead of
// 28.0 us forward, 25.1 instead of 30.8 backward at 26 x 8192 x 64.  Bags of
// several lookups are pooled by pool_bags (rows of at most 256 floats: all rows
// of a bag of up to 7 at once, longer ones in rounds of 8): 19.9 instead of 25.8
// us forward, 27.5 instead of 49.1 backward at 8 tables x 4096 bags of 20 x 128.
// Longer rows keep the loop that asks for four rows of a bag at a time.
#include "forward_body.h"
#include "ss_common.h"

namespace ss {
namespace {

// P below = f4 per lane: 1 for dim <= 256, up to 4 for dim = 64 lanes * 4 * 4 = 1024

template <int G>
__device__ __forceinline__ float group_sum(float v)
{
#pragma unroll
    for (int off = G / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, G);
    return v;
}

__device__ __forceinline__ float hsum(f4 v) { return (v.x + v.y) + (v.z + v.w); }

// Sums of products, and products that later sums use, with their roundings spelled out:
// which of two products of a sum becomes part of an FMA is otherwise the compiler's choice,
// and the kernels that read their vectors and those that pool them must agree bit for bit.
__device__ __forceinline__ float hdot(f4 a, f4 b)
{
    return fmaf(a.x, b.x, a.y * b.y) + fmaf(a.z, b.z, a.w * b.w);
}
__device__ __forceinline__ f4 fma4(f4 a, f4 b, f4 c)
{
    return f4{fmaf(a.x, b.x, c.x), fmaf(a.y, b.y, c.y), fmaf(a.z, b.z, c.z), fmaf(a.w, b.w, c.w)};
}
template <typename A, typename B>
__device__ __forceinline__ A mul_rounded(A a, B b)
{
#pragma clang fp contract(off)
    return a * b;
}

// loads the lane's share of a vector; lanes / slots past the row read nothing
template <int G, int P>
__device__ __forceinline__ void load_row(const f4 *__restrict__ p, int c, int D4, f4 (&v)[P])
{
#pragma unroll
    for (int i = 0; i < P; ++i) {
        const int col = c + i * G;
        v[i] = f4{0.f, 0.f, 0.f, 0.f};
        if (col < D4) v[i] = p[col];
    }
}

// Where the vectors come from: memory, the one row a one-hot bag names, or the bag of
// rows a vector is the sum of (kBagFull: a row fills its group of lanes exactly).
enum XFrom { kMemory, kOneHot, kBag, kBagFull };
struct XSource {
    const float *x;                  // [T][Bcap][dim]
    const float *const *weights;     // tables
    const int32_t *idx;              // [T][Bcap][L]
    int L;
};

// v = sum over the bag of W_t[idx[t][j][l]][:], rows added in bag order; four
// row loads are in flight at a time.
template <int G, int P>
__device__ __forceinline__ void pool_row(const XSource &src, int t, int64_t vec, int c, int D4,
                                         f4 (&v)[P])
{
    const auto W = as_global(reinterpret_cast<const f4 *>(src.weights[t]));
    const int32_t *__restrict__ ip = src.idx + vec * src.L;
    constexpr int U = 4;
#pragma unroll
    for (int i = 0; i < P; ++i) v[i] = f4{0.f, 0.f, 0.f, 0.f};
    for (int l0 = 0; l0 < src.L; l0 += U) {
        int32_t r[U];
        f4 w[U][P];
#pragma unroll
        for (int u = 0; u < U; ++u) r[u] = ip[l0 + u < src.L ? l0 + u : l0];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < P; ++i) {
                const int col = c + i * G;
                w[u][i] = W[(int64_t)r[u] * D4 + (col < D4 ? col : 0)];
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (l0 + u < src.L) {
#pragma unroll
                for (int i = 0; i < P; ++i) v[i] = (l0 + u == 0) ? w[u][i] : v[i] + w[u][i];
            }
    }
    // lanes and slots past the row loaded column 0 to stay in bounds: they hold zeros,
    // as after load_row
#pragma unroll
    for (int i = 0; i < P; ++i)
        if (c + i * G >= D4) v[i] = f4{0.f, 0.f, 0.f, 0.f};
}

// The V vectors j0 + k * NG of table t (those at n or beyond: vector j0 again, which is
// always valid), everything that does not depend on another load requested at once.
template <int G, int P, int V, XFrom FROM, int BITS>
__device__ __forceinline__ void fetch_x(const XSource &src, int t, int Bcap, int j0, int NG,
                                        int n, int c, int D4, f4 (&v)[V][P])
{
    const int64_t base = (int64_t)t * Bcap;
    if constexpr (FROM == kOneHot) {
        const auto W = as_global(reinterpret_cast<const f4 *>(src.weights[t]));
        const int32_t *__restrict__ ip = src.idx + base;
        int32_t r[V];
#pragma unroll
        for (int k = 0; k < V; ++k) r[k] = ip[j0 + k * NG < n ? j0 + k * NG : j0];
#pragma unroll
        for (int k = 0; k < V; ++k)
#pragma unroll
            for (int i = 0; i < P; ++i) {
                const int col = c + i * G;
                v[k][i] = f4{0.f, 0.f, 0.f, 0.f};
                if (col < D4) v[k][i] = W[(int64_t)r[k] * D4 + col];
            }
    } else {
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const int64_t vec = base + (j0 + k * NG < n ? j0 + k * NG : j0);
            if constexpr (P == 1 && (FROM == kBag || FROM == kBagFull)) {
                // lanes past the row form the sum of column 0 and hold zeros, as after load_row
                const auto Wc = as_global(reinterpret_cast<const f4 *>(src.weights[t])) +
                                (FROM == kBagFull || c < D4 ? c : 0);
                const int32_t *__restrict__ const q[1] = {src.idx + vec * src.L};
                pool_bags<G, FROM == kBagFull, BITS, 1>(Wc, q, src.L, FROM == kBagFull ? G : D4,
                                                        v[k]);
                if (FROM == kBag && c >= D4) v[k][0] = f4{0.f, 0.f, 0.f, 0.f};
            } else if constexpr (FROM == kBag)
                pool_row<G, P>(src, t, vec, c, D4, v[k]);
            else
                load_row<G, P>(reinterpret_cast<const f4 *>(src.x) + vec * D4, c, D4, v[k]);
        }
    }
}

// A group takes V vectors of its tile: all their loads are issued before the first of
// them is normalised, which is what a pass that only streams needs most.  More than four
// (two in the backward pass, which reads twice as much per vector) leave too few
// wavefronts to overlap one's loads with another's stores: 24.5 us with eight and 21.0
// with four forward, 27.9 with four, 24.8 with two and 26.0 with one backward, at 26 x 8192
// one-hot vectors of 64 floats.
template <int P, XFrom FROM> constexpr int ln_fwd_vectors()
{
    return P > 1 || FROM == kBag || FROM == kBagFull ? 1 : 4;
}

template <int G, int P, XFrom FROM, int BITS, bool STREAM>
__global__ __launch_bounds__(kWG) void ln_forward_kernel(
    XSource src, int Bcap, const int32_t *__restrict__ n_valid,
    const float *__restrict__ gamma, const float *__restrict__ beta, float eps,
    float *y, float *__restrict__ mean, float *__restrict__ rstd, int D4)
{
    constexpr int NG = kWG / G, V = ln_fwd_vectors<P, FROM>();
    const int t = blockIdx.y;
    const int64_t tile = blockIdx.x + (int64_t)blockIdx.z * gridDim.x;
    const int n = clamp_valid(n_valid, Bcap);
    const int g = threadIdx.x / G, c = threadIdx.x % G;
    if (tile * NG * V >= n) return;
    const int j0 = (int)tile * NG * V + g;    // vectors j0 + k * NG
    if (j0 >= n) return;                      // whole groups leave together
    const float inv_d = 1.0f / (float)(D4 * 4);

    f4 v[V][P];
    fetch_x<G, P, V, FROM, BITS>(src, t, Bcap, j0, NG, n, c, D4, v);
#pragma unroll
    for (int k = 0; k < V; ++k) {
        const int j = j0 + k * NG;
        if (j >= n) break;
        const int64_t vec = (int64_t)t * Bcap + j;
        f4 *yp = reinterpret_cast<f4 *>(y) + vec * D4;       // may be x's own row
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < P; ++i) s += hsum(v[k][i]);
        const float mu = mul_rounded(group_sum<G>(s), inv_d);
        float q = 0.f;
#pragma unroll
        for (int i = 0; i < P; ++i) {
            if (c + i * G < D4) {
                v[k][i] = v[k][i] - mu;
                q += hdot(v[k][i], v[k][i]);
            }
        }
        const float rs = 1.0f / sqrtf(fmaf(group_sum<G>(q), inv_d, eps));
#pragma unroll
        for (int i = 0; i < P; ++i) {
            const int col = c + i * G;
            if (col < D4) {
                f4 o = v[k][i] * rs;
                if (gamma) o = o * reinterpret_cast<const f4 *>(gamma)[(int64_t)t * D4 + col];
                if (beta) o = o + reinterpret_cast<const f4 *>(beta)[(int64_t)t * D4 + col];
                if (STREAM) __builtin_nontemporal_store(o, &yp[col]);
                else yp[col] = o;
            }
        }
        if (c == 0) {
            mean[vec] = mu;
            rstd[vec] = rs;
        }
    }
}

// Workgroup b of a table takes vectors [b * NG * tiles, (b+1) * NG * tiles); group g takes
// every NG-th of them, V at a time (tiles is a multiple of V).  Partial parameter gradients:
// one row of dim floats per workgroup for dgamma and one for dbeta.
template <int P, XFrom FROM> constexpr int ln_bwd_vectors()
{
    return P > 1 || FROM == kBag || FROM == kBagFull ? 1 : 2;
}

template <int G, int P, XFrom FROM, int BITS>
__global__ __launch_bounds__(kWG) void ln_backward_kernel(
    const float *dy, XSource src, int Bcap,
    const int32_t *__restrict__ n_valid, const float *__restrict__ gamma,
    const float *__restrict__ mean, const float *__restrict__ rstd, float *dx, int D4,
    int tiles, int wgs_per_table, f4 *__restrict__ part_dgamma, f4 *__restrict__ part_dbeta)
{
    constexpr int NG = kWG / G, V = ln_bwd_vectors<P, FROM>();
    __shared__ f4 s_red[kWG];
    const int t = blockIdx.x / wgs_per_table;
    const int wg = blockIdx.x - t * wgs_per_table;
    const int n = clamp_valid(n_valid, Bcap);
    const int g = threadIdx.x / G, c = threadIdx.x % G;
    const float inv_d = 1.0f / (float)(D4 * 4);
    const bool want_params = part_dgamma != nullptr;

    f4 gam[P], acc_g[P], acc_b[P];
#pragma unroll
    for (int i = 0; i < P; ++i) {
        const int col = c + i * G;
        gam[i] = f4{1.f, 1.f, 1.f, 1.f};
        if (gamma && col < D4)
            gam[i] = reinterpret_cast<const f4 *>(gamma)[(int64_t)t * D4 + col];
        acc_g[i] = acc_b[i] = f4{0.f, 0.f, 0.f, 0.f};
    }

    for (int k0 = 0; k0 < tiles; k0 += V) {
        const int j0 = (wg * tiles + k0) * NG + g;         // vectors j0 + k * NG
        if (j0 >= n) break;                   // later vectors of this group are past n too
        f4 xv[V][P], dv[V][P];
        float mu[V], rs[V];
#pragma unroll
        for (int k = 0; k < V; ++k) {
            const int64_t vec = (int64_t)t * Bcap + (j0 + k * NG < n ? j0 + k * NG : j0);
            load_row<G, P>(reinterpret_cast<const f4 *>(dy) + vec * D4, c, D4, dv[k]);
            mu[k] = mean[vec];
            rs[k] = rstd[vec];
        }
        fetch_x<G, P, V, FROM, BITS>(src, t, Bcap, j0, NG, n, c, D4, xv);
#pragma unroll
        for (int k = 0; k < V; ++k) {
            if (j0 + k * NG >= n) break;
            const int64_t vec = (int64_t)t * Bcap + j0 + k * NG;
            float s1 = 0.f, s2 = 0.f;
#pragma unroll
            for (int i = 0; i < P; ++i) {
                if (c + i * G < D4) {
                    xv[k][i] = mul_rounded(xv[k][i] - mu[k], rs[k]);             // x-hat
                    const f4 gd = mul_rounded(gam[i], dv[k][i]);
                    s1 += hdot(gam[i], dv[k][i]);
                    s2 += hdot(gd, xv[k][i]);
                    acc_g[i] = fma4(dv[k][i], xv[k][i], acc_g[i]);
                    acc_b[i] = acc_b[i] + dv[k][i];
                }
            }
            const float m1 = mul_rounded(group_sum<G>(s1), inv_d);
            const float m2 = mul_rounded(group_sum<G>(s2), inv_d);
            f4 *op = reinterpret_cast<f4 *>(dx) + vec * D4;      // may be dy's own row
#pragma unroll
            for (int i = 0; i < P; ++i) {
                const int col = c + i * G;
                if (col < D4) {
                    const f4 gd = fma4(gam[i], dv[k][i], f4{-m1, -m1, -m1, -m1});
                    op[col] = fma4(-xv[k][i], f4{m2, m2, m2, m2}, gd) * rs[k];
                }
            }
        }
    }

    if (!want_params) return;
    // column sums over the NG groups, in group order
    const int64_t prow = ((int64_t)t * wgs_per_table + wg) * D4;
#pragma unroll
    for (int i = 0; i < P; ++i) {
        const int col = c + i * G;
        for (int which = 0; which < 2; ++which) {
            s_red[threadIdx.x] = which == 0 ? acc_g[i] : acc_b[i];
            __syncthreads();
            if (g == 0 && col < D4) {
                f4 tot = s_red[c];
                for (int q = 1; q < NG; ++q) tot = tot + s_red[q * G + c];
                (which == 0 ? part_dgamma : part_dbeta)[prow + col] = tot;
            }
            __syncthreads();
        }
    }
}

// out[t][:] = sum over the workgroups' partial rows.  One workgroup per table and
// f4 column block: thread (part, col) adds every kParts-th partial row starting at
// `part`, then the kParts sums of a column are added in part order; the order is
// fixed by the shape alone.
constexpr int kRedCols = 16;                 // f4 columns per workgroup
constexpr int kParts = kWG / kRedCols;       // 16 partial sums per column

__global__ __launch_bounds__(kWG) void ln_param_reduce_kernel(
    const f4 *__restrict__ part_dgamma, const f4 *__restrict__ part_dbeta,
    int wgs_per_table, int D4, float *__restrict__ dgamma, float *__restrict__ dbeta)
{
    __shared__ f4 s_g[kWG], s_b[kWG];
    const int t = blockIdx.y;
    const int part = threadIdx.x / kRedCols;
    const int col = blockIdx.x * kRedCols + threadIdx.x % kRedCols;
    f4 sg = f4{0.f, 0.f, 0.f, 0.f}, sb = sg;
    if (col < D4) {
        const f4 *__restrict__ pg = part_dgamma + (int64_t)t * wgs_per_table * D4 + col;
        const f4 *__restrict__ pb = part_dbeta + (int64_t)t * wgs_per_table * D4 + col;
#pragma unroll 4
        for (int w = part; w < wgs_per_table; w += kParts) {
            sg = sg + pg[(int64_t)w * D4];
            sb = sb + pb[(int64_t)w * D4];
        }
    }
    s_g[threadIdx.x] = sg;
    s_b[threadIdx.x] = sb;
    __syncthreads();
    if (part == 0 && col < D4) {
        for (int q = 1; q < kParts; ++q) {
            sg = sg + s_g[q * kRedCols + threadIdx.x];
            sb = sb + s_b[q * kRedCols + threadIdx.x];
        }
        if (dgamma) reinterpret_cast<f4 *>(dgamma)[(int64_t)t * D4 + col] = sg;
        if (dbeta) reinterpret_cast<f4 *>(dbeta)[(int64_t)t * D4 + col] = sb;
    }
}

// Backward: vectors per lane group, and workgroups per table.  Eight vectors per group
// keep the partial rows of the parameter gradients few; fewer where that would leave under
// two workgroups per compute unit, each a chain of trips to memory (9 tables x 3001 vectors
// of 36 floats pooled from bags of 5: 12.8 us with two per group, 17.6 with eight; 8 x 1000
// of 512 floats: 11.8 and 17.4).  With the border at 1024 or 1600 workgroups 8 x 4096 x 128
// (bags of 20) takes 27.7 or 30.2 us instead of 25.9.
constexpr int kLnMaxTiles = 8;
constexpr int kLnMinWgs = 512;
constexpr int kMaxTiles = 1 << 23;           // forward: workgroups of a table in one grid dimension

struct BackwardPlan {
    int tiles, wgs;
};

BackwardPlan plan_backward(int T, int dim, int Bcap)
{
    const int ng = kWG / lanes_per_row(dim);
    BackwardPlan p;
    p.tiles = kLnMaxTiles;
    while (p.tiles > 2 && (int64_t)T * Bcap < (int64_t)kLnMinWgs * ng * p.tiles) p.tiles /= 2;
    p.wgs = (Bcap + ng * p.tiles - 1) / (ng * p.tiles);
    return p;
}

// Partial rows of all tables that a workspace holds: at least those of every split of this
// and of every smaller batch, so that a program can size it once for its largest.  (A smaller
// batch may get more workgroups: 26 tables of 64 floats take 64 per table at 4096 vectors and
// 79 at 2520.)  With 8 vectors per group T * ceil(Bcap / 8 ng); with fewer, which takes T * Bcap
// below 2 * kLnMinWgs * ng * tiles, at most T * ceil(Bcap / 2 ng) and under 2 * kLnMinWgs + T.
int64_t partial_rows(int T, int dim, int Bcap)
{
    const int ng = kWG / lanes_per_row(dim);
    const auto wgs = [&](int tiles) { return ((int64_t)Bcap + ng * tiles - 1) / (ng * tiles); };
    const int64_t most = T * wgs(kLnMaxTiles), few = T * wgs(2), split = 2 * kLnMinWgs + T;
    const int64_t fine = few < split ? few : split;
    return most > fine ? most : fine;
}

}  // namespace

int32_t launch_layernorm_forward(int T, int dim, const float *x, const float *const *weights,
                                 const int32_t *idx, int L, int Bcap, const int32_t *n_valid,
                                 const float *gamma, const float *beta, float eps, float *y,
                                 float *mean, float *rstd, hipStream_t s)
{
    const XSource src{x, weights, idx, L};
    const int D4 = dim / 4, g = lanes_per_row(dim);
    const int per_tile = (kWG / g) * (D4 <= g && (x || L == 1) ? 4 : 1);     // as V in the kernel
    const int tiles = (Bcap + per_tile - 1) / per_tile;
    if ((int64_t)tiles * T > 0x7fffffffLL)
        return fail(SS_ERR_UNSUPPORTED, "ss_layernorm_forward: grid too large");
    // A launch's threads in one dimension are counted in 32 bits (without an error: the rest of
    // the grid does not run), and one vector per lane group takes 2^24 workgroups for 64 GiB of y.
    const int slices = (tiles - 1) / kMaxTiles + 1;
    const dim3 grid((unsigned)((tiles - 1) / slices + 1), T, slices);
    // y is streamed past the caches where it would not stay in the L2s anyway: whoever reads it
    // next (the dense model) then loses nothing, and the tables' rows are not pushed out.  us per
    // training step, streamed and not, in a graph: 26 x 32768 x 64 (218 MB) with nobody reading y
    // 280 / 291, with a scaling of it 356 / 363, a transposing copy 377 / 388, a concatenation of
    // its tables 382 / 389; 26 x 8192 x 64 (54 MB) 75.6 / 81.2, 99.0 / 100.8, 104.7 / 108.7, 108.5 /
    // 107.1; 26 x 2048 x 64 (14 MB) 39.2 / 40.4, 45.0 / 45.7, 48.3 / 48.5, 47.8 / 46.8; 26 x 512 x 64
    // (3 MB) 28.9 / 29.0, 32.1 / 32.2, 33.8 / 33.6, 35.7 / 34.4.
    const bool stream_y = !x && (int64_t)T * Bcap * dim * 4 >= 32 << 20;
    ProfScope prof(x ? "ln_forward_kernel" : "ln_forward_pool_kernel", s);
#define SS_LN_FWD2(P_, F_, BITS_, S_)                                                        \
    launch(ln_forward_kernel<G, P_, F_, BITS_, S_>, grid, dim3(kWG), s, src, Bcap, n_valid,  \
           gamma, beta, eps, y, mean, rstd, D4)
#define SS_LN_FWD1(P_, F_, BITS_)                                                            \
    if (stream_y) { SS_LN_FWD2(P_, F_, BITS_, true); } else { SS_LN_FWD2(P_, F_, BITS_, false); }
#define SS_LN_FWD(P_)                                                                        \
    if (x) { SS_LN_FWD2(P_, kMemory, 4, false); }                                            \
    else if (L == 1) { SS_LN_FWD1(P_, kOneHot, 4); }                                         \
    else if constexpr (P_ > 1) { SS_LN_FWD1(P_, kBag, 4); }                                  \
    else if (D4 == g) { SS_DISPATCH_LN_BAG(L, SS_LN_FWD1(1, kBagFull, BITS)); }              \
    else { SS_DISPATCH_LN_BAG(L, SS_LN_FWD1(1, kBag, BITS)); }
    SS_DISPATCH_G(g, if constexpr (G < 64) { SS_LN_FWD(1); } else {
        if (D4 <= 64) { SS_LN_FWD(1); } else if (D4 <= 128) { SS_LN_FWD(2); } else { SS_LN_FWD(4); }
    });
#undef SS_LN_FWD
#undef SS_LN_FWD1
#undef SS_LN_FWD2
    return check_launch("ss_layernorm_forward");
}

size_t layernorm_backward_ws_bytes(int T, int dim, int Bcap)
{
    return align_up((size_t)2 * partial_rows(T, dim, Bcap) * dim * sizeof(float), 256);
}

int32_t launch_layernorm_backward(int T, int dim, const float *dy, const float *x,
                                  const float *const *weights, const int32_t *idx, int L,
                                  int Bcap, const int32_t *n_valid, const float *gamma,
                                  const float *mean, const float *rstd, float *dx,
                                  float *dgamma, float *dbeta, void *ws, hipStream_t s)
{
    const XSource src{x, weights, idx, L};
    const int D4 = dim / 4, g = lanes_per_row(dim);
    const BackwardPlan plan = plan_backward(T, dim, Bcap);
    const int wgs = plan.wgs;
    if ((int64_t)wgs * T > 0x7fffffffLL)
        return fail(SS_ERR_UNSUPPORTED, "ss_layernorm_backward: grid too large");
    const bool params = dgamma || dbeta;
    f4 *pg = params ? static_cast<f4 *>(ws) : nullptr;
    f4 *pb = params ? pg + (size_t)T * wgs * D4 : nullptr;
    {
        ProfScope prof(x ? "ln_backward_kernel" : "ln_backward_pool_kernel", s);
#define SS_LN_BWD1(P_, F_, BITS_)                                                                 \
    launch(ln_backward_kernel<G, P_, F_, BITS_>, dim3((unsigned)(wgs * T)), dim3(kWG), s, dy, src,   \
           Bcap, n_valid, gamma, mean, rstd, dx, D4, plan.tiles, wgs, pg, pb)
#define SS_LN_BWD(P_)                                                                        \
    if (x) { SS_LN_BWD1(P_, kMemory, 4); }                                                   \
    else if (L == 1) { SS_LN_BWD1(P_, kOneHot, 4); }                                         \
    else if constexpr (P_ > 1) { SS_LN_BWD1(P_, kBag, 4); }                                  \
    else if (D4 == g) { SS_DISPATCH_LN_BAG(L, SS_LN_BWD1(1, kBagFull, BITS)); }                 \
    else { SS_DISPATCH_LN_BAG(L, SS_LN_BWD1(1, kBag, BITS)); }
        SS_DISPATCH_G(g, if constexpr (G < 64) { SS_LN_BWD(1); } else {
            if (D4 <= 64) { SS_LN_BWD(1); } else if (D4 <= 128) { SS_LN_BWD(2); } else { SS_LN_BWD(4); }
        });
#undef SS_LN_BWD
#undef SS_LN_BWD1
    }
    if (params)
        launch(ln_param_reduce_kernel, dim3((D4 + kRedCols - 1) / kRedCols, T), dim3(kWG), s,
               (const f4 *)pg, (const f4 *)pb, wgs, D4, dgamma, dbeta);
    return check_launch("ss_layernorm_backward");
}

}  // namespace ss
