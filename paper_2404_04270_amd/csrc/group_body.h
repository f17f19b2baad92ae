// Grouping of one table's lookups by row, for tables of up to 16384 lookups
// (stage 1 of the backward pass), as a device function so that it can run as a
// kernel of its own or as one role of the fused forward + grouping launch; and the
// pieces it shares with the grouping of larger tables: ranking inside a wavefront,
// the sentinel for stale rows.  (An LSD radix sort in LDS, which only the larger
// tables take, is here too.)
#pragma once
#include "ss_common.h"

namespace ss {

__device__ __forceinline__ uint64_t lanes_below(int lane)
{
    return (1ull << lane) - 1ull;
}

// Lanes of this wavefront whose digit equals mine (all 64 lanes must call).
__device__ __forceinline__ uint64_t match_digit(uint32_t d, int nbits)
{
    uint64_t m = ~0ull;
    for (int b = 0; b < nbits; ++b) {
        const bool one = (d >> b) & 1u;
        const uint64_t bal = __ballot(one);
        m &= one ? bal : ~bal;
    }
    return m;
}

// Stable rank of this lane's key among the keys its wavefront has seen so far
// with the same digit: the lowest lane of each digit group bumps the
// wavefront's LDS counter once for the whole group and hands the old value to
// the others.  cnt points at the wavefront's counters (one per digit).
__device__ __forceinline__ uint32_t wave_rank(uint32_t *cnt, uint32_t d, int nbits,
                                              int lane)
{
    const uint64_t m = match_digit(d, nbits);
    const uint32_t before = __popcll(m & lanes_below(lane));
    uint32_t base = 0;
    if (before == 0) base = atomicAdd(&cnt[d], (uint32_t)__popcll(m));
    base = __shfl(base, __ffsll((long long)m) - 1);
    return base + before;
}

// Gives the sentinel key to lookups of stale rows.  All bitmap words are
// requested before the first one is used.
template <int N>
__device__ __forceinline__ void drop_stale(gptr<const uint32_t> bt, uint32_t (&key)[N])
{
    if (!bt) return;
    uint32_t word[N];
#pragma unroll
    for (int r = 0; r < N; ++r) word[r] = bt[key[r] == kNoRow ? 0u : key[r] >> 5];
#pragma unroll
    for (int r = 0; r < N; ++r)
        if (key[r] != kNoRow && ((word[r] >> (key[r] & 31)) & 1u)) key[r] = kNoRow;
}

// Bits of the pass-th of npass digits when key_bits are split as evenly as
// possible (earlier passes take the extra bits).
__host__ __device__ inline int pass_bits(int key_bits, int npass, int pass)
{
    return key_bits / npass + (pass < key_bits % npass ? 1 : 0);
}

// LSD radix sort, by a workgroup of NT threads, of m <= NT * ITEMS keys that lie in LDS,
// on `bits` key bits from bit `shift` up; stable.  PACKED: s_keys alone is permuted,
// else s_vals with it.  s_cnt: 2 * (NT / 64) * 64 words, s_dig: 64 words.  All threads
// call; on return the sorted keys are visible to all of them.
// Digits of at most 6 bits: one wavefront can then turn the per-wavefront counters into
// offsets with shuffles alone, which leaves three barriers per pass.
template <int NT, int ITEMS, bool PACKED>
__device__ __forceinline__ void lds_lsd_sort(uint32_t *s_keys, uint32_t *s_vals,
                                             uint32_t *s_cnt, uint32_t *s_dig, uint32_t m,
                                             int bits, int shift)
{
    constexpr int NW = NT / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t key[ITEMS], val[PACKED ? 1 : ITEMS], rank[ITEMS];
    const int rounds = ((int)m + NT - 1) / NT;       // keys per thread, <= ITEMS
    const int npass = (bits + 5) / 6;
    for (int i = tid; i < 2 * NW * 64; i += NT) s_cnt[i] = 0;
    __syncthreads();
    for (int pass = 0; pass < npass; ++pass) {
        uint32_t *cnt = s_cnt + (pass & 1) * (NW * 64);       // this pass
        uint32_t *cnt_next = s_cnt + ((pass + 1) & 1) * (NW * 64);
#pragma unroll
        for (int r = 0; r < ITEMS; ++r)
            if (r < rounds) {
                const uint32_t pos = wave * rounds * 64 + r * 64 + lane;
                key[r] = pos < m ? s_keys[pos] : kNoRow;
                if (!PACKED) val[r] = pos < m ? s_vals[pos] : 0u;
            }
        const int nb = pass_bits(bits, npass, pass);
        const uint32_t dmask = (1u << nb) - 1u;
#pragma unroll
        for (int r = 0; r < ITEMS; ++r)
            if (r < rounds) {
                const uint32_t d = (key[r] >> shift) & dmask;
                rank[r] = wave_rank(cnt + wave * 64, d, nb, lane);
            }
        __syncthreads();
        if (wave == 0) {
            // lane d: offsets of the wavefronts for digit d, then digit starts
            uint32_t run = 0;
            if (lane <= (int)dmask)
                for (int w = 0; w < NW; ++w) {
                    const uint32_t c = cnt[w * 64 + lane];
                    cnt[w * 64 + lane] = run;
                    run += c;
                }
            uint32_t incl = run;
            for (int off = 1; off < 64; off <<= 1) {
                const uint32_t up = __shfl_up(incl, off);
                if (lane >= off) incl += up;
            }
            s_dig[lane] = incl - run;
        }
        if (NW == 1 || wave != 0)
            for (int i = NW == 1 ? tid : tid - 64; i < NW * 64; i += NW == 1 ? NT : NT - 64)
                cnt_next[i] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r)
            if (r < rounds) {
                const uint32_t d = (key[r] >> shift) & dmask;
                const uint32_t p = s_dig[d] + cnt[wave * 64 + d] + rank[r];
                if (p < m) {            // padding keys rank behind every real key
                    s_keys[p] = key[r];
                    if (!PACKED) s_vals[p] = val[r];
                }
            }
        __syncthreads();
        shift += nb;
    }
}

// Row ids times an odd constant, modulo a power of two: rows next to each other, and rows a power
// of two apart, are spread evenly over the product's high bits, and the product can be undone.
constexpr uint32_t kMix = 0x9E3779B1u;
constexpr uint32_t inverse_mod_2_32(uint32_t a)
{
    uint32_t x = a;                        // right to 3 bits; each step doubles them
    for (int i = 0; i < 5; ++i) x *= 2u - a * x;
    return x;
}
constexpr uint32_t kUnmix = inverse_mod_2_32(kMix);
static_assert(kMix * kUnmix == 1u, "the product is undone");

// ---------------------------------------------------------------------------
// Grouping of one workgroup's list: equal rows become neighbours, in sample order inside a
// row.  Nothing else is asked of the order, which is what spares a digit pass per six row
// bits: an entry is a word of its own, (row bits << VB) | position of the lookup, so its place
// among the entries of its bucket is the number of smaller ones, whatever order they arrived in.
//
//   1. 64 entries vote for heavy rows (three or more votes), one from each 64th of the list.
//   2. A heavy row's entries are counted per wavefront with a ballot per row, in list order;
//      every other entry takes a place in one of NB buckets (the high row bits) with an LDS
//      atomic.  (With the heavy rows among them the atomics of a bucket would be taken one
//      after the other.)
//   3. One prefix sum over the heavy rows' and the buckets' counts.
//   4. Heavy entries go straight to their place in the output, the others into their
//      bucket in LDS, and then to the place that counting the smaller ones gives.
//
// What bounds it is latency: a chain of five barriers with a trip to LDS or two between
// each, whatever the row bits, where an LSD radix sort takes three barriers and 70
// instructions per entry for every six of them.  The whole launch with the radix sort and
// with this: 15.1 and 9.0 us for 26 tables x 8192 lookups of a million rows, popular rows next to
// each other, 20 and 11 scattered; 42 and 14, 46 and 17 for 26 x 16384; 11 and 7 for 26 x 2048.
//
// load(i) gives entry i of the list (called before the second barrier only, so s_bucket, m entries
// and kBucketPad more, may be where the list lies), keep(entry) whether it is wanted at all;
// emit(i, entry) is called once for every place i below the number of wanted entries, which is
// returned.  All entries are different.  kFew < m <= NT * R.
// ---------------------------------------------------------------------------
constexpr int kMaxHeavy = 16;          // heavy rows looked for
constexpr uint32_t kMinVotes = 3;      // of 64
constexpr uint32_t kVoteMix = 0x85EBCA6Bu;   // odd; its multiples spread over the 32-bit numbers
constexpr int kBucketPad = 8;

template <bool PACKED>
using group_entry = typename std::conditional<PACKED, uint32_t, uint64_t>::type;

template <int NT, int NB> struct GroupScratch {
    static constexpr int NW = NT / 64, HC = kMaxHeavy * NW, N = HC + NB;
    uint32_t cnt[N + 1];
    uint32_t heavy[kMaxHeavy];
    uint32_t n_heavy;
    uint32_t wave_sum[NW];
};

// Sum over the lanes up to and including this one (all 64 lanes call).
__device__ __forceinline__ uint32_t wave_inclusive_sum(uint32_t x)
{
#define SS_DPP_ADD(ctrl, rows) \
    x += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, ctrl, rows, 0xf, false)
    SS_DPP_ADD(0x111, 0xf);            // row_shr:1, 2, 4, 8: within 16 lanes
    SS_DPP_ADD(0x112, 0xf);
    SS_DPP_ADD(0x114, 0xf);
    SS_DPP_ADD(0x118, 0xf);
    SS_DPP_ADD(0x142, 0xa);            // row_bcast:15 into rows 1 and 3
    SS_DPP_ADD(0x143, 0xc);            // row_bcast:31 into rows 2 and 3
#undef SS_DPP_ADD
    return x;
}

// Lanes of the wavefront below this one whose bit is set in a ballot.
__device__ __forceinline__ uint32_t set_below(uint64_t ballot)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(ballot >> 32),
                                     __builtin_amdgcn_mbcnt_lo((uint32_t)ballot, 0u));
}

template <int NT, int R, int NB, typename E, typename Load, typename Keep, typename Emit>
__device__ __forceinline__ uint32_t group_entries(uint32_t m, int VB, int row_bits, E *s_bucket,
                                                  GroupScratch<NT, NB> &s, Load load, Keep keep,
                                                  Emit emit)
{
    constexpr int NW = NT / 64, HC = GroupScratch<NT, NB>::HC, N = GroupScratch<NT, NB>::N;
    constexpr int NBB = ilog2(NB);
    constexpr uint32_t kIsHeavy = 1u << 24;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int bshift = row_bits > NBB ? row_bits - NBB : 0;
    // entry r of a lane is number first + 64 r
    const uint32_t first = wave * (R * 64) + lane;
    E ent[R];
    bool in[R];
#pragma unroll
    for (int r = 0; r < R; ++r) ent[r] = load(first + r * 64 < m ? first + r * 64 : m - 1);
#pragma unroll
    for (int r = 0; r < R; ++r) in[r] = first + r * 64 < m && keep(ent[r]);
    for (int i = tid; i < N; i += NT) s.cnt[i] = 0;
    if (wave == 0) {
        // By a hash where in its 64th: at even distances the votes meet only some of the rows of a
        // list that repeats itself, and the lookups of a row that is not found are compared each
        // with each (64 tables x 8192 bags of the same two ids: 1245 us, 25 so).
        const uint32_t from = (uint32_t)(((uint64_t)lane * m) >> 6), width = m >> 6;
        const uint32_t place = from + __umulhi((uint32_t)(lane + 1) * kVoteMix, width);
        const uint32_t mine = (uint32_t)(load(place) >> VB);
        // the lanes that have a lane's row, by ten bits of a hash ...
        const uint32_t h = (mine * 0x9E3779B1u) >> 22;
        uint64_t same = ~0ull;
#pragma unroll
        for (int b = 0; b < 10; ++b) {
            const bool one = (h >> b) & 1u;
            const uint64_t bal = __ballot(one);
            same &= one ? bal : ~bal;
        }
        // ... and, where these agree for several rows, by the row: each time round a group of lanes
        // loses those that differ from its first.  (Of two heavy rows the second was not found, and
        // its lookups compared each with each: 64 tables x 16384 lookups of two such rows 2469 us,
        // 35 so.  Places by a hash and this take 0.15 us of a launch: 26 x 8192 uniform 5.93 and 6.09, Zipf
        // 7.5 either way, the slowest of 16 batches 9.5 and 7.7.)
        for (;;) {
            const uint32_t row = (uint32_t)__shfl((int)mine, (int)__builtin_ctzll(same));
            const uint64_t differ = __ballot(mine != row);
            if (!differ) break;
            same &= mine != row ? differ : ~differ;
        }
        const bool heavy = set_below(same) == 0 && __popcll(same) >= (int)kMinVotes;
        const uint64_t found = __ballot(heavy);
        const uint32_t at = set_below(found);
        if (heavy && at < kMaxHeavy) s.heavy[at] = mine;
        uint32_t n = __popcll(found);
        n = n < kMaxHeavy ? n : kMaxHeavy;
        if (lane == 0) s.n_heavy = n;
    }
    __syncthreads();

    // 2: slot[r] = place among the wavefront's entries of heavy row k (kIsHeavy * (k + 1)
    // added), or in the bucket
    const uint32_t nh = __builtin_amdgcn_readfirstlane(s.n_heavy);
    uint32_t slot[R];
#pragma unroll
    for (int r = 0; r < R; ++r) slot[r] = 0;
    for (uint32_t k = 0; k < nh; ++k) {
        const uint32_t row = s.heavy[k];
        uint32_t run = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool eq = in[r] && (uint32_t)(ent[r] >> VB) == row;
            const uint64_t bm = __ballot(eq);
            slot[r] = eq ? (k + 1) * kIsHeavy + run + set_below(bm) : slot[r];
            run += __popcll(bm);
        }
        if (lane == 0) s.cnt[k * NW + wave] = run;
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (in[r] && slot[r] < kIsHeavy)
            slot[r] = atomicAdd(&s.cnt[HC + ((uint32_t)(ent[r] >> VB) >> bshift)], 1u);
    __syncthreads();

    // 3: each thread owns PER neighbouring counts
    constexpr int PER = (N + NT - 1) / NT;
    uint32_t c[PER], sum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        c[q] = tid * PER + q < N ? s.cnt[tid * PER + q] : 0u;
        sum += c[q];
    }
    const uint32_t incl = wave_inclusive_sum(sum);
    if (lane == 63) s.wave_sum[wave] = incl;
    __syncthreads();
    uint32_t start = incl - sum;
#pragma unroll
    for (int w = 0; w < NW; ++w) start += w < wave ? s.wave_sum[w] : 0u;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (tid * PER + q < N) s.cnt[tid * PER + q] = start;
        start += c[q];
    }
    if (tid == NT - 1) s.cnt[N] = start;
    __syncthreads();

    // 4
    const uint32_t n_of_heavy = s.cnt[HC], n_rest = s.cnt[N] - n_of_heavy;
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (in[r]) {
            const uint32_t k = slot[r] / kIsHeavy;
            if (k)
                emit(s.cnt[(k - 1) * NW + wave] + slot[r] % kIsHeavy, ent[r]);
            else
                s_bucket[s.cnt[HC + ((uint32_t)(ent[r] >> VB) >> bshift)] - n_of_heavy + slot[r]] =
                    ent[r];
        }
    if (tid < kBucketPad) s_bucket[n_rest + tid] = (E)~(E)0;
    __syncthreads();
    // Buckets ascend with the row bits: entries of earlier buckets are smaller, of later ones
    // larger, so the bucket may be read in whole aligned pieces.
    typedef E piece __attribute__((ext_vector_type(16 / sizeof(E)), aligned(16)));
    constexpr uint32_t PC = 16 / sizeof(E), U = 2;
    const piece *s_piece = reinterpret_cast<const piece *>(s_bucket);
    for (uint32_t i = tid; i < n_rest; i += NT) {
        const E e = s_bucket[i];
        const uint32_t b = (uint32_t)(e >> VB) >> bshift;
        const uint32_t p0 = (s.cnt[HC + b] - n_of_heavy) / PC;
        const uint32_t p1 = (s.cnt[HC + b + 1] - n_of_heavy + PC - 1) / PC;
        uint32_t place = n_of_heavy + p0 * PC;
        for (uint32_t p = p0; p < p1; p += U) {
            piece v[U];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u) v[u] = s_piece[p + u];
#pragma unroll
            for (uint32_t u = 0; u < U; ++u)
#pragma unroll
                for (uint32_t q = 0; q < PC; ++q)
                    place += v[u][q] < e;
        }
        emit(place, e);
    }
    return n_of_heavy + n_rest;
}

// The same for at most 256 entries that lie in s_list (with room for kBucketPad more): each is
// compared with all the others, by NT / 256 neighbouring lanes that share the list between them.
// One barrier, and a chain a quarter as long as that of the buckets (8 tables x 128 lookups: 8.2 us
// with the radix sort, 5.3 with the buckets, 4 so).
constexpr uint32_t kFew = 256;
template <int NT, int NB, typename E, typename Keep, typename Emit>
__device__ __forceinline__ uint32_t group_few(uint32_t m, E *s_list, GroupScratch<NT, NB> &s,
                                              Keep keep, Emit emit)
{
    constexpr int NW = NT / 64;
    constexpr uint32_t PARTS = NT / kFew, PC = 16 / sizeof(E), U = 4;
    static_assert(NT % kFew == 0 && PARTS <= 4, "whole wavefronts, parts within four lanes");
    typedef E piece __attribute__((ext_vector_type(16 / sizeof(E)), aligned(16)));
    const piece *s_piece = reinterpret_cast<const piece *>(s_list);
    const uint32_t tid = threadIdx.x, i = tid / PARTS, part = tid % PARTS;
    E e = (E)~(E)0;
    bool in = false;
    if (i < m) {
        e = s_list[i];
        in = keep(e);
        if (!in && part == 0) s_list[i] = (E)~(E)0;      // above every entry
    }
    if (tid < kBucketPad) s_list[m + tid] = (E)~(E)0;
    const uint64_t wanted = __ballot(in && part == 0);
    if ((tid & 63) == 0) s.wave_sum[tid >> 6] = __popcll(wanted);
    __syncthreads();
    uint32_t place = 0, total = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) total += s.wave_sum[w];
    const uint32_t pieces = (m + PC - 1) / PC;
    for (uint32_t p0 = part; p0 < pieces; p0 += PARTS * U) {
        piece v[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t p = p0 + u * PARTS;
            v[u] = s_piece[p < pieces ? p : pieces];     // (the pad)
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
#pragma unroll
            for (uint32_t q = 0; q < PC; ++q) place += v[u][q] < e;
    }
#pragma unroll
    for (uint32_t off = 1; off < PARTS; off <<= 1) place += __shfl_xor(place, off);
    if (in && part == 0) emit(place, e);
    return total;
}

// ---------------------------------------------------------------------------
// The apply stage needs equal rows to be neighbours, not ascending rows, so a
// table is cut into classes and each class is grouped by a workgroup of its own.
// Every workgroup reads all lookups of its table (cheap at this size), keeps its
// class, and learns from the same read where its class starts in the output (the
// number of lookups in lower classes).  Only the class's own lookups are looked up in
// the bitmap: the stale ones become sentinels at the end of their class.
//
// The class is the high bits of the mixed row id (kMix), the next bits choose the bucket.
//
// PACKED: the remaining row bits and the position of the lookup fit 32 bits, which is then
// all that is grouped: half the LDS and half the registers.  (64-bit entries, 26 tables of 4 M rows x
// 1024 bags of 16, whole launch: 16.4 us; 13.9 packed, at 1 M rows; with the radix sort 39 and 38.
// Per step through the scheduler, rows of 16 floats: 32.0, 30.3; 76 and 67.)
// ---------------------------------------------------------------------------
template <int NT, int ITEMS, bool PACKED>
__device__ __forceinline__ void class_sort_body(
    int cls, int t, const int32_t *__restrict__ idx, int Bcap, int L,
    const int32_t *__restrict__ n_valid, const uint32_t *const *__restrict__ bits,
    int key_bits, int class_bits, int pos_bits, uint2 *__restrict__ out_ent, int NP, int fill)
{
    using E = group_entry<PACKED>;
    constexpr int NW = NT / 64, CAP = NT * ITEMS, NB = NT;
    __shared__ __attribute__((aligned(16))) E s_list[CAP + 64];
    __shared__ GroupScratch<NT, NB> s_group;
    __shared__ uint32_t s_mine[NW], s_below[NW];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = clamp_valid(n_valid, Bcap) * L;
    const int32_t *__restrict__ ip = idx + (int64_t)t * Bcap * L;
    const auto bt = as_global(bits ? bits[t] : nullptr);
    const int rem_bits = key_bits - class_bits, VB = PACKED ? pos_bits : 32;
    const uint32_t kmask = (1u << key_bits) - 1u, rmask = (1u << rem_bits) - 1u;
    const uint32_t lowest = (uint32_t)cls << rem_bits;      // of the class

    uint32_t key[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int pos = (wave * ITEMS + r) * 64 + lane;
        // requested before n is known (it comes from device memory); used only below n
        key[r] = (uint32_t)ip[pos < Bcap * L ? pos : 0];
    }
    // how far above the class's lowest the mixed row lies: in the class up to rmask, in a
    // lower one from -lowest on
    uint32_t above[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int pos = (wave * ITEMS + r) * 64 + lane;
        above[r] = ((key[r] * kMix) & kmask) - lowest;
        if (pos >= n) above[r] = kmask + 1u - lowest;       // in no class and below none
    }
    // keep my class, in order; count the lookups of lower classes
    uint32_t c_mine = 0, c_below = 0, slot[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const uint64_t bm = __ballot(above[r] <= rmask);
        slot[r] = above[r] <= rmask ? c_mine + set_below(bm) : kNoRow;
        c_mine += __popcll(bm);
        c_below += __popcll(__ballot(above[r] >= 0u - lowest && lowest != 0));
    }
    if (lane == 0) {
        s_mine[wave] = c_mine;
        s_below[wave] = c_below;
    }
    __syncthreads();
    uint32_t woff = 0, m = 0, n_below = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        if (w < wave) woff += s_mine[w];
        m += s_mine[w];
        n_below += s_below[w];
    }
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        // (the places behind the list take what is not in it: no branch per lookup)
        const uint32_t at = slot[r] != kNoRow ? woff + slot[r] : (uint32_t)(CAP + lane);
        s_list[at] = ((E)above[r] << VB) | (uint32_t)((wave * ITEMS + r) * 64 + lane);
    }
    __syncthreads();

    uint2 *__restrict__ oe = out_ent + (int64_t)t * NP;
    const auto load = [&](uint32_t i) { return s_list[i]; };
    const auto row_of = [&](E e) { return ((lowest + (uint32_t)(e >> VB)) * kUnmix) & kmask; };
    const auto keep = [&](E e) {
        if (!bt) return true;
        const uint32_t row = row_of(e);
        return ((bt[row >> 5] >> (row & 31)) & 1u) == 0;
    };
    const auto emit = [&](uint32_t i, E e) {
        const uint32_t pos = (uint32_t)(e & (((E)1 << VB) - 1));
        oe[n_below + i] = make_uint2(row_of(e), L == 1 ? pos : pos / (uint32_t)L);
    };
#define SS_GROUP(R_) \
    real = group_entries<NT, R_, NB>(m, VB, rem_bits, s_list, s_group, load, keep, emit)
    uint32_t real = 0;
    if (m <= kFew) real = group_few<NT, NB>(m, s_list, s_group, keep, emit);
    else if (ITEMS == 1 || m <= NT) SS_GROUP(1);
    else if (ITEMS <= 2 || m <= 2 * NT) SS_GROUP(2);
    else if (ITEMS > 2 && m <= 3 * NT) SS_GROUP(3);
    else if (ITEMS <= 4 || m <= 4 * NT) SS_GROUP(4);
    else if (ITEMS > 4 && m <= 6 * NT) SS_GROUP(6);
    else if (ITEMS <= 8 || m <= 8 * NT) SS_GROUP(8);
    else SS_GROUP(16);
#undef SS_GROUP
    // sentinels: the class's stale lookups, and a share of the padding behind the table, up to
    // the last place that the apply stage reads
    for (uint32_t i = n_below + real + tid; i < n_below + m; i += NT) oe[i] = make_uint2(kNoRow, 0u);
    for (int i = n + cls * NT + tid; i < fill; i += NT << class_bits) oe[i] = make_uint2(kNoRow, 0u);
}

// Host side: how the class sort is configured for a table geometry.
struct ClassSortPlan {
    int threads;      // template NT: 512 or 1024
    int items;        // template ITEMS: 1, 2, 4, 8 or 16
    int class_bits;   // log2 of the number of classes
    int pos_bits;     // bits of a lookup's position
    bool packed;      // row bits below the class + position fit 32 bits
};

// Threads: 1024 from 4097 lookups on, 512 below (26 tables x 8192 lookups in 8 classes each 11.4
// and 13.1 us, x 2048 7.7 and 8.2).  Classes: of at most 256 lookups, but no more than leave every
// class a compute unit of its own, as long as a thread has no more than two lookups of its class: all
// classes of a table read all of its lookups (us by the average class of 256 / 512 / 1024 / 2048
// lookups: 8 tables x 4096 7.7 / 8.4 / 10.2, 8 x 16384 17.9 / 12.5 / 13.8, 26 x 2048 7.7 / 7.7 /
// 9.1, 26 x 8192 21 / 15 / 11.4 / 16, 64 x 8192 41 / 25 / 18.4 / 16.4).
// The classes decide the order of the list, and so where runs of equal rows are cut and how their sums
// round: they depend on the batch alone, not on `threads`, with which a caller asks for a workgroup
// size of its own.
inline ClassSortPlan plan_class_sort(int T, int nnz, int key_bits, int threads = 0)
{
    ClassSortPlan p;
    const int own = nnz > 4096 ? 1024 : 512;
    p.threads = threads ? threads : own;
    const int it = (nnz + p.threads - 1) / p.threads;
    p.items = it <= 1 ? 1 : it <= 2 ? 2 : it <= 4 ? 4 : it <= 8 ? 8 : 16;
    p.class_bits = 0;
    while ((256 << p.class_bits) < nnz && p.class_bits < key_bits &&
           (((int64_t)T << (p.class_bits + 1)) <= 256 || (2 * own) << p.class_bits < nnz))
        ++p.class_bits;
    p.pos_bits = 1;
    while ((1 << p.pos_bits) < nnz) ++p.pos_bits;
    p.packed = (key_bits - p.class_bits) + p.pos_bits <= 32;
    return p;
}

}  // namespace ss
