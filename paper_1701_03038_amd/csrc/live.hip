// Live-state sweeps: the semiring step over the arcs that leave live states.
//
// After a few input symbols only a handful of states of an HMM tagger (or of
// any sparsely connected WFST) carry a finite value: on the 45-tag trigram
// tagger 4 of 2071 states on average, which 8 arcs leave, while the label's
// arc block holds 3450.  The sweeps of sweeps.hip stream the whole block; the
// sweeps here keep the live states as a list and fetch the arcs of
// (label, live source) through an index, so a step costs what its live arcs
// cost.  They are bound by memory latency (one dependent load per step where
// the index is arithmetic, two elsewhere) and by the instructions of a step,
// not by bandwidth, so the design puts one sentence on a wavefront (8 or 16
// lanes of it for narrow labels), many sentences per compute unit, and no
// workgroup barrier in a step; long lists take a workgroup.  4096 sentences of
// the trigram tagger: Viterbi 520 us streaming, 88 here; forward 550 and 98.
// 16384 sentences of the bigram tagger: Viterbi 3500 and 110.
//
// Contributions to one destination meet in an open-addressed table (LDS, or a
// direct table over the states in global memory for long lists).  Every
// combination is order independent: maxima of ordered integers, and sums of
// fixed-point integers, so results have the same bits whatever the schedule,
// the group width or the table.
#pragma once

#include "kernels.h"

namespace wfst {

// One arc as a live step reads it (one 16-byte load); its score is an array
// of its own so that score updates write whole lines.
struct LiveArc {
    int32_t dst;
    int32_t arc;   // arc id
    int32_t src;
    int32_t seg;   // dst's position among the label's destinations (forward segment)
};
// Arcs of (label, source s): when every state has `per` arcs under the label,
// at first + s * per (no lookup); else (per < 0) through the row table
// (entry row + s) or the pair table.
struct LiveLabel {
    int32_t first, per;
    int64_t row;
    int32_t seg_first, n_segs;  // its destinations (forward segments)
};
struct LivePair {  // open-addressed (label, source) -> arcs; label < 0: empty
    int32_t label, src, first, count;
};
struct LiveIndex {
    const LiveArc *arc = nullptr;
    const float *score = nullptr;     // [arc id]
    int32_t listed = 0;               // arcs are listed by (label, source): arc id = position here
    const LiveLabel *label = nullptr;
    const int2 *all = nullptr;        // {first, count} of all arcs of a label
    const int2 *row = nullptr;        // {first, count} per (label, source)
    const LivePair *pair = nullptr;   // ... or hashed
    uint32_t pair_mask = 0;
};

// Score of the arc x at position pos.  L: arcs are listed by (label, source),
// the position is the arc id, and the score is loaded beside the arc; else
// after it (a copy in index order would cost a gather over every arc at each
// score update: 0.8 ms at 50M arcs, against one more load a step).  The two
// are separate kernels: with a branch at run time, every loop waited for all
// its loads in flight each time round, for the sake of the second.
template <bool L>
__device__ __forceinline__ float live_score(const LiveIndex &ix, int32_t pos, const LiveArc &x)
{
    return ix.score[L ? pos : x.arc];
}

__host__ __device__ __forceinline__ uint32_t live_pair_hash(uint32_t label, uint32_t src)
{
    uint32_t h = label * 0x9e3779b1u ^ src * 0x85ebca6bu;
    h ^= h >> 15;
    h *= 0x2c1b3c6du;
    return h ^ (h >> 13);
}

// {first, count} of the arcs of a label leaving state s
__device__ __forceinline__ int2 live_arcs(const LiveIndex &ix, const LiveLabel &l, int32_t a, int32_t s)
{
    if (l.per >= 0) return make_int2(l.first + s * l.per, l.per);
    if (ix.row) return ix.row[l.row + s];
    for (uint32_t h = live_pair_hash((uint32_t)a, (uint32_t)s);; ++h) {  // the table is at most half full
        const LivePair p = ix.pair[h & ix.pair_mask];
        if (p.label < 0) return make_int2(0, 0);
        if (p.label == a && p.src == s) return make_int2(p.first, p.count);
    }
}

// Sentences a sweep works on: all of the batch in processing order, or (n set)
// those an earlier sweep gave up.  Groups take them at a fixed stride: a
// shared queue's atomic costs about 25 ns a sentence on its one address.
struct LiveWork {
    const int32_t *order = nullptr;  // null: 0, 1, 2, ...
    const int32_t *n = nullptr;      // device count; null: B
    int32_t *left = nullptr;         // sentences given up
    int32_t *n_left = nullptr;
};
// Lists of live states (or back-pointers) of every token: entries come from
// one pool in chunks; a group's first chunk is its own (group index), later
// ones are taken with one atomic.
struct LivePool {
    unsigned long long *used = nullptr;
    int64_t cap = 0;
};
constexpr int kLiveChunk = 256;
struct LiveTape {
    int2 *tok = nullptr;         // [N] {first entry, entries} after each token
    int2 *state = nullptr;       // [pool] {state, its position among the label's destinations}
    double *val = nullptr;       // [pool] log alpha
    int32_t *done = nullptr;     // [B] 1: the sentence has a path and its lists are here (2: by the global-memory form)
    double *log_z = nullptr;     // [B]
};

// Table size and list capacity of a group.
struct LiveShape {
    int32_t K = 0;  // live states per step at most (on chip)
    int32_t H = 0;  // table entries
    int32_t rounds = 0;  // a step with more rounds of (lane, 4 arcs) than this is given up
};

// Where contributions to one destination meet: an LDS table indexed by the
// destination's position under the label (labels with few destinations), an
// open-addressed LDS table keyed by state, or a table over all states in
// global memory.
enum LiveTable { kDirect, kHash, kGlobal };

// A group of W lanes working on one sentence.  kGlobal: the whole workgroup.
template <int W, int TB>
struct LiveGroup {
    static constexpr bool GM = TB == kGlobal;
    static_assert(GM || W == 64, "on chip a group is a wavefront");
    int lid;          // lane in the group
    int32_t H, K;
    int32_t *key;             // kHash: [H] state of a table entry, -1 = free
    unsigned long long *mx;   // ordered maximum, 0 = none
    int *cnt;                 // kGlobal: counter in LDS

    __device__ __forceinline__ void sync() const
    {
        if constexpr (GM) {
            __syncthreads();
        } else {  // one wavefront: LDS operations complete in order, only the compiler has to keep it
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    __device__ __forceinline__ bool any(bool p) const
    {
        if constexpr (GM) return __syncthreads_or(p);
        else return __any(p);
    }
    // kHash: the table entry of state d, claimed if it is new (first = this
    // lane claimed it).  The caller keeps the table from filling up.
    __device__ __forceinline__ int claim(int32_t d, bool &first) const
    {
        uint32_t h = ((uint32_t)d * 0x9e3779b1u) >> 7;
        for (;; ++h) {
            const int at = (int)(h & (uint32_t)(H - 1));
            const int old = atomicCAS(&key[at], -1, d);
            first = old == -1;
            if (first || old == d) return at;
        }
    }
    __device__ __forceinline__ int find(int32_t d) const
    {
        for (uint32_t h = ((uint32_t)d * 0x9e3779b1u) >> 7;; ++h) {
            const int at = (int)(h & (uint32_t)(H - 1));
            const int k = key[at];
            if (k == d) return at;
            if (k == -1) return -1;
        }
    }
    // Candidate k for the destination of x: its table entry, and whether it is the first one there
    __device__ __forceinline__ int put(const LiveArc &x, unsigned long long k, bool &first) const
    {
        if constexpr (TB == kHash) {
            const int at = claim(x.dst, first);
            atomicMax(&mx[at], k);
            return at;
        } else {
            const int at = TB == kDirect ? x.seg : x.dst;
            first = atomicMax(&mx[at], k) == 0ull;
            return at;
        }
    }
    __device__ __forceinline__ int at(const LiveArc &x) const
    {
        if constexpr (TB == kHash) return find(x.dst);
        else return TB == kDirect ? x.seg : x.dst;
    }
    __device__ __forceinline__ unsigned long long max_of(int sl) const
    {
        if constexpr (GM) return __hip_atomic_load(&mx[sl], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        else return mx[sl];
    }
    // Consecutive positions for the lanes with p, from n on (n: group-uniform, updated)
    __device__ __forceinline__ int place(bool p, int &n) const
    {
        if constexpr (GM) {
            return p ? atomicAdd(cnt, 1) : 0;
        } else {
            const uint64_t m = __ballot(p);
            const int lane = (int)(threadIdx.x & 63);
            const int at = n + __popcll(m & ((1ull << lane) - 1ull));
            n += __popcll(m);
            return at;
        }
    }
    // log2 of the lanes that share one of n list entries (each takes every
    // 2^share-th arc of it): all W lanes when the list is short
    __device__ __forceinline__ int share(int n) const
    {
        if constexpr (GM) return 0;
        const int bits = n > 1 ? 32 - __clz(n - 1) : 0;
        return bits < 6 ? 6 - bits : 0;
    }
};

template <class T>
__device__ __forceinline__ T gload(const T *p)  // past this CU's cache
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void gstore(unsigned long long *p, unsigned long long v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kLiveGroupThreads = 512;  // the global-memory form
// Fixed point of the shifted exponentials: e in [0, 1] as round(e 2^31); the
// largest term of a sum is exactly 2^31, a term's rounding at most 2^-32 of it.
constexpr float kLiveOne = 2147483648.0f;
__device__ __forceinline__ unsigned int live_fixed(float e) { return (unsigned int)__builtin_rintf(e * kLiveOne); }
constexpr unsigned long long kLivePoison = 1ull << 63;  // a NaN or +inf term went into the sum

__device__ __forceinline__ double live_lse(double m, unsigned long long s)
{
    if (s & kLivePoison) return __builtin_nan("");
    return m + (double)log_e((float)((double)s * (1.0 / 2147483648.0)));
}
// term x under its sum's maximum m (x > -inf) into the sum
__device__ __forceinline__ void live_add_term(unsigned long long *sum, double x, double m)
{
    if (!(x < __builtin_huge_val())) {
        atomicOr(sum, kLivePoison);
        return;
    }
    const unsigned int q = live_fixed(exp_e((float)(x - m)));
    if (q) atomicAdd(sum, (unsigned long long)q);
}
// ... or nothing for x = -inf, without a branch but for NaN and +inf
__device__ __forceinline__ void live_add_any(unsigned long long *sum, double x, double m)
{
    const unsigned int q = x != -__builtin_huge_val() ? live_fixed(exp_e((float)(x - m))) : 0u;
    const bool bad = !(x < __builtin_huge_val());
    atomicAdd(sum, bad ? 0ull : (unsigned long long)q);
    if (bad) atomicOr(sum, kLivePoison);
}
__device__ __forceinline__ unsigned long long live_ord(double x)  // NaN counts as +inf (its sum is poisoned)
{
    return ord_f64(x < __builtin_huge_val() ? x : __builtin_huge_val());
}

// Offsets and tokens of a sentence: WFST_STATUS_*.
template <int W, int TB>
__device__ __forceinline__ int live_check(const LiveGroup<W, TB> &g, const BatchView &bv, int b, int &o0, int &o1)
{
    o0 = bv.offsets[b];
    o1 = bv.offsets[b + 1];
    const bool bad_off = o0 < 0 || o1 < o0 || (int64_t)o1 > bv.N;
    bool bad = false;
    if (!bad_off)
        for (int i = o0 + g.lid; i < o1; i += W) {
            const int a = bv.tokens[i];
            bad |= a < 0 || a >= bv.M;
        }
    bad = g.any(bad);
    return bad_off ? WFST_STATUS_BAD_INPUT : bad ? WFST_STATUS_BAD_TOKEN : WFST_STATUS_OK;
}

// A group's range of the pool for n entries (group-uniform); cap or more: none left.
template <int W, int TB>
__device__ __forceinline__ int64_t live_alloc(const LiveGroup<W, TB> &g, const LivePool &pool, int n, int64_t &at,
                                              int64_t &end, unsigned long long *cell)
{
    if (at + n > end) {
        const unsigned long long want = (unsigned long long)max(n, kLiveChunk);
        if constexpr (TB == kGlobal) {
            __syncthreads();
            if (g.lid == 0) *cell = atomicAdd(pool.used, want);
            __syncthreads();
            at = (int64_t)*cell;
        } else {
            unsigned long long x = 0;
            if (g.lid == 0) x = atomicAdd(pool.used, want);
            at = (int64_t)__shfl(x, 0, W);
        }
        end = at + (int64_t)want;
    }
    const int64_t got = at;
    at += n;
    return got + n <= pool.cap ? got : pool.cap;
}

// Groups of a launch (one a workgroup), this one's index, and its sentences: item, item + groups, ...
__device__ __forceinline__ int live_groups(int &first, int skip = 0)
{
    first = (int)blockIdx.x - skip;
    return (int)gridDim.x - skip;
}

// LDS bytes of a group on chip.
__host__ __device__ constexpr size_t live_viterbi_lds(int K, int H, bool hash)
{
    return (size_t)H * (hash ? 16 : 12) + (size_t)K * 16;
}
__host__ __device__ constexpr size_t live_forward_lds(int K, int H, bool hash)
{
    return (size_t)H * (hash ? 20 : 16) + (size_t)K * 20;
}
__host__ __device__ constexpr size_t live_backward_lds(int K, int H, bool hash)
{
    return (size_t)H * (hash ? 24 : 16) + (size_t)K * (hash ? 24 : 16);
}
// Bytes of a workgroup's slot in the global-memory form.
__host__ __device__ constexpr size_t live_slot(int64_t Q) { return ((size_t)Q * 36 + 255) / 256 * 256; }

// A group's on-chip arrays, one after another.
struct LiveCarve {
    unsigned char *p;
    template <class T>
    __device__ __forceinline__ T *take(int64_t n)
    {
        T *r = reinterpret_cast<T *>(p);
        p += (size_t)n * sizeof(T);
        return r;
    }
};
template <int W, int TB>
__device__ __forceinline__ LiveCarve live_begin(LiveGroup<W, TB> &g, const LiveShape &sh, int32_t Q, unsigned char *lds,
                                                unsigned char *gscratch, int *cnt)
{
    g.lid = threadIdx.x;
    g.cnt = cnt;
    g.key = nullptr;
    if constexpr (TB == kGlobal) {
        g.H = g.K = Q;
        return LiveCarve{gscratch + (size_t)blockIdx.x * live_slot(Q)};
    } else {
        g.H = sh.H;
        g.K = sh.K;
        return LiveCarve{lds};
    }
}

// The arcs of up to W list entries of a workgroup, shared out evenly: numbered
// by a prefix sum over the entries' arc counts, a term's entry found by
// bisection.  Where no entry of the W has more than kLiveSkew arcs, each thread
// takes its own entry's instead.  (One state with 16384 arcs under a label took
// its thread 12 ms a step; the streaming sweeps take 9 us.)
constexpr int kLiveSkew = 16;
constexpr int kLiveStreamArcs = 4096;
// The workgroup form gives a sentence up with more live states than this: the
// streaming sweeps take their turn.  (Ten steps of n states and 4n arcs, forward
// and backward, lists / given up, us.  25011 states, 16 strings: n = Q/8
// 1729 / 6113, Q/4 3537 / 6948, Q/2 7094 / 7636, Q 14668 / 12071.  100003 states,
// 16 strings: Q/4 14645 / 22519, Q/2 32765 / 24554; 256 strings: Q/4
// 75595 / 206190, Q/2 158300 / 80512.)
__host__ __device__ constexpr int32_t live_most(int32_t Q) { return Q / 4 > 1024 ? Q / 4 : 1024; }
template <int W>
struct LiveTile {
    int32_t pre[W], first[W];  // first term of an entry, its first arc minus that
    int32_t tot[W / 64];
    // Numbers the terms of entries with {first, count} rc, one a thread (barriers inside; the total is at most the
    // arcs of a label, so 32 bits hold it).
    __device__ __forceinline__ int number(int2 rc)
    {
        const int lid = threadIdx.x;
        int inc = rc.y;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(inc, o, 64);
            if ((lid & 63) >= o) inc += up;
        }
        if ((lid & 63) == 63) tot[lid >> 6] = inc;
        __syncthreads();
        int off = inc - rc.y, total = 0;
#pragma unroll
        for (int x = 0; x < W / 64; ++x) {
            off += x < (lid >> 6) ? tot[x] : 0;
            total += tot[x];
        }
        pre[lid] = off;
        first[lid] = rc.x - off;
        __syncthreads();
        return total;
    }
    __device__ __forceinline__ int owner(int t) const  // the last entry whose first term is not behind t
    {
        int lo = 0;
#pragma unroll
        for (int step = W / 2; step > 0; step >>= 1)
            if (pre[lo + step] <= t) lo += step;
        return lo;
    }
    // f(entry of the tile, arc position, arc, score) for every term
    template <bool L, class F>
    __device__ __forceinline__ void each(const LiveIndex &ix, int total, F f) const
    {
        for (int t0 = threadIdx.x; t0 < total; t0 += 4 * W) {
            int e[4], pos[4];
            LiveArc x[4];
            float sc[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = min(t0 + u * W, total - 1);
                e[u] = owner(t);
                pos[u] = first[e[u]] + t;
                x[u] = ix.arc[pos[u]];
                sc[u] = live_score<L>(ix, pos[u], x[u]);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (t0 + u * W < total) f(e[u], pos[u], x[u], sc[u]);
        }
    }
};
// f(list entry, arc, score) for every arc of the label leaving the n listed states, by a workgroup
template <int W, bool L, class F>
__device__ __forceinline__ void live_each(const LiveIndex &ix, const LiveLabel &l, int a, const int32_t *state, int n,
                                          LiveTile<W> &tile, F f)
{
    for (int e0 = 0; e0 < n; e0 += W) {
        const int e = e0 + (int)threadIdx.x;
        const int2 rc = e < n ? live_arcs(ix, l, a, state[e]) : make_int2(0, 0);
        if (__syncthreads_or(rc.y > kLiveSkew)) {
            const int total = tile.number(rc);
            tile.template each<L>(ix, total, [&](int k, int, const LiveArc &x, float sc) { f(e0 + k, x, sc); });
            continue;
        }
        for (int r0 = 0; r0 < rc.y; r0 += 4) {
            LiveArc x[4];
            float sc[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (r0 + u < rc.y) {
                    x[u] = ix.arc[rc.x + r0 + u];
                    sc[u] = live_score<L>(ix, rc.x + r0 + u, x[u]);
                }
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (r0 + u < rc.y) f(e, x[u], sc[u]);
        }
    }
}

// What the steps of a sentence need to know beforehand, for 64 of them, one a
// lane, with the next 64 behind them: a step reads its own from registers
// instead of loading token and label one after the other.  A wavefront works on
// one sentence here, so everything is uniform.  Back: step m is that of token
// T - 1 - m, with the list its sources are in.
template <bool Back>
struct LiveWindow {
    int32_t tok[2], first[2], per[2], row_lo[2], row_hi[2], list[2], entries[2];
    int32_t base = 0;
    const BatchView &bv;
    const LiveIndex &ix;
    const int2 *lists;
    const int o0, T;
    __device__ __forceinline__ LiveWindow(const BatchView &b, const LiveIndex &i, const int2 *tok_lists, int off, int n)
        : bv(b), ix(i), lists(tok_lists), o0(off), T(n) {}
    __device__ __forceinline__ void load(int x, int m)  // steps m ... m + 63 into half x
    {
        const int k = min(m + (int)(threadIdx.x & 63), T - 1), i = Back ? T - 1 - k : k;
        tok[x] = bv.tokens[o0 + i];
        if constexpr (Back) {
            const int2 l = lists[o0 + max(i - 1, 0)];
            list[x] = i > 0 ? l.x : 0;
            entries[x] = i > 0 ? l.y : 1;
        }
        const LiveLabel l = ix.label[tok[x]];
        first[x] = l.first;
        per[x] = l.per;
        row_lo[x] = (int32_t)(uint32_t)l.row;
        row_hi[x] = (int32_t)(l.row >> 32);
    }
    __device__ __forceinline__ void start()  // T > 0
    {
        load(0, 0);
        load(1, 64);
    }
    __device__ __forceinline__ void step(int m)  // once for m = 0, 1, ...; then steps m ... m + 63 can be read
    {
        if (m != base + 64) return;
        base = m;
        tok[0] = tok[1], first[0] = first[1], per[0] = per[1], row_lo[0] = row_lo[1], row_hi[0] = row_hi[1];
        if constexpr (Back) list[0] = list[1], entries[0] = entries[1];
        load(1, m + 64);
    }
    __device__ __forceinline__ int32_t get(const int32_t (&v)[2], int m) const
    {
        const int x = __builtin_amdgcn_readfirstlane(m - base);
        return x < 64 ? __builtin_amdgcn_readlane(v[0], x & 63) : __builtin_amdgcn_readlane(v[1], x & 63);
    }
    __device__ __forceinline__ LiveLabel label(int m, int &a) const
    {
        LiveLabel l;
        a = get(tok, m);
        l.first = get(first, m);
        l.per = get(per, m);
        l.row = (int64_t)(((uint64_t)(uint32_t)get(row_hi, m) << 32) | (uint32_t)get(row_lo, m));
        l.seg_first = l.n_segs = 0;
        return l;
    }
};

// =====================================================================
// Viterbi
// =====================================================================
template <int W, int TB, bool L>
__global__ void __launch_bounds__(TB == kGlobal ? W : 64, 4)
live_viterbi(LiveIndex ix, LiveShape sh, int32_t Q, int32_t start, const float *__restrict__ final_score, BatchView bv,
             LiveWork work, LivePool pool, int2 *__restrict__ bp, float *__restrict__ best_score,
             int32_t *__restrict__ best_arcs, int32_t *__restrict__ best_olabels, const int32_t *__restrict__ olabel,
             unsigned char *__restrict__ gscratch)
{
    constexpr int NWV = TB == kGlobal ? W / 64 : 1;
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ int s_cnt;
    __shared__ unsigned long long s_cell, s_red[NWV];
    __shared__ int s_idx[NWV], s_arcs;
    __shared__ LiveTile<TB == kGlobal ? W : 64> s_tile;
    LiveGroup<W, TB> g;
    LiveCarve c = live_begin(g, sh, Q, lds, gscratch, &s_cnt);
    g.mx = c.take<unsigned long long>(g.H);
    if constexpr (TB == kGlobal) c.take<unsigned long long>(Q);  // the forward sweep's sums, which stay zero
    int32_t *pred = c.take<int32_t>(g.H);
    if constexpr (TB == kHash) g.key = c.take<int32_t>(g.H);
    int32_t *cl = c.take<int32_t>(g.K), *cs = c.take<int32_t>(g.K), *fs = c.take<int32_t>(g.K);
    float *fv = c.take<float>(g.K);
    auto clear = [&]() {
        for (int h = g.lid; h < g.H; h += W) {
            g.mx[h] = 0ull;
            if constexpr (TB == kHash) g.key[h] = -1;
        }
    };
    if constexpr (TB != kGlobal) clear();
    g.sync();
    const int32_t limit = work.n ? *work.n : bv.B;
    int item;
    const int stride = live_groups(item);
    int64_t pool_at = TB == kGlobal ? 0 : (int64_t)item * kLiveChunk, pool_end = TB == kGlobal ? 0 : pool_at + kLiveChunk;
    for (; item < limit; item += stride) {
        const int b = work.order ? work.order[item] : item;
        int o0, o1;
        const int st = live_check(g, bv, b, o0, o1);
        if (st != WFST_STATUS_OK) {
            if (g.lid == 0) {
                bv.status[b] = st;
                best_score[b] = WFST_NINF;
            }
            if (st == WFST_STATUS_BAD_TOKEN)
                for (int i = o0 + g.lid; i < o1; i += W) {
                    best_arcs[i] = -1;
                    if (best_olabels) best_olabels[i] = -1;
                }
            continue;
        }
        const int T = o1 - o0;
        if (g.lid == 0) {
            fs[0] = start;
            fv[0] = 0.0f;
        }
        g.sync();
        int n = 1;
        int64_t prev = -1;  // pool position of the current list (-1: the start state)
        bool give_up = false;
        LiveWindow<false> win(bv, ix, nullptr, o0, T);
        if (TB != kGlobal && T > 0) win.start();
        int a_next = TB == kGlobal && T > 0 ? bv.tokens[o0] : 0;
        LiveLabel l_next = TB == kGlobal && T > 0 ? ix.label[a_next] : LiveLabel{};
        int a_next2 = TB == kGlobal && T > 1 ? bv.tokens[o0 + 1] : 0;
        for (int t = 0; t < T && n > 0; ++t) {
            int a = a_next;
            LiveLabel l = l_next;
            if constexpr (TB == kGlobal) {
                a_next = a_next2;
                if (t + 1 < T) l_next = ix.label[a_next];
                if (t + 2 < T) a_next2 = bv.tokens[o0 + t + 2];
            } else {
                win.step(t);
                l = win.label(t, a);
            }
            int nn = 0;
            int rounds = 0;
            if constexpr (TB == kGlobal) {
                if (g.lid == 0) s_cnt = s_arcs = 0;
                __syncthreads();
            }
            if constexpr (TB != kGlobal) {
                // Short lists of sources with few arcs, one arc a lane at most: straight through.  The lane that
                // claims a destination finishes it.
                const int sb = g.share(n), e = g.lid >> sb, sub = g.lid & ((1 << sb) - 1);
                const bool on = e < n;
                const int2 rc = on ? live_arcs(ix, l, a, fs[e]) : make_int2(0, 0);
                if (n <= W && !g.any(rc.y > 1 << sb)) {
                    const float v = on ? fv[e] : (float)0;
                    const bool has = sub < rc.y;
                    const int32_t pos = has ? rc.x + sub : 0;
                    const LiveArc x = ix.arc[pos];
                    const float sc = live_score<L>(ix, pos, x);
                    const float c = v + sc;
                    const bool live = has && c > WFST_NINF;
                    const unsigned long long k =
                        ((unsigned long long)ord_f32(c) << 32) | (0xffffffffu - (uint32_t)(L ? pos : x.arc));
                    bool first = false;
                    int sl = 0;
                    if (live) sl = g.put(x, k, first);
                    const int i = g.place(first, nn);
                    g.sync();
                    // the winner's lane writes the list entry: its place is where the claiming lane put the table entry
                    const bool won = live && g.mx[sl] == k;
                    if (first) pred[sl] = i;
                    g.sync();
                    const int64_t base = live_alloc(g, pool, nn, pool_at, pool_end, &s_cell);
                    const bool fits = base < pool.cap;
                    if (won) {
                        const int j = pred[sl];
                        fs[j] = x.dst;
                        fv[j] = c;
                        if (fits) bp[base + j] = make_int2(L ? pos : x.arc, prev < 0 ? -1 : (int)prev + e);
                        g.mx[sl] = 0ull;
                        if constexpr (TB == kHash) g.key[sl] = -1;
                    }
                    g.sync();
                    n = nn;
                    prev = base;
                    if (fits) continue;
                    give_up = true;
                    break;
                }
            }
            if constexpr (TB == kGlobal) {
                // a step over a quarter of a label's many arcs is the streaming sweep's: it reads little more, and
                // combines in LDS what meets in one place of memory here (16384 arcs into 40 states, 1024 sentences:
                // 3420 us in ten such steps, streaming 320)
                int mine = 0;
                for (int e = g.lid; e < n; e += W) mine += live_arcs(ix, l, a, fs[e]).y;
                if (mine) atomicAdd(&s_arcs, mine);
                __syncthreads();
                const int arcs = s_arcs;
                if (arcs > kLiveStreamArcs && arcs > ix.all[a].y / 4) {
                    give_up = true;
                    break;
                }
                auto key_of = [](float c, int32_t arc) {
                    return ((unsigned long long)ord_f32(c) << 32) | (0xffffffffu - (uint32_t)arc);
                };
                live_each<W, L>(ix, l, a, fs, n, s_tile, [&](int e, const LiveArc &x, float sc) {
                    const float c = fv[e] + sc;
                    if (!(c > WFST_NINF)) return;
                    bool first;
                    const int sl = g.put(x, key_of(c, x.arc), first);
                    if (!first) return;
                    const int at = atomicAdd(&s_cnt, 1);
                    cl[at] = sl;
                    cs[at] = x.dst;
                });
                __syncthreads();
                nn = s_cnt;
                // the winners' list entries
                live_each<W, L>(ix, l, a, fs, n, s_tile, [&](int e, const LiveArc &x, float sc) {
                    const float c = fv[e] + sc;
                    if (!(c > WFST_NINF)) return;
                    const int sl = g.at(x);
                    if (g.max_of(sl) == key_of(c, x.arc)) pred[sl] = e;
                });
            } else {
                // the maximum at every destination; the lanes that share a list entry take up to 4 of its arcs each per
                // round, and the round's winners note their entry (a later round's overwrite it)
                const int sb = g.share(n);
                const int sub = g.lid & ((1 << sb) - 1), S = 1 << sb;
                for (int e0 = 0; e0 < n; e0 += W) {
                    const int e = e0 + (g.lid >> sb);
                    const bool on = e < n;
                    const int2 rc = on ? live_arcs(ix, l, a, fs[e]) : make_int2(0, 0);
                    const float v = on ? fv[e] : 0.0f;
                    for (int r0 = 0; r0 == 0 || g.any(r0 < rc.y); r0 += 4 * S) {
                        if (++rounds > sh.rounds || nn > g.K) {
                            give_up = true;
                            break;
                        }
                        LiveArc x[4];
                        float sc[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int r = r0 + sub + u * S;
                            if (r < rc.y) {
                                x[u] = ix.arc[rc.x + r];
                                sc[u] = live_score<L>(ix, rc.x + r, x[u]);
                            }
                        }
                        int slot[4] = {-1, -1, -1, -1};
                        unsigned long long cand[4] = {0, 0, 0, 0};
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            bool first = false;
                            if (r0 + sub + u * S < rc.y) {
                                const float c = v + sc[u];
                                if (c > WFST_NINF) {
                                    cand[u] = ((unsigned long long)ord_f32(c) << 32) | (0xffffffffu - (uint32_t)x[u].arc);
                                    slot[u] = g.put(x[u], cand[u], first);
                                }
                            }
                            if (u > 0 && !g.any(slot[u] >= 0)) continue;
                            const int at = g.place(first, nn);
                            if (first && at < g.K) {
                                cl[at] = slot[u];
                                cs[at] = x[u].dst;
                            }
                            if (nn > g.K) break;
                        }
                        g.sync();
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            if (slot[u] >= 0 && g.mx[slot[u]] == cand[u]) pred[slot[u]] = e;
                        g.sync();
                    }
                    if (give_up) break;
                }
                if (nn > g.K) give_up = true;
                if (give_up) break;
            }
            g.sync();
            const int64_t base = live_alloc(g, pool, nn, pool_at, pool_end, &s_cell);
            const bool fits = base < pool.cap;
            for (int i = g.lid; i < nn; i += W) {
                const int sl = cl[i];
                const unsigned long long k = g.max_of(sl);
                if (fits)
                    bp[base + i] = make_int2((int32_t)(0xffffffffu - (uint32_t)k), prev < 0 ? -1 : (int)prev + pred[sl]);
                fs[i] = cs[i];
                fv[i] = unord_f32((uint32_t)(k >> 32));
                if constexpr (TB == kGlobal) gstore(&g.mx[sl], 0ull);
                else g.mx[sl] = 0ull;
                if constexpr (TB == kHash) g.key[sl] = -1;
            }
            g.sync();
            n = nn;
            prev = base;
            if (!fits || (TB == kGlobal && n > live_most(Q))) {  // most states live: the streaming sweeps are faster
                give_up = true;
                break;
            }
        }
        if (give_up) {
            if constexpr (TB != kGlobal) {
                clear();
                g.sync();
            }
            if (g.lid == 0) work.left[atomicAdd(work.n_left, 1)] = b;
            continue;
        }
        // final state: the highest score, then the lowest state id
        unsigned long long best = 0ull;
        int at = -1;
        for (int e = g.lid; e < n; e += W) {
            const float f = final_score[fs[e]];
            const float v = fv[e] + f;
            if (f == WFST_NINF || v == WFST_NINF) continue;
            const unsigned long long k = ((unsigned long long)ord_f32(v) << 32) | (0xffffffffu - (uint32_t)fs[e]);
            if (k > best) {
                best = k;
                at = e;
            }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const unsigned long long k = __shfl_xor(best, o, 64);
            const int x = __shfl_xor(at, o, 64);
            if (k > best) {
                best = k;
                at = x;
            }
        }
        if constexpr (TB == kGlobal) {
            if ((threadIdx.x & 63) == 0) {
                s_red[threadIdx.x >> 6] = best;
                s_idx[threadIdx.x >> 6] = at;
            }
            __syncthreads();
            for (int w = 0; w < W / 64; ++w)
                if (s_red[w] > best) {
                    best = s_red[w];
                    at = s_idx[w];
                }
            __syncthreads();
        }
        if (best == 0ull) {
            if (g.lid == 0) {
                bv.status[b] = WFST_STATUS_NO_PATH;
                best_score[b] = WFST_NINF;
            }
            for (int i = o0 + g.lid; i < o1; i += W) {
                best_arcs[i] = -1;
                if (best_olabels) best_olabels[i] = -1;
            }
            continue;
        }
        if (g.lid == 0) {
            bv.status[b] = WFST_STATUS_OK;
            best_score[b] = unord_f32((uint32_t)(best >> 32));
        }
        // backtrace (serial, on device: paper section 5.1)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        if constexpr (TB == kGlobal) __syncthreads();
        if (g.lid == 0 && T > 0) {
            int p = (int)prev + at;
            for (int i = o1 - 1; i >= o0; --i) {
                const int2 x = bp[p];
                best_arcs[i] = x.x;
                p = x.y;
            }
        }
        if (best_olabels) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            if constexpr (TB == kGlobal) __syncthreads();
            else __builtin_amdgcn_wave_barrier();
            for (int i = o0 + g.lid; i < o1; i += W) best_olabels[i] = olabel[best_arcs[i]];
        }
        g.sync();
    }
}

// =====================================================================
// Forward (log semiring)
// =====================================================================
// On-chip tables of the workgroup form, for the steps whose arcs fit them: the
// live sources' (arc, source) terms are numbered by a prefix sum, one thread a
// term, and meet in one hashed table.  A step then costs a few barriers instead
// of atomics in memory; the table over all states is for the steps beyond.
constexpr int kStepTerms = 2048, kStepTable = 4096;
template <bool On>
struct LiveStep {
    static constexpr int W = kLiveGroupThreads;
    unsigned long long mx[kStepTable], sum[kStepTable];
    int32_t key[kStepTable];
    double val[W], list_val[W];       // of the step's sources; of the list it leaves
    int32_t first[W], list_state[W];  // a source's first arc minus its first term
    uint16_t owner[kStepTerms], claimed[kStepTerms];
    int32_t tot[W / 64];
};
template <>
struct LiveStep<false> {};

// One destination's log-sum-exp: the maximum term first (ordered integers),
// then the sum of the shifted exponentials in fixed point.  Terms are
// alpha (FP64) + theta, so no normalisation along the sentence is needed.
template <int W, int TB, bool L>
__global__ void __launch_bounds__(TB == kGlobal ? W : 64, TB == kGlobal ? 2 : 5)
live_forward(LiveIndex ix, LiveShape sh, int32_t Q, int32_t start, const float *__restrict__ final_score, BatchView bv,
             LiveWork work, LivePool pool, LiveTape lt, float *__restrict__ log_z_out,
             unsigned char *__restrict__ gscratch)
{
    constexpr int NWV = TB == kGlobal ? W / 64 : 1;
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ int s_cnt;
    __shared__ unsigned long long s_cell;
    __shared__ double s_rm[NWV];
    __shared__ LiveStep<TB == kGlobal> st_;
    __shared__ LiveTile<TB == kGlobal ? W : 64> s_tile;
    LiveGroup<W, TB> g;
    LiveCarve c = live_begin(g, sh, Q, lds, gscratch, &s_cnt);
    g.mx = c.take<unsigned long long>(g.H);
    unsigned long long *sm = c.take<unsigned long long>(g.H);
    double *fv = c.take<double>(g.K);
    if constexpr (TB == kHash) g.key = c.take<int32_t>(g.H);
    int32_t *cl = c.take<int32_t>(g.K), *cs = c.take<int32_t>(g.K), *fs = c.take<int32_t>(g.K);
    auto clear = [&]() {
        for (int h = g.lid; h < g.H; h += W) {
            g.mx[h] = 0ull;
            sm[h] = 0ull;
            if constexpr (TB == kHash) g.key[h] = -1;
        }
    };
    if constexpr (TB != kGlobal) {
        clear();
    } else {
        for (int h = g.lid; h < kStepTable; h += W) {
            st_.mx[h] = st_.sum[h] = 0ull;
            st_.key[h] = -1;
        }
    }
    g.sync();
    const int32_t limit = work.n ? *work.n : bv.B;
    int item;
    const int stride = live_groups(item);
    int64_t pool_at = TB == kGlobal ? 0 : (int64_t)item * kLiveChunk, pool_end = TB == kGlobal ? 0 : pool_at + kLiveChunk;
    for (; item < limit; item += stride) {
        const int b = work.order ? work.order[item] : item;
        int o0, o1;
        const int st = live_check(g, bv, b, o0, o1);
        if (st != WFST_STATUS_OK) {
            if (g.lid == 0) {
                bv.status[b] = st;
                lt.done[b] = 0;
                log_z_out[b] = WFST_NINF;
                lt.log_z[b] = -__builtin_huge_val();
            }
            continue;
        }
        const int T = o1 - o0;
        if (g.lid == 0) {
            fs[0] = start;
            fv[0] = 0.0;
        }
        g.sync();
        int n = 1;
        bool give_up = false;
        bool in_lds = false;  // (workgroup form) the list is in st_
        LiveWindow<false> win(bv, ix, nullptr, o0, T);
        if (TB != kGlobal && T > 0) win.start();
        int a_next = TB == kGlobal && T > 0 ? bv.tokens[o0] : 0;
        LiveLabel l_next = TB == kGlobal && T > 0 ? ix.label[a_next] : LiveLabel{};
        int a_next2 = TB == kGlobal && T > 1 ? bv.tokens[o0 + 1] : 0;
        for (int t = 0; t < T && n > 0; ++t) {
            int a = a_next;
            LiveLabel l = l_next;
            if constexpr (TB == kGlobal) {
                a_next = a_next2;
                if (t + 1 < T) l_next = ix.label[a_next];
                if (t + 2 < T) a_next2 = bv.tokens[o0 + t + 2];
            } else {
                win.step(t);
                l = win.label(t, a);
            }
            int nn = 0;
            int rounds = 0;
            if constexpr (TB == kGlobal) {
                if (g.lid == 0) s_cnt = 0;
                __syncthreads();
            }
            if constexpr (TB == kGlobal) {
                static_assert(W == kLiveGroupThreads, "one source a thread");
                bool small = n <= W;
                int E = 0;
                if (small) {
                    int2 rc = make_int2(0, 0);
                    double v = 0.0;
                    if (g.lid < n) {
                        rc = live_arcs(ix, l, a, in_lds ? st_.list_state[g.lid] : fs[g.lid]);
                        v = in_lds ? st_.list_val[g.lid] : fv[g.lid];
                    }
                    int inc = rc.y;
#pragma unroll
                    for (int o = 1; o < 64; o <<= 1) {
                        const int up = __shfl_up(inc, o, 64);
                        if ((g.lid & 63) >= o) inc += up;
                    }
                    if ((g.lid & 63) == 63) st_.tot[g.lid >> 6] = inc;
                    const bool huge = __syncthreads_or(rc.y > kStepTerms);  // (the sum stays within 32 bits)
                    int off = inc - rc.y;
#pragma unroll
                    for (int x = 0; x < W / 64; ++x) {
                        off += x < (g.lid >> 6) ? st_.tot[x] : 0;
                        E += st_.tot[x];
                    }
                    small = !huge && E <= kStepTerms;
                    if (small) {
                        st_.first[g.lid] = rc.x - off;
                        st_.val[g.lid] = v;
                        for (int r = 0; r < rc.y; ++r) st_.owner[off + r] = (uint16_t)g.lid;
                    }
                    __syncthreads();
                }
                if (small) {
                    constexpr int R = kStepTerms / W;
                    int sl[R];
                    double y[R];
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const int x = g.lid + r * W;
                        sl[r] = -1;
                        if (x >= E) continue;
                        const int o = st_.owner[x];
                        const int32_t pos = st_.first[o] + x;
                        const LiveArc arc = ix.arc[pos];
                        y[r] = st_.val[o] + (double)live_score<L>(ix, pos, arc);
                        if (y[r] == -__builtin_huge_val()) continue;
                        uint32_t h = ((uint32_t)arc.dst * 0x9e3779b1u) >> 7;
                        for (;; ++h) {  // at most half full
                            const int at = (int)(h & (uint32_t)(kStepTable - 1));
                            const int old = atomicCAS(&st_.key[at], -1, arc.dst);
                            if (old == -1) st_.claimed[atomicAdd(&s_cnt, 1)] = (uint16_t)at;
                            if (old == -1 || old == arc.dst) {
                                sl[r] = at;
                                break;
                            }
                        }
                        atomicMax(&st_.mx[sl[r]], live_ord(y[r]));
                    }
                    __syncthreads();
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        if (sl[r] >= 0) live_add_term(&st_.sum[sl[r]], y[r], unord_f64(st_.mx[sl[r]]));
                    __syncthreads();
                    nn = s_cnt;
                    const int64_t base = live_alloc(g, pool, nn, pool_at, pool_end, &s_cell);
                    const bool fits = base < pool.cap;
                    if (g.lid == 0) lt.tok[o0 + t] = make_int2((int)base, fits ? nn : 0);
                    in_lds = nn <= W;
                    for (int i = g.lid; i < nn; i += W) {
                        const int at = st_.claimed[i];
                        const int32_t d = st_.key[at];
                        const double z = live_lse(unord_f64(st_.mx[at]), st_.sum[at]);
                        st_.mx[at] = st_.sum[at] = 0ull;
                        st_.key[at] = -1;
                        if (fits) {
                            lt.state[base + i] = make_int2(d, 0);
                            lt.val[base + i] = z;
                        }
                        if (in_lds) {
                            st_.list_state[i] = d;
                            st_.list_val[i] = z;
                        } else {
                            fs[i] = d;
                            fv[i] = z;
                        }
                    }
                    __syncthreads();
                    n = nn;
                    if (fits && n <= live_most(Q)) continue;
                    give_up = true;
                    break;
                }
                if (in_lds) {
                    for (int e = g.lid; e < n; e += W) {
                        fs[e] = st_.list_state[e];
                        fv[e] = st_.list_val[e];
                    }
                    in_lds = false;
                    __syncthreads();
                }
            }
            if constexpr (TB != kGlobal) {
                // Short lists of sources with few arcs, one arc a lane at most: straight through.  The lane that
                // claims a destination finishes it.
                const int sb = g.share(n), e = g.lid >> sb, sub = g.lid & ((1 << sb) - 1);
                const bool on = e < n;
                const int2 rc = on ? live_arcs(ix, l, a, fs[e]) : make_int2(0, 0);
                if (n <= W && !g.any(rc.y > 1 << sb)) {
                    const double v = on ? fv[e] : (double)0;
                    const bool has = sub < rc.y;
                    const int32_t pos = has ? rc.x + sub : 0;
                    const LiveArc x = ix.arc[pos];
                    const float sc = live_score<L>(ix, pos, x);
                    const double y = v + (double)sc;
                    const bool live = has && y != -__builtin_huge_val();
                    bool first = false;
                    int sl = 0;
                    if (live) sl = g.put(x, live_ord(y), first);
                    const int i = g.place(first, nn);
                    g.sync();
                    if (live) live_add_term(&sm[sl], y, unord_f64(g.mx[sl]));
                    g.sync();
                    const int64_t base = live_alloc(g, pool, nn, pool_at, pool_end, &s_cell);
                    const bool fits = base < pool.cap;
                    if (g.lid == 0) lt.tok[o0 + t] = make_int2((int)base, fits ? nn : 0);
                    if (first) {
                        const double z = live_lse(unord_f64(g.mx[sl]), sm[sl]);
                        g.mx[sl] = 0ull;
                        sm[sl] = 0ull;
                        if constexpr (TB == kHash) g.key[sl] = -1;
                        fs[i] = x.dst;
                        fv[i] = z;
                        if (fits) {
                            lt.state[base + i] = make_int2(x.dst, TB == kDirect ? sl : 0);
                            lt.val[base + i] = z;
                        }
                    }
                    g.sync();
                    n = nn;
                    if (fits) continue;
                    give_up = true;
                    break;
                }
            }
            if constexpr (TB == kGlobal) {
                live_each<W, L>(ix, l, a, fs, n, s_tile, [&](int e, const LiveArc &x, float sc) {
                    const double y = fv[e] + (double)sc;
                    if (y == -__builtin_huge_val()) return;
                    bool first;
                    const int sl = g.put(x, live_ord(y), first);
                    if (!first) return;
                    const int at = atomicAdd(&s_cnt, 1);
                    cl[at] = sl;
                    cs[at] = x.dst;
                });
                __syncthreads();
                nn = s_cnt;
                live_each<W, L>(ix, l, a, fs, n, s_tile, [&](int e, const LiveArc &x, float sc) {
                    const double y = fv[e] + (double)sc;
                    if (y == -__builtin_huge_val()) return;
                    const int sl = g.at(x);
                    live_add_term(&sm[sl], y, unord_f64(g.max_of(sl)));
                });
            } else {
                // first pass: the maximum at every destination; the lanes that share a list entry take up to 4 of its
                // arcs each per round
                int slot[4];
                double term[4];
                const int sb = g.share(n);
                const int sub = g.lid & ((1 << sb) - 1), S = 1 << sb;
                for (int e0 = 0; e0 < n; e0 += W) {
                    const int e = e0 + (g.lid >> sb);
                    const bool on = e < n;
                    const int2 rc = on ? live_arcs(ix, l, a, fs[e]) : make_int2(0, 0);
                    const double v = on ? fv[e] : 0.0;
                    for (int r0 = 0; r0 == 0 || g.any(r0 < rc.y); r0 += 4 * S) {
                        if (++rounds > sh.rounds || nn > g.K) {
                            give_up = true;
                            break;
                        }
                        LiveArc x[4];
                        float sc[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int r = r0 + sub + u * S;
                            if (r < rc.y) {
                                x[u] = ix.arc[rc.x + r];
                                sc[u] = live_score<L>(ix, rc.x + r, x[u]);
                            }
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            bool first = false;
                            slot[u] = -1;
                            if (r0 + sub + u * S < rc.y) {
                                term[u] = v + (double)sc[u];
                                if (term[u] != -__builtin_huge_val()) slot[u] = g.put(x[u], live_ord(term[u]), first);
                            }
                            if (u > 0 && !g.any(slot[u] >= 0)) continue;
                            const int at = g.place(first, nn);
                            if (first && at < g.K) {
                                cl[at] = slot[u];
                                cs[at] = x[u].dst;
                            }
                            if (nn > g.K) break;
                        }
                    }
                    if (give_up) break;
                }
                if (nn > g.K) give_up = true;
                g.sync();
                if (give_up) break;
                if (rounds == 1) {  // the terms are still in registers
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (slot[u] >= 0) live_add_term(&sm[slot[u]], term[u], unord_f64(g.mx[slot[u]]));
                } else {  // shared the same way, two arcs a lane at a time
                    for (int e0 = 0; e0 < n; e0 += W) {
                        const int e = e0 + (g.lid >> sb);
                        const bool on = e < n;
                        const int2 rc = on ? live_arcs(ix, l, a, fs[e]) : make_int2(0, 0);
                        const double v = on ? fv[e] : 0.0;
                        for (int r = sub; r < rc.y; r += 2 * S) {
                            const int32_t p0 = rc.x + r, p1 = r + S < rc.y ? p0 + S : p0;
                            const LiveArc x0 = ix.arc[p0], x1 = ix.arc[p1];
                            const double y0 = v + (double)live_score<L>(ix, p0, x0), y1 = v + (double)live_score<L>(ix, p1, x1);
                            if (y0 != -__builtin_huge_val()) {
                                const int sl = g.at(x0);
                                live_add_term(&sm[sl], y0, unord_f64(g.mx[sl]));
                            }
                            if (p1 != p0 && y1 != -__builtin_huge_val()) {
                                const int sl = g.at(x1);
                                live_add_term(&sm[sl], y1, unord_f64(g.mx[sl]));
                            }
                        }
                    }
                }
            }
            g.sync();
            const int64_t base = live_alloc(g, pool, nn, pool_at, pool_end, &s_cell);
            const bool fits = base < pool.cap;
            if (g.lid == 0) lt.tok[o0 + t] = make_int2((int)base, fits ? nn : 0);
            for (int i = g.lid; i < nn; i += W) {
                const int sl = cl[i];
                const double v = live_lse(unord_f64(g.max_of(sl)), TB == kGlobal ? gload(&sm[sl]) : sm[sl]);
                if (fits) {
                    lt.state[base + i] = make_int2(cs[i], TB == kDirect ? sl : 0);
                    lt.val[base + i] = v;
                }
                fs[i] = cs[i];
                fv[i] = v;
                if constexpr (TB == kGlobal) {
                    gstore(&g.mx[sl], 0ull);
                    gstore(&sm[sl], 0ull);
                } else {
                    g.mx[sl] = 0ull;
                    sm[sl] = 0ull;
                }
                if constexpr (TB == kHash) g.key[sl] = -1;
            }
            g.sync();
            n = nn;
            if (!fits || (TB == kGlobal && n > live_most(Q))) {  // most states live: the streaming sweeps are faster
                give_up = true;
                break;
            }
        }
        if constexpr (TB == kGlobal) {
            if (in_lds && !give_up) {
                for (int e = g.lid; e < n; e += W) {
                    fs[e] = st_.list_state[e];
                    fv[e] = st_.list_val[e];
                }
                __syncthreads();
            }
        }
        if (give_up) {
            if constexpr (TB != kGlobal) {
                clear();
                g.sync();
            }
            if (g.lid == 0) {
                lt.done[b] = 0;
                work.left[atomicAdd(work.n_left, 1)] = b;
            }
            continue;
        }
        // log Z = LSE over the live states of alpha + f: the largest term, then the
        // fixed-point sum (order independent, like the steps)
        double m = -__builtin_huge_val();
        bool poison = false;
        for (int e = g.lid; e < n; e += W) {
            const float f = final_score[fs[e]];
            const double x = fv[e] + (double)f;
            if (f == WFST_NINF) continue;
            poison |= !(x < __builtin_huge_val());
            m = fmax(m, x);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
        poison = g.any(poison);
        if constexpr (TB == kGlobal) {
            if ((threadIdx.x & 63) == 0) s_rm[threadIdx.x >> 6] = m;
            __syncthreads();
            for (int w = 0; w < W / 64; ++w) m = fmax(m, s_rm[w]);
            if (threadIdx.x == 0) s_cell = 0ull;
            __syncthreads();
        }
        unsigned long long s = 0;
        if (m != -__builtin_huge_val())
            for (int e = g.lid; e < n; e += W) {
                const float f = final_score[fs[e]];
                if (f == WFST_NINF) continue;
                s += live_fixed(exp_e((float)((fv[e] + (double)f) - m)));
            }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if constexpr (TB == kGlobal) {
            if ((threadIdx.x & 63) == 0) atomicAdd(&s_cell, s);
            __syncthreads();
            s = s_cell;
            __syncthreads();
        }
        if (g.lid == 0) {
            if (m == -__builtin_huge_val() && !poison) {
                bv.status[b] = WFST_STATUS_NO_PATH;
                lt.done[b] = 0;
                log_z_out[b] = WFST_NINF;
                lt.log_z[b] = -__builtin_huge_val();
            } else {
                const double lz = poison ? __builtin_nan("") : live_lse(m, s);
                bv.status[b] = WFST_STATUS_OK;
                lt.done[b] = TB == kGlobal ? 2 : 1;
                log_z_out[b] = (float)lz;
                lt.log_z[b] = lz;
            }
        }
        g.sync();
    }
}

// =====================================================================
// Backward, with expected counts
// =====================================================================
struct LiveCounts {
    unsigned long long *acc = nullptr;     // [arcs in index order] fixed-point sums, zero between calls
    int32_t *touched = nullptr;            // positions with a contribution (repeats allowed, -1: unused; null: not kept)
    unsigned long long *n_touched = nullptr;
    int64_t touched_cap = 0;
    const double *scale = nullptr;         // 2^S
    const float *grad_log_z = nullptr;     // g_b (null = 1)
    unsigned long long *fin = nullptr;     // [fin_words][Q] final-state posteriors (null: not wanted)
    int32_t Q = 0;
    int32_t fin_shift = 4;                 // log2 of the exponents that share a word
};

// Final-state posteriors are FP32 terms of any size (a weight g_b times a
// posterior), so no one scale suits them all: a state's terms are summed
// exactly, as integers, in one 64-bit word per 2^shift binary exponents, and
// rounded once in the end.  A term is below 2^(24 + 2^shift - 1) there and a
// sentence adds one term to a state, so 2^24 sentences fit shift 4 and 2^31
// shift 3.  The last word has the signs of infinite terms, and NaN.  Words of
// one range lie side by side: a sentence's terms are mostly of like size, and
// neighbours share lines (512 sentences that end in 2000 states each: 60 us
// less than with a state's words together).  (Fixed
// point at the counts' scale lost weights far below 1: 2^-46 and less were 0.)
__host__ __device__ constexpr int fin_words(int shift) { return (256 >> shift) + 1; }
__device__ __forceinline__ void fin_add(const LiveCounts &ct, int32_t s, float v)
{
    const uint32_t u = __float_as_uint(v), e = (u >> 23) & 255u, frac = u & 0x7fffffu;
    unsigned long long *w = ct.fin + s;
    if (e == 255u) {
        atomicOr(&w[(int64_t)(256 >> ct.fin_shift) * ct.Q], frac ? 4ull : (u >> 31) ? 2ull : 1ull);
        return;
    }
    if (!(u << 1)) return;
    const uint32_t at = e ? e : 1u;  // value = m 2^(at - 150)
    const long long m = (long long)(e ? frac | 0x800000u : frac) << (at & ((1u << ct.fin_shift) - 1u));
    atomicAdd(&w[(int64_t)(at >> ct.fin_shift) * ct.Q], (unsigned long long)((u >> 31) ? -m : m));
}
__device__ __forceinline__ float fin_value(const LiveCounts &ct, int32_t s)
{
    const int n = 256 >> ct.fin_shift;
    double x = 0.0;
    for (int k0 = 0; k0 < n; k0 += 16) {  // (16 or 32 words)
        unsigned long long w[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) w[k] = ct.fin[(int64_t)(k0 + k) * ct.Q + s];
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (w[k]) x += ldexp((double)(long long)w[k], ((k0 + k) << ct.fin_shift) - 150);
    }
    const unsigned long long f = ct.fin[(int64_t)n * ct.Q + s];
    return f == 0ull ? (float)x : f == 1ull ? (float)__builtin_huge_val() : f == 2ull ? WFST_NINF : (float)__builtin_nan("");
}

// The gradient is zero-filled by the first workgroups of the backward sweep's
// launch, beside the sweep: the fill is bound by memory (127 us for the 218M
// arcs of the large tagger, as a launch of its own), the sweep by latency.
struct GradFill {
    float *p = nullptr;
    int64_t n = 0;
    int32_t blocks = 0;
};
__device__ __forceinline__ void live_fill_grad(const GradFill &gf)
{
    typedef float v4f __attribute__((ext_vector_type(4)));
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gf.blocks * blockDim.x;
    const int64_t head = min(gf.n, (int64_t)((16 - ((uintptr_t)gf.p & 15)) & 15) / 4), quads = (gf.n - head) / 4;
    v4f *q = reinterpret_cast<v4f *>(gf.p + head);
    for (int64_t x = i; x < quads; x += step) __builtin_nontemporal_store((v4f){0.0f, 0.0f, 0.0f, 0.0f}, q + x);
    if (i < head) gf.p[i] = 0.0f;
    if (i < gf.n - head - 4 * quads) gf.p[head + 4 * quads + i] = 0.0f;
}

// The lists of the forward pass, from the last token back: the lanes that
// share a live source take its arcs, look their destinations' beta up in the
// table of the step after, and combine them as the forward step does; the
// source's beta goes to the table of the step before.  Nothing a step loads
// depends on beta, so its arcs are loaded two steps ahead and its list entries
// three (one step ahead, with the registers moved along: 130 us for the 4096
// sentences of the trigram tagger, every step waiting for its loads).
template <int W, int TB, bool L>
__global__ void __launch_bounds__(64)
live_backward(LiveIndex ix, LiveShape sh, int32_t Q, int32_t start, const float *__restrict__ final_score, BatchView bv,
              LiveWork work, LiveTape lt, LiveCounts ct, GradFill gf)
{
    extern __shared__ __align__(16) unsigned char lds[];
    if ((int)blockIdx.x < gf.blocks) return live_fill_grad(gf);
    LiveGroup<W, TB> g;
    LiveCarve c = live_begin(g, sh, Q, lds, nullptr, nullptr);
    double *val0 = c.take<double>(g.H), *val1 = c.take<double>(g.H);
    unsigned long long *bm = c.take<unsigned long long>(g.K), *bs = c.take<unsigned long long>(g.K);
    int32_t *key0 = nullptr, *key1 = nullptr, *cl0 = nullptr, *cl1 = nullptr;
    if constexpr (TB == kHash) {
        key0 = c.take<int32_t>(g.H);
        key1 = c.take<int32_t>(g.H);
        cl0 = c.take<int32_t>(g.K);
        cl1 = c.take<int32_t>(g.K);
        for (int h = g.lid; h < g.H; h += W) key0[h] = key1[h] = -1;
    } else {
        for (int h = g.lid; h < g.H; h += W) val0[h] = val1[h] = -__builtin_huge_val();
    }
    for (int k = g.lid; k < g.K; k += W) bm[k] = bs[k] = 0ull;
    g.sync();
    const int32_t limit = work.n ? *work.n : bv.B;
    const double scale = *ct.scale;
    int item;
    const int stride = live_groups(item, gf.blocks);
    int64_t list_at = (int64_t)item * kLiveChunk, list_end = list_at + kLiveChunk;  // range of the touched list
    // the value of a list entry into a table (kHash: entry i of its list)
    auto put_val = [&](double *vals, int32_t *keys, int32_t *cls, int2 sg, int i, double v) {
        if constexpr (TB == kHash) {
            g.key = keys;
            bool first;
            const int at = g.claim(sg.x, first);
            vals[at] = v;
            cls[i] = at;
        } else {
            vals[sg.y] = v;
        }
    };
    for (; item < limit; item += stride) {
        const int b = work.order ? work.order[item] : item;
        if (lt.done[b] != 1) continue;
        const int o0 = bv.offsets[b], o1 = bv.offsets[b + 1];
        const int T = o1 - o0;
        const float gb = ct.grad_log_z ? ct.grad_log_z[b] : 1.0f;
        const double lz = lt.log_z[b];
        if (T == 0) {
            if (ct.fin && g.lid == 0) fin_add(ct, start, gb * exp_e((float)((double)final_score[start] - lz)));
            continue;
        }
        // list i (after token i): {first entry, entries}; list 0 is the start state
        auto list_of = [&](int i) { return i >= 1 ? lt.tok[o0 + i - 1] : make_int2(0, 1); };
        auto entries = [&](int2 tk) { return min(tk.y, g.K); };
        // entry e of list i
        auto entry_of = [&](int i, int2 tk, int e, double &al) {
            const bool in = i >= 1 && e < entries(tk);
            al = in ? lt.val[tk.x + e] : 0.0;
            return in ? lt.state[tk.x + e] : make_int2(start, 0);
        };
        // beta_T = f on the last list
        const int2 last = list_of(T);
        int n_prev = entries(last);
        for (int e = g.lid; e < n_prev; e += W) {
            double al;
            const int2 sg = entry_of(T, last, e, al);
            const float f = final_score[sg.x];
            if (ct.fin && f != WFST_NINF) fin_add(ct, sg.x, gb * exp_e((float)((al + (double)f) - lz)));
            put_val(val0, key0, cl0, sg, e, (double)f);
        }
        g.sync();
        // a posterior into its arc's accumulator, and the arc's position noted for the conversion
        auto count = [&](long long q, int32_t pos) {
            if (q) atomicAdd(&ct.acc[pos], (unsigned long long)q);
            if (!ct.touched) return;
            const uint64_t mk = __ballot(q != 0);
            const int tot = __popcll(mk);
            if (list_at + tot > list_end) {  // a new chunk; the old one's tail holds no slots
                for (int64_t j = list_at + g.lid; j < min(list_end, ct.touched_cap); j += W) ct.touched[j] = -1;
                unsigned long long ch = 0;
                if (g.lid == 0) ch = atomicAdd(ct.n_touched, (unsigned long long)kLiveChunk);
                list_at = (int64_t)__shfl(ch, 0, W);
                list_end = list_at + kLiveChunk;
            }
            const int64_t at = list_at + __popcll(mk & ((1ull << (threadIdx.x & 63)) - 1ull));
            if (q && at < ct.touched_cap) ct.touched[at] = pos;
            list_at += tot;
        };
        // Step m takes the arcs of token T - 1 - m from the list before it.  Nothing it loads depends on beta: its arcs
        // are loaded two steps ahead, its list entries three, in registers that a step's number mod 4 names (moving
        // them from step to step made every step wait for all loads in flight).
        LiveWindow<true> win(bv, ix, lt.tok, o0, T);
        win.start();
        int2 sg_[4], rc_[4];
        double al_[4];
        LiveArc x_[4];
        float sc_[4];
        auto fetch_entries = [&](int m, int p) {
            const int2 tk = make_int2(win.get(win.list, m), win.get(win.entries, m));
            const int n = entries(tk), e = g.lid >> g.share(n);
            const bool in = m < T - 1 && e < n;
            const int at = in ? tk.x + e : 0;
            sg_[p] = lt.state[at];
            al_[p] = lt.val[at];
        };
        auto fetch_arcs = [&](int m, int p) {
            const int n = min(win.get(win.entries, m), g.K), sb = g.share(n), sub = g.lid & ((1 << sb) - 1);
            int a;
            const LiveLabel l = win.label(m, a);
            if (m >= T - 1) {  // list 0 is the start state
                sg_[p] = make_int2(start, 0);
                al_[p] = 0.0;
            }
            rc_[p] = m < T && (g.lid >> sb) < n ? live_arcs(ix, l, a, sg_[p].x) : make_int2(0, 0);
            const int32_t pos = sub < rc_[p].y ? rc_[p].x + sub : 0;
            x_[p] = ix.arc[pos];
            sc_[p] = live_score<L>(ix, pos, x_[p]);
        };
#pragma unroll
        for (int p = 0; p < 3; ++p) fetch_entries(p, p);
#pragma unroll
        for (int p = 0; p < 2; ++p) fetch_arcs(p, p);
        for (int m0 = 0; m0 < T; m0 += 4) {
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const int m = m0 + p;
                if (m >= T) break;
                double *vp = (p & 1) ? val1 : val0, *vc = (p & 1) ? val0 : val1;
                int32_t *kp = (p & 1) ? key1 : key0, *kc = (p & 1) ? key0 : key1;
                int32_t *cp = (p & 1) ? cl1 : cl0, *cc = (p & 1) ? cl0 : cl1;
                win.step(m);
                const int2 k0 = make_int2(win.get(win.list, m), win.get(win.entries, m));
                int a0;
                const LiveLabel l0 = win.label(m, a0);
                const int n = entries(k0);
                const int sb = g.share(n), S = 1 << sb, sub = g.lid & (S - 1);
                fetch_arcs(m + 2, (p + 2) & 3);
                fetch_entries(m + 3, (p + 3) & 3);
                if (n <= W && !g.any(rc_[p].y > S)) {  // one arc a lane at most: straight through
                    const int e = g.lid >> sb;
                    const bool on = e < n, has = sub < rc_[p].y;
                    g.key = kp;
                    double y = -__builtin_huge_val();
                    if (has) {
                        const int at = g.at(x_[p]);
                        if (at >= 0 && sc_[p] > WFST_NINF) y = (double)sc_[p] + vp[at];
                    }
                    double mx = y;
                    if (S > 1) {
                        if (y != -__builtin_huge_val()) atomicMax(&bm[e], live_ord(y));
                        g.sync();
                        const unsigned long long k = bm[on ? e : 0];
                        mx = on && k ? unord_f64(k) : -__builtin_huge_val();
                    }
                    unsigned long long sum = 0;
                    long long q = 0;
                    if (y != -__builtin_huge_val()) {
                        sum = !(y < __builtin_huge_val()) ? kLivePoison
                                                          : live_fixed(exp_e((float)(y - mx)));
                        q = __double2ll_rn((double)(gb * exp_e((float)((al_[p] + y) - lz))) * scale);
                    }
                    if (S > 1) {
                        if (sum & kLivePoison) atomicOr(&bs[e], kLivePoison);
                        else if (sum) atomicAdd(&bs[e], sum);
                        g.sync();
                        sum = bs[on ? e : 0];
                    }
                    if (on && sub == 0) {
                        put_val(vc, kc, cc, sg_[p], e, mx == -__builtin_huge_val() ? mx : live_lse(mx, sum));
                        if (S > 1) bm[e] = bs[e] = 0ull;
                    }
                    count(q, rc_[p].x + sub);
                } else {
                    for (int e0 = 0; e0 < n; e0 += W) {
                        const int e = e0 + (g.lid >> sb);
                        const bool on = e < n;
                        int2 sg = sg_[p];
                        double al = al_[p];
                        int2 rc = rc_[p];
                        if (e0 > 0) {
                            sg = entry_of(T - 1 - m, k0, e, al);
                            rc = on ? live_arcs(ix, l0, a0, sg.x) : make_int2(0, 0);
                        }
                        g.key = kp;
                        auto beta_of = [&](const LiveArc &x, float sc) {
                            const int at = g.at(x);
                            return at >= 0 && sc > WFST_NINF ? (double)sc + vp[at] : -__builtin_huge_val();
                        };
                        double y0 = -__builtin_huge_val(), mx = -__builtin_huge_val();
                        LiveArc xf = x_[p];
                        float scf = sc_[p];
                        if (e0 > 0 && sub < rc.y) {
                            xf = ix.arc[rc.x + sub];
                            scf = live_score<L>(ix, rc.x + sub, xf);
                        }
                        if (sub < rc.y) y0 = beta_of(xf, scf);
                        mx = y0;
                        for (int r = sub + S; r < rc.y; r += S) {
                            const LiveArc x = ix.arc[rc.x + r];
                            mx = fmax(mx, beta_of(x, live_score<L>(ix, rc.x + r, x)));
                        }
                        if (S > 1) {
                            if (mx != -__builtin_huge_val()) atomicMax(&bm[e], live_ord(mx));
                            g.sync();
                            if (on) mx = bm[e] ? unord_f64(bm[e]) : -__builtin_huge_val();
                        }
                        // sums and posteriors
                        unsigned long long sum = 0;
                        for (int r = sub; r == sub || g.any(r < rc.y); r += S) {
                            long long q = 0;
                            LiveArc x = xf;
                            if (r < rc.y) {
                                float sc = scf;
                                double y = y0;
                                if (r != sub) {
                                    x = ix.arc[rc.x + r];
                                    sc = live_score<L>(ix, rc.x + r, x);
                                    y = beta_of(x, sc);
                                }
                                if (y != -__builtin_huge_val()) {
                                    if (!(y < __builtin_huge_val())) sum |= kLivePoison;
                                    else sum += live_fixed(exp_e((float)(y - mx)));
                                    q = __double2ll_rn((double)(gb * exp_e((float)((al + y) - lz))) * scale);
                                }
                            }
                            count(q, rc.x + r);
                        }
                        if (S > 1) {
                            if (sum & kLivePoison) atomicOr(&bs[e], kLivePoison);
                            else if (sum) atomicAdd(&bs[e], sum);
                            g.sync();
                            if (on) sum = bs[e];
                        }
                        if (on && sub == 0) {
                            put_val(vc, kc, cc, sg, e, mx == -__builtin_huge_val() ? mx : live_lse(mx, sum));
                            if (S > 1) bm[e] = bs[e] = 0ull;
                        }
                    }
                }
                g.sync();
                if constexpr (TB == kHash) {
                    for (int e = g.lid; e < n_prev; e += W) kp[cp[e]] = -1;
                    g.sync();
                }
                n_prev = n;
            }
        }
        if constexpr (TB == kHash) {  // the start state's entry
            int32_t *kl = (T & 1) ? key1 : key0, *cll = (T & 1) ? cl1 : cl0;
            for (int e = g.lid; e < n_prev; e += W) kl[cll[e]] = -1;
            g.sync();
        }
    }
    if (ct.touched)
        for (int64_t j = list_at + g.lid; j < min(list_end, ct.touched_cap); j += W) ct.touched[j] = -1;
}

// The workgroup form.  As in the forward sweep, a step whose lists and arcs fit
// runs on chip: terms numbered by a prefix sum, one thread a term, beta of the
// step after in a hashed table.  The others take a thread per list entry and
// keep beta in vectors over the states in memory (only entries of the lists are
// read).  The next step's list and label are loaded during a step.  24 strings
// over 1M states: 338 us (in memory throughout, one atomic per touched arc: 736).
constexpr int kBackTable = 2 * kStepTerms;
struct LiveBackStep {
    static constexpr int W = kLiveGroupThreads;
    double val[2][kBackTable];
    int32_t key[2][kBackTable];
    unsigned long long mx[W], sum[W];  // of a source, zero between steps
    double alpha[W];
    int32_t first[W];
    uint16_t owner[kStepTerms], claimed[2][kStepTerms];
    int32_t tot[W / 64];
    LiveTile<W> tile;
    int n_claimed[2];
    long long list_at, list_end;  // this workgroup's range of the touched list
};

template <int W, bool L>
__global__ void __launch_bounds__(W)
live_backward_wide(LiveIndex ix, int32_t Q, int32_t start, const float *__restrict__ final_score, BatchView bv,
                   LiveWork work, LiveTape lt, LiveCounts ct, unsigned char *__restrict__ gscratch)
{
    static_assert(W == kLiveGroupThreads, "one source a thread");
    __shared__ LiveBackStep st;
    // past the tables of the other sweeps, which stay zero
    double *val0 = reinterpret_cast<double *>(gscratch + (size_t)blockIdx.x * live_slot(Q)) + 2 * (int64_t)Q;
    double *val1 = val0 + Q;
    const int lid = threadIdx.x;
    const int32_t limit = work.n ? *work.n : bv.B;
    const double scale = *ct.scale;
    for (int h = lid; h < kBackTable; h += W) st.key[0][h] = st.key[1][h] = -1;
    st.mx[lid] = st.sum[lid] = 0ull;
    if (lid == 0) {
        st.n_claimed[0] = st.n_claimed[1] = 0;
        st.list_at = st.list_end = 0;
    }
    __syncthreads();
    auto insert = [&](int x, int32_t s, double v) {  // a state of its own into table x
        for (uint32_t h = ((uint32_t)s * 0x9e3779b1u) >> 7;; ++h) {  // at most half full
            const int at = (int)(h & (uint32_t)(kBackTable - 1));
            if (atomicCAS(&st.key[x][at], -1, s) == -1) {
                st.val[x][at] = v;
                st.claimed[x][atomicAdd(&st.n_claimed[x], 1)] = (uint16_t)at;
                return;
            }
        }
    };
    auto drop = [&](int x) {  // (between barriers)
        for (int i = lid; i < st.n_claimed[x]; i += W) st.key[x][st.claimed[x][i]] = -1;
        __syncthreads();
        if (lid == 0) st.n_claimed[x] = 0;
    };
    // room for `need` more entries of the touched list in this workgroup's range (uniform)
    auto reserve = [&](int need) {
        if (st.list_at + need > st.list_end) {
            const long long from = st.list_at, to = min((long long)ct.touched_cap, st.list_end);
            for (long long j = from + lid; j < to; j += W) ct.touched[j] = -1;
            __syncthreads();
            if (lid == 0) {
                const unsigned long long want = (unsigned long long)max(need, 4 * kLiveChunk);
                st.list_at = (long long)atomicAdd(ct.n_touched, want);
                st.list_end = st.list_at + (long long)want;
            }
            __syncthreads();
        }
    };
    auto count = [&](double gb, double x, int32_t pos, bool reserved) {
        const long long q = __double2ll_rn((double)((float)gb * exp_e((float)x)) * scale);
        if (!q) return;
        atomicAdd(&ct.acc[pos], (unsigned long long)q);
        if (!ct.touched) return;
        const long long at = reserved ? (long long)atomicAdd((unsigned long long *)&st.list_at, 1ull)
                                      : (long long)atomicAdd(ct.n_touched, 1ull);
        if (at < ct.touched_cap) ct.touched[at] = pos;
    };
    for (int item = blockIdx.x; item < limit; item += gridDim.x) {
        const int b = work.order ? work.order[item] : item;
        if (lt.done[b] != 2) continue;
        const int o0 = bv.offsets[b], o1 = bv.offsets[b + 1];
        const int T = o1 - o0;
        const float gb = ct.grad_log_z ? ct.grad_log_z[b] : 1.0f;
        const double lz = lt.log_z[b];
        if (T == 0) {
            if (ct.fin && lid == 0) fin_add(ct, start, gb * exp_e((float)((double)final_score[start] - lz)));
            continue;
        }
        const int2 last = lt.tok[o1 - 1];
        __syncthreads();
        bool in_lds = last.y <= kStepTerms;  // beta of the step after is in table (T - t) & 1, else in its vector
        for (int e = lid; e < last.y; e += W) {
            const int32_t s = lt.state[last.x + e].x;
            const float f = final_score[s];
            if (ct.fin && f != WFST_NINF) fin_add(ct, s, gb * exp_e((float)((lt.val[last.x + e] + (double)f) - lz)));
            if (in_lds) insert(0, s, (double)f);
            else val0[s] = (double)f;
        }
        // list 0 is the start state
        auto list_of = [&](int i) { return i >= 1 ? lt.tok[o0 + i - 1] : make_int2(0, 1); };
        auto state_of = [&](int i, int2 k) { return i >= 1 ? lt.state[k.x + min(lid, max(k.y - 1, 0))].x : start; };
        auto alpha_of = [&](int i, int2 k) { return i >= 1 ? lt.val[k.x + min(lid, max(k.y - 1, 0))] : 0.0; };
        int a0 = bv.tokens[o1 - 1], a1 = bv.tokens[max(o1 - 2, o0)], a2 = bv.tokens[max(o1 - 3, o0)];
        LiveLabel l0 = ix.label[a0], l1 = ix.label[a1];
        int2 k_prev = last, k0 = list_of(T - 1), k1 = list_of(T - 2), k2 = list_of(T - 3);
        int32_t s0 = state_of(T - 1, k0), s1 = state_of(T - 2, k1);
        double al0 = alpha_of(T - 1, k0), al1 = alpha_of(T - 2, k1);
        int2 rc0 = lid < k0.y ? live_arcs(ix, l0, a0, s0) : make_int2(0, 0);
        __syncthreads();
        for (int t = T; t >= 1; --t) {
            const int pv = (T - t) & 1, cv = pv ^ 1;
            double *vp = pv ? val1 : val0, *vc = pv ? val0 : val1;
            // in flight during this step
            const int a3 = bv.tokens[max(o0 + t - 4, o0)];
            const LiveLabel l2 = ix.label[a2];
            const int2 k3 = list_of(t - 4);
            const int32_t s2 = state_of(t - 3, k2);
            const double al2 = alpha_of(t - 3, k2);
            const int2 rc1 = t >= 2 && lid < k1.y ? live_arcs(ix, l1, a1, s1) : make_int2(0, 0);
            bool small = k0.y <= W && k_prev.y <= kStepTerms;
            int E = 0;
            if (small) {
                const int2 rc = rc0;
                int inc = rc.y;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const int up = __shfl_up(inc, o, 64);
                    if ((lid & 63) >= o) inc += up;
                }
                if ((lid & 63) == 63) st.tot[lid >> 6] = inc;
                const bool huge = __syncthreads_or(rc.y > kStepTerms);
                int off = inc - rc.y;
#pragma unroll
                for (int x = 0; x < W / 64; ++x) {
                    off += x < (lid >> 6) ? st.tot[x] : 0;
                    E += st.tot[x];
                }
                small = !huge && E <= kStepTerms;
                if (small) {
                    st.first[lid] = rc.x - off;
                    st.alpha[lid] = al0;
                    for (int r = 0; r < rc.y; ++r) st.owner[off + r] = (uint16_t)lid;
                    if (!in_lds)  // from its vector into the table
                        for (int e = lid; e < k_prev.y; e += W) {
                            const int32_t s = lt.state[k_prev.x + e].x;
                            insert(pv, s, vp[s]);
                        }
                }
                __syncthreads();
                if (small && ct.touched) reserve(E);
            }
            if (small) {
                constexpr int R = kStepTerms / W;
                double y[R];
                int32_t own[R];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int x = lid + r * W;
                    y[r] = -__builtin_huge_val();
                    own[r] = 0;
                    if (x >= E) continue;
                    own[r] = st.owner[x];
                    const int32_t pos = st.first[own[r]] + x;
                    const LiveArc arc = ix.arc[pos];
                    const float sc = live_score<L>(ix, pos, arc);
                    for (uint32_t h = ((uint32_t)arc.dst * 0x9e3779b1u) >> 7;; ++h) {
                        const int at = (int)(h & (uint32_t)(kBackTable - 1));
                        const int32_t k = st.key[pv][at];
                        if (k == arc.dst && sc > WFST_NINF) y[r] = (double)sc + st.val[pv][at];
                        if (k == arc.dst || k == -1) break;
                    }
                    if (y[r] != -__builtin_huge_val()) atomicMax(&st.mx[own[r]], live_ord(y[r]));
                }
                __syncthreads();
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if (y[r] == -__builtin_huge_val()) continue;
                    live_add_term(&st.sum[own[r]], y[r], unord_f64(st.mx[own[r]]));
                    count(gb, (st.alpha[own[r]] + y[r]) - lz, st.first[own[r]] + lid + r * W, true);
                }
                __syncthreads();
                if (lid < k0.y) {
                    const unsigned long long m = st.mx[lid];
                    insert(cv, s0, m ? live_lse(unord_f64(m), st.sum[lid]) : -__builtin_huge_val());
                    st.mx[lid] = st.sum[lid] = 0ull;
                }
                drop(pv);
                in_lds = true;
            } else {
                if (in_lds) {  // from the table to its vector
                    for (int i = lid; i < st.n_claimed[pv]; i += W) {
                        const int at = st.claimed[pv][i];
                        vp[st.key[pv][at]] = st.val[pv][at];
                    }
                    __syncthreads();
                    drop(pv);
                    __syncthreads();
                }
                for (int e0 = 0; e0 < k0.y; e0 += W) {
                    const int e = e0 + lid;
                    const bool on = e < k0.y;
                    const int32_t s = e0 == 0 ? s0 : on ? lt.state[k0.x + e].x : start;
                    const double al = e0 == 0 ? al0 : on ? lt.val[k0.x + e] : 0.0;
                    const int2 rc = e0 == 0 ? rc0 : on ? live_arcs(ix, l0, a0, s) : make_int2(0, 0);
                    auto beta_of = [&](const LiveArc &x, float sc) {
                        return sc > WFST_NINF ? (double)sc + vp[x.dst] : -__builtin_huge_val();
                    };
                    if (__syncthreads_or(rc.y > kLiveSkew)) {
                        const int total = st.tile.number(rc);
                        st.alpha[lid] = al;
                        __syncthreads();
                        if (ct.touched) reserve(total);
                        st.tile.template each<L>(ix, total, [&](int k, int, const LiveArc &x, float sc) {
                            const double y = beta_of(x, sc);
                            if (y != -__builtin_huge_val()) atomicMax(&st.mx[k], live_ord(y));
                        });
                        __syncthreads();
                        st.tile.template each<L>(ix, total, [&](int k, int pos, const LiveArc &x, float sc) {
                            const double y = beta_of(x, sc);
                            if (y == -__builtin_huge_val()) return;
                            live_add_term(&st.sum[k], y, unord_f64(st.mx[k]));
                            count(gb, (st.alpha[k] + y) - lz, pos, true);
                        });
                        __syncthreads();
                        const unsigned long long m = st.mx[lid];
                        if (on) vc[s] = m ? live_lse(unord_f64(m), st.sum[lid]) : -__builtin_huge_val();
                        st.mx[lid] = st.sum[lid] = 0ull;
                        continue;
                    }
                    double m = -__builtin_huge_val();
                    for (int r = 0; r < rc.y; ++r) {
                        const LiveArc x = ix.arc[rc.x + r];
                        m = fmax(m, beta_of(x, live_score<L>(ix, rc.x + r, x)));
                    }
                    unsigned long long sum = 0;
                    for (int r = 0; r < rc.y; ++r) {
                        const LiveArc x = ix.arc[rc.x + r];
                        const double y = beta_of(x, live_score<L>(ix, rc.x + r, x));
                        if (y == -__builtin_huge_val()) continue;
                        if (!(y < __builtin_huge_val())) sum |= kLivePoison;
                        else sum += live_fixed(exp_e((float)(y - m)));
                        count(gb, (al + y) - lz, rc.x + r, false);
                    }
                    if (on) vc[s] = m == -__builtin_huge_val() ? m : live_lse(m, sum);
                }
                in_lds = false;
            }
            __syncthreads();
            k_prev = k0, k0 = k1, k1 = k2, k2 = k3;
            a0 = a1, a1 = a2, a2 = a3;
            l0 = l1, l1 = l2;
            s0 = s1, s1 = s2, al0 = al1, al1 = al2, rc0 = rc1;
        }
        if (in_lds) {  // the start state's entry
            drop(T & 1);
            __syncthreads();
        }
    }
    if (ct.touched)
        for (long long j = st.list_at + lid; j < min((long long)ct.touched_cap, st.list_end); j += W) ct.touched[j] = -1;
}

// =====================================================================
// Narrow labels: at most W destinations per label (W = 8 or 16), and for each
// of them at most U arcs per lane under another label (U = 2 or 4)
// =====================================================================
// Then no list is needed: the live states after a token are among its label's
// destinations, so a step's sources, and with them every address it loads,
// follow from the tokens alone.  narrow_prep looks them up for all tokens in
// parallel; the sweeps then load a step's arcs kNarrowAhead steps ahead, and
// nothing in their chain waits for memory (one step ahead left the bigram
// tagger's Viterbi sweep at 1.6 us a step, one memory latency; now 0.55 us).
// A sentence
// takes W lanes, 64 / W sentences a wavefront: lane d holds destination d's
// value, lane j * S + k takes the k-th, (k + S)-th, ... arc of source j.
constexpr int kNarrowAhead = 4;
struct NarrowView {
    const int32_t *seg_key = nullptr;  // states of the forward segments
    int32_t D = 0;                     // most destinations of a label (stride of the per-token values)
    int32_t share = 0;                 // log2 S, S = W / D rounded down to a power of two
    const int2 *prep = nullptr;        // [N * D] {first, count}: arcs of token i from source j
    const int32_t *verdict = nullptr;  // [B] WFST_STATUS_* of offsets and tokens (Viterbi and forward)
};

// The labels that occur most in a large batch: their arcs' counts are summed in
// LDS by every workgroup of the backward sweep and added to the accumulators
// once.  Without that the sweep is bound by its atomics: at most about three
// lines a nanosecond over the device, and one line takes about 13 ns each time
// (16384 sentences of the bigram tagger, word frequencies ~ 1/rank^1.1: 6.5M
// posteriors in 3.3M line updates, 81 thousand of them on the hottest line;
// 1174 us, with the cells 299).  The 100 most frequent words are 56% of the
// tokens.
struct HotLabel {
    int32_t label, first, n, cell;  // arcs [first, first + n) in cells [cell, cell + n)
};
struct HotView {
    const HotLabel *label = nullptr;
    const int32_t *n = nullptr;  // null: no cells
    int32_t cells = 0;
};
constexpr int kHotMax = 255, kHotMap = 512;       // labels, LDS map entries
constexpr int kHotCells = 9728;                   // accumulators of a workgroup: with the map 80 KiB, two a compute unit
constexpr int kHotSample = 8192, kHotTable = 8192;

// One workgroup: the most frequent labels of kHotSample tokens spread evenly over the batch whose arcs fit `cells`.
struct HotOut {
    HotLabel *label = nullptr;  // null: not wanted
    int32_t *n = nullptr;
    int32_t cells = 0;
};
__device__ __forceinline__ void hot_of(const int32_t *__restrict__ tokens, int64_t N, int32_t M,
                                       const int2 *__restrict__ all, const HotOut &ho)
{
    const int32_t cells = ho.cells;
    HotLabel *out = ho.label;
    __shared__ int32_t s_key[kHotTable], s_cnt[kHotTable];
    __shared__ int s_need[256];  // cells of the labels seen this often
    __shared__ int s_from, s_n, s_used;
    const int tid = threadIdx.x;
    for (int h = tid; h < kHotTable; h += 1024) {
        s_key[h] = -1;
        s_cnt[h] = 0;
    }
    if (tid < 256) s_need[tid] = 0;
    if (tid == 0) s_n = s_used = 0;
    __syncthreads();
    const int S = (int)min(N, (int64_t)kHotSample);
    int lab[kHotSample / 1024];
#pragma unroll
    for (int u = 0; u < kHotSample / 1024; ++u) {
        const int k = tid + u * 1024;
        lab[u] = k < S ? tokens[N * k / S] : -1;
    }
#pragma unroll
    for (int u = 0; u < kHotSample / 1024; ++u) {
        const int a = lab[u];
        if (a < 0 || a >= M) continue;
        uint32_t h = (uint32_t)a * 0x9e3779b1u >> 7;
        for (int probe = 0; probe < 16; ++probe, ++h) {  // what finds no place is rare
            const int at = (int)(h & (kHotTable - 1)), old = atomicCAS(&s_key[at], -1, a);
            if (old == -1 || old == a) {
                atomicAdd(&s_cnt[at], 1);
                break;
            }
        }
    }
    __syncthreads();
    int need[kHotTable / 1024];
#pragma unroll
    for (int u = 0; u < kHotTable / 1024; ++u) {
        const int h = tid + u * 1024;
        need[u] = s_cnt[h] >= 2 ? all[s_key[h]].y : 0;
        if (need[u] > cells / 4) need[u] = 0;
        if (need[u]) atomicAdd(&s_need[min(s_cnt[h], 255)], need[u]);
    }
    __syncthreads();
    if (tid < 64) {  // labels seen at least s_from times all fit: lane x sums the counts 255 - 4 x - {0, 1, 2, 3}
        int v[4], sum = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) sum += v[r] = s_need[255 - 4 * tid - r];
        int before = sum;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int up = __shfl_up(before, o, 64);
            if (tid >= o) before += up;
        }
        before -= sum;
        int fit = 0;  // counts of this lane that fit with all above them
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            before += v[r];
            if (before <= cells) ++fit;
        }
        const uint64_t part = __ballot(fit < 4);  // its first lane holds the limit
        const int x = part ? __ffsll((unsigned long long)part) - 1 : 63;
        const int from = 256 - 4 * x - __shfl(fit, x, 64);
        if (tid == 0) s_from = max(from, 2);
    }
    __syncthreads();
    for (int pass = 0; pass < 2; ++pass) {  // those, then what fits of the next
#pragma unroll
        for (int u = 0; u < kHotTable / 1024; ++u) {
            const int h = tid + u * 1024, c = min(s_cnt[h], 255);
            if (!need[u] || (pass == 0 ? c < s_from : c != s_from - 1)) continue;
            const int cell = atomicAdd(&s_used, need[u]);
            if (cell + need[u] > cells) continue;
            const int at = atomicAdd(&s_n, 1);
            if (at < kHotMax) out[at] = HotLabel{s_key[h], all[s_key[h]].x, need[u], cell};
        }
        __syncthreads();
    }
    if (tid == 0) *ho.n = min(s_n, kHotMax);
}

// One wavefront per sentence: its verdict, and the arcs of every (token, source).
// Where an order is wanted (workgroups of 1024), the first workgroup makes it
// meanwhile (13 us for 16384 sentences, as a launch of its own), and with Hot
// the second one picks the frequent labels for the backward sweep (23 us, as a
// launch of its own; the whole takes 37, without Hot 33).
template <bool Hot>
__global__ void __launch_bounds__(1024)
narrow_prep(LiveIndex ix, const int32_t *__restrict__ seg_key, int32_t D, int32_t start, BatchView bv,
            int2 *__restrict__ prep, int32_t *__restrict__ verdict, int32_t *__restrict__ order, HotOut ho)
{
    if (order && blockIdx.x == 0) return order_of(bv.offsets, bv.B, order);
    if constexpr (Hot)
        if (blockIdx.x == 1) return hot_of(bv.tokens, bv.N, bv.M, ix.all, ho);
    const int lane = threadIdx.x & 63, skip = Hot ? 2 : order ? 1 : 0, waves = (int)blockDim.x / 64;
    for (int b = ((int)blockIdx.x - skip) * waves + (int)(threadIdx.x >> 6); b < bv.B;
         b += ((int)gridDim.x - skip) * waves) {
        const int o0 = bv.offsets[b], o1 = bv.offsets[b + 1];
        if (o0 < 0 || o1 < o0 || (int64_t)o1 > bv.N) {
            if (lane == 0) verdict[b] = WFST_STATUS_BAD_INPUT;
            continue;
        }
        bool bad = false;
        for (int i = o0 + lane; i < o1; i += 64) {
            const int a = bv.tokens[i], before = i > o0 ? bv.tokens[i - 1] : 0;
            const bool ok = a >= 0 && a < bv.M;
            bad |= !ok;
            const bool both = ok && before >= 0 && before < bv.M;
            const LiveLabel l = ix.label[both ? a : 0], lb = ix.label[both ? before : 0];
            const int n = i > o0 ? lb.n_segs : 1;
            for (int j = 0; j < D; ++j) {
                int2 rc = make_int2(0, 0);
                if (both && j < n) rc = live_arcs(ix, l, a, i > o0 ? seg_key[lb.seg_first + j] : start);
                prep[(int64_t)i * D + j] = rc;
            }
        }
        bad = __any(bad);
        if (lane == 0) verdict[b] = bad ? WFST_STATUS_BAD_TOKEN : WFST_STATUS_OK;
    }
}

// A lane's arcs of one step.
template <int U>
struct NarrowArcs {
    int32_t seg[U], arc[U];
    float sc[U];
    int32_t pos, n;  // position of the first; how many (<= 0: none)
};
// The steps in flight.  L (arcs listed by (label, source)): step m + 2 K's
// {first, count} and step m + K's arcs with their scores are loaded as step m
// ends; else the scores, which need the arc id, follow K steps after their
// arcs.  All loads are unconditional (arc 0 where there is none), so that the
// number in flight is known and only the oldest are waited for.
template <int U, bool L>
struct NarrowPipe {
    static constexpr int K = kNarrowAhead;
    NarrowArcs<U> q[K], nx[L ? 1 : K];
    int2 rc[K];
    const LiveIndex &ix;
    const int sub, share;
    const bool on;  // this lane has a source.  What is loaded is looked at only when it is used: a select at the load of
                    // the last step of a round made every round wait for all loads in flight (forward sweep of
                    // 16384 sentences: 152 us, 142 without)
    __device__ __forceinline__ NarrowPipe(const LiveIndex &index, int sub_, int share_, bool on_)
        : ix(index), sub(sub_), share(share_), on(on_) {}
    __device__ __forceinline__ int32_t at(const NarrowArcs<U> &v, int u) const { return u < v.n ? v.pos + (u << share) : 0; }
    __device__ __forceinline__ void arcs(NarrowArcs<U> &v, int2 r) const
    {
        v.pos = r.x + sub;
        v.n = on ? (r.y - sub + (1 << share) - 1) >> share : 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            // (A < 2^28: byte offsets are 32 bits)
            const LiveArc *x = reinterpret_cast<const LiveArc *>(reinterpret_cast<const char *>(ix.arc) +
                                                                 (uint32_t)at(v, u) * (uint32_t)sizeof(LiveArc));
            v.seg[u] = x->seg;
            v.arc[u] = L ? at(v, u) : x->arc;
        }
    }
    __device__ __forceinline__ void scores(NarrowArcs<U> &v) const
    {
#pragma unroll
        for (int u = 0; u < U; ++u)
            v.sc[u] = *reinterpret_cast<const float *>(reinterpret_cast<const char *>(ix.score) +
                                                       (uint32_t)v.arc[u] * (uint32_t)sizeof(float));
    }
    // steps 0, 1, ...; of(m): {first, count} of step m (any m: steps past the last may be anything valid)
    template <class Of>
    __device__ __forceinline__ void start(const Of &of)
    {
#pragma unroll
        for (int k = 0; k < K; ++k) rc[k] = of(k);
        if constexpr (!L) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                arcs(nx[k], rc[k]);
                rc[k] = of(K + k);
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k) next(k, k - K, of);
    }
    // step m, kept at k, is done
    template <class Of>
    __device__ __forceinline__ void next(int k, int m, const Of &of)
    {
        if constexpr (L) {
            arcs(q[k], rc[k]);
            scores(q[k]);
            rc[k] = of(m + 2 * K);
        } else {
            q[k] = nx[k];
            scores(q[k]);
            arcs(nx[k], rc[k]);
            rc[k] = of(m + 3 * K);
        }
    }
};

// The sentences of a wavefront: neighbours of the order.
template <int W>
struct NarrowGroup {
    int lid, gi, item, stride, j, sub;
    __device__ __forceinline__ explicit NarrowGroup(int share, int skip = 0)  // skip: workgroups that are no groups
    {
        const int per = (int)blockDim.x / W;  // groups of a workgroup
        lid = threadIdx.x % W;
        gi = threadIdx.x % 64 / W;
        item = ((int)blockIdx.x - skip) * per + (int)threadIdx.x / W;
        stride = ((int)gridDim.x - skip) * per;
        j = lid >> share;  // source of this lane's arcs
        sub = lid & ((1 << share) - 1);
    }
    __device__ __forceinline__ static void sync()
    {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    __device__ __forceinline__ bool any(bool p) const
    {
        return (__ballot(p) & (((1ull << W) - 1ull) << (gi * W))) != 0ull;
    }
    // {first, count} of this lane's source at token i (lanes past the sources: the last one's, which the pipe ignores)
    __device__ __forceinline__ int2 arcs(const NarrowView &nv, int64_t i) const
    {
        return nv.prep[i * nv.D + min(j, nv.D - 1)];
    }
};

// Viterbi.  A candidate's key is its score, then its arc id (28 bits), then
// its source (4 bits), so one maximum per destination is the whole step.
// pred[i * W + d]: source of the winner at destination d of token i;
// win[i * D + d]: its arc.
template <int W, int U, bool L>
__global__ void __launch_bounds__(64)
narrow_viterbi(LiveIndex ix, NarrowView nv, int32_t start, const float *__restrict__ final_score, BatchView bv,
               const int32_t *__restrict__ order, uint8_t *__restrict__ pred, int32_t *__restrict__ win,
               float *__restrict__ best_score, int32_t *__restrict__ best_arcs, int32_t *__restrict__ best_olabels,
               const int32_t *__restrict__ olabel)
{
    constexpr int K = kNarrowAhead;
    __shared__ unsigned long long s_mx[128];
    NarrowGroup<W> g(nv.share);
    unsigned long long *mx = s_mx + g.gi * W;
    const int none = 64 + (int)threadIdx.x - g.gi * W;  // where this lane's missing arcs go
    mx[g.lid] = 0ull;
    g.sync();
    for (int item = g.item; item < bv.B; item += g.stride) {
        const int b = order ? order[item] : item;
        const int o0 = bv.offsets[b], o1 = bv.offsets[b + 1], T = o1 - o0;
        const int stt = nv.verdict[b];
        if (stt != WFST_STATUS_OK) {
            if (g.lid == 0) {
                bv.status[b] = stt;
                best_score[b] = WFST_NINF;
            }
            if (stt == WFST_STATUS_BAD_TOKEN)
                for (int i = o0 + g.lid; i < o1; i += W) {
                    best_arcs[i] = -1;
                    if (best_olabels) best_olabels[i] = -1;
                }
            continue;
        }
        float v = g.lid == 0 ? 0.0f : WFST_NINF;  // lane d: value of destination d of the last token
        if (T > 0) {
            NarrowPipe<U, L> pipe(ix, g.sub, nv.share, g.j < nv.D);
            auto of = [&](int m) { return g.arcs(nv, o0 + min(m, T - 1)); };
            pipe.start(of);
            for (int t0 = 0; t0 < T; t0 += K) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const int t = t0 + k;
                    const NarrowArcs<U> &q = pipe.q[k];
                    if (t < T) {
                        const float vs = __shfl(v, g.j, W);
#pragma unroll
                        for (int u = 0; u < U; ++u) {  // key 0: none
                            const float c = vs + q.sc[u];
                            const unsigned long long key = ((unsigned long long)ord_f32(c) << 32) |
                                                           ((0x0fffffffu - (uint32_t)q.arc[u]) << 4) | (uint32_t)g.j;
                            atomicMax(&mx[u < q.n ? q.seg[u] : none], u < q.n && c > WFST_NINF ? key : 0ull);
                        }
                        g.sync();
                        const unsigned long long key = mx[g.lid];
                        mx[g.lid] = 0ull;
                        v = key ? unord_f32((uint32_t)(key >> 32)) : WFST_NINF;
                        pred[(int64_t)(o0 + t) * W + g.lid] = (uint8_t)(key & 15u);
                        if (key) win[(int64_t)(o0 + t) * nv.D + g.lid] = (int32_t)(0x0fffffffu - ((uint32_t)key >> 4));
                        g.sync();
                    }
                    pipe.next(k, t, of);
                }
            }
        }
        // final state: the highest score, then the lowest state id
        unsigned long long best = 0ull;
        int at = g.lid;
        if (v > WFST_NINF) {
            const int st = T > 0 ? nv.seg_key[ix.label[bv.tokens[o1 - 1]].seg_first + g.lid] : start;
            const float f = final_score[st];
            const float y = v + f;
            if (f != WFST_NINF && y != WFST_NINF)
                best = ((unsigned long long)ord_f32(y) << 32) | (0xffffffffu - (uint32_t)st);
        }
#pragma unroll
        for (int o = W / 2; o > 0; o >>= 1) {
            const unsigned long long k = __shfl_xor(best, o, W);
            const int x = __shfl_xor(at, o, W);
            if (k > best) best = k, at = x;
        }
        if (best == 0ull) {
            if (g.lid == 0) {
                bv.status[b] = WFST_STATUS_NO_PATH;
                best_score[b] = WFST_NINF;
            }
            for (int i = o0 + g.lid; i < o1; i += W) {
                best_arcs[i] = -1;
                if (best_olabels) best_olabels[i] = -1;
            }
            continue;
        }
        if (g.lid == 0) {
            bv.status[b] = WFST_STATUS_OK;
            best_score[b] = unord_f32((uint32_t)(best >> 32));
        }
        // backtrace, W tokens at a time: lane l holds all sources of token hi - l (their
        // addresses do not depend on the path), the chain is one shift and mask a token
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        auto row = [&](int t, int h) {
            return reinterpret_cast<const unsigned long long *>(pred + (int64_t)(o0 + max(t, 0)) * W)[h];
        };
        unsigned long long w0 = T > 0 ? row(T - 1 - g.lid, 0) : 0ull, w1 = W == 16 && T > 0 ? row(T - 1 - g.lid, 1) : 0ull;
        for (int hi = T - 1; hi >= 0; hi -= W) {
            const int t = hi - g.lid;
            const unsigned long long n0 = row(t - W, 0), n1 = W == 16 ? row(t - W, 1) : 0ull;  // the next tokens'
            int mine = 0;
#pragma unroll
            for (int l = 0; l < W; ++l) {
                mine = l == g.lid ? at : mine;
                unsigned long long w = __shfl(w0, l, W);
                if constexpr (W == 16) {
                    const unsigned long long y = __shfl(w1, l, W);
                    w = at >= 8 ? y : w;
                }
                at = (int)(w >> (8 * (at & 7))) & 15;
            }
            w0 = n0, w1 = n1;
            if (t >= 0) {
                const int arc = win[(int64_t)(o0 + t) * nv.D + mine];
                best_arcs[o0 + t] = arc;
                if (best_olabels) best_olabels[o0 + t] = olabel[arc];
            }
        }
    }
}

// Forward (log semiring); val[i * D + d]: log alpha of destination d after token i.
template <int W, int U, bool L>
__global__ void __launch_bounds__(64)
narrow_forward(LiveIndex ix, NarrowView nv, int32_t start, const float *__restrict__ final_score, BatchView bv,
               const int32_t *__restrict__ order, double *__restrict__ val, int32_t *__restrict__ done,
               double *__restrict__ log_z, float *__restrict__ log_z_out)
{
    constexpr int K = kNarrowAhead;
    __shared__ unsigned long long s_mx[128], s_sm[128];
    NarrowGroup<W> g(nv.share);
    unsigned long long *mx = s_mx + g.gi * W, *sm = s_sm + g.gi * W;
    const int none = 64 + (int)threadIdx.x - g.gi * W;  // where this lane's missing arcs go
    mx[g.lid] = 0ull;
    sm[g.lid] = 0ull;
    g.sync();
    for (int item = g.item; item < bv.B; item += g.stride) {
        const int b = order ? order[item] : item;
        const int o0 = bv.offsets[b], o1 = bv.offsets[b + 1], T = o1 - o0;
        const int stt = nv.verdict[b];
        if (stt != WFST_STATUS_OK) {
            if (g.lid == 0) {
                bv.status[b] = stt;
                done[b] = 0;
                log_z_out[b] = WFST_NINF;
                log_z[b] = -__builtin_huge_val();
            }
            continue;
        }
        double v = g.lid == 0 ? 0.0 : -__builtin_huge_val();
        if (T > 0) {
            NarrowPipe<U, L> pipe(ix, g.sub, nv.share, g.j < nv.D);
            auto of = [&](int m) { return g.arcs(nv, o0 + min(m, T - 1)); };
            pipe.start(of);
            for (int t0 = 0; t0 < T; t0 += K) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    const int t = t0 + k;
                    const NarrowArcs<U> &q = pipe.q[k];
                    if (t < T) {
                        const double vs = __shfl(v, g.j, W);
                        double y[U];
                        int at[U];
#pragma unroll
                        for (int u = 0; u < U; ++u) {  // key 0: none
                            y[u] = u < q.n ? vs + (double)q.sc[u] : -__builtin_huge_val();
                            at[u] = u < q.n ? q.seg[u] : none;
                            atomicMax(&mx[at[u]], y[u] != -__builtin_huge_val() ? live_ord(y[u]) : 0ull);
                        }
                        g.sync();
#pragma unroll
                        for (int u = 0; u < U; ++u) live_add_any(&sm[at[u]], y[u], unord_f64(mx[at[u]]));
                        g.sync();
                        const unsigned long long key = mx[g.lid];
                        const double lse = live_lse(unord_f64(key), sm[g.lid]);
                        v = key ? lse : -__builtin_huge_val();
                        mx[g.lid] = 0ull;
                        sm[g.lid] = 0ull;
                        if (g.lid < nv.D) val[(int64_t)(o0 + t) * nv.D + g.lid] = v;
                        g.sync();
                    }
                    pipe.next(k, t, of);
                }
            }
        }
        // log Z = LSE of alpha + f, the sum in fixed point like a step's
        float f = WFST_NINF;
        if (v != -__builtin_huge_val())
            f = final_score[T > 0 ? nv.seg_key[ix.label[bv.tokens[o1 - 1]].seg_first + g.lid] : start];
        const double x = f != WFST_NINF ? v + (double)f : -__builtin_huge_val();
        const bool poison = g.any(!(x < __builtin_huge_val()));
        double m = x;
#pragma unroll
        for (int o = W / 2; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, W));
        unsigned long long sum = x != -__builtin_huge_val() ? live_fixed(exp_e((float)(x - m))) : 0u;
#pragma unroll
        for (int o = W / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o, W);
        if (g.lid == 0) {
            const bool ok = m != -__builtin_huge_val() || poison;
            const double lz = poison ? __builtin_nan("") : ok ? live_lse(m, sum) : -__builtin_huge_val();
            bv.status[b] = ok ? WFST_STATUS_OK : WFST_STATUS_NO_PATH;
            done[b] = ok ? 1 : 0;
            log_z_out[b] = ok ? (float)lz : WFST_NINF;
            log_z[b] = lz;
        }
    }
}

// The forward pass of one sentence spread over a workgroup, for the latency
// entry point.  The sentence is cut into up to kScanChunks chunks.  The states
// that can enter a chunk are the few destinations of the token before it, so a
// chunk's matrix is one forward pass per such state, all of them at once; the
// chunks' matrices are then applied one after another to the start vector, and
// a last pass from each chunk's true entry vector writes log alpha.  Long
// sentences go window by window (as many tokens as the lookups' LDS holds).
// Bound by the chain of 2 T / chunks + chunks dependent steps of about 0.3 us
// and, before it, by five dependent loads.  Sixteen chunks: T = 200 gives 13 +
// 16 + 13 steps, 27 us in all (matrices of every token and 8 levels of products:
// 450 us); the waves of the workgroup hold 32 to 64 rows at once.
constexpr int kScanChunks = 16, kNarrowScanThreads = 512, kScanArcs = 4096;
template <int W, int U, bool L>
__global__ void __launch_bounds__(kNarrowScanThreads)
narrow_scan(LiveIndex ix, NarrowView nv, int32_t start, const float *__restrict__ final_score, BatchView bv,
            float *__restrict__ log_z, float *__restrict__ alpha, int32_t Q)
{
    constexpr int K = kNarrowAhead, NT = kNarrowScanThreads, G = NT / W;
    __shared__ int2 s_rc[kScanArcs];              // {first, count} of (token, source)
    __shared__ uint8_t s_dst[kScanArcs];          // state of (token, destination); Q is at most 64
    __shared__ float s_alpha[kScanArcs];
    __shared__ unsigned long long s_mx[2 * NT], s_sm[2 * NT];
    __shared__ double s_row[kScanChunks][W][W];   // value at destination d after chunk k entered at source j
    __shared__ double s_in[kScanChunks + 1][W];   // true vectors before each chunk
    const int tid = threadIdx.x, D = nv.D;
    NarrowGroup<W> g(nv.share);
    const int gi = tid / W;
    unsigned long long *mx = s_mx + gi * W, *sm = s_sm + gi * W;
    const int none = NT + tid - gi * W;  // where this lane's missing arcs go
    mx[g.lid] = 0ull;
    sm[g.lid] = 0ull;
    const int window = kScanArcs / D;
    for (int b = blockIdx.x; b < bv.B; b += gridDim.x) {
        const int o0 = bv.offsets[b], o1 = bv.offsets[b + 1], T = o1 - o0;
        const bool bad_off = o0 < 0 || o1 < o0 || (int64_t)o1 > bv.N;
        bool bad = false;
        if (!bad_off)
            for (int i = o0 + tid; i < o1; i += NT) bad |= bv.tokens[i] < 0 || bv.tokens[i] >= bv.M;
        bad = __syncthreads_or(bad);
        if (bad_off || bad) {
            if (tid == 0) {
                bv.status[b] = bad_off ? WFST_STATUS_BAD_INPUT : WFST_STATUS_BAD_TOKEN;
                log_z[b] = WFST_NINF;
            }
            continue;
        }
        if (tid < W) s_in[0][tid] = tid == 0 ? 0.0 : -__builtin_huge_val();
        for (int w0 = 0; w0 < T; w0 += window) {
            const int n = min(window, T - w0), C = (n + kScanChunks - 1) / kScanChunks, nc = (n + C - 1) / C;
            __syncthreads();  // the last window's tables are read
            for (int x = tid; x < n * D; x += NT) {
                const int t = x / D, j = x - t * D, i = o0 + w0 + t;
                const int a = bv.tokens[i], before = i > o0 ? bv.tokens[i - 1] : 0;
                const LiveLabel l = ix.label[a], lb = ix.label[before];
                int2 rc = make_int2(0, 0);
                if (j < (i > o0 ? lb.n_segs : 1)) rc = live_arcs(ix, l, a, i > o0 ? nv.seg_key[lb.seg_first + j] : start);
                s_rc[x] = rc;
                s_dst[x] = j < l.n_segs ? (uint8_t)nv.seg_key[l.seg_first + j] : 255;
            }
            if (alpha)
                for (int64_t x = tid; x < (int64_t)n * Q; x += NT) alpha[(int64_t)(o0 + w0) * Q + x] = WFST_NINF;
            __syncthreads();
            auto arcs = [&](int t) { return s_rc[t * D + min(g.j, D - 1)]; };
            // the steps of tokens [c0, c1) from the vector v (lane d: destination d)
            auto run = [&](int c0, int c1, double v, bool keep) {
                NarrowPipe<U, L> pipe(ix, g.sub, nv.share, g.j < nv.D);
                auto of = [&](int m) { return arcs(min(c0 + m, c1 - 1)); };
                pipe.start(of);
                for (int t0 = c0; t0 < c1; t0 += K) {
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        const int t = t0 + k;
                        const NarrowArcs<U> &q = pipe.q[k];
                        if (t < c1) {
                            const double vs = __shfl(v, g.j, W);
                            double y[U];
                            int at[U];
#pragma unroll
                            for (int u = 0; u < U; ++u) {  // key 0: none
                                y[u] = u < q.n ? vs + (double)q.sc[u] : -__builtin_huge_val();
                                at[u] = u < q.n ? q.seg[u] : none;
                                atomicMax(&mx[at[u]], y[u] != -__builtin_huge_val() ? live_ord(y[u]) : 0ull);
                            }
                            g.sync();
#pragma unroll
                            for (int u = 0; u < U; ++u) live_add_any(&sm[at[u]], y[u], unord_f64(mx[at[u]]));
                            g.sync();
                            const unsigned long long key = mx[g.lid];
                            const double lse = live_lse(unord_f64(key), sm[g.lid]);
                            v = key ? lse : -__builtin_huge_val();
                            mx[g.lid] = 0ull;
                            sm[g.lid] = 0ull;
                            if (keep && g.lid < D) s_alpha[t * D + g.lid] = (float)v;
                            g.sync();
                        }
                        pipe.next(k, t - c0, of);
                    }
                }
                return v;
            };
            // rows: chunk 0 from its true vector, the others from each source that has arcs
            for (int item = gi; item < nc * D; item += G) {
                const int j = item / nc, k = item - j * nc;
                double v = -__builtin_huge_val();
                if (k == 0 ? j == 0 : s_rc[k * C * D + j].y > 0) {
                    if (k == 0) v = s_in[0][g.lid];
                    else if (g.lid == j) v = 0.0;
                    v = run(k * C, min((k + 1) * C, n), v, alpha && k == 0);
                }
                if (k > 0 || j == 0) s_row[k][j][g.lid] = v;
            }
            __syncthreads();
            // true vectors, one chunk after another: lane (j, d) of the first wavefront
            if (tid < 64) {
                const int d = tid % W, j0 = tid / W;
                constexpr int R = W * W / 64;  // sources of a lane
                double v = s_row[0][0][d];
                for (int k = 1;; ++k) {
                    if (j0 == 0) s_in[k][d] = v;
                    if (k == nc) break;
                    double x[R], m = -__builtin_huge_val(), sum = 0.0;
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const int j = j0 + r * (64 / W);
                        x[r] = j < D ? __shfl(v, j, W) + s_row[k][j][d] : -__builtin_huge_val();
                        m = fmax(m, x[r]);
                    }
#pragma unroll
                    for (int o = W; o < 64; o <<= 1) m = fmax(m, __shfl_xor(m, o, 64));
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        if (x[r] != -__builtin_huge_val()) sum += (double)exp_e((float)(x[r] - m));
#pragma unroll
                    for (int o = W; o < 64; o <<= 1) sum += __shfl_xor(sum, o, 64);
                    v = sum == 0.0 ? -__builtin_huge_val() : m + (double)log_e((float)sum);  // NaN and +inf: NaN
                }
            }
            __syncthreads();
            if (alpha) {
                for (int k = 1 + gi; k < nc; k += G) run(k * C, min((k + 1) * C, n), s_in[k][g.lid], true);
                __syncthreads();
                for (int x = tid; x < n * D; x += NT)
                    if (s_dst[x] != 255) alpha[(int64_t)(o0 + w0 + x / D) * Q + s_dst[x]] = s_alpha[x];
            }
            if (tid < W) s_in[0][tid] = s_in[nc][tid];
        }
        __syncthreads();
        if (tid < W) {  // log Z = LSE of alpha + f
            const int d = tid;
            const double v = s_in[0][d];
            float f = WFST_NINF;
            if (v != -__builtin_huge_val())
                f = final_score[T > 0 ? nv.seg_key[ix.label[bv.tokens[o1 - 1]].seg_first + d] : start];
            const double x = f != WFST_NINF ? v + (double)f : -__builtin_huge_val();
            double m = x;
#pragma unroll
            for (int o = W / 2; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, W));
            double sum = x != -__builtin_huge_val() ? exp(x - m) : 0.0;
#pragma unroll
            for (int o = W / 2; o > 0; o >>= 1) sum += __shfl_xor(sum, o, W);
            if (d == 0) {
                const bool ok = sum != 0.0;
                bv.status[b] = ok ? WFST_STATUS_OK : WFST_STATUS_NO_PATH;
                log_z[b] = ok ? (float)(m + log(sum)) : WFST_NINF;
            }
        }
    }
}

// Backward with expected counts: beta of an arc's destination is fetched from
// the lanes that held it in the step after; the lanes of one source combine
// by shuffles.  Workgroups of one wavefront, or (C) of as many as share a compute
// unit, with cells for the batch's most frequent labels.
template <int W, int U, bool L, bool C>
__global__ void __launch_bounds__(C ? 512 : 64)
narrow_backward(LiveIndex ix, NarrowView nv, int32_t start, const float *__restrict__ final_score, BatchView bv,
                const int32_t *__restrict__ order, const double *__restrict__ val, const int32_t *__restrict__ done,
                const double *__restrict__ log_z, LiveCounts ct, GradFill gf, HotView hot)
{
    constexpr int K = kNarrowAhead;
    extern __shared__ __align__(16) unsigned char lds[];
    if ((int)blockIdx.x < gf.blocks) return live_fill_grad(gf);
    unsigned long long *cell = reinterpret_cast<unsigned long long *>(lds);
    int2 *map = reinterpret_cast<int2 *>(cell + hot.cells);  // {label (-1: none), position - cell}
    const int n_hot = C ? *hot.n : 0;
    if constexpr (C) {
        for (int x = threadIdx.x; x < hot.cells; x += blockDim.x) cell[x] = 0ull;
        for (int x = threadIdx.x; x < kHotMap; x += blockDim.x) map[x] = make_int2(-1, 0);
        __syncthreads();
        for (int x = threadIdx.x; x < n_hot; x += blockDim.x) {
            const HotLabel l = hot.label[x];
            for (uint32_t h = (uint32_t)l.label * 0x9e3779b1u >> 7;; ++h) {  // at most half full
                int2 &e = map[h & (kHotMap - 1)];
                if (atomicCAS(&e.x, -1, l.label) == -1) {
                    e.y = l.first - l.cell;
                    break;
                }
            }
        }
        __syncthreads();
    }
    constexpr int32_t kCold = INT32_MIN;
    auto cells_of = [&](int a) {  // position - cell of a label's arcs
        if constexpr (!C) return kCold;
        for (uint32_t h = (uint32_t)a * 0x9e3779b1u >> 7;; ++h) {
            const int2 e = map[h & (kHotMap - 1)];
            if (e.x == a) return e.y;
            if (e.x < 0) return kCold;
        }
    };
    NarrowGroup<W> g(nv.share, gf.blocks);
    const double scale = *ct.scale;
    int64_t list_at = (int64_t)g.item * kLiveChunk, list_end = list_at + kLiveChunk;
    for (int item = g.item; item < bv.B; item += g.stride) {
        const int b = order ? order[item] : item;
        if (done[b] != 1) continue;
        const int o0 = bv.offsets[b], T = bv.offsets[b + 1] - o0;
        const float gb = ct.grad_log_z ? ct.grad_log_z[b] : 1.0f;
        const double lz = log_z[b];
        auto final_count = [&](int s, double al) {
            const float f = final_score[s];
            if (f != WFST_NINF) fin_add(ct, s, gb * exp_e((float)((al + (double)f) - lz)));
        };
        if (T == 0) {
            if (ct.fin && g.lid == 0) final_count(start, 0.0);
            continue;
        }
        // log alpha of this lane's source at token t (destination j of the token before): loaded, and when it is used
        auto alpha = [&](int t) { return val[(int64_t)(o0 + max(t - 1, 0)) * nv.D + min(g.j, nv.D - 1)]; };
        auto alpha_of = [&](int t, double x) {
            return t <= 0 ? (g.j == 0 ? 0.0 : -__builtin_huge_val()) : g.j < nv.D ? x : -__builtin_huge_val();
        };
        double beta = -__builtin_huge_val();  // of the destination held by this lane: lid >> held
        {
            const LiveLabel l = ix.label[bv.tokens[o0 + T - 1]];
            if (g.lid < l.n_segs) {
                const int s = nv.seg_key[l.seg_first + g.lid];
                beta = (double)final_score[s];
                if (ct.fin) {
                    const double al = val[(int64_t)(o0 + T - 1) * nv.D + g.lid];
                    if (al != -__builtin_huge_val()) final_count(s, al);
                }
            }
        }
        int held = 0;
        NarrowPipe<U, L> pipe(ix, g.sub, nv.share, g.j < nv.D);
        auto of = [&](int m) { return g.arcs(nv, o0 + max(T - 1 - m, 0)); };
        pipe.start(of);
        double al[K];
        int lab[K] = {};
#pragma unroll
        for (int k = 0; k < K; ++k) {
            al[k] = alpha(T - 1 - k);
            if constexpr (C) lab[k] = bv.tokens[o0 + max(T - 1 - k, 0)];
        }
        for (int t0 = T - 1; t0 >= 0; t0 -= K) {
#pragma unroll
            for (int k = 0; k < K; ++k) {
                const int t = t0 - k;
                const NarrowArcs<U> &q = pipe.q[k];
                if (t >= 0) {
                    const double a = alpha_of(t, al[k]);
                    const int32_t base = cells_of(lab[k]);
                    const bool on = a != -__builtin_huge_val();
                    double y[U], m = -__builtin_huge_val();
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const bool has = u < q.n && q.sc[u] > WFST_NINF;
                        const double bt = __shfl(beta, has ? q.seg[u] << held : 0, W);
                        y[u] = has ? (double)q.sc[u] + bt : -__builtin_huge_val();
                        m = fmax(m, y[u]);
                    }
                    for (int o = 1 << nv.share; o > 1; o >>= 1) m = fmax(m, __shfl_xor(m, o >> 1, W));
                    unsigned long long sum = 0ull;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        long long c = 0;
                        if (y[u] != -__builtin_huge_val()) {
                            if (!(y[u] < __builtin_huge_val())) sum |= kLivePoison;
                            else sum += live_fixed(exp_e((float)(y[u] - m)));
                            if (on) c = __double2ll_rn((double)(gb * exp_e((float)((a + y[u]) - lz))) * scale);
                        }
                        const int32_t pos = q.pos + (u << nv.share);
                        if (C && c && base != kCold) atomicAdd(&cell[pos - base], (unsigned long long)c);
                        else if (c) atomicAdd(&ct.acc[pos], (unsigned long long)c);
                        if (!C && ct.touched) {
                            const uint64_t mk = __ballot(c != 0) & (((1ull << W) - 1ull) << (g.gi * W));
                            const int tot = __popcll(mk);
                            if (list_at + tot > list_end) {
                                for (int64_t x = list_at + g.lid; x < min(list_end, ct.touched_cap); x += W)
                                    ct.touched[x] = -1;
                                unsigned long long ch = 0;
                                if (g.lid == 0) ch = atomicAdd(ct.n_touched, (unsigned long long)kLiveChunk);
                                list_at = (int64_t)__shfl(ch, 0, W);
                                list_end = list_at + kLiveChunk;
                            }
                            const int64_t at = list_at + __popcll(mk & ((1ull << (threadIdx.x & 63)) - 1ull));
                            if (c && at < ct.touched_cap) ct.touched[at] = q.pos + (u << nv.share);
                            list_at += tot;
                        }
                    }
                    for (int o = 1 << nv.share; o > 1; o >>= 1) {
                        const unsigned long long w = __shfl_xor(sum, o >> 1, W);
                        sum = ((sum | w) & kLivePoison) | ((sum & ~kLivePoison) + (w & ~kLivePoison));
                    }
                    beta = m == -__builtin_huge_val() ? m : live_lse(m, sum);
                    held = nv.share;
                }
                pipe.next(k, T - 1 - t, of);
                al[k] = alpha(t - K);
                if constexpr (C) lab[k] = bv.tokens[o0 + max(t - K, 0)];
            }
        }
    }
    if (!C && ct.touched)
        for (int64_t x = list_at + g.lid; x < min(list_end, ct.touched_cap); x += W) ct.touched[x] = -1;
    if constexpr (!C) return;
    __syncthreads();
    for (int x = threadIdx.x / 64; x < n_hot; x += blockDim.x / 64) {
        const HotLabel l = hot.label[x];
        for (int k = threadIdx.x % 64; k < l.n; k += 64) {
            const unsigned long long c = cell[l.cell + k];
            if (c) atomicAdd(&ct.acc[l.first + k], c);
        }
    }
}

// Counters of a pass, zero but for what the groups own from the start: pool
// entries (mode 0), or ranges of the touched list (mode 1: a backward pass,
// which keeps the lists of sentences left over; mode 2: nothing to keep).
__device__ __forceinline__ void live_set_counters(int32_t *__restrict__ cnt, int32_t n, int32_t owned, int32_t mode)
{
    const int i = threadIdx.x;
    unsigned long long *c = reinterpret_cast<unsigned long long *>(cnt);
    const int own = mode == 0 ? 2 : 3;  // 64-bit cell
    if (i == 2 * own) c[own] = (unsigned long long)owned;
    else if (i < n && i != 2 * own + 1 && (mode != 1 || i == 8)) cnt[i] = 0;
}
__global__ void live_counters(int32_t *__restrict__ cnt, int32_t n, int32_t owned, int32_t mode)
{
    live_set_counters(cnt, n, owned, mode);
}

// The gradient of the touched arcs from their accumulators, which go back to
// zero.  Every accumulator is looked at when no list was kept or it
// overflowed, or when sentences were left to the streaming sweeps (which keep
// none); else only the listed ones.  every: the gradient of the others is
// written too (zero; it was not filled before).  Then the final states'.
__global__ void __launch_bounds__(256) live_counts_to_grad(LiveCounts ct, LiveIndex ix, int64_t n, bool every,
                                                           const int32_t *__restrict__ n_left, float *__restrict__ grad,
                                                           int32_t Q, float *__restrict__ grad_final)
{
    const double inv = 1.0 / *ct.scale;
    if (grad_final)
        for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < Q; q += gridDim.x * blockDim.x)
            grad_final[q] = fin_value(ct, q);
    const int64_t used = (int64_t)min(*ct.n_touched, (unsigned long long)ct.touched_cap + 1ull);
    const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    if (ct.touched && used <= ct.touched_cap && *n_left == 0) {
        for (int64_t i = i0; i < used; i += step) {
            const int32_t at = ct.touched[i];
            if (at < 0) continue;
            const unsigned long long q = atomicExch(&ct.acc[at], 0ull);  // whichever repeat comes first
            if (q) grad[ix.listed ? at : ix.arc[at].arc] = (float)((double)(long long)q * inv);
        }
    } else {
        for (int64_t e = i0; e < n; e += step) {
            const unsigned long long q = ct.acc[e];
            if (q) ct.acc[e] = 0ull;
            else if (!every) continue;
            grad[ix.listed ? e : ix.arc[e].arc] = (float)((double)(long long)q * inv);
        }
    }
}

// Before the backward sweeps: the accumulators' scale, the final states' sums
// cleared, the pass's counters set (mode: as live_counters).
__global__ void __launch_bounds__(256) live_backward_begin(const float *__restrict__ g, int32_t B, int64_t N,
                                                           double *__restrict__ scale,
                                                           unsigned long long *__restrict__ fin, int64_t fin_n,
                                                           int32_t *__restrict__ cnt, int32_t n, int32_t owned, int32_t mode)
{
    if (fin)
        for (int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < fin_n; q += (int64_t)gridDim.x * blockDim.x)
            fin[q] = 0ull;
    if (blockIdx.x > 0) return;
    live_set_counters(cnt, n, owned, mode);
    fx_scale_of(g, B, N, scale);
}

// =====================================================================
// Input lattices
// =====================================================================
// The live form of lattice_forward: a node's vector is the list of its live
// states (48 of 2071 at the median on confusion networks of the trigram
// tagger).  A node's work is its (incoming arc, live source state) pairs: an
// epsilon arc contributes the source's value, a labelled arc one term per FST
// arc of (label, state).  The pairs' terms are numbered by a prefix sum, one
// thread a term, and all of them meet in one hashed LDS table, maxima first,
// then fixed-point sums; nothing is merged lattice arc by lattice arc.  Bound
// by the latency of a node (waves wait 71% of their cycles): one dependent arc
// load and seven barriers.  4096 networks of 10 to 40 words, streaming form
// 3180 us: 712 us here.  (With FP32 exponentials, 737 us with one thread a pair
// and its terms one after another, 665 with numbered terms.)  What outgrows 384
// states then takes 319 us, beside the last of the others, with 1024 threads a
// lattice (FP32: 310; 375 with 256 threads; 1225 when the streaming form took
// it).
struct LiveLattices {
    LatticeView lv;
    const int32_t *order = nullptr;  // null: 0, 1, ...
    const int32_t *n = nullptr;      // device count (null: all)
    int32_t *left = nullptr, *n_left = nullptr;
    int32_t *count = nullptr;        // [nodes] the lists of nodes read later than by the next one
    int32_t *state = nullptr;        // [nodes * keep]
    double *val = nullptr;
    int32_t keep = 0;                // states of a kept list at most
    double one = 0.0, unit = 0.0;    // 2^S and 2^-S: fixed point of a term at its destination's maximum
};
// List entries and table entries (a power of two) of the first form, of the
// one that takes what outgrows it (a slot of 4 words of 8 tags after another:
// at most 32 by 32 states of a trigram tagger; 1280 leaves room for what epsilon
// arcs add).
constexpr int kLatK = 384, kLatH = 512, kLatK2 = 1280, kLatH2 = 2048;
constexpr int kLatWin = 64;                      // lattice arcs staged at a time
constexpr int kLatPer = 8;                       // FST arcs of a pair, in the form that numbers the terms
// A destination meets at most kLatWin * kLatK2 * (arcs of a label from one
// state) terms, each at most 2^S: S is the largest that keeps their sum below
// 2^62 (45 for one arc, 42 for a tagger's eight).  Exponentials and logarithms
// are FP64, so a term's error is its rounding, 2^-(S + 1) of the largest, and
// the bits do not depend on the order.  Below 31 bits the streaming form runs.
constexpr int kLatBitsMin = 31, kLatBitsMax = 51;
__host__ __device__ constexpr int lat_bits(int64_t arcs_of_pair)
{
    int s = 62;
    for (int64_t n = (int64_t)kLatWin * kLatK2 * (arcs_of_pair > 0 ? arcs_of_pair : 1); n > 1; n = (n + 1) / 2) --s;
    return s < kLatBitsMax ? s : kLatBitsMax;
}
// e^d for d <= 0, in FP64: d = k ln 2 + r with |r| <= ln 2 / 2, Taylor's
// polynomial of degree 11 in r (relative error below 2^-46), scaled by 2^k.
// (4096 networks, whole pass: 878 us; with the library's exp and log, 130
// registers and three wavefronts a SIMD instead of four, 1070; with FP32
// exponentials and logarithms, less than the merge of lattice_forward has, 845.)
__device__ __forceinline__ double lat_exp(double d)
{
    d = fmax(d, -800.0);
    const double k = rint(d * 1.4426950408889634);
    const double r = fma(k, -2.3190468138462996e-17, fma(k, -0.6931471805599453, d));
    double p = 1.0 / 39916800.0;
    p = fma(p, r, 1.0 / 3628800.0);
    p = fma(p, r, 1.0 / 362880.0);
    p = fma(p, r, 1.0 / 40320.0);
    p = fma(p, r, 1.0 / 5040.0);
    p = fma(p, r, 1.0 / 720.0);
    p = fma(p, r, 1.0 / 120.0);
    p = fma(p, r, 1.0 / 24.0);
    p = fma(p, r, 1.0 / 6.0);
    p = fma(p, r, 0.5);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return ldexp(p, (int)k);
}
// log x for x >= 1, in FP64: one Newton step from the FP32 logarithm y, whose
// error f = x e^-y - 1 is about 2^-22, with log(1 + f) = f - f^2 / 2 (+ 2^-67)
__device__ __forceinline__ double lat_log(double x)
{
    const double y = (double)log_e((float)x);
    const double f = fma(x, lat_exp(-y), -1.0);
    return y + fma(-0.5 * f, f, f);
}
// term x under its destination's maximum m (x > -inf) into the sum
__device__ __forceinline__ void lat_add_term(unsigned long long *sum, double x, double m, double one)
{
    if (!(x < __builtin_huge_val())) {
        atomicOr(sum, kLivePoison);
        return;
    }
    // rounded to an integer by the addition: the product is below 2^52, the sum's unit is 1
    const double r = fma(lat_exp(x - m), one, 4503599627370496.0);
    const unsigned long long q = (unsigned long long)__double_as_longlong(r) & 0xfffffffffffffull;
    if (q) atomicAdd(sum, q);
}
__device__ __forceinline__ double lat_lse(double m, unsigned long long s, double unit)
{
    if (s & kLivePoison) return __builtin_nan("");
    return m + lat_log((double)s * unit);
}

template <int NT, int K, int H, bool L>
__global__ void __launch_bounds__(NT)
live_lattice(LiveIndex ix, int32_t Q, int32_t start, int32_t M, const float *__restrict__ final_score, LiveLattices w,
             float *__restrict__ log_z, float *__restrict__ node_alpha, int32_t *__restrict__ status)
{
    // Pairs and terms of a node, in the form that numbers the terms; R: terms of a thread kept for the second pass.
    constexpr int NW = NT / 64, R = 4, kLatPairs = 2 * NT, kLatTerms = 8 * NT;
    const LatticeView &lv = w.lv;
    __shared__ unsigned long long s_mx[H], s_sm[H];
    __shared__ int32_t s_key[H];
    __shared__ double s_val[2][K];     // live values of the last node and of the one being built
    __shared__ int32_t s_state[2][K];
    __shared__ uint16_t s_cl[K];       // table entries claimed
    __shared__ int32_t w_from[kLatWin], w_to[kLatWin], w_lab[kLatWin];
    __shared__ float w_wt[kLatWin];
    __shared__ LiveLabel w_ll[kLatWin];
    __shared__ double p_val[kLatPairs];      // a pair's value with the lattice weight
    __shared__ int32_t p_first[kLatPairs];   // its first arc minus its first term; an epsilon arc's state as ~state
    __shared__ uint16_t s_owner[kLatTerms];  // pair of a term
    __shared__ int s_n, s_item, s_arcs, s_tot[NW], s_first[kLatWin + 1];
    __shared__ unsigned long long s_max, s_sum;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t limit = w.n ? min(*w.n, lv.B) : lv.B;
    if (limit <= 0) return;
    for (int h = tid; h < H; h += NT) {
        s_mx[h] = s_sm[h] = 0ull;
        s_key[h] = -1;
    }
    auto find = [&](int32_t d) {
        for (uint32_t h = ((uint32_t)d * 0x9e3779b1u) >> 7;; ++h) {
            const int at = (int)(h & (uint32_t)(H - 1));
            if (s_key[at] == d) return at;
        }
    };
    // term z of destination d: its table entry, -1 when the list is full
    auto put = [&](int32_t d, double z) {
        if (s_n > K) return -1;
        uint32_t h = ((uint32_t)d * 0x9e3779b1u) >> 7;
        int at, old;
        for (int tries = 0;; ++h, ++tries) {
            at = (int)(h & (uint32_t)(H - 1));
            old = atomicCAS(&s_key[at], -1, d);
            if (old == -1 || old == d) break;
            if (tries >= H) {  // the table is full: far beyond the list
                atomicMax(&s_n, K + 1);
                return -1;
            }
        }
        if (old == -1) {
            const int place = atomicAdd(&s_n, 1);
            if (place < K) s_cl[place] = (uint16_t)at;
        }
        atomicMax(&s_mx[at], live_ord(z));
        return at;
    };
    for (;;) {
        __syncthreads();
        if (tid == 0) s_item = atomicAdd(lv.queue, 1);
        __syncthreads();
        const int item = s_item;
        if (item < 0 || item >= limit) break;
        const int b = w.order ? w.order[item] : item;
        const int n0 = lv.node_off[b], n1 = lv.node_off[b + 1];
        const int a0 = lv.arc_off[b], a1 = lv.arc_off[b + 1];
        const int n = n1 - n0;
        int bad = (*lv.offs_bad || n0 < 0 || n < 1 || (int64_t)n1 > lv.n_nodes || a0 < 0 || a1 < a0 ||
                   (int64_t)a1 > lv.n_arcs) ? 1 : 0;
        int badtok = 0, far = 0;
        if (!bad)
            for (int e = a0 + tid; e < a1; e += NT) {
                const int u = lv.from[e], v = lv.to[e], a = lv.label[e];
                const float x = lv.weight[e];
                bad |= u < 0 || v <= u || v >= n || (e > a0 && lv.to[e - 1] > v) || isnan(x) || x == -WFST_NINF;
                badtok |= a < -1 || a >= M;
                far |= v > u + 1;
            }
        bad = __syncthreads_or(bad);
        badtok = __syncthreads_or(badtok);
        far = __syncthreads_or(far);  // lists are kept in global memory only if some arc skips a node
        if (bad || badtok) {
            if (tid == 0) {
                status[b] = bad ? WFST_STATUS_BAD_INPUT : WFST_STATUS_BAD_TOKEN;
                log_z[b] = WFST_NINF;
            }
            continue;
        }
        auto keep_list = [&](int v, int buf, int count) {
            const int64_t at = (int64_t)(n0 + v) * w.keep;
            if (tid == 0) w.count[n0 + v] = count;
            for (int x = tid; x < count; x += NT) {
                w.state[at + x] = s_state[buf][x];
                w.val[at + x] = s_val[buf][x];
            }
            __threadfence_block();
            __syncthreads();  // read again by this workgroup
        };
        if (tid == 0) {
            s_state[0][0] = start;
            s_val[0][0] = 0.0;
            if (node_alpha) node_alpha[(int64_t)n0 * Q + start] = 0.0f;
        }
        __syncthreads();
        if (far) keep_list(0, 0, 1);
        int np = 1;           // entries of the last node's list
        int wb = a0, wn = 0;  // staged arcs [wb, wb + wn)
        int e = a0;           // next arc
        bool give_up = false;
        for (int v = 1; v < n; ++v) {
            const int cur = v & 1, last = cur ^ 1;
            // the node's arcs: staged with their labels, up to kLatWin at a time
            if (wb + wn < a1 && (wn == 0 || (e > wb && w_to[wn - 1] <= v))) {
                __syncthreads();
                wb = e;
                wn = min(kLatWin, a1 - wb);
                if (tid < wn) {
                    const int a = lv.label[wb + tid];
                    w_from[tid] = lv.from[wb + tid];
                    w_to[tid] = lv.to[wb + tid];
                    w_wt[tid] = lv.weight[wb + tid];
                    w_lab[tid] = a;
                    w_ll[tid] = ix.label[max(a, 0)];
                }
                __syncthreads();
            }
            // first pair of every arc
            if (tid < 64) {
                const int k = e - wb + lane;
                const bool mine = k < wn && w_to[k] == v;
                int c = 0;
                if (mine) c = w_from[k] == v - 1 ? np : gload(&w.count[n0 + w_from[k]]);
                int inc = c;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const int up = __shfl_up(inc, o, 64);
                    if (lane >= o) inc += up;
                }
                s_first[lane + 1] = inc;
                const int arcs = __popcll(__ballot(mine));
                if (lane == 0) {
                    s_first[0] = 0;
                    s_n = 0;
                    s_arcs = arcs;
                }
            }
            __syncthreads();
            const int arcs = s_arcs;
            if (e + arcs == wb + wn && wb + wn < a1 && lv.to[e + arcs] == v) {  // more arcs than are staged
                give_up = true;
                break;
            }
            const int P = s_first[arcs];
            const int top = arcs > 1 ? 1 << (31 - __clz(arcs - 1)) : 0;
            // pair p: its source state, its value, its FST arcs (an epsilon arc: count -1)
            auto pair = [&](int p, int &s, double &x, bool &eps) {
                int k = 0;  // the last arc whose first pair is not behind p
                for (int step = top; step > 0; step >>= 1)
                    if (s_first[k + step] <= p) k += step;
                const int a = e - wb + k, u = w_from[a], x_at = p - s_first[k];
                if (u == v - 1) {
                    s = s_state[last][x_at];
                    x = s_val[last][x_at];
                } else {
                    s = gload(&w.state[(int64_t)(n0 + u) * w.keep + x_at]);
                    x = gload(&w.val[(int64_t)(n0 + u) * w.keep + x_at]);
                }
                x += (double)w_wt[a];
                eps = w_lab[a] < 0;
                return eps ? make_int2(0, 1) : live_arcs(ix, w_ll[a], w_lab[a], s);
            };
            // number the terms: two pairs a thread
            int2 rc[2];
            int st[2] = {0, 0};
            double pv[2] = {0.0, 0.0};
            bool eps[2] = {false, false};
            bool wide = P > kLatPairs;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int p = 2 * tid + u;
                rc[u] = make_int2(0, 0);
                if (p < P && p < kLatPairs) rc[u] = pair(p, st[u], pv[u], eps[u]);
                wide |= rc[u].y > kLatPer;
            }
            const int mine = rc[0].y + rc[1].y;
            int inc = mine;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int up = __shfl_up(inc, o, 64);
                if (lane >= o) inc += up;
            }
            if (lane == 63) s_tot[wave] = inc;
            wide = __syncthreads_or(wide);
            int off = inc - mine, E = 0;
#pragma unroll
            for (int x = 0; x < NW; ++x) {
                off += x < wave ? s_tot[x] : 0;
                E += s_tot[x];
            }
            wide |= E > kLatTerms;
            int slot[R];
            double term[R];
#pragma unroll
            for (int r = 0; r < R; ++r) slot[r] = -1;
            if (!wide) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int p = 2 * tid + u;
                    if (rc[u].y > 0) {
                        p_val[p] = pv[u];
                        p_first[p] = eps[u] ? ~st[u] : rc[u].x - off;
                    }
                    for (int r = 0; r < rc[u].y; ++r) s_owner[off + r] = (uint16_t)(p | (eps[u] ? 0x8000 : 0));
                    off += rc[u].y;
                }
                __syncthreads();
                auto one = [&](int t, int32_t &d, double &z) {
                    const int o = s_owner[t], p = o & 0x7fff;
                    z = p_val[p];
                    if (o & 0x8000) {
                        d = ~p_first[p];
                    } else {
                        const int32_t at = p_first[p] + t;
                        const LiveArc x = ix.arc[at];
                        z += (double)live_score<L>(ix, at, x);
                        d = x.dst;
                    }
                };
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int t = tid + r * NT;
                    int32_t d;
                    if (t < E) {
                        one(t, d, term[r]);
                        if (term[r] != -__builtin_huge_val()) slot[r] = put(d, term[r]);
                    }
                }
                for (int t = tid + R * NT; t < E; t += NT) {
                    int32_t d;
                    double z;
                    one(t, d, z);
                    if (z != -__builtin_huge_val()) put(d, z);
                }
                __syncthreads();
                if (s_n > K) {
                    give_up = true;
                    break;
                }
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (slot[r] >= 0) lat_add_term(&s_sm[slot[r]], term[r], unord_f64(s_mx[slot[r]]), w.one);
                for (int t = tid + R * NT; t < E; t += NT) {
                    int32_t d;
                    double z;
                    one(t, d, z);
                    if (z == -__builtin_huge_val()) continue;
                    const int at = find(d);
                    lat_add_term(&s_sm[at], z, unord_f64(s_mx[at]), w.one);
                }
            } else {
                // A node over half of its labels' many arcs is the streaming form's.  (Where other nodes are small, lists
                // are faster in all for larger nodes too: 1024 of 2071 states in a slot of frequent words.)
                if (tid == 0) s_max = s_sum = 0ull;
                __syncthreads();
                unsigned long long terms = 0;
                for (int p = tid; p < P; p += NT) {
                    int s;
                    double x;
                    bool ep;
                    const int2 c = pair(p, s, x, ep);
                    terms += ep ? 0ull : (unsigned long long)c.y;
                }
                if (terms) atomicAdd(&s_max, terms);
                if (tid < arcs && w_lab[e - wb + tid] >= 0)
                    atomicAdd(&s_sum, (unsigned long long)ix.all[w_lab[e - wb + tid]].y);
                __syncthreads();
                if (s_max > kLiveStreamArcs && s_max > s_sum / 2) {
                    give_up = true;
                    break;
                }
                // many pairs, or pairs with many arcs: NT pairs at a time, twice; a thread a pair, or (one of them has
                // more than kLatPer arcs) their terms numbered and a term's pair found by bisection
                auto one = [&](int pass, int32_t d, double z) {
                    if (z == -__builtin_huge_val()) return;
                    if (pass == 0) {
                        put(d, z);
                    } else {
                        const int at = find(d);
                        lat_add_term(&s_sm[at], z, unord_f64(s_mx[at]), w.one);
                    }
                };
                int32_t *pre = p_first, *base = p_first + NT;  // first term of a pair, its first arc minus that
                for (int pass = 0; pass < 2; ++pass) {
                    for (int p0 = 0; p0 < P; p0 += NT) {
                        int s = 0;
                        double x = 0.0;
                        bool ep = false;
                        const int2 c = p0 + tid < P ? pair(p0 + tid, s, x, ep) : make_int2(0, 0);
                        if (!__syncthreads_or(c.y > kLatPer)) {
                            if (ep) one(pass, s, x);
                            else
                                for (int r = 0; r < c.y && (pass > 0 || s_n <= K); ++r) {
                                    const LiveArc y = ix.arc[c.x + r];
                                    one(pass, y.dst, x + (double)live_score<L>(ix, c.x + r, y));
                                }
                            continue;
                        }
                        int upto = c.y;
#pragma unroll
                        for (int o = 1; o < 64; o <<= 1) {
                            const int up = __shfl_up(upto, o, 64);
                            if (lane >= o) upto += up;
                        }
                        if (lane == 63) s_tot[wave] = upto;
                        __syncthreads();
                        int at0 = upto - c.y, total = 0;
#pragma unroll
                        for (int y = 0; y < NW; ++y) {
                            at0 += y < wave ? s_tot[y] : 0;
                            total += s_tot[y];
                        }
                        pre[tid] = at0;
                        base[tid] = ep ? ~s : c.x - at0;
                        p_val[tid] = x;
                        s_owner[tid] = ep;
                        __syncthreads();
                        for (int t = tid; t < total && (pass > 0 || s_n <= K); t += NT) {
                            int o = 0;
#pragma unroll
                            for (int step = NT / 2; step > 0; step >>= 1)
                                if (pre[o + step] <= t) o += step;
                            if (s_owner[o]) {
                                one(pass, ~base[o], p_val[o]);
                            } else {
                                const int32_t pos = base[o] + t;
                                const LiveArc y = ix.arc[pos];
                                one(pass, y.dst, p_val[o] + (double)live_score<L>(ix, pos, y));
                            }
                        }
                    }
                    __syncthreads();
                    if (s_n > K) break;
                }
                if (s_n > K) {
                    give_up = true;
                    break;
                }
            }
            __syncthreads();
            const int nn = s_n;
            for (int x = tid; x < nn; x += NT) {
                const int at = s_cl[x];
                const int32_t d = s_key[at];
                const double y = lat_lse(unord_f64(s_mx[at]), s_sm[at], w.unit);
                s_state[cur][x] = d;
                s_val[cur][x] = y;
                if (node_alpha) node_alpha[(int64_t)(n0 + v) * Q + d] = (float)y;
                s_mx[at] = s_sm[at] = 0ull;
                s_key[at] = -1;
            }
            __syncthreads();
            if (far) keep_list(v, cur, nn);
            np = nn;
            e += arcs;
        }
        if (give_up) {
            __syncthreads();
            for (int h = tid; h < H; h += NT) {
                s_mx[h] = s_sm[h] = 0ull;
                s_key[h] = -1;
            }
            if (tid == 0) w.left[atomicAdd(w.n_left, 1)] = b;
            continue;
        }
        // log Z = LSE of the last node's values + f, the sum in fixed point like a node's
        const int lb = (n - 1) & 1;
        if (tid == 0) s_max = s_sum = 0ull;
        __syncthreads();
        for (int x = tid; x < np; x += NT) {
            const float f = final_score[s_state[lb][x]];
            const double y = s_val[lb][x] + (double)f;
            if (f != WFST_NINF && y != -__builtin_huge_val()) atomicMax(&s_max, live_ord(y));
        }
        __syncthreads();
        const double m = unord_f64(s_max);
        for (int x = tid; x < np; x += NT) {
            const float f = final_score[s_state[lb][x]];
            const double y = s_val[lb][x] + (double)f;
            if (f != WFST_NINF && y != -__builtin_huge_val()) lat_add_term(&s_sum, y, m, w.one);
        }
        __syncthreads();
        if (tid == 0) {
            const bool ok = s_max != 0ull;
            status[b] = ok ? WFST_STATUS_OK : WFST_STATUS_NO_PATH;
            log_z[b] = ok ? (float)lat_lse(m, s_sum, w.unit) : WFST_NINF;
        }
    }
}

// =====================================================================
// Sentences left to the streaming sweeps
// =====================================================================
// Their compact per-step storage: offsets of every token, each sentence's
// range taken from one counter (at most tokens x the widest label in all).
// stale: the sliced layouts' scores are current from here on, if any pass reads them.
__global__ void __launch_bounds__(64) rest_offsets(DevLayout fl, BatchView bv, unsigned long long *__restrict__ total,
                                                   int64_t *__restrict__ tok_off, int32_t *__restrict__ stale)
{
    const int lane = threadIdx.x;
    const int32_t limit = bv.count();
    if (blockIdx.x == 0 && lane == 0 && limit > 0) *stale = 0;
    for (int x = blockIdx.x; x < limit; x += gridDim.x) {
        const int b = bv.order[x];  // checked by the live sweep
        const int o0 = bv.offsets[b], o1 = bv.offsets[b + 1];
        unsigned long long sum = 0;
        for (int i = o0 + lane; i < o1; i += 64) sum += (unsigned long long)fl.label[bv.tokens[i]].n_segs;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        unsigned long long at = 0;
        if (lane == 0) at = atomicAdd(total, sum);
        at = __shfl(at, 0, 64);
        for (int i0 = o0; i0 < o1; i0 += 64) {
            const int i = i0 + lane;
            const int n = i < o1 ? fl.label[bv.tokens[i]].n_segs : 0;
            int inc = n;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int up = __shfl_up(inc, o, 64);
                if (lane >= o) inc += up;
            }
            if (i < o1) tok_off[i] = (int64_t)at + inc - n;
            at += (unsigned long long)__shfl(inc, 63, 64);
        }
    }
}

// Their final-state posteriors, from the tape of the streaming sweep, into
// the fixed-point sums of the live ones (one wavefront per sentence).
// list: sentences of a batch of which `bv` holds only these (else null).
__device__ __forceinline__ void rest_final_of(const BatchView &bv, const TapeView &tp, const DevLayout &fl,
                                              int32_t start, const float *__restrict__ final_score,
                                              const LiveCounts &ct, int b, int tid, int nt)
{
    const int o0 = bv.offsets[b], o1 = bv.offsets[b + 1];
    const float g = ct.grad_log_z ? ct.grad_log_z[b] : 1.0f;
    if (o1 == o0) {
        const float f = final_score[start];
        if (tid == 0 && f != WFST_NINF) fin_add(ct, start, g * exp_e(f + (float)(0.0 - tp.log_z[b])));
        return;
    }
    const int i = o1 - 1;
    const LabelInfo lf = fl.label[bv.tokens[i]];
    const float *ta = tp.alpha + (tp.ck_off ? tp.ck_off[i] : bv.tok_off[i]);
    const float c = tp.a_max[i], o = (float)(tp.a_log[i] - tp.log_z[b]);
    for (int j = tid; j < lf.n_segs; j += nt) {
        const int s = fl.seg_key[lf.seg_first + j];
        const float y = ta[j], f = final_score[s];
        if (y == WFST_NINF || f == WFST_NINF) continue;
        fin_add(ct, s, g * exp_e(((y - c) + f) + o));
    }
}
__global__ void rest_final(BatchView bv, TapeView tp, DevLayout fl, int32_t start,
                           const float *__restrict__ final_score, LiveCounts ct)
{
    const int32_t limit = bv.count();
    for (int x = blockIdx.x; x < limit; x += gridDim.x) {
        const int b = bv.n ? bv.order[x] : x;
        if (bv.status[b] == WFST_STATUS_OK) rest_final_of(bv, tp, fl, start, final_score, ct, b, threadIdx.x, 64);
    }
}

// Backward pass and expected counts of the sentences left to the streaming
// sweeps.  backward_sweep picks the segments of the states that matter and
// gives each to a thread, which suits few of them, and adds every posterior to
// its accumulator with an atomic.  A sentence is left because most states are
// live: 512 strings over 2000 states and 20 labels took 8.4 ms that way, 4.1 ms
// of it gathering slices out of order and the rest 183M atomics.  Here
// rest_backward streams each label's reverse slices in order, as the forward
// sweep does, and only keeps beta; the visits are grouped by label and counted
// by rest_counts.  Same arithmetic as backward_sweep, segment by segment, and
// the same rounding of each posterior: the same bits.

// The counts of left sentences that backward_sweep took by reverse-layout slot
// (neighbouring arcs of a step share lines there; indexed by (label, source)
// its atomics took 22 ms instead of 12.7 for a string over 20000 of 25011 live
// states) added to the others'; the slots' sums go back to zero.
__global__ void __launch_bounds__(256) rest_slot_counts(unsigned long long *__restrict__ slot, int64_t n,
                                                        const int32_t *__restrict__ pos,
                                                        const int32_t *__restrict__ n_left,
                                                        unsigned long long *__restrict__ acc)
{
    if (n_left && *n_left <= 0) return;
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const unsigned long long c = slot[e];
        if (!c) continue;
        slot[e] = 0ull;
        acc[pos[e]] += c;
    }
}

// A token's place among the left tokens of its label.
__global__ void rest_rank(BatchView bv, RestGroups rg)
{
    const int32_t limit = bv.count();
    for (int x = blockIdx.x; x < limit; x += gridDim.x) {
        const int b = bv.order[x];
        if (bv.status[b] != WFST_STATUS_OK) continue;
        for (int i = bv.offsets[b] + (int)threadIdx.x; i < bv.offsets[b + 1]; i += blockDim.x)
            rg.rank[i] = atomicAdd(&rg.label_n[bv.tokens[i]], 1);
    }
}

template <int NT>
__global__ void __launch_bounds__(NT)
rest_backward(DevLayout fl, DevLayout rl, int32_t Q, int32_t start, const float *__restrict__ final_score,
              const float *__restrict__ final_max, BatchView bv, TapeView tp, RestGroups rg, LiveCounts ct)
{
    extern __shared__ __align__(16) unsigned char lds[];
    float *val0 = reinterpret_cast<float *>(lds);
    float *val1 = val0 + (Q + 1);
    const RestCarve at = rest_carve(Q, rl.max_segs, rl.max_slots);
    double *vval = reinterpret_cast<double *>(lds + at.lse.vval);
    double *part = reinterpret_cast<double *>(lds + at.lse.part);
    int32_t *vkey = reinterpret_cast<int32_t *>(lds + at.lse.vkey);
    float *part_s = reinterpret_cast<float *>(lds + at.part_s);
    uint8_t *marks = lds + at.marks;  // [3][Q+1] states of a step, steps mod 3
    __shared__ int s_item;
    __shared__ unsigned long long s_cmax[3];
    const int tid = threadIdx.x, lane = tid & 63, wave = wave_uniform(tid >> 6);
    const int32_t limit = bv.count();
    if (limit <= 0) return;
    const float fmax0 = *final_max;
    for (;;) {
        if (tid == 0) s_item = atomicAdd(bv.queue, 1);
        __syncthreads();
        const int item = wave_uniform(s_item);
        __syncthreads();
        if (item < 0 || item >= limit) break;
        const int b = bv.order[item];
        if (bv.status[b] != WFST_STATUS_OK) continue;
        const int o0 = bv.offsets[b], o1 = bv.offsets[b + 1], T = o1 - o0;
        if (ct.fin) rest_final_of(bv, tp, fl, start, final_score, ct, b, tid, NT);
        if (T == 0) {
            if (tid == 0) tp.log_z_bwd[b] = (double)final_score[start];
            continue;
        }
        for (int i = o0 + tid; i < o1; i += NT) rg.tok[rg.first[bv.tokens[i]] + rg.rank[i]] = make_int2(i, b);
        float *vT = (T & 1) ? val1 : val0, *vO = (T & 1) ? val0 : val1;
        for (int q = tid; q <= Q; q += NT) {  // beta^_T = f - max f, with C = max f
            const float f = q < Q ? final_score[q] : WFST_NINF;
            vT[q] = f != WFST_NINF ? f - fmax0 : WFST_NINF;
            vO[q] = WFST_NINF;
        }
        for (int q = tid; q < 3 * (Q + 1); q += NT) marks[q] = 0;
        if (tid < 3) s_cmax[tid] = 0ull;
        __syncthreads();
        // states of step t - 1: the destinations of token t - 1, or the start state
        auto mark = [&](int t, int2 l) {
            uint8_t *m = marks + (t % 3) * (Q + 1);
            if (t >= 2) {
                for (int j = tid; j < l.y; j += NT) m[fl.seg_key[l.x + j]] = 1;
            } else if (tid == 0) {
                m[start] = 1;
            }
        };
        auto dests = [&](int i) {  // {first segment, segments} of a token's destinations
            const LabelInfo *l = fl.label + bv.tokens[max(i, o0)];
            return make_int2(l->seg_first, l->n_segs);
        };
        LabelInfo li = rl.label[bv.tokens[o1 - 1]];
        int2 f0 = dests(o1 - 1), f1 = dests(o1 - 2), f2 = dests(o1 - 3);  // of tokens t, t - 1, t - 2
        mark(T, f1);
        for (int j = tid; j < f0.y; j += NT) tp.beta[bv.tok_off[o1 - 1] + j] = vT[fl.seg_key[f0.x + j]];
        if (tid == 0) {
            tp.b_max[o1 - 1] = 0.0f;
            tp.b_log[o1 - 1] = (double)fmax0;
        }
        double C = (double)fmax0;
        __syncthreads();
        for (int t = T; t >= 1; --t) {
            float *prev = (t & 1) ? val1 : val0, *cur = (t & 1) ? val0 : val1;
            const int i = o0 + t - 1;
            // in flight during this step
            const LabelInfo li_next = rl.label[bv.tokens[max(i - 1, o0)]];
            const int2 f3 = dests(i - 3);
            if (t >= 2) mark(t - 1, f2);
            const uint8_t *m = marks + (t % 3) * (Q + 1);
            const double mx = lse_step<NT, 4, true>(rl, li, prev, part, vval, vkey, lane, wave, Q, part_s,
                                                    [&](int32_t q) { return m[q] != 0; });
            // beta^_t is read: its tape, and its support cleared (everything at the first step)
            if (t == T) {
                for (int q = tid; q < Q; q += NT) prev[q] = WFST_NINF;
            } else {
                uint8_t *old = marks + ((t + 1) % 3) * (Q + 1);
                float *tape = tp.beta + bv.tok_off[i];
                for (int j = tid; j < f0.y; j += NT) {
                    const int q = fl.seg_key[f0.x + j];
                    tape[j] = prev[q];
                    prev[q] = WFST_NINF;
                    old[q] = 0;
                }
            }
            if (tid == 0) s_cmax[(t + 1) % 3] = 0ull;
            block_max_d(mx, &s_cmax[t % 3], lane);
            __syncthreads();
            double c = unord_f64(s_cmax[t % 3]);
            if (!(c > -__builtin_huge_val())) c = 0.0;
            for (int j = tid; j < li.n_segs; j += NT) {
                const double v = vval[j];
                const int32_t q = vkey[j];
                cur[q] = v == -__builtin_huge_val() ? WFST_NINF : (float)(v - c);
                if (t == 1 && q == start) tp.log_z_bwd[b] = v == -__builtin_huge_val() ? v : C + v;
            }
            C += c;
            if (t >= 2 && tid == 0) {
                tp.b_max[i - 1] = 0.0f;  // the tape is normalised
                tp.b_log[i - 1] = C;
            }
            __syncthreads();
            li = uniform_label(li_next);
            f0 = f1;
            f1 = f2;
            f2 = f3;
        }
    }
}

// Counts.  A workgroup takes kRestV visits and kRestR arcs a thread of one
// label: the arcs stay in registers with their sums over all those visits, the
// visits' alpha and beta vectors are staged in LDS, TT of them at a time, one
// row of TT values a state, and an arc meets its accumulator once: 0.52 ms for
// the 183M posteriors, bound by their exponentials and roundings.
constexpr int kRestV = 64, kRestR = 8, kRestThreads = 512;
constexpr int kRestArcs = kRestR * kRestThreads;

__host__ __device__ __forceinline__ int rest_items(int visits, int arcs)
{
    return ((visits + kRestV - 1) / kRestV) * ((arcs + kRestArcs - 1) / kRestArcs);
}

// Offsets of the labels' visits and work items (one workgroup), and their counters back to zero.
__global__ void __launch_bounds__(1024)
rest_group(RestGroups rg, const int2 *__restrict__ all, int32_t M, const int32_t *__restrict__ n_left)
{
    __shared__ int3 s_sum[1024];
    if (*n_left <= 0) return;
    const int tid = threadIdx.x, per = (M + 1023) / 1024;
    const int a0 = min(tid * per, M), a1 = min(a0 + per, M);
    int3 sum = make_int3(0, 0, 0);  // visits, labels, items
    for (int a = a0; a < a1; ++a) {
        const int n = rg.label_n[a];
        if (n == 0) continue;
        sum.x += n;
        sum.y += 1;
        sum.z += rest_items(n, all[a].y);
    }
    s_sum[tid] = sum;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        int3 x = make_int3(0, 0, 0);
        if (tid >= o) x = s_sum[tid - o];
        __syncthreads();
        s_sum[tid] = make_int3(s_sum[tid].x + x.x, s_sum[tid].y + x.y, s_sum[tid].z + x.z);
        __syncthreads();
    }
    int3 at = make_int3(s_sum[tid].x - sum.x, s_sum[tid].y - sum.y, s_sum[tid].z - sum.z);
    for (int a = a0; a < a1; ++a) {
        const int n = rg.label_n[a];
        if (n == 0) continue;
        rg.label_n[a] = 0;
        rg.first[a] = at.x;
        rg.label[at.y] = RestLabel{a, at.x, n, at.z};
        at.x += n;
        at.y += 1;
        at.z += rest_items(n, all[a].y);
    }
    if (tid == 1023) {
        rg.label[at.y] = RestLabel{-1, at.x, 0, at.z};
        *rg.n_label = at.y;
    }
}

template <int TT>
__global__ void __launch_bounds__(kRestThreads)
rest_counts(LiveIndex ix, DevLayout fl, int32_t Q, int32_t start, BatchView bv, TapeView tp, RestGroups rg,
            LiveCounts ct)
{
    constexpr int NT = kRestThreads;
    extern __shared__ __align__(16) unsigned char lds[];
    float *av = reinterpret_cast<float *>(lds);  // [Q][TT] alpha before the visit
    float *bw = av + (int64_t)Q * TT;            // [Q][TT] beta after it, with the visit's scale
    __shared__ int2 s_tok[kRestV];
    __shared__ LabelInfo s_prev[kRestV];
    __shared__ float s_cm[kRestV], s_o[kRestV], s_g[kRestV];
    if (*bv.n <= 0) return;
    const int tid = threadIdx.x, nl = *rg.n_label;
    const int items = rg.label[nl].item;
    const double fx = *ct.scale;
    for (int item = blockIdx.x; item < items; item += gridDim.x) {
        int lo = 0, hi = nl;  // the last label whose first item is not behind this one
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (rg.label[mid].item <= item) lo = mid; else hi = mid;
        }
        const RestLabel rl = rg.label[lo];
        const int2 all = ix.all[rl.label];
        const LabelInfo lf = fl.label[rl.label];
        const int chunks = (all.y + kRestArcs - 1) / kRestArcs, x = item - rl.item;
        const int v0 = (x / chunks) * kRestV, nv = min(kRestV, rl.n - v0);
        const int p0 = all.x + (x % chunks) * kRestArcs, p1 = all.x + all.y;
        int src[kRestR], dst[kRestR];
        float sc[kRestR];
        long long sum[kRestR];
#pragma unroll
        for (int r = 0; r < kRestR; ++r) {
            const int p = p0 + r * NT + tid;
            src[r] = -1;
            dst[r] = 0;
            sc[r] = 0.0f;
            sum[r] = 0;
            if (p < p1) {
                const LiveArc y = ix.arc[p];
                src[r] = y.src * TT;
                dst[r] = y.dst * TT;
                sc[r] = ix.listed ? live_score<true>(ix, p, y) : live_score<false>(ix, p, y);
            }
        }
        __syncthreads();  // the last item's vectors are read
        if (tid < nv) {
            const int2 t = rg.tok[rl.first + v0 + tid];
            const bool first = t.x == bv.offsets[t.y];
            s_tok[tid] = make_int2(t.x, first ? 1 : 0);
            LabelInfo lp{};
            if (!first) lp = fl.label[bv.tokens[t.x - 1]];
            s_prev[tid] = lp;
            s_cm[tid] = first ? 0.0f : tp.a_max[t.x - 1];
            s_o[tid] = (float)((first ? 0.0 : tp.a_log[t.x - 1]) + tp.b_log[t.x] - tp.log_z[t.y]);
            s_g[tid] = ct.grad_log_z ? ct.grad_log_z[t.y] : 1.0f;
        }
        for (int64_t y = tid; y < (int64_t)Q * TT; y += NT) bw[y] = WFST_NINF;
        for (int t0 = 0; t0 < nv; t0 += TT) {
            __syncthreads();  // s_tok is there; the last tile's vectors are read
            for (int64_t y = tid; y < (int64_t)Q * TT; y += NT) av[y] = WFST_NINF;
            __syncthreads();
#pragma unroll
            for (int u = 0; u < TT; ++u) {
                const int k = t0 + u;
                if (k < nv) {
                    const int2 t = s_tok[k];
                    const LabelInfo lp = s_prev[k];
                    const float cm = s_cm[k], o = s_o[k];
                    const float *ta = t.y ? nullptr : tp.alpha + bv.tok_off[t.x - 1], *tb = tp.beta + bv.tok_off[t.x];
                    if (t.y) {
                        if (tid == 0) av[start * TT + u] = 0.0f;
                    } else {
                        for (int j = tid; j < lp.n_segs; j += NT) av[fl.seg_key[lp.seg_first + j] * TT + u] = ta[j] - cm;
                    }
                    for (int j = tid; j < lf.n_segs; j += NT) bw[fl.seg_key[lf.seg_first + j] * TT + u] = tb[j] + o;
                }
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < kRestR; ++r) {
                if (src[r] < 0) continue;
                float a[TT], b[TT];
#pragma unroll
                for (int u = 0; u < TT; ++u) {
                    a[u] = av[src[r] + u];
                    b[u] = bw[dst[r] + u];
                }
#pragma unroll
                for (int u = 0; u < TT; ++u)
                    if (a[u] != WFST_NINF && b[u] != WFST_NINF)  // av is -inf past the last visit
                        sum[r] += __double2ll_rn((double)(s_g[t0 + u] * exp_e((a[u] + sc[r]) + b[u])) * fx);
            }
        }
#pragma unroll
        for (int r = 0; r < kRestR; ++r)
            if (sum[r]) atomicAdd(&ct.acc[p0 + r * NT + tid], (unsigned long long)sum[r]);
    }
}

// =====================================================================
// Building the index from the sliced layouts
// =====================================================================
__device__ __forceinline__ void seg_chunks(const DevLayout &L, const LabelInfo &li, int j, int &c0, int &nc)
{
    if (j < li.n_multi) {
        const SegChunk sc = L.seg_chunk[li.seg_first + j];
        c0 = sc.first;
        nc = sc.count;
    } else {
        c0 = li.n_slots + (j - li.n_multi);
        nc = 1;
    }
}

// arcs of every segment of a layout (one thread per segment, one workgroup per label)
__global__ void live_seg_sizes(DevLayout L, int32_t M, int32_t *__restrict__ size)
{
    for (int a = blockIdx.x; a < M; a += gridDim.x) {
        const LabelInfo li = L.label[a];
        for (int j = threadIdx.x; j < li.n_segs; j += blockDim.x) {
            int c0, nc, n = 0;
            seg_chunks(L, li, j, c0, nc);
            for (int c = c0; c < c0 + nc; ++c) {
                const SliceInfo si = L.slice[li.slice_first + (c >> 6)];
                const int col = si.base + (c & 63);
                int h = si.height;  // padding rows are at the end of the chunk
                while (h > 0 && L.elem_arc[col + (h - 1) * si.width] < 0) --h;
                n += h;
            }
            size[li.seg_first + j] = n;
        }
    }
}

// every arc's destination segment, counted within its label (forward layout)
__global__ void live_segs(DevLayout fl, int32_t M, int32_t *__restrict__ seg_of)
{
    for (int a = blockIdx.x; a < M; a += gridDim.x) {
        const LabelInfo li = fl.label[a];
        for (int j = threadIdx.x; j < li.n_segs; j += blockDim.x) {
            int c0, nc;
            seg_chunks(fl, li, j, c0, nc);
            for (int c = c0; c < c0 + nc; ++c) {
                const SliceInfo si = fl.slice[li.slice_first + (c >> 6)];
                for (int r = 0; r < si.height; ++r) {
                    const int id = fl.elem_arc[si.base + (c & 63) + r * si.width];
                    if (id < 0) break;
                    seg_of[id] = j;
                }
            }
        }
    }
}

// The arcs by (label, source), and where each reverse slot's arc went.  first[] = exclusive
// prefix sums of the reverse layout's segment sizes.
__global__ void live_fill(DevLayout fl, DevLayout rl, int32_t M, int32_t Q, const int32_t *__restrict__ size,
                          const int32_t *__restrict__ first, const int32_t *__restrict__ seg_of,
                          LiveArc *__restrict__ arc, float *__restrict__ score,
                          int32_t *__restrict__ pos, LiveLabel *__restrict__ label, int2 *__restrict__ all,
                          int32_t *__restrict__ unsorted)
{
    __shared__ int s_same;
    for (int a = blockIdx.x; a < M; a += gridDim.x) {
        const LabelInfo li = rl.label[a];
        __syncthreads();
        if (threadIdx.x == 0) s_same = li.n_segs == Q;
        __syncthreads();
        const int per = li.n_segs > 0 ? size[li.seg_first] : 0;
        for (int j = threadIdx.x; j < li.n_segs; j += blockDim.x) {
            if (size[li.seg_first + j] != per) s_same = 0;
            int c0, nc, at = first[li.seg_first + j];
            seg_chunks(rl, li, j, c0, nc);
            for (int c = c0; c < c0 + nc; ++c) {
                const SliceInfo si = rl.slice[li.slice_first + (c >> 6)];
                for (int r = 0; r < si.height; ++r) {
                    const int e = si.base + (c & 63) + r * si.width;
                    const int id = rl.elem_arc[e];
                    if (id < 0) break;
                    arc[at] = LiveArc{rl.other[e], id, rl.seg_key[li.seg_first + j], seg_of[id]};
                    pos[e] = at;
                    score[id] = rl.score[e];
                    if (id != at) *unsorted = 1;
                    ++at;
                }
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            LiveLabel l;
            l.first = li.n_segs > 0 ? first[li.seg_first] : 0;
            // same size and every state present: segments are in state order
            l.per = li.n_segs == 0 ? 0 : (s_same ? per : -1);
            l.row = (int64_t)a * Q;
            l.seg_first = fl.label[a].seg_first;
            l.n_segs = fl.label[a].n_segs;
            const int end = li.seg_first + li.n_segs - 1;
            all[a] = make_int2(l.first, li.n_segs > 0 ? first[end] + size[end] - l.first : 0);
            label[a] = l;
            if (l.per < 0) unsorted[1] = 1;
        }
    }
}

// {first, count} of every (label, source): the row table (zeroed before) or the pair table (label = -1 before).
__global__ void live_lookup(DevLayout rl, int32_t M, int32_t Q, const int32_t *__restrict__ size,
                            const int32_t *__restrict__ first, int2 *__restrict__ row, LivePair *__restrict__ pair,
                            uint32_t mask)
{
    for (int a = blockIdx.x; a < M; a += gridDim.x) {
        const LabelInfo li = rl.label[a];
        for (int j = threadIdx.x; j < li.n_segs; j += blockDim.x) {
            const int s = rl.seg_key[li.seg_first + j], f = first[li.seg_first + j], c = size[li.seg_first + j];
            if (row) {
                row[(int64_t)a * Q + s] = make_int2(f, c);
            } else {
                for (uint32_t h = live_pair_hash((uint32_t)a, (uint32_t)s);; ++h) {
                    LivePair *p = pair + (h & mask);
                    if (atomicCAS(&p->label, -1, a) == -1) {  // pairs are distinct: a taken entry is another pair's
                        p->src = s;
                        p->first = f;
                        p->count = c;
                        break;
                    }
                }
            }
        }
    }
}

// New scores in arc-id order (-0 stored as +0); the sliced layouts are stale from here on.
__global__ void __launch_bounds__(256) live_scores(float *__restrict__ out, int64_t n, const float *__restrict__ score,
                                                   int32_t wide, int32_t *__restrict__ stale)
{
    const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    if (i0 == 0) *stale = 1;
    int64_t done = 0;
    if (wide) {  // both 16-byte aligned
        const float4 *in4 = reinterpret_cast<const float4 *>(score);
        float4 *out4 = reinterpret_cast<float4 *>(out);
        const int64_t n4 = n / 4;
        for (int64_t i = i0; i < n4; i += 4 * step) {  // four loads in flight
            float4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = in4[min(i + u * step, n4 - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                v[u].x = v[u].x == 0.0f ? 0.0f : v[u].x;
                v[u].y = v[u].y == 0.0f ? 0.0f : v[u].y;
                v[u].z = v[u].z == 0.0f ? 0.0f : v[u].z;
                v[u].w = v[u].w == 0.0f ? 0.0f : v[u].w;
                if (i + u * step < n4) out4[i + u * step] = v[u];
            }
        }
        done = 4 * n4;
    }
    for (int64_t i = done + i0; i < n; i += step) out[i] = score[i] == 0.0f ? 0.0f : score[i];
}
// The sliced layouts' scores are current.
__global__ void live_fresh(int32_t *__restrict__ stale)
{
    if (threadIdx.x == 0) *stale = 0;
}

// A sentence list's tokens copied one after another (one workgroup per sentence).
__global__ void live_gather(const int32_t *__restrict__ list, int32_t n, const int32_t *__restrict__ offsets,
                            const int32_t *__restrict__ tokens, const int32_t *__restrict__ sub_off,
                            int32_t *__restrict__ sub_tok)
{
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        const int o = offsets[list[i]], s0 = sub_off[i], T = sub_off[i + 1] - s0;
        for (int t = threadIdx.x; t < T; t += blockDim.x) sub_tok[s0 + t] = tokens[o + t];
    }
}
// ... and results put back: one 4-byte value per sentence, or per token.
__global__ void live_scatter(const int32_t *__restrict__ list, int32_t n, const int32_t *__restrict__ offsets,
                             const int32_t *__restrict__ sub_off, const uint32_t *__restrict__ sub,
                             uint32_t *__restrict__ out, int32_t per_token)
{
    for (int i = blockIdx.x; i < n; i += gridDim.x) {
        if (!per_token) {
            if (threadIdx.x == 0) out[list[i]] = sub[i];
            continue;
        }
        const int o = offsets[list[i]], s0 = sub_off[i], T = sub_off[i + 1] - s0;
        for (int t = threadIdx.x; t < T; t += blockDim.x) out[o + t] = sub[s0 + t];
    }
}
// ... a value of each listed sentence.
__global__ void live_pick(const int32_t *__restrict__ list, int32_t n, const float *__restrict__ in,
                          float *__restrict__ out)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) out[i] = in[list[i]];
}
}  // namespace wfst
