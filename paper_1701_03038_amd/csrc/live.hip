// Live-state sweeps: the semiring step over the arcs that leave live states.
//
// After a few input symbols only a handful of states of an HMM tagger (or of
// any sparsely connected WFST) carry a finite value: on the 45-tag trigram
// tagger 4 of 2071 states on average, which 8 arcs leave, while the label's
// arc block holds 3450.  The sweeps of sweeps.hip stream the whole block; the
// sweeps here keep the live states as a list and fetch the arcs of
// (label, live source) through an index, so a step costs what its live arcs
// cost.  They are bound by memory latency (one dependent load per step where
// the index is arithmetic, two elsewhere), not by bandwidth, so the design
// puts one sentence on 16 or 64 lanes of a wavefront, many sentences per
// compute unit, and no workgroup barrier in a step.
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
    int32_t slot;  // its slot in the reverse layout (count accumulators)
    int32_t pad;
};
// Arcs of (label, source s): when every state has `per` arcs under the label,
// at first + s * per (no lookup); else (per < 0) through the row table
// (entry row + s) or the pair table.
struct LiveLabel {
    int32_t first, per;
    int64_t row;
};
struct LivePair {  // open-addressed (label, source) -> arcs; label < 0: empty
    int32_t label, src, first, count;
};
struct LiveIndex {
    const LiveArc *arc = nullptr;
    const float *score = nullptr;
    const LiveLabel *label = nullptr;
    const int2 *row = nullptr;        // {first, count} per (label, source)
    const LivePair *pair = nullptr;   // ... or hashed
    uint32_t pair_mask = 0;
};

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
// those an earlier sweep gave up.
struct LiveWork {
    const int32_t *order = nullptr;  // null: 0, 1, 2, ...
    const int32_t *n = nullptr;      // device count; null: B
    int32_t *queue = nullptr;
    int32_t *left = nullptr;         // sentences given up
    int32_t *n_left = nullptr;
};
// Lists of live states (or back-pointers) of every token: entries come from
// one pool, in chunks a group takes with one atomic.
struct LivePool {
    unsigned long long *used = nullptr;
    int64_t cap = 0;
};
constexpr int kLiveChunk = 256;
struct LiveTape {
    int2 *tok = nullptr;         // [N] {first entry, entries} after each token
    int32_t *state = nullptr;    // [pool]
    double *val = nullptr;       // [pool] log alpha
    int32_t *done = nullptr;     // [B] 1: the sentence has a path and its lists are here (2: by the global-memory form)
    double *log_z = nullptr;     // [B]
};

// Table size and list capacity of a group.
struct LiveShape {
    int32_t K = 0;  // live states per step at most (on chip)
    int32_t H = 0;  // table entries, a power of two >= K + lanes
    int32_t rounds = 0;  // a step with more rounds of (lane, 4 arcs) than this is given up
};

// A group of W lanes working on one sentence.  GM: the whole workgroup, with
// its list and its table (direct over the states) in a slot of global memory.
template <int W, bool GM>
struct LiveGroup {
    int lid;          // lane in the group
    uint64_t mask;    // the group's lanes of the wavefront (wavefront form)
    int32_t H, K;
    int32_t *key;             // [H] state of a table entry, -1 = free (wavefront form)
    unsigned long long *mx;   // [H] or [Q]: ordered maximum, 0 = none
    int *cnt;                 // GM: counter in LDS

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
        else return (__ballot(p) & mask) != 0ull;
    }
    // The table entry of state d, claimed if it is new (first = this lane
    // claimed it).  The caller keeps the table from filling up.
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
    // Consecutive positions for the lanes with p, from n on (n: group-uniform, updated)
    __device__ __forceinline__ int place(bool p, int &n) const
    {
        if constexpr (GM) {
            return p ? atomicAdd(cnt, 1) : 0;
        } else {
            const uint64_t m = __ballot(p) & mask;
            const int lane = (int)(threadIdx.x & 63);
            const int at = n + __popcll(m & ((1ull << lane) - 1ull));
            n += __popcll(m);
            return at;
        }
    }
};

__device__ __forceinline__ unsigned long long gload(const unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void gstore(unsigned long long *p, unsigned long long v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

constexpr int kLiveGroupThreads = 512;  // the global-memory form
// Fixed point of the shifted exponentials: e in [0, 1] as round(e 2^31); the
// largest term of a sum is exactly 2^31, a term's rounding 2^-32 of it.
constexpr float kLiveOne = 2147483648.0f;
constexpr unsigned long long kLivePoison = 1ull << 63;  // a NaN or +inf term went into the sum

__device__ __forceinline__ double live_lse(double m, unsigned long long s)
{
    if (s & kLivePoison) return __builtin_nan("");
    return m + (double)log_e((float)((double)s * (1.0 / 2147483648.0)));
}

// Offsets and tokens of a sentence: WFST_STATUS_*.
template <int W, bool GM>
__device__ __forceinline__ int live_check(const LiveGroup<W, GM> &g, const BatchView &bv, int b, int &o0, int &o1)
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
template <int W, bool GM>
__device__ __forceinline__ int64_t live_alloc(const LiveGroup<W, GM> &g, const LivePool &pool, int n, int64_t &at,
                                              int64_t &end, unsigned long long *cell)
{
    if (at + n > end) {
        const unsigned long long want = (unsigned long long)max(n, kLiveChunk);
        if constexpr (GM) {
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

// Next sentence of a group (-1: none).  Wavefront form: the groups of a
// wavefront take neighbours of the order (similar lengths) with one atomic.
template <int W, bool GM>
__device__ __forceinline__ int live_pop(const LiveWork &w, int32_t limit, int *cell, bool &more)
{
    int base = 0;
    constexpr int G = GM ? 1 : 64 / (W > 64 ? 64 : W);
    if constexpr (GM) {
        __syncthreads();
        if (threadIdx.x == 0) *cell = atomicAdd(w.queue, 1);
        __syncthreads();
        base = *cell;
    } else {
        if (threadIdx.x == 0) base = atomicAdd(w.queue, G);
        base = __builtin_amdgcn_readfirstlane(base);
    }
    more = base >= 0 && base < limit;
    const int item = GM ? base : base + (int)(threadIdx.x / (W > 64 ? 64 : W));
    if (!more || item >= limit) return -1;
    return w.order ? w.order[item] : item;
}

// LDS bytes of a group in the wavefront form.
__host__ __device__ constexpr size_t live_viterbi_lds(int K, int H) { return (size_t)H * 16 + (size_t)K * 12; }
__host__ __device__ constexpr size_t live_forward_lds(int K, int H) { return (size_t)H * 20 + (size_t)K * 16; }
__host__ __device__ constexpr size_t live_backward_lds(int K, int H) { return (size_t)H * 24 + (size_t)K * 8; }
// Bytes of a workgroup's slot in the global-memory form.
__host__ __device__ constexpr size_t live_slot(int64_t Q) { return ((size_t)Q * 32 + 255) / 256 * 256; }

// =====================================================================
// Viterbi
// =====================================================================
template <int W, bool GM>
__global__ void __launch_bounds__(GM ? W : 64)
live_viterbi(LiveIndex ix, LiveShape sh, int32_t Q, int32_t start, const float *__restrict__ final_score, BatchView bv,
             LiveWork work, LivePool pool, int2 *__restrict__ bp, float *__restrict__ best_score,
             int32_t *__restrict__ best_arcs, int32_t *__restrict__ best_olabels, const int32_t *__restrict__ olabel,
             unsigned char *__restrict__ gscratch)
{
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ int s_cnt, s_item;
    __shared__ unsigned long long s_cell, s_red[GM ? W / 64 : 1];
    __shared__ int s_idx[GM ? W / 64 : 1];
    LiveGroup<W, GM> g;
    int32_t *cl, *fs, *pred;
    float *fv;
    if constexpr (GM) {
        unsigned char *p = gscratch + (size_t)blockIdx.x * live_slot(Q);
        g.lid = threadIdx.x;
        g.mask = ~0ull;
        g.H = g.K = Q;
        g.key = nullptr;
        g.mx = reinterpret_cast<unsigned long long *>(p);
        pred = reinterpret_cast<int32_t *>(p + (size_t)Q * 16);  // past the table of the forward sweep, which stays zero
        cl = pred + Q;
        fs = cl + Q;
        fv = reinterpret_cast<float *>(fs + Q);
        g.cnt = &s_cnt;
    } else {
        const int gi = threadIdx.x / W;
        unsigned char *p = lds + (size_t)gi * live_viterbi_lds(sh.K, sh.H);
        g.lid = threadIdx.x % W;
        g.mask = W == 64 ? ~0ull : ((1ull << (W & 63)) - 1ull) << (gi * W);
        g.H = sh.H;
        g.K = sh.K;
        g.mx = reinterpret_cast<unsigned long long *>(p);
        g.key = reinterpret_cast<int32_t *>(p + (size_t)sh.H * 8);
        pred = g.key + sh.H;
        cl = pred + sh.H;
        fs = cl + sh.K;
        fv = reinterpret_cast<float *>(fs + sh.K);
        for (int h = g.lid; h < g.H; h += W) {
            g.key[h] = -1;
            g.mx[h] = 0ull;
        }
    }
    g.sync();
    const int32_t limit = work.n ? *work.n : bv.B;
    int64_t pool_at = 0, pool_end = 0;
    bool more = true;
    while (true) {
        const int b = live_pop<W, GM>(work, limit, &s_item, more);
        if (!more) break;
        if (b < 0) continue;
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
        int a_next = T > 0 ? bv.tokens[o0] : 0;
        LiveLabel l_next = T > 0 ? ix.label[a_next] : LiveLabel{};
        int a_next2 = T > 1 ? bv.tokens[o0 + 1] : 0;
        for (int t = 0; t < T && n > 0; ++t) {
            const int a = a_next;
            const LiveLabel l = l_next;
            a_next = a_next2;
            if (t + 1 < T) l_next = ix.label[a_next];
            if (t + 2 < T) a_next2 = bv.tokens[o0 + t + 2];
            int nn = 0;
            int rounds = 0;
            if constexpr (GM) {
                if (g.lid == 0) s_cnt = 0;
                __syncthreads();
            }
            // first pass: the best candidate of every destination (highest score, then
            // lowest arc id); a lane takes 4 arcs of its live state per round
            int slot[4];
            unsigned long long cand[4];
            int entry = 0;
            for (int e0 = 0; e0 < n; e0 += W) {
                const int e = e0 + g.lid;
                const bool on = e < n;
                const int2 rc = on ? live_arcs(ix, l, a, fs[e]) : make_int2(0, 0);
                const float v = on ? fv[e] : WFST_NINF;
                for (int r0 = 0; r0 == 0 || (GM ? r0 < rc.y : g.any(r0 < rc.y)); r0 += 4) {
                    if (!GM && (++rounds > sh.rounds || nn > g.K)) {
                        give_up = true;
                        break;
                    }
                    LiveArc x[4];
                    float sc[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (r0 + u < rc.y) {
                            x[u] = ix.arc[rc.x + r0 + u];
                            sc[u] = ix.score[rc.x + r0 + u];
                        }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        bool first = false;
                        slot[u] = -1;
                        if (r0 + u < rc.y) {
                            const float c = v + sc[u];
                            if (c > WFST_NINF) {
                                cand[u] = ((unsigned long long)ord_f32(c) << 32) | (0xffffffffu - (uint32_t)x[u].arc);
                                if constexpr (GM) {
                                    slot[u] = x[u].dst;
                                    first = atomicMax(&g.mx[slot[u]], cand[u]) == 0ull;
                                } else {
                                    slot[u] = g.claim(x[u].dst, first);
                                    atomicMax(&g.mx[slot[u]], cand[u]);
                                }
                            }
                        }
                        const int at = g.place(first, nn);
                        if (first && at < g.K) cl[at] = slot[u];
                        if (!GM && nn > g.K) break;
                    }
                    entry = e;
                }
                if (give_up) break;
            }
            if (!GM && nn > g.K) give_up = true;
            g.sync();
            if (give_up) break;
            if constexpr (GM) nn = s_cnt;
            // second pass: the winner's live state (the last round is still in registers)
            if (!GM && rounds == 1) {
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (slot[u] >= 0 && g.mx[slot[u]] == cand[u]) pred[slot[u]] = entry;
            } else {
                for (int e = g.lid; e < n; e += W) {
                    const int2 rc = live_arcs(ix, l, a, fs[e]);
                    const float v = fv[e];
                    for (int r = 0; r < rc.y; ++r) {
                        const LiveArc x = ix.arc[rc.x + r];
                        const float c = v + ix.score[rc.x + r];
                        if (!(c > WFST_NINF)) continue;
                        const unsigned long long k =
                            ((unsigned long long)ord_f32(c) << 32) | (0xffffffffu - (uint32_t)x.arc);
                        const int sl = GM ? x.dst : g.find(x.dst);
                        if ((GM ? gload(&g.mx[sl]) : g.mx[sl]) == k) pred[sl] = e;
                    }
                }
            }
            g.sync();
            const int64_t base = live_alloc(g, pool, nn, pool_at, pool_end, &s_cell);
            const bool fits = base < pool.cap;
            for (int i = g.lid; i < nn; i += W) {
                const int sl = cl[i];
                const unsigned long long k = GM ? gload(&g.mx[sl]) : g.mx[sl];
                const int32_t d = GM ? sl : g.key[sl];
                if (fits)
                    bp[base + i] = make_int2((int32_t)(0xffffffffu - (uint32_t)k), prev < 0 ? -1 : (int)prev + pred[sl]);
                fs[i] = d;
                fv[i] = unord_f32((uint32_t)(k >> 32));
                if constexpr (GM) {
                    gstore(&g.mx[sl], 0ull);
                } else {
                    g.mx[sl] = 0ull;
                    g.key[sl] = -1;
                }
            }
            g.sync();
            n = nn;
            prev = base;
            if (!fits) {
                give_up = true;
                break;
            }
            if (GM && n > max(1024, Q / 4)) {  // most states live: the streaming sweeps are faster
                give_up = true;
                break;
            }
        }
        if (give_up) {
            if constexpr (!GM) {
                for (int h = g.lid; h < g.H; h += W) {
                    g.key[h] = -1;
                    g.mx[h] = 0ull;
                }
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
        for (int o = (W > 64 ? 64 : W) / 2; o > 0; o >>= 1) {
            const unsigned long long k = __shfl_xor(best, o, 64);
            const int x = __shfl_xor(at, o, 64);
            if (k > best) {
                best = k;
                at = x;
            }
        }
        if constexpr (GM) {
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
        if constexpr (GM) __syncthreads();
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
            if constexpr (GM) __syncthreads();
            else __builtin_amdgcn_wave_barrier();
            for (int i = o0 + g.lid; i < o1; i += W) best_olabels[i] = olabel[best_arcs[i]];
        }
        g.sync();
    }
}

// =====================================================================
// Forward (log semiring)
// =====================================================================
// One destination's log-sum-exp: the maximum term first (ordered integers),
// then the sum of the shifted exponentials in fixed point.  Terms are
// alpha (FP64) + theta, so no normalisation along the sentence is needed.
template <int W, bool GM>
__global__ void __launch_bounds__(GM ? W : 64)
live_forward(LiveIndex ix, LiveShape sh, int32_t Q, int32_t start, const float *__restrict__ final_score, BatchView bv,
             LiveWork work, LivePool pool, LiveTape lt, float *__restrict__ log_z_out,
             unsigned char *__restrict__ gscratch)
{
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ int s_cnt, s_item;
    __shared__ unsigned long long s_cell;
    __shared__ double s_rm[GM ? W / 64 : 1];
    LiveGroup<W, GM> g;
    int32_t *cl, *fs;
    unsigned long long *sm;
    double *fv;
    if constexpr (GM) {
        unsigned char *p = gscratch + (size_t)blockIdx.x * live_slot(Q);
        g.lid = threadIdx.x;
        g.mask = ~0ull;
        g.H = g.K = Q;
        g.key = nullptr;
        g.mx = reinterpret_cast<unsigned long long *>(p);
        sm = g.mx + Q;
        fv = reinterpret_cast<double *>(sm + Q);
        cl = reinterpret_cast<int32_t *>(fv + Q);
        fs = cl + Q;
        g.cnt = &s_cnt;
    } else {
        const int gi = threadIdx.x / W;
        unsigned char *p = lds + (size_t)gi * live_forward_lds(sh.K, sh.H);
        g.lid = threadIdx.x % W;
        g.mask = W == 64 ? ~0ull : ((1ull << (W & 63)) - 1ull) << (gi * W);
        g.H = sh.H;
        g.K = sh.K;
        g.mx = reinterpret_cast<unsigned long long *>(p);
        sm = g.mx + sh.H;
        fv = reinterpret_cast<double *>(sm + sh.H);
        g.key = reinterpret_cast<int32_t *>(fv + sh.K);
        cl = g.key + sh.H;
        fs = cl + sh.K;
        for (int h = g.lid; h < g.H; h += W) {
            g.key[h] = -1;
            g.mx[h] = 0ull;
            sm[h] = 0ull;
        }
    }
    g.sync();
    const int32_t limit = work.n ? *work.n : bv.B;
    int64_t pool_at = 0, pool_end = 0;
    bool more = true;
    // the shifted exponential of term x under the maximum m
    auto add_term = [&](int sl, double x, double m) {
        if (!(x < __builtin_huge_val())) {
            atomicOr(&sm[sl], kLivePoison);
            return;
        }
        const unsigned int q = (unsigned int)(exp_e((float)(x - m)) * kLiveOne);
        if (q) atomicAdd(&sm[sl], (unsigned long long)q);
    };
    while (true) {
        const int b = live_pop<W, GM>(work, limit, &s_item, more);
        if (!more) break;
        if (b < 0) continue;
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
        int a_next = T > 0 ? bv.tokens[o0] : 0;
        LiveLabel l_next = T > 0 ? ix.label[a_next] : LiveLabel{};
        int a_next2 = T > 1 ? bv.tokens[o0 + 1] : 0;
        for (int t = 0; t < T && n > 0; ++t) {
            const int a = a_next;
            const LiveLabel l = l_next;
            a_next = a_next2;
            if (t + 1 < T) l_next = ix.label[a_next];
            if (t + 2 < T) a_next2 = bv.tokens[o0 + t + 2];
            int nn = 0;
            int rounds = 0;
            if constexpr (GM) {
                if (g.lid == 0) s_cnt = 0;
                __syncthreads();
            }
            int slot[4];
            double term[4];
            for (int e0 = 0; e0 < n; e0 += W) {
                const int e = e0 + g.lid;
                const bool on = e < n;
                const int2 rc = on ? live_arcs(ix, l, a, fs[e]) : make_int2(0, 0);
                const double v = on ? fv[e] : 0.0;
                for (int r0 = 0; r0 == 0 || (GM ? r0 < rc.y : g.any(r0 < rc.y)); r0 += 4) {
                    if (!GM && (++rounds > sh.rounds || nn > g.K)) {
                        give_up = true;
                        break;
                    }
                    int32_t d[4];
                    float sc[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (r0 + u < rc.y) {
                            d[u] = ix.arc[rc.x + r0 + u].dst;
                            sc[u] = ix.score[rc.x + r0 + u];
                        }
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        bool first = false;
                        slot[u] = -1;
                        if (r0 + u < rc.y) {
                            term[u] = v + (double)sc[u];
                            if (term[u] != -__builtin_huge_val()) {
                                const unsigned long long k =
                                    ord_f64(term[u] < __builtin_huge_val() ? term[u] : __builtin_huge_val());
                                if constexpr (GM) {
                                    slot[u] = d[u];
                                    first = atomicMax(&g.mx[slot[u]], k) == 0ull;
                                } else {
                                    slot[u] = g.claim(d[u], first);
                                    atomicMax(&g.mx[slot[u]], k);
                                }
                            }
                        }
                        const int at = g.place(first, nn);
                        if (first && at < g.K) cl[at] = slot[u];
                        if (!GM && nn > g.K) break;
                    }
                }
                if (give_up) break;
            }
            if (!GM && nn > g.K) give_up = true;
            g.sync();
            if (give_up) break;
            if constexpr (GM) nn = s_cnt;
            if (!GM && rounds == 1) {  // the terms are still in registers
#pragma unroll
                for (int u = 0; u < 4; ++u)
                    if (slot[u] >= 0) add_term(slot[u], term[u], unord_f64(g.mx[slot[u]]));
            } else {
                for (int e = g.lid; e < n; e += W) {
                    const int2 rc = live_arcs(ix, l, a, fs[e]);
                    const double v = fv[e];
                    for (int r = 0; r < rc.y; ++r) {
                        const double x = v + (double)ix.score[rc.x + r];
                        if (x == -__builtin_huge_val()) continue;
                        const int32_t dd = ix.arc[rc.x + r].dst;
                        const int sl = GM ? dd : g.find(dd);
                        add_term(sl, x, unord_f64(GM ? gload(&g.mx[sl]) : g.mx[sl]));
                    }
                }
            }
            g.sync();
            const int64_t base = live_alloc(g, pool, nn, pool_at, pool_end, &s_cell);
            const bool fits = base < pool.cap;
            if (g.lid == 0) lt.tok[o0 + t] = make_int2((int)base, fits ? nn : 0);
            for (int i = g.lid; i < nn; i += W) {
                const int sl = cl[i];
                const double m = unord_f64(GM ? gload(&g.mx[sl]) : g.mx[sl]);
                const double v = live_lse(m, GM ? gload(&sm[sl]) : sm[sl]);
                const int32_t d = GM ? sl : g.key[sl];
                if (fits) {
                    lt.state[base + i] = d;
                    lt.val[base + i] = v;
                }
                fs[i] = d;
                fv[i] = v;
                if constexpr (GM) {
                    gstore(&g.mx[sl], 0ull);
                    gstore(&sm[sl], 0ull);
                } else {
                    g.mx[sl] = 0ull;
                    sm[sl] = 0ull;
                    g.key[sl] = -1;
                }
            }
            g.sync();
            n = nn;
            if (!fits || (GM && n > max(1024, Q / 4))) {
                give_up = true;
                break;
            }
        }
        if (give_up) {
            if constexpr (!GM) {
                for (int h = g.lid; h < g.H; h += W) {
                    g.key[h] = -1;
                    g.mx[h] = 0ull;
                    sm[h] = 0ull;
                }
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
        for (int o = (W > 64 ? 64 : W) / 2; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
        poison = g.any(poison);
        if constexpr (GM) {
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
                s += (unsigned long long)(unsigned int)(exp_e((float)((fv[e] + (double)f) - m)) * kLiveOne);
            }
#pragma unroll
        for (int o = (W > 64 ? 64 : W) / 2; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
        if constexpr (GM) {
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
                lt.done[b] = GM ? 2 : 1;
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
    unsigned long long *acc = nullptr;     // [reverse slots] fixed-point sums, zero between calls
    int32_t *touched = nullptr;            // slots with a contribution (repeats allowed, -1: unused)
    unsigned long long *n_touched = nullptr;
    int64_t touched_cap = 0;
    const double *scale = nullptr;         // 2^S
    const float *grad_log_z = nullptr;     // g_b (null = 1)
    unsigned long long *fin = nullptr;     // [Q] fixed-point final-state posteriors (null: not wanted)
};

// The lists of the forward pass, from the last token back: a lane takes a
// live source, looks its destinations' beta up in the table of the step
// after, and keeps its own beta for the step before.  Every destination of a
// live arc is on the next list.
template <int W, bool GM>
__global__ void __launch_bounds__(GM ? W : 64)
live_backward(LiveIndex ix, LiveShape sh, int32_t Q, int32_t start, const float *__restrict__ final_score, BatchView bv,
              LiveWork work, LiveTape lt, LiveCounts ct, unsigned char *__restrict__ gscratch)
{
    extern __shared__ __align__(16) unsigned char lds[];
    __shared__ int s_item;
    LiveGroup<W, GM> g;
    double *val0, *val1;
    int32_t *key0 = nullptr, *key1 = nullptr, *cl0 = nullptr, *cl1 = nullptr;
    if constexpr (GM) {
        unsigned char *p = gscratch + (size_t)blockIdx.x * live_slot(Q);
        g.lid = threadIdx.x;
        g.mask = ~0ull;
        g.H = g.K = Q;
        val0 = reinterpret_cast<double *>(p) + 2 * (int64_t)Q;  // past the table, which stays zero
        val1 = val0 + Q;
    } else {
        const int gi = threadIdx.x / W;
        unsigned char *p = lds + (size_t)gi * live_backward_lds(sh.K, sh.H);
        g.lid = threadIdx.x % W;
        g.mask = W == 64 ? ~0ull : ((1ull << (W & 63)) - 1ull) << (gi * W);
        g.H = sh.H;
        g.K = sh.K;
        val0 = reinterpret_cast<double *>(p);
        val1 = val0 + sh.H;
        key0 = reinterpret_cast<int32_t *>(val1 + sh.H);
        key1 = key0 + sh.H;
        cl0 = key1 + sh.H;
        cl1 = cl0 + sh.K;
        for (int h = g.lid; h < g.H; h += W) key0[h] = key1[h] = -1;
    }
    g.sync();
    const int32_t limit = work.n ? *work.n : bv.B;
    const double scale = *ct.scale;
    int64_t list_at = 0, list_end = 0;  // this group's (GM: lane's) range of the touched list
    bool more = true;
    while (true) {
        const int b = live_pop<W, GM>(work, limit, &s_item, more);
        if (!more) break;
        if (b < 0) continue;
        if (lt.done[b] != (GM ? 2 : 1)) continue;
        const int o0 = bv.offsets[b], o1 = bv.offsets[b + 1];
        const int T = o1 - o0;
        const float gb = ct.grad_log_z ? ct.grad_log_z[b] : 1.0f;
        const double lz = lt.log_z[b];
        if (T == 0) {
            if (ct.fin && g.lid == 0) {
                const long long q = __double2ll_rn((double)(gb * exp_e((float)((double)final_score[start] - lz))) * scale);
                if (q) atomicAdd(&ct.fin[start], (unsigned long long)q);
            }
            continue;
        }
        // beta_T = f on the last list
        const int2 last = lt.tok[o1 - 1];
        int n_prev = GM ? last.y : min(last.y, g.K);  // entries of the list the table holds
        for (int e = g.lid; e < n_prev; e += W) {
            const int32_t s = lt.state[last.x + e];
            const float f = final_score[s];
            const double bt = (double)f;
            if (ct.fin && f != WFST_NINF) {
                const float p = gb * exp_e((float)((lt.val[last.x + e] + bt) - lz));
                const long long q = __double2ll_rn((double)p * scale);
                if (q) atomicAdd(&ct.fin[s], (unsigned long long)q);
            }
            if constexpr (GM) {
                val0[s] = bt;
            } else {
                g.key = key0;
                bool first;
                const int at = g.claim(s, first);
                val0[at] = bt;
                cl0[e] = at;
            }
        }
        g.sync();
        int a_next = bv.tokens[o1 - 1];
        LiveLabel l_next = ix.label[a_next];
        int2 tok_next = T >= 2 ? lt.tok[o1 - 2] : make_int2(0, 1);
        int32_t s_next = 0;
        double al_next = 0.0;
        {
            const int n = GM ? tok_next.y : min(tok_next.y, g.K);
            s_next = T >= 2 ? (g.lid < n ? lt.state[tok_next.x + g.lid] : 0) : start;
            al_next = T >= 2 && g.lid < n ? lt.val[tok_next.x + g.lid] : 0.0;
        }
        int a_next2 = T >= 2 ? bv.tokens[o1 - 2] : 0;
        int2 tok_next2 = T >= 3 ? lt.tok[o1 - 3] : make_int2(0, 1);
        for (int t = T; t >= 1; --t) {
            double *vp = ((T - t) & 1) ? val1 : val0, *vc = ((T - t) & 1) ? val0 : val1;
            int32_t *kp = ((T - t) & 1) ? key1 : key0, *kc = ((T - t) & 1) ? key0 : key1;
            int32_t *cp = ((T - t) & 1) ? cl1 : cl0, *cc = ((T - t) & 1) ? cl0 : cl1;
            const int a = a_next;
            const LiveLabel l = l_next;
            const int2 tk = tok_next;
            const int n = GM ? tk.y : min(tk.y, g.K);
            const int32_t s_first = s_next;
            const double al_first = al_next;
            // the next step's label and list, and the list range of the one after, in flight during this step
            if (t >= 2) {
                a_next = a_next2;
                l_next = ix.label[a_next];
                tok_next = tok_next2;
                const int nx = GM ? tok_next.y : min(tok_next.y, g.K);
                s_next = t >= 3 ? (g.lid < nx ? lt.state[tok_next.x + g.lid] : 0) : start;
                al_next = t >= 3 && g.lid < nx ? lt.val[tok_next.x + g.lid] : 0.0;
                if (t >= 3) a_next2 = bv.tokens[o0 + t - 3];
                tok_next2 = t >= 4 ? lt.tok[o0 + t - 4] : make_int2(0, 1);
            }
            for (int e0 = 0; e0 < n; e0 += W) {
                const int e = e0 + g.lid;
                const bool on = e < n;
                int32_t s = s_first;
                double al = al_first;
                if (e0 > 0 && on) {
                    s = lt.state[tk.x + e];
                    al = lt.val[tk.x + e];
                }
                const int2 rc = on ? live_arcs(ix, l, a, s) : make_int2(0, 0);
                LseD acc{-__builtin_huge_val(), 0.0f};
                for (int r0 = 0; r0 == 0 || (GM ? r0 < rc.y : g.any(r0 < rc.y)); r0 += 4) {
                    LiveArc x[4];
                    float sc[4];
                    double y[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (r0 + u < rc.y) {
                            x[u] = ix.arc[rc.x + r0 + u];
                            sc[u] = ix.score[rc.x + r0 + u];
                        }
                    double m = -__builtin_huge_val();
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        y[u] = -__builtin_huge_val();
                        if (r0 + u < rc.y) {
                            if constexpr (GM) {
                                y[u] = (double)sc[u] + vp[x[u].dst];
                            } else {
                                g.key = kp;
                                const int at = g.find(x[u].dst);
                                if (at >= 0) y[u] = (double)sc[u] + vp[at];
                            }
                        }
                        m = fmax(m, y[u]);
                    }
                    float sum = 0.0f;
                    long long q[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        q[u] = 0;
                        if (y[u] != -__builtin_huge_val()) {
                            sum += exp_e((float)(y[u] - m));
                            q[u] = __double2ll_rn((double)(gb * exp_e((float)((al + y[u]) - lz))) * scale);
                        }
                    }
                    if (m != -__builtin_huge_val()) acc = lse_merge_d(acc, LseD{m, sum});
                    // posteriors: added to the arc's accumulator, its slot noted for the conversion
                    int mine = 0;
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (q[u]) {
                            atomicAdd(&ct.acc[x[u].slot], (unsigned long long)q[u]);
                            ++mine;
                        }
                    int64_t at = 0;
                    if constexpr (GM) {
                        if (mine) at = (int64_t)atomicAdd(ct.n_touched, (unsigned long long)mine);
                    } else {
                        int tot = 0, pre = 0;
                        const uint64_t below = (1ull << (threadIdx.x & 63)) - 1ull;
#pragma unroll
                        for (int k = 0; k < 3; ++k) {
                            const uint64_t mk = __ballot((mine >> k) & 1) & g.mask;
                            pre += __popcll(mk & below) << k;
                            tot += __popcll(mk) << k;
                        }
                        if (list_at + tot > list_end) {  // a new chunk; the old one's tail holds no slots
                            for (int64_t j = list_at + g.lid; j < min(list_end, ct.touched_cap); j += W)
                                ct.touched[j] = -1;
                            unsigned long long c = 0;
                            if (g.lid == 0) c = atomicAdd(ct.n_touched, (unsigned long long)kLiveChunk);
                            list_at = (int64_t)__shfl(c, 0, W);
                            list_end = list_at + kLiveChunk;
                        }
                        at = list_at + pre;
                        list_at += tot;
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (q[u]) {
                            if (at < ct.touched_cap) ct.touched[at] = x[u].slot;
                            ++at;
                        }
                }
                if (on) {
                    const double v = lse_value_d(acc);
                    if constexpr (GM) {
                        vc[s] = v;
                    } else {
                        g.key = kc;
                        bool first;
                        const int at = g.claim(s, first);
                        vc[at] = v;
                        cc[e] = at;
                    }
                }
            }
            g.sync();
            if constexpr (!GM) {
                for (int e = g.lid; e < n_prev; e += W) kp[cp[e]] = -1;
                g.sync();
            }
            n_prev = n;
        }
        if constexpr (!GM) {  // the start state's entry
            int32_t *kl = (T & 1) ? key1 : key0, *cll = (T & 1) ? cl1 : cl0;
            for (int e = g.lid; e < n_prev; e += W) kl[cll[e]] = -1;
            g.sync();
        }
    }
    if constexpr (!GM)
        for (int64_t j = list_at + g.lid; j < min(list_end, ct.touched_cap); j += W) ct.touched[j] = -1;
}

// Work queues and the touched count of a backward pass.
__global__ void live_reset(int32_t *__restrict__ cnt)
{
    if (threadIdx.x == 0) cnt[0] = cnt[2] = cnt[6] = cnt[7] = cnt[8] = 0;  // the lists left stay
}

// The gradient of the touched arcs from their accumulators, which go back to
// zero.  When the list overflowed, or sentences were left to the streaming
// sweeps (which keep no list), every accumulator is looked at.
__global__ void __launch_bounds__(256) live_counts_to_grad(LiveCounts ct, const int32_t *__restrict__ elem_arc,
                                                           int64_t n_slots, const int32_t *__restrict__ n_left,
                                                           float *__restrict__ grad)
{
    const double inv = 1.0 / *ct.scale;
    const unsigned long long used = *ct.n_touched;
    const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    if (used <= (unsigned long long)ct.touched_cap && *n_left == 0) {
        for (int64_t i = i0; i < (int64_t)used; i += step) {
            const int32_t sl = ct.touched[i];
            if (sl < 0) continue;
            const unsigned long long q = atomicExch(&ct.acc[sl], 0ull);  // whichever repeat comes first
            if (q) grad[elem_arc[sl]] = (float)((double)(long long)q * inv);
        }
    } else {
        for (int64_t e = i0; e < n_slots; e += step) {
            const unsigned long long q = ct.acc[e];
            if (!q) continue;
            ct.acc[e] = 0ull;
            grad[elem_arc[e]] = (float)((double)(long long)q * inv);
        }
    }
}

__global__ void live_final_to_grad(const unsigned long long *__restrict__ fin, int32_t Q,
                                   const double *__restrict__ scale, float *__restrict__ out)
{
    const double inv = 1.0 / *scale;
    for (int q = blockIdx.x * blockDim.x + threadIdx.x; q < Q; q += gridDim.x * blockDim.x)
        out[q] = (float)((double)(long long)fin[q] * inv);
}

// =====================================================================
// Sentences left to the streaming sweeps
// =====================================================================
// Their compact per-step storage: offsets of every token, each sentence's
// range taken from one counter (at most tokens x the widest label in all).
__global__ void __launch_bounds__(64) rest_offsets(DevLayout fl, BatchView bv, unsigned long long *__restrict__ total,
                                                   int64_t *__restrict__ tok_off)
{
    const int lane = threadIdx.x;
    const int32_t limit = bv.count();
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
__global__ void rest_final(BatchView bv, TapeView tp, DevLayout fl, int32_t start,
                           const float *__restrict__ final_score, LiveCounts ct)
{
    const int lane = threadIdx.x & 63;
    const int32_t limit = bv.count();
    for (int x = blockIdx.x; x < limit; x += gridDim.x) {
        const int b = bv.n ? bv.order[x] : x;
        if (bv.status[b] != WFST_STATUS_OK) continue;
        const int o0 = bv.offsets[b], o1 = bv.offsets[b + 1];
        const float g = ct.grad_log_z ? ct.grad_log_z[b] : 1.0f;
        if (o1 == o0) {
            const float f = final_score[start];
            const long long q = __double2ll_rn((double)(g * exp_e(f + (float)(0.0 - tp.log_z[b]))) * *ct.scale);
            if (lane == 0 && f != WFST_NINF && q) atomicAdd(&ct.fin[start], (unsigned long long)q);
            continue;
        }
        const int i = o1 - 1;
        const LabelInfo lf = fl.label[bv.tokens[i]];
        const float *ta = tp.alpha + (tp.ck_off ? tp.ck_off[i] : bv.tok_off[i]);
        const float c = tp.a_max[i], o = (float)(tp.a_log[i] - tp.log_z[b]);
        for (int j = lane; j < lf.n_segs; j += 64) {
            const int s = fl.seg_key[lf.seg_first + j];
            const float y = ta[j], f = final_score[s];
            if (y == WFST_NINF || f == WFST_NINF) continue;
            const long long q = __double2ll_rn((double)(g * exp_e(((y - c) + f) + o)) * *ct.scale);
            if (q) atomicAdd(&ct.fin[s], (unsigned long long)q);
        }
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

// The arcs by (label, source), and the lookup tables.  first[] = exclusive
// prefix sums of the reverse layout's segment sizes.
__global__ void live_fill(DevLayout rl, int32_t M, int32_t Q, const int32_t *__restrict__ size,
                          const int32_t *__restrict__ first, LiveArc *__restrict__ arc, float *__restrict__ score,
                          int32_t *__restrict__ arc_id, LiveLabel *__restrict__ label, int32_t *__restrict__ unsorted)
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
                    arc[at] = LiveArc{rl.other[e], id, e, 0};
                    score[at] = rl.score[e];
                    arc_id[at] = id;
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

__global__ void __launch_bounds__(256) live_scores(float *__restrict__ out, const int32_t *__restrict__ arc_id,
                                                   int64_t n, const float *__restrict__ score)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const float s = score[arc_id ? arc_id[i] : i];
        out[i] = s == 0.0f ? 0.0f : s;
    }
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
