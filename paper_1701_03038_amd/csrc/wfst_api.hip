// C ABI of the library (declared in include/wfst.h): argument validation,
// device layouts, workspace and kernel launches.
//
// Memory: every FST owns its layouts plus a grow-only workspace and a pool of
// tape buffers.  A call only allocates when it needs more than any earlier
// call on the same FST (then it synchronises its stream, frees the smaller
// buffer and allocates a larger one); in steady state calls allocate nothing.
// Consequently calls on one FST must not overlap: issue them on one stream.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <fstream>
#include <mutex>
#include <sstream>
#include <string>
#include <vector>

#include "../../include/wfst.h"
#include "kernels.h"
#include "layout.h"
#include "prims.hip"
#include "sweeps.hip"
#include "live.hip"

using namespace wfst;

namespace {

thread_local std::string g_err;

int set_err(int code, const std::string &msg)
{
    g_err = msg;
    return code;
}
int set_err_nothrow(int code, const char *msg) noexcept
{
    try {
        g_err = msg;
    } catch (...) {  // no room for the message: its code is left
        g_err.clear();
    }
    return code;
}

// Ends every entry point of the C ABI (a function try block): no C++ exception crosses it.
#define C_GUARD                                                                                   \
    catch (const std::bad_alloc &) { return set_err_nothrow(WFST_ENOMEM, "host allocation failed"); } \
    catch (const std::exception &e) { return set_err_nothrow(WFST_EINVAL, e.what()); }                \
    catch (...) { return set_err_nothrow(WFST_EINVAL, "unknown exception"); }

// The same for a part of an entry point that has to clean up behind it.
template <class F>
int guarded(F f) noexcept
try {
    return f();
}
C_GUARD

#define HIP_OK(expr)                                                                      \
    do {                                                                                  \
        hipError_t e_ = (expr);                                                           \
        if (e_ != hipSuccess)                                                             \
            return set_err(WFST_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)

#define TRY(expr)                       \
    do {                                \
        int rc_ = (expr);               \
        if (rc_ != WFST_OK) return rc_; \
    } while (0)

inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

inline int grid_for(int64_t n, int nt, int cap = 65535)
{
    const int64_t g = (n + nt - 1) / nt;
    return (int)std::max<int64_t>(1, std::min<int64_t>(g, cap));
}

// A grow-only device buffer.
struct Buf {
    void *p = nullptr;
    size_t cap = 0;
    bool dirty = false;              // a buffer kept zero between calls: a call left it otherwise
    const int64_t *limit = nullptr;  // largest allocation allowed (testing hook of the owning FST; 0: any)
};

int ensure(Buf &b, size_t bytes, hipStream_t s)
{
    bytes = std::max<size_t>(bytes, 256);
    if (b.cap >= bytes) return WFST_OK;
    if (b.limit && *b.limit > 0 && bytes > (size_t)*b.limit)
        return set_err(WFST_ENOMEM, "allocation of " + std::to_string(bytes) + " bytes refused (testing limit)");
    if (b.p) {
        HIP_OK(hipStreamSynchronize(s));
        HIP_OK(hipFree(b.p));
        b.p = nullptr;
        b.cap = 0;
    }
    const size_t want = bytes + bytes / 4;
    hipError_t e = hipMalloc(&b.p, want);
    if (e != hipSuccess) {
        (void)hipGetLastError();  // a launch check of the pass that runs instead would find it
        b.p = nullptr;
        return set_err(WFST_ENOMEM, "hipMalloc(" + std::to_string(want) + " bytes): " + hipGetErrorString(e));
    }
    b.cap = want;
    return WFST_OK;
}

template <class T>
int ensure_t(Buf &b, int64_t count, hipStream_t s, T **out)
{
    TRY(ensure(b, (size_t)std::max<int64_t>(count, 1) * sizeof(T), s));
    *out = reinterpret_cast<T *>(b.p);
    return WFST_OK;
}

enum WsSlot {
    W_ORDER, W_TOKOFF, W_TILES, W_COUNTERS, W_BP, W_PATH, W_BETA, W_BMAX, W_BLOG, W_LZB, W_TOKSENT,
    W_KEY0, W_KEY1, W_VAL0, W_VAL1, W_HIST, W_GRPLO, W_GRPN, W_NIP, W_ITEMBASE, W_ITEMS, W_ITEMSLOT,
    W_PARTIAL, W_SPLITE, W_SEOFF, W_VINFO, W_FROWS, W_FSUM, W_ABUF0, W_ABUF1, W_BBUF0, W_BBUF1,
    W_ILIST, W_ILOFF, W_RKEY0, W_RKEY1, W_RVAL0, W_RVAL1, W_GSCRATCH, W_FXACC, W_FXSCALE, W_EMSUM, W_SCAN0,
    W_SCAN1, W_LATNODE, W_LATSCALE, W_BSTEP, W_TVEC, W_TPMAX, W_TPZ, W_TPART, W_TBAR, W_LATFAR, W_TWORK, W_RTILE,
    W_LCNT, W_LORDER, W_LBP, W_LLEFT, W_LSUB, W_LSUBOUT, W_LSCRATCH, W_LWIN, W_LPREP, W_LVERDICT, W_LATTOK, W_LATSTATE, W_LATVAL, W_LACC, W_LTOUCH, W_LFIN,
    W_LSLOT, W_RGN, W_RGRANK, W_RGFIRST, W_RGTOK, W_RGLABEL, W_NUM
};

// Global memory for the per-workgroup state of sweeps whose state vectors do
// not fit on chip: at most this many bytes (the persistent grid shrinks to fit).
constexpr int64_t kStateScratchBudget = (int64_t)16 << 30;

// Matrices of the time-parallel scan: at most this many bytes (two per token).
constexpr int64_t kScanBudgetBytes = (int64_t)32 << 30;

// small device counters kept together (one allocation)
enum Counter { C_QUEUE = 0, C_NITEMS = 1, C_SLOTS = 2, C_ITEMQ = 3, C_TOTAL = 4 /* int64 at byte 16 */,
               C_SETOTAL = 6 /* int64 at byte 24 */, C_RECS = 8 /* uint64 at byte 32 */,
               C_RTOTAL = 10 /* uint64 at byte 40 */, C_COUNT = 12 };

struct TapeBufs {
    Buf order, tok_off, alpha, a_max, a_log, log_z, tiles, total, ck_size, ck_off, blk_size, blk_base;
    Buf l_cnt, l_tok, l_state, l_val, l_done, l_left, l_sub, l_out;  // live lists, and the sentences they leave
    std::vector<Buf *> all()
    {
        return {&order, &tok_off, &alpha, &a_max, &a_log, &log_z, &tiles, &total, &ck_size, &ck_off, &blk_size,
                &blk_base, &l_cnt, &l_tok, &l_state, &l_val, &l_done, &l_left, &l_sub, &l_out};
    }
    void free_all();
};

// device counters of a live sweep (one allocation)
enum LiveCounter { L_LEFT = 1, L_LEFT2 = 3, L_USED = 4 /* uint64 at byte 16 */,
                   L_TOUCHED = 6 /* uint64 at byte 24 */, L_QUEUE3 = 8, L_GROUPS = 9, L_ROFF = 10 /* uint64 at byte 40 */,
                   L_COUNT = 12 };

// The live-state index of an FST (live.hip) and the shape of its sweeps.
struct LiveFst {
    bool on = false;
    LiveIndex ix;
    LiveArc *arc = nullptr;
    float *score = nullptr;     // [arc id] the FST's scores; the sliced layouts' copies follow when a pass reads them
    int32_t *stale = nullptr;   // device: those copies are older than `score`
    bool dense_stale = false;   // ... as far as the host knows
    bool dense_check = false;   // scores may change without the host knowing (updates inside a capture)
    LiveLabel *label = nullptr;
    int2 *all = nullptr;
    int2 *row = nullptr;
    LivePair *pair = nullptr;
    LiveShape sh;
    int narrow = 0;      // lanes per sentence of the narrow-label sweeps (8 or 16; 0: lists)
    int narrow_arcs = 0, narrow_share = 0;  // arcs a lane takes (2 or 4); log2 of the lanes per source
    int32_t *pos = nullptr;  // [reverse slots] the slot's arc's position in the index
    bool hash = false;   // destinations meet in a hashed table
    bool wide = false;   // sentences the on-chip form gives up go to the global-memory form
    bool safe = false;   // the on-chip form can not give a sentence up, whatever the input
    int64_t pool = 0;    // list entries an earlier call needed beyond the default
    int32_t per = 0;     // most arcs of a label leaving one state
    bool refused = false;  // (while a graph is made) no room for a live pass: its sequence streams
};

}  // namespace

struct wfst_fst {
    int device = 0;
    int32_t Q = 0, M = 0, start = 0, chunk = 16, nt = 256;
    int32_t ckpt_mode = 0;                        // wfst_options.checkpoint
    int32_t state_mem = 0;                        // wfst_options.state_memory
    bool fx_counts = false;                       // counts by fixed-point accumulation (count_records = -2)
    bool graph_mode = false;                      // capturing a graph: no host read-back, no records
    int32_t live_graphs = 0;                      // graphs made on this FST and not destroyed
    int32_t *em_order = nullptr;                  // EM: arc ids grouped by source state
    EmItem *em_item = nullptr;                    // ... cut into segments, in the order they are summed
    int64_t em_items = 0;
    int64_t *em_seg = nullptr;                    // ... first segment of each state [Q+1]
    int32_t *em_src = nullptr;                    // ... source state of each arc
    uint64_t score_version = 0;                   // bumped by every score update
    int64_t tape_budget = (int64_t)8 << 30;       // bytes of alpha + beta tape before auto checkpointing
    int64_t A = 0;
    DevLayout fwd, rev;
    float *final_score = nullptr;
    float *final_max = nullptr;
    int32_t *olabel = nullptr;
    int2 *label_range = nullptr;  // [M] lowest and highest arc id of each label (score updates)
    bool stage_scores = false;    // score updates staged per label through LDS
    int64_t rec_cap = 0;          // record slots per backward call (0: from the batch size); grows
    int64_t rec_max = 0;          // most records a call may use before the grouped count kernel is used
    bool rec_off = false;         // grouped count kernel only
    uint32_t *health = nullptr;  // sticky health bits of the kernels (see wfst_fst_health)
    int64_t bytes = 0;
    int cu_count = 0;
    size_t max_lds = 0;
    bool coop = false;  // cooperative launches supported (team sweeps)
    LiveFst live;
    int32_t *pin = nullptr;  // pinned host memory: counters read back by the live sweeps
    int32_t team_spin = 0;  // team barrier poll limit (0: the default)
    int64_t alloc_limit = 0;  // testing hook: larger allocations of the workspace and the tapes fail (0: none)
    std::vector<std::pair<void *, size_t>> allocs;  // owned device arrays and their bytes
    Buf ws[W_NUM];
    std::vector<TapeBufs *> tape_pool;
    // per-kernel timing (wfst_fst_profile): event pairs recorded around the main kernels
    std::vector<int32_t> label_arcs, label_fwd_segs, label_rev_segs;  // host copies for reporting
    bool prof = false;
    struct Mark {
        int kind;
        hipEvent_t a, b;
    };
    std::vector<Mark> marks, spare;
};

struct wfst_tape {
    const wfst_fst *fst = nullptr;
    uint64_t score_version = 0;  // the FST's scores the forward pass ran with
    int32_t B = 0;
    int64_t N = 0, total = 0;
    const int32_t *offsets = nullptr, *tokens = nullptr;
    int32_t *status = nullptr;
    TapeBufs *bufs = nullptr;
    int32_t *order = nullptr;
    int64_t *tok_off = nullptr;
    float *alpha = nullptr, *a_max = nullptr;
    double *a_log = nullptr, *log_z = nullptr;
    // checkpointed tape (ck_c > 0): alpha~ kept every ck_c steps and at the last step
    int32_t ck_c = 0, ck_K = 1;
    int64_t *ck_off = nullptr;    // [N] offset of a kept token's alpha~, -1 otherwise
    int64_t *blk_base = nullptr;  // [B] start of each sentence in a block buffer
    int64_t blk_total = 0;        // floats of one block buffer
    // live lists (live.hip): the tape of every sentence but those left over, whose
    // tape is the compact one above (list mode) or that of a batch of their own
    bool live = false;
    LiveTape lists;
    bool wide = false;            // the workgroup form ran on the sentences the wavefront form gave up
    bool direct = false;          // ... on all of them
    const int32_t *left = nullptr, *n_left = nullptr;  // list mode: sentences left over, and their number
    bool reserved = false;        // not list mode, but a call like this inside a capture would be: its buffers are sized
    int32_t n_rest = 0;
    const int32_t *rest_list = nullptr;  // device list, increasing (null: all of the batch)
    wfst_tape *rest = nullptr;
};

struct wfst_graph {
    wfst_fst *fst = nullptr;
    wfst_graph_args args{};
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    Buf ws[W_NUM];                   // the graph's own workspace (eager calls never resize it)
    std::vector<TapeBufs *> pool;    // ... and tape buffers
};

namespace {

void free_buf(Buf &b)
{
    if (b.p) (void)hipFree(b.p);
    b.p = nullptr;
    b.cap = 0;
}

void TapeBufs::free_all()
{
    for (Buf *b : all()) free_buf(*b);
}

// A grow-only buffer that is zero between calls: cleared when it is
// (re)allocated, or when the call before did not get to leave it zero.
template <class T>
int ensure_zeroed(Buf &b, int64_t count, hipStream_t s, T **out)
{
    const size_t had = b.cap;
    TRY(ensure_t(b, count, s, out));
    if (b.cap != had || b.dirty)
        hipLaunchKernelGGL(fill_i32, dim3(grid_for((int64_t)(b.cap / 4), 256, 8192)), dim3(256), 0, s,
                           reinterpret_cast<int32_t *>(b.p), (int64_t)(b.cap / 4), 0);
    return WFST_OK;
}

// Held by a call while the kernels it queues write such a buffer: unless the
// kernel that clears it again was queued too (done), the next call clears it.
// (Inside a capture nothing runs: a buffer that was not zero before stays marked.)
struct ZeroHold {
    Buf &b;
    const bool still;
    ZeroHold(Buf &buf, bool capturing) : b(buf), still(buf.dirty && capturing) { b.dirty = true; }
    void done() { b.dirty = still; }
};

template <class T>
int dev_upload(wfst_fst *f, T **dst, const T *src, int64_t count, hipStream_t s)
{
    const size_t bytes = (size_t)std::max<int64_t>(count, 1) * sizeof(T);
    void *p = nullptr;
    HIP_OK(hipMalloc(&p, bytes));
    f->allocs.emplace_back(p, bytes);
    f->bytes += (int64_t)bytes;
    if (src && count > 0) HIP_OK(hipMemcpyAsync(p, src, (size_t)count * sizeof(T), hipMemcpyHostToDevice, s));
    *dst = reinterpret_cast<T *>(p);
    return WFST_OK;
}

int upload_layout(wfst_fst *f, const HostLayout &h, DevLayout &d, hipStream_t s)
{
    TRY(dev_upload(f, &d.other, h.other.data(), (int64_t)h.other.size(), s));
    TRY(dev_upload(f, &d.score, h.score.data(), (int64_t)h.score.size(), s));
    TRY(dev_upload(f, &d.elem_arc, h.elem_arc.data(), (int64_t)h.elem_arc.size(), s));
    TRY(dev_upload(f, &d.slice, h.slice.data(), (int64_t)h.slice.size(), s));
    TRY(dev_upload(f, &d.seg_key, h.seg_key.data(), (int64_t)h.seg_key.size(), s));
    TRY(dev_upload(f, &d.seg_chunk, h.seg_chunk.data(), (int64_t)h.seg_chunk.size(), s));
    TRY(dev_upload(f, &d.label, h.label.data(), (int64_t)h.label.size(), s));
    d.n_elem = (int64_t)h.other.size();
    d.n_slice = (int64_t)h.slice.size();
    d.n_seg = (int64_t)h.seg_key.size();
    d.max_segs = h.max_segs;
    d.max_slots = h.max_slots;
    d.max_elems = h.max_elems;
    d.max_height = h.max_height;
    d.max_slices = h.max_slices;
    return WFST_OK;
}

// Free one device array owned by the FST (nullptr-safe).
void free_owned(wfst_fst *f, void *p)
{
    if (!p) return;
    for (size_t i = 0; i < f->allocs.size(); ++i)
        if (f->allocs[i].first == p) {
            f->bytes -= (int64_t)f->allocs[i].second;
            f->allocs.erase(f->allocs.begin() + (ptrdiff_t)i);
            break;
        }
    (void)hipFree(p);
}

void free_layout(wfst_fst *f, DevLayout &d)
{
    for (void *p : {(void *)d.other, (void *)d.score, (void *)d.elem_arc, (void *)d.elem_loc, (void *)d.slice,
                    (void *)d.seg_key, (void *)d.seg_chunk, (void *)d.label})
        free_owned(f, p);
    d = DevLayout();
}

// The 2-byte label-relative arc offsets of both layouts, for score updates
// staged per label (built when the FST's labels are staged).
int build_elem_locs(wfst_fst *f, hipStream_t s)
{
    if (!f->stage_scores) return WFST_OK;
    for (DevLayout *d : {&f->fwd, &f->rev}) {
        if (d->n_elem == 0) continue;
        TRY(dev_upload<uint16_t>(f, &d->elem_loc, nullptr, d->n_elem, s));
        hipLaunchKernelGGL(build_elem_loc, dim3(grid_for(d->n_slice, 1, 65535)), dim3(256), 0, s,
                           (const SliceInfo *)d->slice, d->n_slice, (const int32_t *)d->elem_arc,
                           (const int2 *)f->label_range, d->elem_loc);
    }
    HIP_OK(hipGetLastError());
    return WFST_OK;
}

void free_fst(wfst_fst *f)
{
    if (!f) return;
    int cur = 0;
    const bool other = hipGetDevice(&cur) == hipSuccess && cur != f->device;
    if (other) (void)hipSetDevice(f->device);
    (void)hipDeviceSynchronize();
    for (auto &a : f->allocs) (void)hipFree(a.first);
    for (Buf &b : f->ws) free_buf(b);
    for (TapeBufs *t : f->tape_pool) {
        t->free_all();
        delete t;
    }
    if (f->pin) (void)hipHostFree(f->pin);
    for (auto &m : f->marks) { (void)hipEventDestroy(m.a); (void)hipEventDestroy(m.b); }
    for (auto &m : f->spare) { (void)hipEventDestroy(m.a); (void)hipEventDestroy(m.b); }
    if (other) (void)hipSetDevice(cur);
    delete f;
}

// Brackets one main-kernel launch with timing events when profiling is on.
struct ProfScope {
    wfst_fst *f;
    hipStream_t s;
    int kind;
    wfst_fst::Mark m{};
    bool on = false;
    ProfScope(const wfst_fst *fc, hipStream_t st, int k) : f(const_cast<wfst_fst *>(fc)), s(st), kind(k)
    {
        if (!f->prof || k < 0) return;
        if (!f->spare.empty()) {
            m = f->spare.back();
            f->spare.pop_back();
        } else if (hipEventCreate(&m.a) != hipSuccess || hipEventCreate(&m.b) != hipSuccess) {
            return;
        }
        m.kind = kind;
        on = hipEventRecord(m.a, s) == hipSuccess;
    }
    ~ProfScope()
    {
        if (on && hipEventRecord(m.b, s) == hipSuccess) f->marks.push_back(m);
    }
};

// Marked segments per backward step: at most the destinations of one label.
int32_t backward_list_cap(const wfst_fst *f) { return std::max(f->fwd.max_segs, 1); }

// Bytes of each sweep's per-sentence state for this FST (LDS, or one slot of
// the global scratch when the vectors do not fit on chip).
size_t lds_viterbi(const wfst_fst *f, bool gmem)
{
    // two FP32 value vectors and their segment indices, then the chunk partials
    return (gmem ? viterbi_state_bytes<true>(f->Q) : viterbi_state_bytes<false>(f->Q)) +
           (size_t)std::max(f->fwd.max_slots, 1) * sizeof(VPart);
}
size_t lds_backward(const wfst_fst *f)
{
    // three FP32 vectors (8-byte aligned end), the segment list and its values,
    // then the 16-bit step stamps
    const size_t q1 = (size_t)f->Q + 1;
    return ((3 * q1 * sizeof(float) + 7) & ~(size_t)7) +
           (size_t)backward_list_cap(f) * (sizeof(int2) + sizeof(double)) + q1 * sizeof(uint16_t);
}
size_t lds_lse(const wfst_fst *f, const DevLayout &l) { return lse_carve(f->Q, l.max_segs, l.max_slots).end; }
size_t lds_counts(const wfst_fst *f)
{
    return (size_t)(f->Q + 1) * 2 * sizeof(CEnt) + (size_t)f->Q * sizeof(int32_t) +
           (size_t)2 * f->fwd.max_segs * sizeof(float) + (size_t)std::max(f->rev.max_slots, 1) * sizeof(int32_t);
}

template <class K>
int persistent_grid(const wfst_fst *f, K kernel, int nt, size_t lds, int64_t work, int *grid)
{
    if (lds > f->max_lds)
        return set_err(WFST_EUNSUPPORTED, "FST needs " + std::to_string(lds) +
                                              " bytes of LDS per workgroup; the device offers " +
                                              std::to_string(f->max_lds));
    if (lds > 65536)
        HIP_OK(hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    int per_cu = 0;
    HIP_OK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, nt, lds));
    if (per_cu < 1) return set_err(WFST_EUNSUPPORTED, "kernel does not fit on a compute unit");
    *grid = (int)std::max<int64_t>(1, std::min<int64_t>(work, (int64_t)per_cu * f->cu_count));
    return WFST_OK;
}

// Where a sweep keeps its per-sentence state, and its persistent grid.
struct SweepShape {
    bool gmem = false;
    int grid = 0;
    size_t lds = 0;                      // dynamic LDS bytes
    int64_t slot = 0;                    // bytes of one workgroup's global slot (gmem)
    unsigned char *scratch = nullptr;    // grid * slot bytes (gmem)
};

int refuse_lds(const wfst_fst *f, size_t bytes)
{
    return set_err(WFST_EUNSUPPORTED, "the FST's state vectors need " + std::to_string(bytes) +
                                          " bytes of LDS per workgroup (the device offers " +
                                          std::to_string(f->max_lds) + "); state_memory=1 forbids the "
                                          "global-memory form");
}

// State memory of a sweep whose state takes lds_bytes on chip or slot_bytes
// in global memory: LDS unless the options ask for global memory, the state
// does not fit, or the sweep needs the wide form (need_wide).  The global
// form's grid is capped so that its slots fit kStateScratchBudget.
template <class KL, class KG>
int sweep_shape(wfst_fst *f, hipStream_t s, KL k_lds, KG k_gmem, int nt, size_t lds_bytes, size_t slot_bytes,
                bool need_wide, int64_t work, SweepShape &sh)
{
    const bool fits = lds_bytes <= f->max_lds && !need_wide;
    sh.gmem = f->state_mem >= 2 || (f->state_mem == 0 && !fits);
    if (!sh.gmem) {
        if (!fits) return refuse_lds(f, lds_bytes);
        sh.lds = lds_bytes;
        return persistent_grid(f, k_lds, nt, lds_bytes, work, &sh.grid);
    }
    sh.slot = (int64_t)((slot_bytes + 255) / 256 * 256);
    TRY(persistent_grid(f, k_gmem, nt, 0, work, &sh.grid));
    const int64_t fit = std::max<int64_t>(1, kStateScratchBudget / sh.slot);
    sh.grid = (int)std::min<int64_t>(sh.grid, fit);
    TRY(ensure_t(f->ws[W_GSCRATCH], sh.grid * sh.slot, s, &sh.scratch));
    return WFST_OK;
}

int check_batch(const wfst_fst *f, int32_t batch, int64_t num_tokens, const void *offsets, const void *tokens)
{
    if (!f) return set_err(WFST_EINVAL, "fst is NULL");
    if (batch < 0) return set_err(WFST_EINVAL, "batch < 0");
    if (num_tokens < 0 || num_tokens >= INT32_MAX) return set_err(WFST_EINVAL, "num_tokens outside [0, 2^31-1)");
    if (batch > 0 && !offsets) return set_err(WFST_EINVAL, "offsets is NULL");
    if (num_tokens > 0 && !tokens) return set_err(WFST_EINVAL, "tokens is NULL");
    return WFST_OK;
}

// Exclusive prefix sum of src over n elements into out; the grand total is
// written to *total (device) when total != nullptr.  tiles: scratch of
// ceil(n / kScanTile) int64.
template <class OutT>
int launch_scan(hipStream_t s, ScanSource src, int64_t n, int64_t *tiles, OutT *out, int64_t *total)
{
    const int64_t ntiles = std::max<int64_t>(1, (n + kScanTile - 1) / kScanTile);
    if (n > 0) hipLaunchKernelGGL(scan_tile_sums, dim3((unsigned)ntiles), dim3(kScanThreads), 0, s, src, n, tiles);
    else hipLaunchKernelGGL(fill_i64, dim3(1), dim3(64), 0, s, tiles, (int64_t)1, (int64_t)0);
    hipLaunchKernelGGL(scan_tiles, dim3(1), dim3(kScanThreads), 0, s, tiles, ntiles, total);
    if (n > 0) hipLaunchKernelGGL((scan_apply<OutT>), dim3((unsigned)ntiles), dim3(kScanThreads), 0, s, src, n,
                                  (const int64_t *)tiles, out);
    HIP_OK(hipGetLastError());
    return WFST_OK;
}

inline int64_t scan_tiles_for(int64_t n) { return std::max<int64_t>(1, (n + kScanTile - 1) / kScanTile); }

struct Plan {
    int32_t *order = nullptr;
    int64_t *tok_off = nullptr;
    int64_t total = 0;  // capacity needed for compact per-(token, segment) storage
};

// Sentence order (length buckets, longest first) and per-token offsets of the
// compact per-step storage.  The storage size is the exact total (read back,
// one synchronisation) when the cheap bound N * max_segs exceeds `bound_cap`.
int make_plan(const wfst_fst *f, hipStream_t s, int32_t B, int64_t N, const int32_t *offsets,
              const int32_t *tokens, int32_t *order, int64_t *tok_off, int64_t *tiles, int64_t *dev_total,
              int64_t bound_cap_elems, Plan &p)
{
    p.order = order;
    p.tok_off = tok_off;
    hipLaunchKernelGGL(order_by_length, dim3(1), dim3(1024), 0, s, offsets, B, order);
    ScanSource src;
    src.tokens = tokens;
    src.label = f->fwd.label;
    src.M = f->M;
    TRY(launch_scan<int64_t>(s, src, N, tiles, tok_off, dev_total));
    const int64_t bound = N * (int64_t)std::max(f->fwd.max_segs, 1);
    if (bound <= bound_cap_elems) {
        p.total = bound;
    } else if (f->graph_mode) {
        return set_err(WFST_EUNSUPPORTED, "a graph sizes its buffers by the bound tokens x largest label (" +
                                              std::to_string(bound) + " entries), which exceeds " +
                                              std::to_string(bound_cap_elems) + "; use a smaller batch");
    } else {
        int64_t t = 0;
        HIP_OK(hipMemcpyAsync(&t, dev_total, sizeof(int64_t), hipMemcpyDeviceToHost, s));
        HIP_OK(hipStreamSynchronize(s));
        p.total = t;
    }
    return WFST_OK;
}

constexpr int64_t kBoundCapBytes = (int64_t)2 << 30;

TapeView tape_view(const wfst_tape *t)
{
    TapeView tp;
    tp.alpha = t->alpha;
    tp.a_max = t->a_max;
    tp.a_log = t->a_log;
    tp.log_z = t->log_z;
    tp.ck_off = t->ck_c > 0 ? t->ck_off : nullptr;
    return tp;
}

// Decide whether the forward tape keeps every alpha~ or only checkpoints
// (every c = ceil(sqrt(T_max)) steps and the last step), and lay out the
// checkpointed tape and the per-sentence block buffers.  *alpha_elems gets the
// tape size.  Auto mode checkpoints when alpha + beta tapes would exceed the
// FST's budget; deciding then needs the exact sizes from the device.
int plan_checkpoints(wfst_fst *f, hipStream_t s, wfst_tape *t, int64_t *tiles, int64_t *dev_total,
                     const Plan &p, int64_t *alpha_elems)
{
    const int32_t B = t->B;
    const int64_t N = t->N;
    t->ck_c = 0;
    t->ck_K = 1;
    if (f->ckpt_mode == 2 || N == 0) return WFST_OK;
    const int64_t bytes_bound = 2 * (int64_t)sizeof(float) * p.total;
    if (f->ckpt_mode != 1 && bytes_bound <= f->tape_budget) return WFST_OK;
    if (f->graph_mode)
        return set_err(WFST_EUNSUPPORTED, "a graph keeps the whole forward tape (checkpointing plans from "
                                          "device totals); its bound exceeds the tape budget or checkpointing "
                                          "is forced");
    // exact tape size and longest sentence
    int32_t *dev_tmax = reinterpret_cast<int32_t *>(dev_total + 1);
    hipLaunchKernelGGL(batch_max_len, dim3(1), dim3(1024), 0, s, t->offsets, B, dev_tmax);
    int64_t host[2] = {0, 0};
    HIP_OK(hipMemcpyAsync(host, dev_total, 2 * sizeof(int64_t), hipMemcpyDeviceToHost, s));
    HIP_OK(hipStreamSynchronize(s));
    const int64_t total = host[0];
    int32_t tmax;
    std::memcpy(&tmax, &host[1], sizeof(int32_t));
    if (f->ckpt_mode != 1 && 2 * (int64_t)sizeof(float) * total <= f->tape_budget) {
        t->total = total;
        return WFST_OK;
    }
    if (tmax <= 0) return WFST_OK;
    int32_t c = 1;
    while ((int64_t)c * c < tmax) ++c;
    t->ck_c = c;
    t->ck_K = (tmax + c - 1) / c;
    if ((int64_t)f->M * t->ck_K >= INT32_MAX)
        return set_err(WFST_EUNSUPPORTED, "labels x checkpoint blocks exceed 2^31");
    TapeBufs *tb = t->bufs;
    int64_t *size, *bsize;
    TRY(ensure_t(tb->ck_size, N, s, &size));
    TRY(ensure_t(tb->ck_off, N, s, &t->ck_off));
    TRY(ensure_t(tb->blk_size, B, s, &bsize));
    TRY(ensure_t(tb->blk_base, B, s, &t->blk_base));
    hipLaunchKernelGGL(ckpt_sizes, dim3(grid_for(B, 256)), dim3(256), 0, s, t->offsets, B, t->tokens,
                       (const LabelInfo *)f->fwd.label, f->M, c, size);
    ScanSource src;
    src.i64 = size;
    TRY(launch_scan<int64_t>(s, src, N, tiles, t->ck_off, dev_total));
    hipLaunchKernelGGL(ckpt_mark, dim3(grid_for(N, 256, 8192)), dim3(256), 0, s, (const int64_t *)size, N,
                       t->ck_off);
    hipLaunchKernelGGL(block_sizes, dim3(grid_for(B, 256)), dim3(256), 0, s, t->offsets, B, t->tokens,
                       (const LabelInfo *)f->fwd.label, f->M, (const int64_t *)t->tok_off, c, bsize);
    ScanSource bsrc;
    bsrc.i64 = bsize;
    TRY(launch_scan<int64_t>(s, bsrc, B, tiles, t->blk_base, dev_total + 1));
    HIP_OK(hipMemcpyAsync(host, dev_total, 2 * sizeof(int64_t), hipMemcpyDeviceToHost, s));
    HIP_OK(hipStreamSynchronize(s));
    *alpha_elems = host[0];
    t->blk_total = host[1];
    t->total = total;
    return WFST_OK;
}

// (size_only: allocate what the launch would need, and launch nothing)
template <int NT>
int launch_viterbi(const wfst_fst *fc, hipStream_t s, const BatchView &bv, int2 *bp, int32_t *path_tmp,
                   float *best_score, int32_t *best_arcs, int32_t *best_olabels, bool no_alloc = false,
                   bool size_only = false)
{
    wfst_fst *f = const_cast<wfst_fst *>(fc);
    SweepShape sh;
    // on chip, segment indices are 16 bits (Q + 1 < 2^16); wider FSTs take the global form
    const bool wide = f->Q + 1 > 0xffff;
    if (no_alloc) {  // on-chip form only: its grid needs no memory beyond the caller's scratch
        if (wide || f->state_mem >= 2 || lds_viterbi(f, false) > f->max_lds)
            return set_err(WFST_EUNSUPPORTED, "the no-allocation Viterbi runs only the on-chip form "
                                              "(state vectors in LDS); this FST needs the global-memory form");
        sh.lds = lds_viterbi(f, false);
        TRY(persistent_grid(f, viterbi_sweep<NT, false>, NT, sh.lds, bv.B, &sh.grid));
    } else {
        TRY(sweep_shape(f, s, viterbi_sweep<NT, false>, viterbi_sweep<NT, true>, NT, lds_viterbi(f, false),
                        lds_viterbi(f, true), wide, bv.B, sh));
    }
    if (size_only) return WFST_OK;
    ProfScope prof(f, s, no_alloc || bv.n ? -1 : WFST_KERNEL_VITERBI);  // sentences left over: timed by the caller
    if (sh.gmem)
        hipLaunchKernelGGL((viterbi_sweep<NT, true>), dim3(sh.grid), dim3(NT), 0, s, f->fwd, f->Q, f->start,
                           (const float *)f->final_score, bv, bp, path_tmp, best_score, best_arcs, best_olabels,
                           (const int32_t *)f->olabel, sh.scratch, sh.slot);
    else
        hipLaunchKernelGGL((viterbi_sweep<NT, false>), dim3(sh.grid), dim3(NT), sh.lds, s, f->fwd, f->Q, f->start,
                           (const float *)f->final_score, bv, bp, path_tmp, best_score, best_arcs, best_olabels,
                           (const int32_t *)f->olabel, nullptr, (int64_t)0);
    HIP_OK(hipGetLastError());
    return WFST_OK;
}

// The team form of the forward sweep runs when its state must be in global
// memory (auto mode) or the options ask for it, the device launches
// cooperatively, and no graph is being captured.  One team per XCD (8 on
// this device), each of all the workgroups that fit on that XCD's CUs.
constexpr int kTeamsPerDevice = 8;

bool team_forward_wanted(const wfst_fst *f)
{
    if (f->graph_mode || !f->coop) return false;
    return f->state_mem == 3 || (f->state_mem == 0 && lds_lse(f, f->fwd) > f->max_lds);
}

template <int NT>
int launch_team_forward(wfst_fst *f, hipStream_t s, const BatchView &bv, const TapeView &tp, const BlockView &bk,
                        float *log_z)
{
    int per_cu = 0;
    HIP_OK(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, team_forward_sweep<NT>, NT, 0));
    const int G = per_cu * f->cu_count / kTeamsPerDevice;
    if (G < 1) return set_err(WFST_EUNSUPPORTED, "team sweep does not fit the device");
    TeamView tv;
    tv.G = G;
    tv.n_teams = kTeamsPerDevice;
    if (f->team_spin > 0) tv.spin_limit = f->team_spin;
    tv.q1 = ((int64_t)f->Q + 1 + 63) / 64 * 64;
    unsigned int *bar = nullptr;
    TRY(ensure_t(f->ws[W_TVEC], (int64_t)tv.n_teams * 3 * tv.q1, s, &tv.vec));
    TRY(ensure_t(f->ws[W_TPMAX], (int64_t)tv.n_teams * 2 * G, s, &tv.pmax));
    TRY(ensure_t(f->ws[W_TPZ], (int64_t)tv.n_teams * 2 * G, s, &tv.pz));
    TRY(ensure_t(f->ws[W_TPART], (int64_t)tv.n_teams * std::max(f->fwd.max_slots, 1), s, &tv.part));
    TRY(ensure_t(f->ws[W_TBAR], (int64_t)tv.n_teams + 1, s, &bar));
    TRY(ensure_t(f->ws[W_TWORK], (int64_t)tv.n_teams * 2, s, &tv.work));
    tv.bar = bar;
    tv.abort = reinterpret_cast<int32_t *>(bar + tv.n_teams);
    hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, reinterpret_cast<int32_t *>(bar), (int64_t)tv.n_teams + 1, 0);
    hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, tv.work, (int64_t)tv.n_teams * 2, 0);
    ProfScope prof(f, s, WFST_KERNEL_FORWARD);
    DevLayout fl = f->fwd;
    int32_t Q = f->Q, start = f->start;
    const float *final_score = (const float *)f->final_score;
    BatchView bv_ = bv;
    TapeView tp_ = tp;
    BlockView bk_ = bk;
    void *args[] = {&fl, &Q, &start, &final_score, &bv_, &tp_, &bk_, &log_z, &tv};
    HIP_OK(hipLaunchCooperativeKernel((const void *)team_forward_sweep<NT>, dim3(tv.n_teams * G), dim3(NT), args, 0,
                                      s));
    return WFST_OK;
}

template <int NT>
int launch_forward(const wfst_fst *fc, hipStream_t s, const BatchView &bv, const TapeView &tp, const BlockView &bk,
                   float *log_z, bool size_only = false)
{
    wfst_fst *f = const_cast<wfst_fst *>(fc);
    if (!size_only && !bv.n && team_forward_wanted(f)) return launch_team_forward<NT>(f, s, bv, tp, bk, log_z);
    SweepShape sh;
    const size_t bytes = lds_lse(f, f->fwd);
    TRY(sweep_shape(f, s, forward_sweep<NT, false>, forward_sweep<NT, true>, NT, bytes, bytes, false, bv.B, sh));
    if (size_only) return WFST_OK;
    ProfScope prof(f, s, bv.n ? -1 : WFST_KERNEL_FORWARD);
    if (sh.gmem)
        hipLaunchKernelGGL((forward_sweep<NT, true>), dim3(sh.grid), dim3(NT), 0, s, f->fwd, f->Q, f->start,
                           (const float *)f->final_score, bv, tp, bk, log_z, sh.scratch, sh.slot);
    else
        hipLaunchKernelGGL((forward_sweep<NT, false>), dim3(sh.grid), dim3(NT), sh.lds, s, f->fwd, f->Q, f->start,
                           (const float *)f->final_score, bv, tp, bk, log_z, nullptr, (int64_t)0);
    HIP_OK(hipGetLastError());
    return WFST_OK;
}

// The backward sweep keeps its state in global memory (and the counts take
// the fixed-point form) when the options say so or its state exceeds LDS.
bool backward_in_gmem(const wfst_fst *f)
{
    return f->state_mem >= 2 || (f->state_mem == 0 && lds_backward(f) > f->max_lds);
}

template <int NT>
int launch_backward(const wfst_fst *fc, hipStream_t s, const BatchView &bv, const TapeView &tp, const BlockView &bk,
                    const RecordSink &rs, bool size_only = false)
{
    wfst_fst *f = const_cast<wfst_fst *>(fc);
    SweepShape sh;
    const size_t bytes = lds_backward(f);
    TRY(sweep_shape(f, s, backward_sweep<NT, false>, backward_sweep<NT, true>, NT, bytes, bytes, false, bv.B, sh));
    if (sh.gmem && rs.key)
        return set_err(WFST_EUNSUPPORTED, "count records need the on-chip backward sweep");
    BwdStep *steps = nullptr;
    TRY(ensure_t(f->ws[W_BSTEP], std::max<int64_t>(bv.N, 1), s, &steps));
    if (size_only) return WFST_OK;
    // the sweep zero-fills the gradient only when its grid covers the device
    // (the grid is at most one workgroup per sentence); else one fill kernel
    RecordSink sink = rs;
    if (sink.fill && sh.grid < 2 * f->cu_count) {
        ProfScope prof(f, s, WFST_KERNEL_GRAD_FILL);
        hipLaunchKernelGGL(fill_f32, dim3(grid_for(sink.fill_n, 256, 8192)), dim3(256), 0, s, sink.fill, sink.fill_n,
                           0.0f);
        sink.fill = nullptr;
    }
    ProfScope prof(f, s, bv.n ? -1 : WFST_KERNEL_BACKWARD);
    hipLaunchKernelGGL(bwd_step_table, dim3(grid_for(bv.B, 1)), dim3(64), 0, s, f->fwd, f->rev, bv, tp, bk,
                       (int32_t)(rs.key != nullptr || rs.acc != nullptr), steps);
    if (sh.gmem)
        hipLaunchKernelGGL((backward_sweep<NT, true>), dim3(sh.grid), dim3(NT), 0, s, f->fwd, f->rev, f->Q,
                           f->start, (const float *)f->final_score, (const float *)f->final_max, bv, tp, bk,
                           backward_list_cap(f), sink, (const BwdStep *)steps, sh.scratch, sh.slot);
    else
        hipLaunchKernelGGL((backward_sweep<NT, false>), dim3(sh.grid), dim3(NT), sh.lds, s, f->fwd, f->rev, f->Q,
                           f->start, (const float *)f->final_score, (const float *)f->final_max, bv, tp, bk,
                           backward_list_cap(f), sink, (const BwdStep *)steps, nullptr, (int64_t)0);
    HIP_OK(hipGetLastError());
    return WFST_OK;
}

// Arguments of the count kernel that stay the same over its launches.
struct CountLaunch {
    const CountItem *items;
    const int32_t *n_items;
    const int32_t *list, *list_off;  // per-block item lists (checkpointing), else null
    int32_t *item_queue;
    int64_t items_bound;
    const VisitInfo *vinfo;
    float *grad, *partial;
    int32_t *item_slot, *slot_counter;
    CountCaps caps;
};

template <int NT, int CH>
int launch_counts_nt(const wfst_fst *f, hipStream_t s, const BatchView &bv, const TapeView &tp,
                     const CountLaunch &c, int32_t blk)
{
    const size_t lds = lds_counts(f);
    int grid = 0;
    TRY(persistent_grid(f, counts_kernel<NT, CH>, NT, lds, c.items_bound, &grid));
    ProfScope prof(f, s, WFST_KERNEL_COUNTS);
    hipLaunchKernelGGL((counts_kernel<NT, CH>), dim3(grid), dim3(NT), lds, s, f->fwd, f->rev, f->Q, f->start, bv,
                       tp, c.items, c.n_items, c.list, c.list_off, blk, c.item_queue, c.vinfo, c.grad, c.partial,
                       c.item_slot, c.slot_counter, c.caps);
    HIP_OK(hipGetLastError());
    return WFST_OK;
}

// Workgroup size of the count kernel: enough wavefronts for the widest label
// of the reverse layout to fit one pass (KPP slices per wavefront).
template <int CH>
int launch_counts_ch(const wfst_fst *f, hipStream_t s, const BatchView &bv, const TapeView &tp,
                     const CountLaunch &c, int32_t blk)
{
    constexpr int KPP = count_slices_per_wave(CH);
    const int waves = (f->rev.max_slices + KPP - 1) / KPP;
    if (waves > 8) return launch_counts_nt<1024, CH>(f, s, bv, tp, c, blk);
    if (waves > 4) return launch_counts_nt<512, CH>(f, s, bv, tp, c, blk);
    return launch_counts_nt<256, CH>(f, s, bv, tp, c, blk);
}

// CH = slice height bound of the reverse layout
int launch_counts(const wfst_fst *f, hipStream_t s, const BatchView &bv, const TapeView &tp, const CountLaunch &c,
                  int32_t blk)
{
    const int ch = f->rev.max_height;
    if (ch <= 4) return launch_counts_ch<4>(f, s, bv, tp, c, blk);
    if (ch <= 8) return launch_counts_ch<8>(f, s, bv, tp, c, blk);
    if (ch <= 16) return launch_counts_ch<16>(f, s, bv, tp, c, blk);
    if (ch <= 32) return launch_counts_ch<32>(f, s, bv, tp, c, blk);
    return launch_counts_ch<64>(f, s, bv, tp, c, blk);
}

#define DISPATCH_NT(rc, nt, fn, ...)                  \
    switch (nt) {                                     \
    case 64: rc = fn<64>(__VA_ARGS__); break;         \
    case 128: rc = fn<128>(__VA_ARGS__); break;       \
    case 256: rc = fn<256>(__VA_ARGS__); break;       \
    case 512: rc = fn<512>(__VA_ARGS__); break;       \
    default: rc = fn<1024>(__VA_ARGS__); break;       \
    }

BatchView make_view(const wfst_fst *f, int32_t B, int64_t N, const int32_t *offsets, const int32_t *tokens,
                    const int32_t *order, const int64_t *tok_off, int32_t *queue, int32_t *status)
{
    BatchView bv;
    bv.B = B;
    bv.M = f->M;
    bv.N = N;
    bv.offsets = offsets;
    bv.tokens = tokens;
    bv.order = order;
    bv.tok_off = tok_off;
    bv.queue = queue;
    bv.status = status;
    bv.health = f->health;
    return bv;
}

// Stable sort of token positions by label: visits[] lists positions grouped by
// label, in increasing position inside each label; skeys[] their labels.
int sort_visits(wfst_fst *f, hipStream_t s, int64_t N, const int32_t *tokens, const int32_t *offsets, int32_t B,
                int32_t c, int32_t K, int32_t **visits_out, int32_t **skeys_out, int32_t *tok_sent)
{
    int32_t *k0, *k1, *v0, *v1;
    TRY(ensure_t(f->ws[W_KEY0], N, s, &k0));
    TRY(ensure_t(f->ws[W_KEY1], N, s, &k1));
    TRY(ensure_t(f->ws[W_VAL0], N, s, &v0));
    TRY(ensure_t(f->ws[W_VAL1], N, s, &v1));
    hipLaunchKernelGGL(token_owner, dim3(grid_for(N, 256)), dim3(256), 0, s, offsets, B, N, tokens, tok_sent, k0,
                       v0, f->M, c, K);
    int bits = 1;  // keys are < M * K + 1
    while (bits < 31 && ((int64_t)1 << bits) <= (int64_t)f->M * K) ++bits;
    const int passes = (bits + 7) / 8;
    const int64_t ntiles = (N + kSortTile - 1) / kSortTile;
    int64_t *hist, *tiles;
    TRY(ensure_t(f->ws[W_HIST], 256 * ntiles, s, &hist));
    TRY(ensure_t(f->ws[W_TILES], scan_tiles_for(256 * ntiles), s, &tiles));
    for (int p = 0; p < passes; ++p) {
        const int shift = 8 * p;
        hipLaunchKernelGGL(radix_hist<int32_t>, dim3((unsigned)ntiles), dim3(kSortThreads), 0, s, (const int32_t *)k0,
                           N, shift, ntiles, hist);
        ScanSource src;
        src.i64 = hist;
        TRY(launch_scan<int64_t>(s, src, 256 * ntiles, tiles, hist, nullptr));
        hipLaunchKernelGGL(radix_scatter<int32_t>, dim3((unsigned)ntiles), dim3(kSortThreads), 0, s, (const int32_t *)k0,
                           (const int32_t *)v0, N, shift, ntiles, (const int64_t *)hist, k1, v1, f->health);
        std::swap(k0, k1);
        std::swap(v0, v1);
    }
    HIP_OK(hipGetLastError());
    *skeys_out = k0;
    *visits_out = v0;
    return WFST_OK;
}

// d(sum_b g_b log Z_b)/d final_score into out[Q], from the forward tape.
int final_posteriors(wfst_fst *f, const wfst_tape *tape, const float *grad_log_z, float *out, hipStream_t s)
{
    const int32_t Q = f->Q, B = tape->B;
    constexpr int32_t G = 64;
    if (B == 0) {
        hipLaunchKernelGGL(fill_f32, dim3(grid_for(Q, 256)), dim3(256), 0, s, out, (int64_t)Q, 0.0f);
        HIP_OK(hipGetLastError());
        return WFST_OK;
    }
    // sentences per block: dense rows of at most 256 MiB
    int64_t nb_max = ((int64_t)256 << 20) / ((int64_t)Q * (int64_t)sizeof(float));
    nb_max = std::max<int64_t>(G, nb_max / G * G);
    nb_max = std::min<int64_t>(nb_max, B);
    float *rows, *S;
    TRY(ensure_t(f->ws[W_FROWS], nb_max * Q, s, &rows));
    TRY(ensure_t(f->ws[W_FSUM], (nb_max + G - 1) / G * Q, s, &S));
    const TapeView tp = tape_view(tape);
    const BatchView bv = make_view(f, B, tape->N, tape->offsets, tape->tokens, tape->order, tape->tok_off, nullptr,
                                   tape->status);
    for (int64_t b0 = 0; b0 < B; b0 += nb_max) {
        const int32_t nb = (int32_t)std::min<int64_t>(nb_max, B - b0);
        const int32_t ng = (nb + G - 1) / G;
        hipLaunchKernelGGL(fill_f32, dim3(grid_for((int64_t)nb * Q, 256, 8192)), dim3(256), 0, s, rows,
                           (int64_t)nb * Q, 0.0f);
        hipLaunchKernelGGL(final_rows, dim3(grid_for(nb, 4)), dim3(256), 0, s, bv, tp, f->fwd, Q, f->start,
                           (const float *)f->final_score, grad_log_z, (int32_t)b0, nb, rows);
        hipLaunchKernelGGL(sum_row_groups, dim3(grid_for((int64_t)ng * Q, 256, 16384)), dim3(256), 0, s,
                           (const float *)rows, nb, Q, G, S);
        hipLaunchKernelGGL(sum_groups, dim3(grid_for(Q, 256)), dim3(256), 0, s, (const float *)S, ng, Q,
                           (int32_t)(b0 > 0), out);
    }
    HIP_OK(hipGetLastError());
    return WFST_OK;
}

// Group n expected-count records by reverse-layout slot (radix sort on the
// slot part of the keys slot:position) and sum each slot's run into its arc's
// gradient as 64-bit fixed-point integers, whose sum does not depend on the
// order of the run (arcs without records keep the zero fill).
int reduce_records(wfst_fst *f, hipStream_t s, int64_t n, int64_t N, uint64_t *k0, float *v0, uint64_t *k1,
                   float *v1, float *grad, const float *grad_log_z, int32_t B)
{
    if (n == 0) return WFST_OK;
    const int64_t ntiles = (n + kSortTile - 1) / kSortTile;
    int64_t *hist, *tiles;
    double *scale;
    TRY(ensure_t(f->ws[W_HIST], 256 * ntiles, s, &hist));
    TRY(ensure_t(f->ws[W_TILES], scan_tiles_for(256 * ntiles), s, &tiles));
    TRY(ensure_t(f->ws[W_FXSCALE], 1, s, &scale));
    hipLaunchKernelGGL(fx_scale_kernel, dim3(1), dim3(256), 0, s, grad_log_z, B, N, scale);
    // digits from the slot part (bits 32 and up) on its significant bits;
    // 2^arc_bits > every slot, so the all-ones sentinel keys sort after all records
    int arc_bits = 1;
    while (arc_bits < 32 && ((int64_t)1 << arc_bits) <= f->rev.n_elem) ++arc_bits;
    std::vector<int> shifts;
    for (int sh = 0; sh < arc_bits; sh += 8) shifts.push_back(32 + sh);
    int32_t *iv0 = reinterpret_cast<int32_t *>(v0), *iv1 = reinterpret_cast<int32_t *>(v1);
    for (int sh : shifts) {
        hipLaunchKernelGGL(radix_hist<uint64_t>, dim3((unsigned)ntiles), dim3(kSortThreads), 0, s,
                           (const uint64_t *)k0, n, sh, ntiles, hist);
        ScanSource src;
        src.i64 = hist;
        TRY(launch_scan<int64_t>(s, src, 256 * ntiles, tiles, hist, nullptr));
        hipLaunchKernelGGL(radix_scatter<uint64_t>, dim3((unsigned)ntiles), dim3(kSortThreads), 0, s,
                           (const uint64_t *)k0, (const int32_t *)iv0, n, sh, ntiles, (const int64_t *)hist, k1, iv1,
                           f->health);
        std::swap(k0, k1);
        std::swap(iv0, iv1);
    }
    const int64_t nrt = (n + 63) / 64;  // tiles of 64 sorted records
    RecTile *rt;
    TRY(ensure_t(f->ws[W_RTILE], nrt, s, &rt));
    hipLaunchKernelGGL(record_tiles, dim3(grid_for(nrt * 64, 256, 16384)), dim3(256), 0, s, (const uint64_t *)k0,
                       (const float *)reinterpret_cast<float *>(iv0), n, (const int32_t *)f->rev.elem_arc,
                       (const double *)scale, grad, rt, nrt);
    hipLaunchKernelGGL(record_runs, dim3(grid_for(nrt, 256, 16384)), dim3(256), 0, s, (const RecTile *)rt, nrt,
                       (const int32_t *)f->rev.elem_arc, (const double *)scale, grad);
    HIP_OK(hipGetLastError());
    return WFST_OK;
}

constexpr int64_t kRecordsMax = (int64_t)1 << 28;  // records per call before the grouped count kernel is used

// ---------------------------------------------------------------------
// Live-state sweeps (live.hip)
// ---------------------------------------------------------------------

// List capacity and table size of a sentence's group, in the on-chip form:
// 64 entries cover the taggers' live sets (at most 32 on the 45-tag trigram
// tagger) at 7 KB of LDS; FSTs too large for the on-chip streaming sweeps
// take 512 (94% of the strings of the 1M-state power-law WFST stay below).
// A step of more rounds of 256 arcs goes on to the next form: from four on that
// is the streaming sweeps, or, for the large FSTs, a workgroup from 32 on.
// (1024 strings with ten steps over one state's many arcs, forward and backward,
// kept / given up at once, us; on chip, 512 arcs: 352 / 485, 1024: 401 / 537,
// 2048: 566 / 642 (Viterbi 164 / 125), 4096: 1000 / 865; large, 2048: 565 / 2993,
// 8192: 1859 / 4340 (Viterbi 478 / 381), 16384: 3576 / 8225 (Viterbi 898 / 446).)
constexpr int kLiveRounds = 4, kLiveRoundsWide = 32;
// Labels with at most this many destinations get a table with an entry for
// each (no keys, one LDS atomic per contribution instead of two).  Its size sets
// how many wavefronts share a compute unit: 4096 sentences of 12 on an FST with
// so many destinations a label, Viterbi, direct / hashed, us: 256: 122 / 124,
// 512: 144 / 145, 768: 153 / 153, 1024: 194 / 161, 2048: 279 / 218.
constexpr int kLiveDirect = 512;

void free_live(wfst_fst *f)
{
    LiveFst &v = f->live;
    for (void *p : {(void *)v.arc, (void *)v.score, (void *)v.stale, (void *)v.label, (void *)v.row, (void *)v.pair,
                    (void *)v.pos, (void *)v.all})
        free_owned(f, p);
    const int64_t pool = v.pool;
    const bool check = v.dense_check;
    v = LiveFst();
    v.pool = pool;
    v.dense_check = check;
}

// Build the index from the reverse layout, on the device.  Without room for
// it the FST keeps to the streaming sweeps.
int build_live(wfst_fst *f, hipStream_t s)
{
    free_live(f);
    const DevLayout &rl = f->rev;
    if (f->A == 0 || f->state_mem >= 2) return WFST_OK;
    LiveFst &v = f->live;
    int32_t *size = nullptr, *first = nullptr, *flags = nullptr, *seg_of = nullptr;
    int64_t *tiles = nullptr;
    const int64_t ntiles = scan_tiles_for(rl.n_seg);
    auto temps = [&]() {
        for (void *p : {(void *)size, (void *)first, (void *)flags, (void *)seg_of, (void *)tiles})
            if (p) (void)hipFree(p);
    };
    auto fail = [&](int rc) {
        temps();
        free_live(f);
        if (rc == WFST_ENOMEM) return (int)WFST_OK;
        return rc;
    };
    auto temp = [&](auto **p, int64_t n) {
        return hipMalloc((void **)p, (size_t)std::max<int64_t>(n, 1) * sizeof(**p)) == hipSuccess;
    };
    auto owned = [&](auto **p, int64_t n) {
        void *q = nullptr;
        const size_t bytes = (size_t)std::max<int64_t>(n, 1) * sizeof(**p);
        if (hipMalloc(&q, bytes) != hipSuccess) return false;
        f->allocs.emplace_back(q, bytes);
        f->bytes += (int64_t)bytes;
        *p = reinterpret_cast<std::remove_reference_t<decltype(*p)>>(q);
        return true;
    };
    if (!temp(&size, rl.n_seg) || !temp(&first, rl.n_seg) || !temp(&flags, 2) || !temp(&seg_of, f->A) ||
        !temp(&tiles, ntiles) ||
        !owned(&v.arc, f->A) || !owned(&v.score, f->A) || !owned(&v.stale, 1) || !owned(&v.pos, rl.n_elem) || !owned(&v.label, f->M) ||
        !owned(&v.all, f->M)) {
        (void)hipGetLastError();
        return fail(WFST_ENOMEM);
    }
    const dim3 per_label((unsigned)std::min(f->M, 65535));
    hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, flags, (int64_t)2, 0);
    hipLaunchKernelGGL(live_segs, per_label, dim3(256), 0, s, f->fwd, f->M, seg_of);
    hipLaunchKernelGGL(live_seg_sizes, per_label, dim3(256), 0, s, rl, f->M, size);
    ScanSource src;
    src.i32 = size;
    int rc = launch_scan<int32_t>(s, src, rl.n_seg, tiles, first, nullptr);
    if (rc != WFST_OK) return fail(rc);
    hipLaunchKernelGGL(live_fill, per_label, dim3(256), 0, s, f->fwd, rl, f->M, f->Q, (const int32_t *)size,
                       (const int32_t *)first, (const int32_t *)seg_of, v.arc, v.score, v.pos, v.label, v.all,
                       flags);
    hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, v.stale, (int64_t)1, 0);
    int32_t host[2] = {0, 0};
    std::vector<int32_t> sizes;
    try {
        sizes.resize((size_t)rl.n_seg);
    } catch (const std::bad_alloc &) {
        return fail(WFST_ENOMEM);
    }
    if (hipMemcpyAsync(host, flags, sizeof(host), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipMemcpyAsync(sizes.data(), size, sizes.size() * sizeof(int32_t), hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return fail(set_err(WFST_EHIP, "building the live-state index"));
    v.ix.listed = !host[0];
    if (host[1]) {
        // Some label does not have the same number of arcs from every state: a
        // direct row per (label, source) where those rows cost at most about
        // twice the arcs themselves, else a hash table of the pairs that exist.
        const double rows = (double)f->M * (double)f->Q * sizeof(int2);
        if (rows <= 32.0 * (double)f->A + (double)((int64_t)64 << 20)) {
            const int64_t n = (int64_t)f->M * f->Q;
            if (!owned(&v.row, n)) {
                (void)hipGetLastError();
                return fail(WFST_ENOMEM);
            }
            hipLaunchKernelGGL(fill_i64, dim3(grid_for(n, 256, 8192)), dim3(256), 0, s,
                               reinterpret_cast<int64_t *>(v.row), n, (int64_t)0);
        } else {
            int64_t n = 64;
            while (n < 2 * rl.n_seg) n *= 2;
            if (!owned(&v.pair, n)) {
                (void)hipGetLastError();
                return fail(WFST_ENOMEM);
            }
            hipLaunchKernelGGL(fill_i32, dim3(grid_for(4 * n, 256, 8192)), dim3(256), 0, s,
                               reinterpret_cast<int32_t *>(v.pair), 4 * n, -1);
            v.ix.pair_mask = (uint32_t)(n - 1);
        }
        hipLaunchKernelGGL(live_lookup, per_label, dim3(256), 0, s, rl, f->M, f->Q, (const int32_t *)size,
                           (const int32_t *)first, v.row, v.pair, v.ix.pair_mask);
    }
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
        return fail(set_err(WFST_EHIP, "building the live-state index"));
    temps();
    size = first = flags = seg_of = nullptr;
    tiles = nullptr;
    if (!f->pin && hipHostMalloc((void **)&f->pin, L_COUNT * sizeof(int32_t), hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        f->pin = nullptr;
        return fail(WFST_ENOMEM);
    }
    v.ix.arc = v.arc;
    v.ix.score = v.score;
    v.ix.label = v.label;
    v.ix.all = v.all;
    v.ix.row = v.row;
    v.ix.pair = v.pair;
    v.wide = lds_lse(f, f->fwd) > f->max_lds;
    const int32_t D = f->fwd.max_segs;
    int32_t per = 0;  // most arcs of a label leaving one state
    for (int32_t x : sizes) per = std::max(per, x);
    v.per = per;
    // Narrow labels: the fewest lanes and arcs per lane that hold every step (28-bit arc ids in the keys).
    for (int w : {8, 16})
        for (int u : {2, 4}) {
            int sh = 0;
            while ((w >> (sh + 1)) >= D) ++sh;
            if (v.narrow || f->A >= (int64_t)1 << 28 || D > w || per > (u << sh)) continue;
            v.narrow = w;
            v.narrow_arcs = u;
            v.narrow_share = sh;
        }
    v.sh.K = v.wide ? 512 : 64;
    v.hash = D > kLiveDirect;
    v.sh.H = !v.hash ? (D + 1) / 2 * 2 : v.sh.K >= 256 ? 2 * v.sh.K : 4 * v.sh.K;
    v.sh.rounds = v.wide ? kLiveRoundsWide : kLiveRounds;
    v.safe = v.narrow || (D <= v.sh.K && (int64_t)((D + 63) / 64) * ((per + 3) / 4) <= v.sh.rounds);
    v.on = true;
    return WFST_OK;
}

bool stream_capturing(hipStream_t s)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &st) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return st != hipStreamCaptureStatusNone;
}

// Whether a pass takes the live-state sweeps: not when the options name a
// form of the streaming sweeps, nor when those would be refused.
bool live_wanted(const wfst_fst *f, size_t dense_lds)
{
    return f->live.on && !f->live.refused && !(f->state_mem == 1 && dense_lds > f->max_lds);
}

// A live pass that found no room for its buffers (rc): the streaming sweeps,
// which need less of them, run instead, after what live passes keep has been
// given back.  Not inside a capture, where nothing can be allocated.
bool live_no_room(wfst_fst *f, hipStream_t s, int rc)
{
    if (rc != WFST_ENOMEM || stream_capturing(s) || hipStreamSynchronize(s) != hipSuccess) return false;
    for (int i : {W_LBP, W_LWIN, W_LPREP, W_LVERDICT, W_LSUB, W_LSUBOUT, W_LSCRATCH, W_LATSTATE, W_LATVAL, W_LACC,
                  W_LTOUCH, W_LFIN, W_LSLOT})
        free_buf(f->ws[i]);
    for (TapeBufs *t : f->tape_pool)  // (of tapes that were freed)
        for (Buf *b : {&t->l_tok, &t->l_state, &t->l_val}) free_buf(*b);
    f->live.pool = 0;
    f->live.refused = f->graph_mode;
    return true;
}

// How sentences that the live sweeps give up are run.  List mode: the
// streaming sweeps take them from a device list in the same call, with no
// read-back; their storage is sized by the bound tokens x widest label.
// Otherwise the host reads their number and runs them as a batch of their own
// (state vectors too large for LDS, whose bound is huge and whose forward
// pass runs as teams; checkpointed tapes).  Inside a capture nothing can be
// read back.
bool live_list_fits(const wfst_fst *f, int64_t N, int64_t cap, bool tape)
{
    const int64_t bound = N * (int64_t)std::max(f->fwd.max_segs, 1);
    if (bound > cap) return false;
    return !tape || f->ckpt_mode == 2 ||
           (f->ckpt_mode != 1 && 2 * (int64_t)sizeof(float) * bound <= f->tape_budget);
}
bool live_list_mode(const wfst_fst *f, hipStream_t s, int64_t N, int64_t cap, bool tape)
{
    if (f->graph_mode || stream_capturing(s)) return true;
    return !f->live.wide && live_list_fits(f, N, cap, tape);
}

// Write the scores (arc-id order) into both sliced layouts, if the gate is open.
int scatter_layouts(wfst_fst *f, hipStream_t s, const float *score, ScoreGate gate)
{
    const int64_t quads = (f->fwd.n_elem + 3) / 4 + (f->rev.n_elem + 3) / 4;
    int64_t tiles = (quads + 255) / 256;
    tiles = (tiles + kXcds - 1) / kXcds * kXcds;
    if (tiles > INT32_MAX) return set_err(WFST_EUNSUPPORTED, "too many arc slots for one score update");
    // a gated launch mostly ends at once: one grid of resident workgroups
    if (f->stage_scores) {
        const unsigned grid = (unsigned)(gate.stale ? std::min<int64_t>(f->M, 4 * f->cu_count) : f->M);
        hipLaunchKernelGGL(scatter_scores_by_label, dim3(grid), dim3(kScoreThreads), kScoreStage * sizeof(float), s,
                           (const LabelInfo *)f->fwd.label, (const LabelInfo *)f->rev.label,
                           (const int2 *)f->label_range, f->fwd.score, (const int32_t *)f->fwd.elem_arc,
                           (const uint16_t *)f->fwd.elem_loc, f->rev.score, (const int32_t *)f->rev.elem_arc,
                           (const uint16_t *)f->rev.elem_loc, score, f->M, gate);
    } else {
        const unsigned grid = (unsigned)(gate.stale ? std::min<int64_t>(tiles, 8 * f->cu_count / kXcds * kXcds) : tiles);
        hipLaunchKernelGGL(scatter_scores, dim3(grid), dim3(256), 0, s, f->fwd.score,
                           (const int32_t *)f->fwd.elem_arc, f->fwd.n_elem, f->rev.score,
                           (const int32_t *)f->rev.elem_arc, f->rev.n_elem, score, tiles, gate);
    }
    HIP_OK(hipGetLastError());
    return WFST_OK;
}

// Before a pass that reads the sliced layouts' scores: bring them up to date
// (n: device count of the sentences that pass has; none, no update; the pass's next kernel then notes that they are).
int refresh_layouts(wfst_fst *f, hipStream_t s, const int32_t *n)
{
    LiveFst &v = f->live;
    if (!v.on) return WFST_OK;
    const bool capture = f->graph_mode || stream_capturing(s);
    if (!v.dense_stale && !v.dense_check && !capture) return WFST_OK;
    ScoreGate gate;
    gate.stale = v.stale;
    gate.n = n;
    TRY(scatter_layouts(f, s, v.score, gate));
    if (!n) hipLaunchKernelGGL(live_fresh, dim3(1), dim3(64), 0, s, v.stale);
    if (!n && !capture) v.dense_stale = false;
    return WFST_OK;
}

// Grid of the on-chip form: every sentence at once if the LDS and the
// wavefront slots of the device hold them.
int live_grid(const wfst_fst *f, size_t lds, int32_t B)
{
    const int64_t per_cu = std::max<int64_t>(1, std::min<int64_t>(32, (int64_t)(f->max_lds / lds)));
    return (int)std::max<int64_t>(1, std::min<int64_t>(B, per_cu * f->cu_count));
}

// Workgroups (and their scratch) of the global-memory form.
int live_wide_grid(wfst_fst *f, hipStream_t s, int32_t B, int *grid, unsigned char **scratch)
{
    const int64_t slot = (int64_t)live_slot(f->Q);
    *grid = (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(B, f->cu_count), kStateScratchBudget / slot));
    return ensure_zeroed(f->ws[W_LSCRATCH], *grid * slot, s, scratch);
}

// The most entries a pool may have (positions are 32-bit).
constexpr int64_t kLivePoolMax = (int64_t)1 << 30;
constexpr int64_t kForwardEntry = sizeof(int2) + sizeof(double);  // of a forward pass: state, log alpha

// Bytes the lists (or narrow tables) of a forward pass may take: the tape
// budget, but at least 64 MiB, which a pass needs to get anywhere; where the
// options rule checkpointing out, as many as positions allow.
int64_t live_tape_bytes(const wfst_fst *f)
{
    if (f->ckpt_mode == 2) return kLivePoolMax * kForwardEntry;
    return std::max<int64_t>(f->tape_budget, (int64_t)64 << 20);
}
int64_t narrow_tape_bytes(const wfst_fst *f, int64_t N)
{
    return (int64_t)sizeof(double) * N * std::max(f->fwd.max_segs, 1);
}

// Pool entries of a pass: the most the on-chip form can need (lists of at most
// min(widest label, K) entries, of which a chunk leaves fewer than that
// unused), unless that is above max_entries or the global-memory form may add
// lists of any length: then a default, which grows when a pass used it up.
int64_t live_pool_entries(const wfst_fst *f, int32_t B, int64_t N, int64_t max_entries, bool *bounded)
{
    const int64_t L = std::min<int64_t>(std::max(f->fwd.max_segs, 1), f->live.sh.K);
    const int64_t groups = std::min<int64_t>((int64_t)f->cu_count * 32, B) + 1;
    const int64_t chunk = std::max<int64_t>(kLiveChunk, L);
    const int64_t most = L < kLiveChunk ? (N * L / (kLiveChunk - L + 1) + 1 + groups) * chunk : (2 * N + 1 + groups) * chunk;
    *bounded = (f->live.safe || !f->live.wide) && most <= max_entries;
    if (*bounded) return most;
    return std::min(max_entries, std::max<int64_t>(f->live.pool, 32 * N + groups * chunk + 65536));
}

// The sentences a live pass gave up, as a batch of their own.
struct LiveRest {
    int32_t n = 0;
    int64_t N = 0;
    const int32_t *list = nullptr;  // null: the whole batch
    const int32_t *off = nullptr, *tok = nullptr;
};

// left: device list of n sentences (any order).  Their offsets and tokens are
// copied into buf, in increasing sentence order, so that what is summed in
// batch order does not depend on the schedule.
int live_rest(wfst_fst *f, hipStream_t s, Buf &buf, int32_t B, int64_t N, const int32_t *offsets,
              const int32_t *tokens, const int32_t *left, int32_t n, LiveRest &r)
{
    r.n = n;
    if (n == B) {
        r.N = N;
        r.off = offsets;
        r.tok = tokens;
        return WFST_OK;
    }
    std::vector<int32_t> list((size_t)n), off((size_t)B + 1), up(2 * (size_t)n + 1);
    HIP_OK(hipMemcpyAsync(list.data(), left, list.size() * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    HIP_OK(hipMemcpyAsync(off.data(), offsets, off.size() * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    HIP_OK(hipStreamSynchronize(s));
    std::sort(list.begin(), list.end());
    int32_t at = 0;
    for (int32_t i = 0; i < n; ++i) {
        const int32_t b = list[(size_t)i];
        up[(size_t)i] = b;
        up[(size_t)n + i] = at;
        at += off[(size_t)b + 1] - off[(size_t)b];
    }
    up[2 * (size_t)n] = at;
    int32_t *p;
    TRY(ensure_t(buf, 2 * (int64_t)n + 1 + at, s, &p));
    HIP_OK(hipMemcpyAsync(p, up.data(), up.size() * sizeof(int32_t), hipMemcpyHostToDevice, s));
    HIP_OK(hipStreamSynchronize(s));  // `up` goes out of scope
    r.N = at;
    r.list = p;
    r.off = p + n;
    r.tok = p + 2 * (int64_t)n + 1;
    hipLaunchKernelGGL(live_gather, dim3(grid_for(n, 1)), dim3(64), 0, s, r.list, n, offsets, tokens, r.off,
                       p + 2 * (int64_t)n + 1);
    HIP_OK(hipGetLastError());
    return WFST_OK;
}

void live_put_back(hipStream_t s, const LiveRest &r, const int32_t *offsets, const void *sub, void *out, bool per_token)
{
    if (!out || !sub) return;
    hipLaunchKernelGGL(live_scatter, dim3(grid_for(r.n, 1)), dim3(64), 0, s, r.list, r.n, offsets, r.off,
                       (const uint32_t *)sub, (uint32_t *)out, (int32_t)per_token);
}

// Processing order: longest first where a wavefront takes several sentences
// or not all of them run at once.
int live_order(wfst_fst *f, hipStream_t s, int32_t B, const int32_t *offsets, Buf &buf, int64_t at_once,
               const int32_t **order)
{
    *order = nullptr;
    if (B <= at_once) return WFST_OK;
    int32_t *p;
    TRY(ensure_t(buf, B, s, &p));
    hipLaunchKernelGGL(order_by_length, dim3(1), dim3(1024), 0, s, offsets, B, p);
    *order = p;
    return WFST_OK;
}

// f(std::true_type or std::false_type): arcs listed by (label, source) or not
template <class F>
auto by_listed(const LiveFst &v, F f)
{
    return v.ix.listed ? f(std::true_type()) : f(std::false_type());
}
#define LIVE_LAUNCH(kernel, v, grid, lds, s, ...)                                                            \
    by_listed(v, [&](auto listed) {                                                                          \
        constexpr bool L = decltype(listed)::value;                                                          \
        if (!(v).hash)                                                                                       \
            hipLaunchKernelGGL((kernel<64, kDirect, L>), dim3(grid), dim3(64), lds, s, __VA_ARGS__);         \
        else                                                                                                 \
            hipLaunchKernelGGL((kernel<64, kHash, L>), dim3(grid), dim3(64), lds, s, __VA_ARGS__);           \
    })
#define WIDE_LAUNCH(kernel, v, grid, s, ...)                                                                 \
    by_listed(v, [&](auto listed) {                                                                          \
        hipLaunchKernelGGL((kernel<kLiveGroupThreads, kGlobal, decltype(listed)::value>), dim3(grid),        \
                           dim3(kLiveGroupThreads), 0, s, __VA_ARGS__);                                      \
    })
template <int W, int U, bool L>
constexpr auto narrow_backward_hot = narrow_backward<W, U, L, true>;
template <int W, int U, bool L>
constexpr auto narrow_backward_cold = narrow_backward<W, U, L, false>;
#define NARROW_LAUNCH(kernel, v, grid, nt, lds, s, ...)                                                      \
    by_listed(v, [&](auto listed) {                                                                          \
        constexpr bool L = decltype(listed)::value;                                                          \
        if ((v).narrow == 8 && (v).narrow_arcs == 2)                                                         \
            hipLaunchKernelGGL((kernel<8, 2, L>), dim3(grid), dim3(nt), lds, s, __VA_ARGS__);                \
        else if ((v).narrow == 8)                                                                            \
            hipLaunchKernelGGL((kernel<8, 4, L>), dim3(grid), dim3(nt), lds, s, __VA_ARGS__);                \
        else if ((v).narrow_arcs == 2)                                                                       \
            hipLaunchKernelGGL((kernel<16, 2, L>), dim3(grid), dim3(nt), lds, s, __VA_ARGS__);               \
        else                                                                                                 \
            hipLaunchKernelGGL((kernel<16, 4, L>), dim3(grid), dim3(nt), lds, s, __VA_ARGS__);               \
    })

// Wavefronts of a narrow sweep: every sentence at once, up to all wavefront slots.
int narrow_grid(const wfst_fst *f, int32_t B)
{
    const int64_t per = 64 / f->live.narrow;
    return (int)std::min<int64_t>(((int64_t)B + per - 1) / per, (int64_t)f->cu_count * 32);
}
NarrowView narrow_view(const wfst_fst *f)
{
    NarrowView v;
    v.seg_key = f->fwd.seg_key;
    v.D = std::max(f->fwd.max_segs, 1);
    v.share = f->live.narrow_share;
    return v;
}
// Cells for the most frequent labels: from this many tokens a compute unit on (fewer repeat too little to pay for
// clearing and adding the cells: forward and backward, cells / none, us: 256 tokens a compute unit 170 / 149 with a
// vocabulary of 2000, 178 / 168 with 20000; 512: 173 / 221 and 180 / 253; 1024: 198 / 428 with 20000), when no list of touched arcs is kept, one cell a token of a workgroup; workgroups of
// the wavefronts that share a compute unit.
constexpr int64_t kHotTokens = 512;
bool touched_kept(const wfst_fst *f, int64_t N) { return N < f->A / 128; }
struct HotPlan {
    int nt = 64, grid = 0;
    int32_t cells = 0;
    size_t lds = 0;
};
bool narrow_hot_plan(const wfst_fst *f, int32_t B, int64_t N, HotPlan &p)
{
    const int waves = narrow_grid(f, B);
    p.grid = waves;
    if (touched_kept(f, N) || N / f->cu_count < kHotTokens || B <= 64 / f->live.narrow) return false;
    const int per = std::min(8, (waves + f->cu_count - 1) / f->cu_count);
    p.nt = 64 * per;
    p.grid = (waves + per - 1) / per;
    p.cells = (int32_t)std::min<int64_t>(kHotCells, N / p.grid);
    p.lds = (size_t)p.cells * sizeof(unsigned long long) + kHotMap * sizeof(int2);
    return true;
}

// Look up every (token, source) of a batch, and order its sentences unless one wavefront takes them all.
int narrow_prepare(wfst_fst *f, hipStream_t s, const BatchView &bv, Buf &prep_buf, Buf &verdict_buf, Buf &order_buf,
                   NarrowView &v, const int32_t **order, const HotOut &ho = HotOut())
{
    int2 *prep;
    int32_t *verdict, *ord = nullptr;
    v = narrow_view(f);
    TRY(ensure_t(prep_buf, bv.N * v.D, s, &prep));
    TRY(ensure_t(verdict_buf, bv.B, s, &verdict));
    if (bv.B > 64 / f->live.narrow) TRY(ensure_t(order_buf, bv.B, s, &ord));
    v.prep = prep;
    v.verdict = verdict;
    *order = ord;
    const int nt = ord ? 1024 : 64;
    const int grid = grid_for((int64_t)bv.B * 64, nt, f->cu_count * 32 * 64 / nt);
    if (ho.label)
        hipLaunchKernelGGL(narrow_prep<true>, dim3(grid + 2), dim3(nt), 0, s, f->live.ix, v.seg_key, v.D, f->start, bv,
                           prep, verdict, ord, ho);
    else
        hipLaunchKernelGGL(narrow_prep<false>, dim3(grid + (ord ? 1 : 0)), dim3(nt), 0, s, f->live.ix, v.seg_key, v.D,
                           f->start, bv, prep, verdict, ord, ho);
    return WFST_OK;
}

int viterbi_dense(wfst_fst *f, int32_t batch, int64_t N, const int32_t *offsets, const int32_t *tokens,
                  float *best_score, int32_t *best_arcs, int32_t *best_olabels, int32_t *status, hipStream_t s);
int forward_dense(wfst_fst *f, int32_t batch, int64_t N, const int32_t *offsets, const int32_t *tokens, float *log_z,
                  int32_t *status, wfst_tape **tape_out, hipStream_t s);
int backward_dense(wfst_fst *f, const wfst_tape *tape, const float *grad_log_z, float *grad_arc_score,
                   float *grad_final, hipStream_t s, const LiveCounts *into = nullptr);

// The launches of one live pass: the on-chip form over the batch, then (wide
// FSTs) the global-memory form over what it gave up.  When no storage bound
// holds and the counters may be read back, a pass that used its pool up is
// run again with a larger one.  *n_rest: sentences left, -1 if not read back.
struct LivePass {
    int32_t *cnt = nullptr, *left = nullptr;
    int grid = 0, wgrid = 0;
    unsigned char *scratch = nullptr;
    LiveWork w, w2;
    LivePool pool;
    bool leaves = false;  // sentences may be left over
    const int32_t *final_left() const { return wgrid ? w2.left : w.left; }
    const int32_t *final_n() const { return wgrid ? w2.n_left : w.n_left; }
};
template <class Sized, class Launch>
int live_pass(wfst_fst *f, hipStream_t s, int32_t B, int64_t N, const int32_t *offsets, bool list_mode, bool direct,
              Buf &cnt_buf,
              Buf &left_buf, Buf &order_buf, size_t lds, int64_t max_entries, LivePass &p, Sized sized, Launch launch,
              int32_t *n_rest)
{
    const LiveFst &v = f->live;
    TRY(ensure_t(cnt_buf, L_COUNT, s, &p.cnt));
    TRY(ensure_t(left_buf, 2 * (int64_t)B, s, &p.left));
    p.grid = direct ? 0 : live_grid(f, lds, B);
    TRY(live_order(f, s, B, offsets, order_buf, direct ? f->cu_count : p.grid, &p.w.order));
    p.w.left = p.left;
    p.w.n_left = p.cnt + L_LEFT;
    if (direct || (v.wide && !v.safe)) TRY(live_wide_grid(f, s, B, &p.wgrid, &p.scratch));
    p.w2.order = direct ? p.w.order : p.left;
    p.w2.n = direct ? nullptr : p.cnt + L_LEFT;
    p.w2.left = p.left + B;
    p.w2.n_left = p.cnt + L_LEFT2;
    p.pool.used = reinterpret_cast<unsigned long long *>(p.cnt + L_USED);
    bool bounded = false;
    p.pool.cap = live_pool_entries(f, B, N, max_entries, &bounded);
    p.leaves = !(v.safe && bounded);
    const bool read_back = !list_mode && p.leaves;
    *n_rest = p.leaves ? -1 : 0;
    for (int attempt = 0;; ++attempt) {
        TRY(sized(p.pool.cap));
        hipLaunchKernelGGL(live_counters, dim3(1), dim3(64), 0, s, p.cnt, (int32_t)L_COUNT,
                           p.grid * kLiveChunk, 0);
        TRY(launch(p));
        HIP_OK(hipGetLastError());
        if (!read_back) return WFST_OK;
        HIP_OK(hipMemcpyAsync(f->pin, p.cnt, L_COUNT * sizeof(int32_t), hipMemcpyDeviceToHost, s));
        HIP_OK(hipStreamSynchronize(s));
        unsigned long long used;
        std::memcpy(&used, f->pin + L_USED, sizeof(used));
        *n_rest = f->pin[p.wgrid ? L_LEFT2 : L_LEFT];
        if ((int64_t)used <= p.pool.cap || attempt == 2 || p.pool.cap >= max_entries) return WFST_OK;
        f->live.pool = std::min<int64_t>((int64_t)used + (int64_t)used / 4, kLivePoolMax);
        p.pool.cap = std::min(f->live.pool, max_entries);
    }
}

int viterbi_live(wfst_fst *f, int32_t B, int64_t N, const int32_t *offsets, const int32_t *tokens, float *best_score,
                 int32_t *best_arcs, int32_t *best_olabels, int32_t *status, hipStream_t s)
{
    const LiveFst &v = f->live;
    const BatchView bv = make_view(f, B, N, offsets, tokens, nullptr, nullptr, nullptr, status);
    if (v.narrow) {
        uint8_t *pred;
        int32_t *win;
        const int32_t *order;
        TRY(ensure_t(f->ws[W_LBP], N * v.narrow, s, &pred));
        TRY(ensure_t(f->ws[W_LWIN], N * (int64_t)std::max(f->fwd.max_segs, 1), s, &win));
        ProfScope prof(f, s, WFST_KERNEL_VITERBI);
        NarrowView nv;
        TRY(narrow_prepare(f, s, bv, f->ws[W_LPREP], f->ws[W_LVERDICT], f->ws[W_LORDER], nv, &order));
        NARROW_LAUNCH(narrow_viterbi, v, narrow_grid(f, B), 64, 0, s, v.ix, nv, f->start,
                      (const float *)f->final_score, bv, order, pred, win, best_score, best_arcs, best_olabels,
                      (const int32_t *)f->olabel);
        HIP_OK(hipGetLastError());
        return WFST_OK;
    }
    const bool list_mode = live_list_mode(f, s, N, kBoundCapBytes / 8, false);
    const size_t lds = live_viterbi_lds(v.sh.K, v.sh.H, v.hash);
    int2 *bp = nullptr;
    LivePass p;
    int32_t n_rest = 0;
    TRY(live_pass(
        f, s, B, N, offsets, list_mode, false, f->ws[W_LCNT], f->ws[W_LLEFT], f->ws[W_LORDER], lds, kLivePoolMax, p,
        [&](int64_t cap) { return ensure_t(f->ws[W_LBP], cap, s, &bp); },
        [&](const LivePass &x) -> int {
            const bool rest = list_mode && x.leaves;
            int32_t *path_tmp = nullptr;
            int64_t *tok_off = nullptr;
            int2 *bpd = nullptr;
            // (also when a later call may need them inside a capture, where nothing can be allocated)
            const int64_t bound = N * (int64_t)std::max(f->fwd.max_segs, 1);
            if (rest || (x.leaves && live_list_fits(f, N, kBoundCapBytes / 8, false))) {
                TRY(ensure_t(f->ws[W_PATH], N, s, &path_tmp));
                TRY(ensure_t(f->ws[W_TOKOFF], N, s, &tok_off));
                TRY(ensure_t(f->ws[W_BP], bound, s, &bpd));
            }
            ProfScope prof(f, s, WFST_KERNEL_VITERBI);
            LIVE_LAUNCH(live_viterbi, v, x.grid, lds, s, v.ix, v.sh, f->Q, f->start,
                        (const float *)f->final_score, bv, x.w, x.pool, bp, best_score, best_arcs, best_olabels,
                        (const int32_t *)f->olabel, (unsigned char *)nullptr);
            if (x.wgrid)
                WIDE_LAUNCH(live_viterbi, v, x.wgrid,
                                   s, v.ix, v.sh, f->Q, f->start, (const float *)f->final_score, bv, x.w2, x.pool, bp,
                                   best_score, best_arcs, best_olabels, (const int32_t *)f->olabel, x.scratch);
            int rc = WFST_OK;
            if (!rest && bpd)
                DISPATCH_NT(rc, f->nt, launch_viterbi, f, s, bv, bpd, path_tmp, best_score, best_arcs, best_olabels,
                            false, true)
            if (!rest) return rc;
            BatchView rv = bv;
            rv.order = x.final_left();
            rv.n = x.final_n();
            rv.tok_off = tok_off;
            rv.queue = x.cnt + L_QUEUE3;
            TRY(refresh_layouts(f, s, x.final_n()));
            hipLaunchKernelGGL(rest_offsets, dim3(grid_for(B, 1, 1024)), dim3(64), 0, s, f->fwd, rv,
                               reinterpret_cast<unsigned long long *>(x.cnt + L_ROFF), tok_off, f->live.stale);
            DISPATCH_NT(rc, f->nt, launch_viterbi, f, s, rv, bpd, path_tmp, best_score, best_arcs, best_olabels)
            return rc;
        },
        &n_rest));
    if (n_rest <= 0) return WFST_OK;
    LiveRest r;
    TRY(live_rest(f, s, f->ws[W_LSUB], B, N, offsets, tokens, p.final_left(), n_rest, r));
    if (!r.list) return viterbi_dense(f, B, N, offsets, tokens, best_score, best_arcs, best_olabels, status, s);
    int32_t *out;
    TRY(ensure_t(f->ws[W_LSUBOUT], 2 * (int64_t)r.n + 2 * std::max<int64_t>(r.N, 1), s, &out));
    float *sc = reinterpret_cast<float *>(out);
    int32_t *st = out + r.n, *arcs = out + 2 * (int64_t)r.n, *ol = best_olabels ? arcs + r.N : nullptr;
    TRY(viterbi_dense(f, r.n, r.N, r.off, r.tok, sc, arcs, ol, st, s));
    live_put_back(s, r, offsets, sc, best_score, false);
    live_put_back(s, r, offsets, st, status, false);
    live_put_back(s, r, offsets, arcs, best_arcs, true);
    live_put_back(s, r, offsets, ol, best_olabels, true);
    HIP_OK(hipGetLastError());
    return WFST_OK;
}

int forward_live(wfst_fst *f, wfst_tape *t, float *log_z, int32_t *status, hipStream_t s)
{
    const LiveFst &v = f->live;
    TapeBufs *tb = t->bufs;
    const int32_t B = t->B;
    const int64_t N = t->N;
    t->live = true;
    TRY(ensure_t(tb->l_done, B, s, &t->lists.done));
    TRY(ensure_t(tb->log_z, B, s, &t->log_z));
    t->lists.log_z = t->log_z;
    const BatchView bv = make_view(f, B, N, t->offsets, t->tokens, nullptr, nullptr, nullptr, status);
    if (v.narrow) {
        const int32_t *order;
        TRY(ensure_t(tb->l_val, N * (int64_t)std::max(f->fwd.max_segs, 1), s, &t->lists.val));
        ProfScope prof(f, s, WFST_KERNEL_FORWARD);
        NarrowView nv;  // kept with the tape: the backward pass reads it too
        HotPlan plan;
        HotOut ho;
        if (narrow_hot_plan(f, B, N, plan)) {
            TRY(ensure_t(tb->l_state, kHotMax + 1, s, &ho.label));
            ho.n = reinterpret_cast<int32_t *>(ho.label + kHotMax);
            ho.cells = plan.cells;
        }
        TRY(narrow_prepare(f, s, bv, tb->l_tok, tb->l_left, tb->order, nv, &order, ho));
        t->order = const_cast<int32_t *>(order);
        NARROW_LAUNCH(narrow_forward, v, narrow_grid(f, B), 64, 0, s, v.ix, nv, f->start,
                      (const float *)f->final_score, bv, order, t->lists.val, t->lists.done, t->lists.log_z, log_z);
        HIP_OK(hipGetLastError());
        return WFST_OK;
    }
    TRY(ensure_t(tb->l_tok, N, s, &t->lists.tok));
    const bool list_mode = live_list_mode(f, s, N, kBoundCapBytes / 4, true);
    const size_t lds = live_forward_lds(v.sh.K, v.sh.H, v.hash);
    // Wide FSTs, at most a sentence a compute unit: every sentence to a workgroup at once, since the last string's
    // steps are then all that is waited for; more strings than that fill the chip with wavefronts (only the longest
    // lists again by a workgroup).  Forward and backward over 1M states, workgroup each / wavefront first, us: 24
    // strings 722 / 1318, 128 5795 / 6654, 256 2846 / 3784 (other strings), 512 4525 / 5231, 1024 12934 / 12121;
    // 200000 states: 256 4944 / 5588, 512 5307 / 5780, 1024 8306 / 7258; 8 strings 698 / 481.
    const bool direct = v.wide && !v.safe && B <= f->cu_count;
    LivePass p;
    int32_t n_rest = 0;
    TRY(live_pass(
        f, s, B, N, t->offsets, list_mode, direct, tb->l_cnt, tb->l_left, tb->order, lds,
        std::min(kLivePoolMax, live_tape_bytes(f) / kForwardEntry), p,
        [&](int64_t cap) -> int {
            TRY(ensure_t(tb->l_state, cap, s, &t->lists.state));
            return ensure_t(tb->l_val, cap, s, &t->lists.val);
        },
        [&](const LivePass &x) -> int {
            const bool rest = list_mode && x.leaves;
            t->total = N * (int64_t)std::max(f->fwd.max_segs, 1);
            if (rest) {
                t->left = x.final_left();
                t->n_left = x.final_n();
            }
            if (rest || (x.leaves && live_list_fits(f, N, kBoundCapBytes / 4, true))) {  // as for Viterbi
                TRY(ensure_t(tb->tok_off, N, s, &t->tok_off));
                TRY(ensure_t(tb->alpha, t->total, s, &t->alpha));
                TRY(ensure_t(tb->a_max, N, s, &t->a_max));
                TRY(ensure_t(tb->a_log, N, s, &t->a_log));
            }
            ProfScope prof(f, s, WFST_KERNEL_FORWARD);
            if (x.grid)
                LIVE_LAUNCH(live_forward, v, x.grid, lds, s, v.ix, v.sh, f->Q, f->start,
                        (const float *)f->final_score, bv, x.w, x.pool, t->lists, log_z, (unsigned char *)nullptr);
            if (x.wgrid)
                WIDE_LAUNCH(live_forward, v, x.wgrid,
                                   s, v.ix, v.sh, f->Q, f->start, (const float *)f->final_score, bv, x.w2, x.pool,
                                   t->lists, log_z, x.scratch);
            int rc = WFST_OK;
            t->reserved = !rest && t->alpha;
            if (t->reserved) DISPATCH_NT(rc, f->nt, launch_forward, f, s, bv, tape_view(t), BlockView(), log_z, true)
            if (!rest) return rc;
            BatchView rv = bv;
            rv.order = x.final_left();
            rv.n = x.final_n();
            rv.tok_off = t->tok_off;
            rv.queue = x.cnt + L_QUEUE3;
            TRY(refresh_layouts(f, s, x.final_n()));
            hipLaunchKernelGGL(rest_offsets, dim3(grid_for(B, 1, 1024)), dim3(64), 0, s, f->fwd, rv,
                               reinterpret_cast<unsigned long long *>(x.cnt + L_ROFF), t->tok_off, f->live.stale);
            DISPATCH_NT(rc, f->nt, launch_forward, f, s, rv, tape_view(t), BlockView(), log_z)
            return rc;
        },
        &n_rest));
    t->order = const_cast<int32_t *>(p.w.order);
    t->wide = p.wgrid > 0;
    t->direct = direct;
    if (n_rest <= 0) return WFST_OK;
    LiveRest r;
    TRY(live_rest(f, s, tb->l_sub, B, N, t->offsets, t->tokens, p.final_left(), n_rest, r));
    t->n_rest = r.n;
    t->rest_list = r.list;
    t->n_left = p.final_n();
    if (!r.list) return forward_dense(f, B, N, t->offsets, t->tokens, log_z, status, &t->rest, s);
    int32_t *out;  // log Z, status, and later the weights of these sentences
    TRY(ensure_t(tb->l_out, 3 * (int64_t)r.n, s, &out));
    float *lz = reinterpret_cast<float *>(out);
    TRY(forward_dense(f, r.n, r.N, r.off, r.tok, lz, out + r.n, &t->rest, s));
    live_put_back(s, r, t->offsets, lz, log_z, false);
    live_put_back(s, r, t->offsets, out + r.n, status, false);
    HIP_OK(hipGetLastError());
    return WFST_OK;
}

// Visits of left sentences staged at a time by rest_counts: one if the states' alpha and beta fit LDS, several if two
// workgroups then still fit a compute unit; 0: they (or rest_backward's state) do not fit, backward_sweep runs.
size_t lds_rest(const wfst_fst *f, int tile) { return 2 * sizeof(float) * (size_t)tile * (size_t)f->Q; }
size_t lds_rest_backward(const wfst_fst *f) { return rest_carve(f->Q, f->rev.max_segs, f->rev.max_slots).end; }
int rest_tile(const wfst_fst *f)
{
    int tile = 0;
    for (int t : {1, 2, 4})
        if (lds_rest(f, t) + 4096 <= f->max_lds / (t == 1 ? 1 : 2)) tile = t;
    return !backward_in_gmem(f) && lds_rest_backward(f) + 256 <= f->max_lds ? tile : 0;
}
// Group the visits of the sentences bv lists by label.
int rest_groups(wfst_fst *f, hipStream_t s, const BatchView &bv, int32_t *cnt, RestGroups &g, bool size_only = false)
{
    TRY(ensure_zeroed(f->ws[W_RGN], f->M, s, &g.label_n));
    TRY(ensure_t(f->ws[W_RGRANK], bv.N, s, &g.rank));
    TRY(ensure_t(f->ws[W_RGFIRST], f->M, s, &g.first));
    TRY(ensure_t(f->ws[W_RGTOK], bv.N, s, &g.tok));
    TRY(ensure_t(f->ws[W_RGLABEL], std::min<int64_t>(f->M, bv.N) + 1, s, &g.label));
    if (size_only) return WFST_OK;
    ZeroHold hold(f->ws[W_RGN], stream_capturing(s));
    g.n_label = cnt + L_GROUPS;
    hipLaunchKernelGGL(rest_rank, dim3(grid_for(bv.B, 1, f->cu_count * 8)), dim3(64), 0, s, bv, g);
    hipLaunchKernelGGL(rest_group, dim3(1), dim3(1024), 0, s, g, (const int2 *)f->live.all, f->M, bv.n);
    HIP_OK(hipGetLastError());
    hold.done();
    return WFST_OK;
}
template <int NT>
int launch_rest_backward(const wfst_fst *f, hipStream_t s, const BatchView &bv, const TapeView &tp, const RestGroups &g,
                         const LiveCounts &ct)
{
    int grid = 0;
    const size_t lds = lds_rest_backward(f);
    TRY(persistent_grid(f, rest_backward<NT>, NT, lds, bv.B, &grid));
    hipLaunchKernelGGL(rest_backward<NT>, dim3(grid), dim3(NT), lds, s, f->fwd, f->rev, f->Q, f->start,
                       (const float *)f->final_score, (const float *)f->final_max, bv, tp, g, ct);
    HIP_OK(hipGetLastError());
    return WFST_OK;
}
template <int TT>
int launch_rest_counts(const wfst_fst *f, hipStream_t s, const BatchView &bv, const TapeView &tp, const RestGroups &g,
                       const LiveCounts &ct)
{
    int grid = 0;
    TRY(persistent_grid(f, rest_counts<TT>, kRestThreads, lds_rest(f, TT), INT32_MAX, &grid));
    hipLaunchKernelGGL(rest_counts<TT>, dim3(grid), dim3(kRestThreads), lds_rest(f, TT), s, f->live.ix, f->fwd, f->Q,
                       f->start, bv, tp, g, ct);
    HIP_OK(hipGetLastError());
    return WFST_OK;
}

// Counts of left sentences by backward_sweep (pass(sink)), into the live passes' accumulators.
// n: device count of those sentences (null: there are some).
template <class Pass>
int slot_counts(wfst_fst *f, hipStream_t s, const LiveCounts &ct, const int32_t *n, Pass pass)
{
    RecordSink rs;
    TRY(ensure_zeroed(f->ws[W_LSLOT], f->rev.n_elem, s, &rs.acc));
    ZeroHold hold(f->ws[W_LSLOT], stream_capturing(s));
    rs.fx_scale = ct.scale;
    rs.grad_log_z = ct.grad_log_z;
    TRY(pass(rs));
    hipLaunchKernelGGL(rest_slot_counts, dim3(grid_for(f->rev.n_elem, 256, n ? 4 * f->cu_count : 8192)), dim3(256), 0, s,
                       rs.acc, f->rev.n_elem, (const int32_t *)f->live.pos, n, ct.acc);
    HIP_OK(hipGetLastError());
    hold.done();
    return WFST_OK;
}

int backward_live(wfst_fst *f, const wfst_tape *t, const float *grad_log_z, float *grad_arc_score, float *grad_final,
                  hipStream_t s)
{
    const LiveFst &v = f->live;
    const int32_t B = t->B;
    const int64_t N = t->N;
    // state_memory = 1 refuses what the streaming sweep could not hold on chip, whichever sweeps would run
    if (N > 0 && f->state_mem == 1 && lds_backward(f) > f->max_lds) return refuse_lds(f, lds_backward(f));
    int32_t *cnt;
    TRY(ensure_t(t->bufs->l_cnt, L_COUNT, s, &cnt));  // (the forward pass's, but for narrow labels)
    LiveCounts ct;
    double *scale;
    TRY(ensure_zeroed(f->ws[W_LACC], f->A, s, &ct.acc));
    ZeroHold hold(f->ws[W_LACC], stream_capturing(s));  // from the first count to the conversion
    // A list of the arcs a small batch touches saves scanning every accumulator (16 bytes
    // read at random and a write against 8 in order, for about 8 touched arcs a token).
    const size_t lds = live_backward_lds(v.sh.K, v.sh.H, v.hash);
    const int grid = v.narrow ? narrow_grid(f, B) : live_grid(f, lds, B);
    const int64_t owned = (int64_t)grid * (v.narrow ? 64 / v.narrow : 1) * kLiveChunk;
    ct.touched_cap = 16 * N + owned + 65536;
    if (touched_kept(f, N)) TRY(ensure_t(f->ws[W_LTOUCH], ct.touched_cap, s, &ct.touched));
    TRY(ensure_t(f->ws[W_FXSCALE], 1, s, &scale));
    ct.scale = scale;
    ct.n_touched = reinterpret_cast<unsigned long long *>(cnt + L_TOUCHED);
    ct.grad_log_z = grad_log_z;
    ct.Q = f->Q;
    ct.fin_shift = B <= 1 << 24 ? 4 : 3;
    const int64_t fin_n = f->Q * (int64_t)fin_words(ct.fin_shift);
    if (grad_final) TRY(ensure_t(f->ws[W_LFIN], fin_n, s, &ct.fin));
    hipLaunchKernelGGL(live_backward_begin, dim3(grad_final ? grid_for(fin_n, 256, 4096) : 1), dim3(256), 0, s,
                       grad_log_z, B, std::max<int64_t>(N, 1), scale, ct.fin, fin_n, cnt, (int32_t)L_COUNT, (int32_t)owned,
                       v.narrow ? 2 : 1);
    // A conversion that looks at every accumulator in arc order writes the whole gradient; else it is filled beside the
    // sweep, by a wavefront a compute unit (large tagger, sweep and fill of 1 and of 4096 sentences: 109 and 164 us;
    // with half as many 137 and 144, twice 112 and 187, four times 116 and 221).
    const bool every = !ct.touched && v.ix.listed;
    GradFill gf;
    if (!every) {
        gf.p = grad_arc_score;
        gf.n = f->A;
        gf.blocks = (int)std::min<int64_t>(f->cu_count, (f->A + 1023) / 1024);
    }
    const BatchView bv = make_view(f, B, N, t->offsets, t->tokens, nullptr, nullptr, nullptr, t->status);
    LiveWork w;
    w.order = t->order;
    TapeView tp = tape_view(t);
    if (t->left || t->reserved) {
        TRY(ensure_t(f->ws[W_BETA], t->total, s, &tp.beta));
        TRY(ensure_t(f->ws[W_BMAX], N, s, &tp.b_max));
        TRY(ensure_t(f->ws[W_BLOG], N, s, &tp.b_log));
        TRY(ensure_t(f->ws[W_LZB], B, s, &tp.log_z_bwd));
    }
    if (t->reserved) {
        RestGroups rg;
        int rc = WFST_OK;
        if (rest_tile(f)) {
            rc = rest_groups(f, s, bv, cnt, rg, true);
        } else {
            unsigned long long *slot;
            TRY(ensure_zeroed(f->ws[W_LSLOT], f->rev.n_elem, s, &slot));
            DISPATCH_NT(rc, f->nt, launch_backward, f, s, bv, tp, BlockView(), RecordSink(), true)
        }
        if (rc != WFST_OK) return rc;
    }
    {
        ProfScope prof(f, s, WFST_KERNEL_BACKWARD);
        if (v.narrow) {
            NarrowView nv = narrow_view(f);
            nv.prep = reinterpret_cast<const int2 *>(t->bufs->l_tok.p);
            HotView hot;
            HotPlan plan;
            if (narrow_hot_plan(f, B, N, plan)) {
                hot.label = reinterpret_cast<const HotLabel *>(t->bufs->l_state.p);  // picked by the forward pass
                hot.n = reinterpret_cast<const int32_t *>(hot.label + kHotMax);
                hot.cells = plan.cells;
                if (plan.lds > 65536) {  // (of the one kernel that is launched)
                    const hipError_t e = by_listed(v, [&](auto listed) {
                        constexpr bool L = decltype(listed)::value;
                        const void *k = v.narrow == 8 ? (v.narrow_arcs == 2 ? (const void *)narrow_backward_hot<8, 2, L>
                                                                            : (const void *)narrow_backward_hot<8, 4, L>)
                                                      : (v.narrow_arcs == 2 ? (const void *)narrow_backward_hot<16, 2, L>
                                                                            : (const void *)narrow_backward_hot<16, 4, L>);
                        return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)plan.lds);
                    });
                    HIP_OK(e);
                }
            }
            if (hot.n)
                NARROW_LAUNCH(narrow_backward_hot, v, plan.grid + gf.blocks, plan.nt, plan.lds, s, v.ix, nv, f->start, (const float *)f->final_score, bv,
                              (const int32_t *)t->order, (const double *)t->lists.val, (const int32_t *)t->lists.done,
                              (const double *)t->lists.log_z, ct, gf, hot);
            else
                NARROW_LAUNCH(narrow_backward_cold, v, plan.grid + gf.blocks, plan.nt, plan.lds, s, v.ix, nv, f->start, (const float *)f->final_score, bv,
                              (const int32_t *)t->order, (const double *)t->lists.val, (const int32_t *)t->lists.done,
                              (const double *)t->lists.log_z, ct, gf, hot);
        } else {
            LIVE_LAUNCH(live_backward, v, grid + gf.blocks, lds, s, v.ix, v.sh, f->Q, f->start, (const float *)f->final_score,
                        bv, w, t->lists, ct, gf);
        }
        if (t->wide) {
            int wgrid = 0;
            unsigned char *scratch = nullptr;
            TRY(live_wide_grid(f, s, B, &wgrid, &scratch));
            if (!t->direct) {
                w.order = reinterpret_cast<const int32_t *>(t->bufs->l_left.p);
                w.n = cnt + L_LEFT;
            }
            by_listed(v, [&](auto listed) {
                hipLaunchKernelGGL((live_backward_wide<kLiveGroupThreads, decltype(listed)::value>), dim3(wgrid),
                                   dim3(kLiveGroupThreads), 0, s, v.ix,
                               f->Q, f->start, (const float *)f->final_score, bv, w, t->lists, ct, scratch);
            });
        }
        if (t->left) {  // the streaming sweep adds to the same accumulators
            BatchView rv = bv;
            rv.order = t->left;
            rv.n = t->n_left;
            rv.tok_off = t->tok_off;
            rv.queue = cnt + L_QUEUE3;
            int rc;
            if (int tile = rest_tile(f)) {
                RestGroups rg;
                TRY(rest_groups(f, s, rv, cnt, rg));
                DISPATCH_NT(rc, f->nt, launch_rest_backward, f, s, rv, tp, rg, ct)
                if (rc != WFST_OK) return rc;
                if (tile == 4) TRY(launch_rest_counts<4>(f, s, rv, tp, rg, ct));
                if (tile == 2) TRY(launch_rest_counts<2>(f, s, rv, tp, rg, ct));
                if (tile == 1) TRY(launch_rest_counts<1>(f, s, rv, tp, rg, ct));
            } else {
                if (grad_final)
                    hipLaunchKernelGGL(rest_final, dim3(grid_for(B, 1, 1024)), dim3(64), 0, s, rv, tp, f->fwd,
                                       f->start, (const float *)f->final_score, ct);
                TRY(slot_counts(f, s, ct, rv.n, [&](const RecordSink &rs) -> int {
                    DISPATCH_NT(rc, f->nt, launch_backward, f, s, rv, tp, BlockView(), rs)
                    return rc;
                }));
            }
        }
    }
    if (t->rest) {
        float *g = nullptr;
        if (grad_log_z && t->rest_list) {
            g = reinterpret_cast<float *>(t->bufs->l_out.p) + 2 * (int64_t)t->n_rest;
            hipLaunchKernelGGL(live_pick, dim3(grid_for(t->n_rest, 256)), dim3(256), 0, s, t->rest_list, t->n_rest,
                               grad_log_z, g);
        }
        LiveCounts into = ct;
        into.grad_log_z = t->rest_list ? g : grad_log_z;
        TRY(backward_dense(f, t->rest, into.grad_log_z, nullptr, nullptr, s, &into));
    }
    {
        ProfScope prof(f, s, WFST_KERNEL_COUNTS);
        hipLaunchKernelGGL(live_counts_to_grad, dim3(grid_for(ct.touched ? ct.touched_cap : f->A, 256, 4096)),
                           dim3(256), 0, s, ct, v.ix, f->A, every,
                           t->n_left ? t->n_left : (const int32_t *)(cnt + L_QUEUE3), grad_arc_score, f->Q, grad_final);
    }
    HIP_OK(hipGetLastError());
    hold.done();
    return WFST_OK;
}

// The backward pass of a live tape by the streaming sweeps: their forward pass
// first (into scratch outputs), whose tape they read.  Synchronises the stream.
int backward_again(wfst_fst *f, const wfst_tape *t, const float *grad_log_z, float *grad_arc_score, float *grad_final,
                   hipStream_t s)
{
    Buf out;
    float *log_z;
    wfst_tape *d = nullptr;
    int rc = ensure_t(out, 2 * (int64_t)t->B, s, &log_z);
    if (rc == WFST_OK)
        rc = guarded([&]() -> int {
            TRY(forward_dense(f, t->B, t->N, t->offsets, t->tokens, log_z, reinterpret_cast<int32_t *>(log_z + t->B), &d,
                              s));
            return backward_dense(f, d, grad_log_z, grad_arc_score, grad_final, s);
        });
    wfst_tape_free(d);
    if (hipStreamSynchronize(s) != hipSuccess && rc == WFST_OK) rc = set_err(WFST_EHIP, "hipStreamSynchronize");
    free_buf(out);
    return rc;
}

// What a graph refuses (its bounds and options are those of the streaming sweeps, whichever sweeps it captures).
int graph_limits(const wfst_fst *f, int64_t N, int64_t cap, bool tape)
{
    const int64_t bound = N * (int64_t)std::max(f->fwd.max_segs, 1);
    if (bound > cap)
        return set_err(WFST_EUNSUPPORTED, "a graph sizes its buffers by the bound tokens x largest label (" +
                                              std::to_string(bound) + " entries), which exceeds " +
                                              std::to_string(cap) + "; use a smaller batch");
    if (tape && N > 0 && f->ckpt_mode != 2 &&
        (f->ckpt_mode == 1 || 2 * (int64_t)sizeof(float) * bound > f->tape_budget))
        return set_err(WFST_EUNSUPPORTED, "a graph keeps the whole forward tape (checkpointing plans from "
                                          "device totals); its bound exceeds the tape budget or checkpointing "
                                          "is forced");
    return WFST_OK;
}

}  // namespace

// Scratch of wfst_viterbi_noalloc: one array per GPU, held until the process
// ends; every call on a GPU reuses (and overwrites) that GPU's copy.  Host
// code never passes the array's name to a kernel: it is only a host-side
// stand-in; the device address comes from hipGetSymbolAddress, per device.
constexpr size_t kStaticScratchBytes = (size_t)256 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {

std::mutex g_scratch_mu;
std::vector<unsigned char *> g_scratch_ptr;  // device address of `scratch`, per device (null: not looked up)

// The current device's address of `scratch` (looked up once per device, with
// that device current).
int static_scratch(int dev, unsigned char **out)
{
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if ((int)g_scratch_ptr.size() <= dev) g_scratch_ptr.resize((size_t)dev + 1, nullptr);
    if (!g_scratch_ptr[(size_t)dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return set_err(WFST_EHIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        g_scratch_ptr[(size_t)dev] = static_cast<unsigned char *>(p);
    }
    *out = g_scratch_ptr[(size_t)dev];
    return WFST_OK;
}

// Count path of later calls: 0 records (with fallbacks), -1 label-grouped
// kernel, -2 fixed-point accumulation.
void set_count_mode(wfst_fst *f, int32_t mode)
{
    f->rec_off = mode < 0;
    f->fx_counts = mode == -2;
}

int32_t count_mode(const wfst_fst *f) { return f->fx_counts ? -2 : (f->rec_off ? -1 : 0); }

// The FST's arcs in id order (label, source, destination, current score),
// read back from the forward layout: its slot (row r, lane l) of slice s
// holds chunk s*64 + l of its label, whose segment's key is the destination.
// Synchronises the stream.
int read_arcs(wfst_fst *f, hipStream_t s, std::vector<int32_t> &src, std::vector<int32_t> &dst,
              std::vector<int32_t> &ilabel, std::vector<float> &sc)
{
    const DevLayout &d = f->fwd;
    TRY(refresh_layouts(f, s, nullptr));
    HIP_OK(hipStreamSynchronize(s));
    std::vector<int32_t> other((size_t)d.n_elem), earc((size_t)d.n_elem), seg_key((size_t)d.n_seg);
    std::vector<float> score((size_t)d.n_elem);
    std::vector<SliceInfo> slice((size_t)d.n_slice);
    std::vector<SegChunk> seg_chunk((size_t)d.n_seg);
    std::vector<LabelInfo> label((size_t)f->M);
    HIP_OK(hipMemcpy(other.data(), d.other, other.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
    HIP_OK(hipMemcpy(earc.data(), d.elem_arc, earc.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
    HIP_OK(hipMemcpy(score.data(), d.score, score.size() * sizeof(float), hipMemcpyDeviceToHost));
    HIP_OK(hipMemcpy(seg_key.data(), d.seg_key, seg_key.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
    HIP_OK(hipMemcpy(slice.data(), d.slice, slice.size() * sizeof(SliceInfo), hipMemcpyDeviceToHost));
    HIP_OK(hipMemcpy(seg_chunk.data(), d.seg_chunk, seg_chunk.size() * sizeof(SegChunk), hipMemcpyDeviceToHost));
    HIP_OK(hipMemcpy(label.data(), d.label, label.size() * sizeof(LabelInfo), hipMemcpyDeviceToHost));
    src.assign((size_t)f->A, 0);
    dst.assign((size_t)f->A, 0);
    ilabel.assign((size_t)f->A, 0);
    sc.assign((size_t)f->A, 0.0f);
    std::vector<int32_t> chunk_seg;
    for (int32_t a = 0; a < f->M; ++a) {
        const LabelInfo &li = label[(size_t)a];
        chunk_seg.assign((size_t)std::max(li.n_slots, 1), 0);
        for (int32_t j = 0; j < li.n_multi; ++j) {
            const SegChunk &c = seg_chunk[(size_t)(li.seg_first + j)];
            for (int32_t p = 0; p < c.count; ++p) chunk_seg[(size_t)(c.first + p)] = j;
        }
        for (int32_t sl = 0; sl < li.n_slices; ++sl) {
            const SliceInfo &si = slice[(size_t)(li.slice_first + sl)];
            for (int32_t l = 0; l < si.width; ++l) {
                const int32_t c = sl * 64 + l;
                const int32_t j = c < li.n_slots ? chunk_seg[(size_t)c] : li.n_multi + (c - li.n_slots);
                const int32_t key = seg_key[(size_t)(li.seg_first + j)];
                for (int32_t r = 0; r < si.height; ++r) {
                    const int64_t e = (int64_t)si.base + (int64_t)r * si.width + l;
                    const int32_t k = earc[(size_t)e];
                    if (k < 0) continue;
                    src[(size_t)k] = other[(size_t)e];
                    dst[(size_t)k] = key;
                    ilabel[(size_t)k] = a;
                    sc[(size_t)k] = score[(size_t)e];
                }
            }
        }
    }
    return WFST_OK;
}

// Rebuild both layouts with another chunk length from the arcs read back
// from the forward layout (with their current scores), so the FST keeps no
// host copy of its arcs.  Synchronises the stream.
int rebuild_layouts(wfst_fst *f, int32_t chunk, hipStream_t s)
{
    if (chunk == f->chunk) return WFST_OK;
    if (chunk < 1 || chunk > 64) return set_err(WFST_EINVAL, "chunk_arcs must be in [1, 64]");
    if (f->live_graphs > 0)
        return set_err(WFST_EINVAL, "the FST has graphs that point at its layouts; destroy them before a rebuild");
    std::vector<int32_t> src, dst, ilabel;
    std::vector<float> sc;
    TRY(read_arcs(f, s, src, dst, ilabel, sc));
    std::string err;
    HostLayout hf, hr;
    int rc = build_layout(f->Q, f->M, f->A, src.data(), dst.data(), ilabel.data(), sc.data(), 0, chunk, hf, err);
    if (rc == WFST_OK)
        rc = build_layout(f->Q, f->M, f->A, src.data(), dst.data(), ilabel.data(), sc.data(), 1, chunk, hr, err);
    if (rc != WFST_OK) return set_err(rc, err);
    free_layout(f, f->fwd);
    free_layout(f, f->rev);
    TRY(upload_layout(f, hf, f->fwd, s));
    TRY(upload_layout(f, hr, f->rev, s));
    TRY(build_elem_locs(f, s));
    TRY(build_live(f, s));
    HIP_OK(hipStreamSynchronize(s));
    f->chunk = chunk;
    f->score_version += 1;  // tapes made on the old layouts are not used again
    return WFST_OK;
}

// By-source index of the arcs for the EM M-step (built once per FST): arc
// ids grouped by source state (increasing id inside a state), the group
// starts, and each arc's source.
int ensure_source_index(wfst_fst *f, hipStream_t s)
{
    if (f->em_src) return WFST_OK;
    std::vector<int32_t> src, dst, ilabel;
    std::vector<float> sc;
    TRY(read_arcs(f, s, src, dst, ilabel, sc));
    std::vector<int64_t> start((size_t)f->Q + 1, 0);
    for (int64_t k = 0; k < f->A; ++k) start[(size_t)src[(size_t)k] + 1] += 1;
    for (int32_t q = 0; q < f->Q; ++q) start[(size_t)q + 1] += start[(size_t)q];
    std::vector<int64_t> fill(start.begin(), start.end() - 1);
    std::vector<int32_t> order((size_t)std::max<int64_t>(f->A, 1));
    for (int64_t k = 0; k < f->A; ++k) order[(size_t)fill[(size_t)src[(size_t)k]]++] = (int32_t)k;
    TRY(dev_upload(f, &f->em_order, order.data(), f->A, s));
    // segments of every state, by segment number first (segment i of all states that have one)
    std::vector<int64_t> seg((size_t)f->Q + 1, 0);
    for (int32_t q = 0; q < f->Q; ++q)
        seg[(size_t)q + 1] = seg[(size_t)q] + (start[(size_t)q + 1] - start[(size_t)q] + kEmSegment - 1) / kEmSegment;
    std::vector<EmItem> item;
    item.reserve((size_t)seg[(size_t)f->Q]);
    std::vector<int32_t> live;
    for (int32_t q = 0; q < f->Q; ++q)
        if (seg[(size_t)q + 1] > seg[(size_t)q]) live.push_back(q);
    for (int64_t i = 0; !live.empty(); ++i) {
        size_t keep = 0;
        for (int32_t q : live) {
            const int64_t lo = start[(size_t)q] + i * kEmSegment;
            item.push_back(EmItem{lo, std::min<int64_t>(lo + kEmSegment, start[(size_t)q + 1]), seg[(size_t)q] + i});
            if (seg[(size_t)q] + i + 1 < seg[(size_t)q + 1]) live[keep++] = q;
        }
        live.resize(keep);
    }
    f->em_items = (int64_t)item.size();
    TRY(dev_upload(f, &f->em_item, item.data(), f->em_items, s));
    TRY(dev_upload(f, &f->em_seg, seg.data(), (int64_t)seg.size(), s));
    TRY(dev_upload(f, &f->em_src, src.data(), f->A, s));
    HIP_OK(hipStreamSynchronize(s));
    return WFST_OK;
}

// Autotune cache: one JSON object, one entry per line,
//   "key": {"threads_per_sentence": 64, "count_records": -2, "chunk_arcs": 16, "ms": 4.5},
struct TuneEntry {
    int32_t nt = 0, mode = 0, chunk = 0;
    float ms = -1.0f;
};

std::vector<std::pair<std::string, TuneEntry>> read_tune_cache(const char *path)
{
    std::vector<std::pair<std::string, TuneEntry>> out;
    std::ifstream in(path);
    std::string line;
    while (std::getline(in, line)) {
        const size_t q0 = line.find('"');
        if (q0 == std::string::npos) continue;
        const size_t q1 = line.find('"', q0 + 1);
        if (q1 == std::string::npos) continue;
        TuneEntry e;
        if (std::sscanf(line.c_str() + q1 + 1,
                        ": {\"threads_per_sentence\": %d, \"count_records\": %d, \"chunk_arcs\": %d, \"ms\": %f",
                        &e.nt, &e.mode, &e.chunk, &e.ms) == 4)
            out.emplace_back(line.substr(q0 + 1, q1 - q0 - 1), e);
    }
    return out;
}

int write_tune_cache(const char *path, const std::vector<std::pair<std::string, TuneEntry>> &entries)
{
    const std::string tmp = std::string(path) + ".tmp";
    {
        std::ofstream o(tmp, std::ios::trunc);
        if (!o) return set_err(WFST_EINVAL, std::string("can not write the autotune cache ") + path);
        o << "{\n";
        for (size_t i = 0; i < entries.size(); ++i) {
            const TuneEntry &e = entries[i].second;
            char buf[160];
            std::snprintf(buf, sizeof(buf),
                          ": {\"threads_per_sentence\": %d, \"count_records\": %d, \"chunk_arcs\": %d, \"ms\": %.4f}",
                          e.nt, e.mode, e.chunk, e.ms);
            o << "\"" << entries[i].first << "\"" << buf << (i + 1 < entries.size() ? ",\n" : "\n");
        }
        o << "}\n";
        if (!o) return set_err(WFST_EINVAL, std::string("can not write the autotune cache ") + path);
    }
    if (std::rename(tmp.c_str(), path) != 0)
        return set_err(WFST_EINVAL, std::string("can not replace the autotune cache ") + path);
    return WFST_OK;
}

// Cache key: device architecture, FST shape and the batch's shape (sentences,
// tokens, mean arcs per token, log2 histogram of sentence lengths).
int tune_key(const wfst_fst *f, int32_t B, int64_t N, const int32_t *offsets, const int32_t *tokens,
             int32_t flags, hipStream_t s, std::string &key)
{
    std::vector<int32_t> off((size_t)B + 1), tok((size_t)std::max<int64_t>(N, 1));
    HIP_OK(hipStreamSynchronize(s));
    HIP_OK(hipMemcpy(off.data(), offsets, off.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
    if (N > 0) HIP_OK(hipMemcpy(tok.data(), tokens, (size_t)N * sizeof(int32_t), hipMemcpyDeviceToHost));
    int hist[12] = {0};
    for (int32_t b = 0; b < B; ++b) {
        const int32_t T = off[(size_t)b + 1] - off[(size_t)b];
        int k = 0;
        while (k < 11 && (1 << k) <= T) ++k;
        hist[k] += 1;
    }
    double arcs = 0.0;
    for (int64_t i = 0; i < N; ++i) {
        const int32_t a = tok[(size_t)i];
        if (a >= 0 && a < f->M) arcs += f->label_arcs[(size_t)a];
    }
    hipDeviceProp_t prop;
    HIP_OK(hipGetDeviceProperties(&prop, f->device));
    std::ostringstream k;
    k << prop.gcnArchName << " Q=" << f->Q << " M=" << f->M << " A=" << f->A << " B=" << B << " N=" << N
      << " Aw=" << (int64_t)std::llround(N > 0 ? arcs / (double)N : 0.0) << " len=";
    for (int i = 0; i < 12; ++i) k << (i ? "," : "") << hist[i];
    k << " chunks=" << ((flags & WFST_TUNE_CHUNK) ? "tuned" : std::to_string(f->chunk));
    if (f->live.on) k << " live";  // (choices made where every sentence streams do not carry over)
    key = k.str();
    for (char &c : key)
        if (c == '"' || c == '\\') c = '_';
    return WFST_OK;
}

// The streaming sweeps over a whole batch.
int viterbi_dense(wfst_fst *f, int32_t batch, int64_t N, const int32_t *offsets, const int32_t *tokens,
                  float *best_score, int32_t *best_arcs, int32_t *best_olabels, int32_t *status, hipStream_t s)
{
    TRY(refresh_layouts(f, s, nullptr));
    int32_t *order, *counters, *path_tmp;
    int64_t *tok_off, *tiles;
    TRY(ensure_t(f->ws[W_ORDER], batch, s, &order));
    TRY(ensure_t(f->ws[W_TOKOFF], N, s, &tok_off));
    TRY(ensure_t(f->ws[W_TILES], scan_tiles_for(N), s, &tiles));
    TRY(ensure_t(f->ws[W_COUNTERS], C_COUNT, s, &counters));
    TRY(ensure_t(f->ws[W_PATH], N, s, &path_tmp));
    int64_t *dev_total = reinterpret_cast<int64_t *>(counters + C_TOTAL);
    Plan p;
    TRY(make_plan(f, s, batch, N, offsets, tokens, order, tok_off, tiles, dev_total, kBoundCapBytes / 8, p));
    int2 *bp;
    TRY(ensure_t(f->ws[W_BP], p.total, s, &bp));
    hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, counters + C_QUEUE, (int64_t)1, 0);
    const BatchView bv = make_view(f, batch, N, offsets, tokens, order, tok_off, counters + C_QUEUE, status);
    int rc;
    DISPATCH_NT(rc, f->nt, launch_viterbi, f, s, bv, bp, path_tmp, best_score, best_arcs, best_olabels)
    return rc;
}

wfst_tape *new_tape(wfst_fst *f, int32_t batch, int64_t N, const int32_t *offsets, const int32_t *tokens,
                    int32_t *status)
{
    TapeBufs *tb;
    if (!f->tape_pool.empty()) {
        tb = f->tape_pool.back();
        f->tape_pool.pop_back();
    } else {
        tb = new TapeBufs();
        if (!f->graph_mode)
            for (Buf *b : tb->all()) b->limit = &f->alloc_limit;
    }
    wfst_tape *t = new wfst_tape();
    t->fst = f;
    t->score_version = f->score_version;
    t->B = batch;
    t->N = N;
    t->offsets = offsets;
    t->tokens = tokens;
    t->status = status;
    t->bufs = tb;
    return t;
}

int forward_dense(wfst_fst *f, int32_t batch, int64_t N, const int32_t *offsets, const int32_t *tokens, float *log_z,
                  int32_t *status, wfst_tape **tape_out, hipStream_t s)
{
    TRY(refresh_layouts(f, s, nullptr));
    wfst_tape *t = new_tape(f, batch, N, offsets, tokens, status);
    TapeBufs *tb = t->bufs;
    int rc = WFST_OK;
    if (batch > 0) {
        int32_t *counters;
        int64_t *tiles, *dev_total;
        rc = ensure_t(tb->order, batch, s, &t->order);
        if (rc == WFST_OK) rc = ensure_t(tb->tok_off, N, s, &t->tok_off);
        if (rc == WFST_OK) rc = ensure_t(tb->tiles, scan_tiles_for(std::max<int64_t>(N, batch)), s, &tiles);
        if (rc == WFST_OK) rc = ensure_t(tb->total, 2, s, &dev_total);
        if (rc == WFST_OK) rc = ensure_t(f->ws[W_COUNTERS], C_COUNT, s, &counters);
        Plan p;
        if (rc == WFST_OK)
            rc = make_plan(f, s, batch, N, offsets, tokens, t->order, t->tok_off, tiles, dev_total,
                           kBoundCapBytes / 4, p);
        int64_t alpha_elems = p.total;
        if (rc == WFST_OK) {
            t->total = p.total;
            rc = plan_checkpoints(f, s, t, tiles, dev_total, p, &alpha_elems);
        }
        if (rc == WFST_OK) rc = ensure_t(tb->alpha, std::max<int64_t>(alpha_elems, 1), s, &t->alpha);
        if (rc == WFST_OK) rc = ensure_t(tb->a_max, N, s, &t->a_max);
        if (rc == WFST_OK) rc = ensure_t(tb->a_log, N, s, &t->a_log);
        if (rc == WFST_OK) rc = ensure_t(tb->log_z, batch, s, &t->log_z);
        if (rc == WFST_OK) {
            hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, counters + C_QUEUE, (int64_t)1, 0);
            const BatchView bv =
                make_view(f, batch, N, offsets, tokens, t->order, t->tok_off, counters + C_QUEUE, status);
            const TapeView tp = tape_view(t);
            DISPATCH_NT(rc, f->nt, launch_forward, f, s, bv, tp, BlockView(), log_z)
        }
    }
    if (rc != WFST_OK) {
        wfst_tape_free(t);
        return rc;
    }
    *tape_out = t;
    return WFST_OK;
}

// The streaming sweeps' backward pass.  With `into` its expected counts (and
// final-state posteriors) are added to those fixed-point sums, and no gradient is written.
int backward_dense(wfst_fst *f, const wfst_tape *tape, const float *grad_log_z, float *grad_arc_score,
                   float *grad_final, hipStream_t s, const LiveCounts *into)
{
    if (grad_final) TRY(final_posteriors(f, tape, grad_log_z, grad_final, s));
    const int32_t B = tape->B;
    const int64_t N = tape->N;
    // expected counts by fixed-point accumulation in the backward sweep: asked
    // for, or forced by a backward state too large for LDS
    // (a graph takes fixed-point counts where the records would need a read-back)
    const bool fx = f->A > 0 && B > 0 && N > 0 &&
                    (into || f->fx_counts || backward_in_gmem(f) || (f->graph_mode && !f->rec_off));
    // on the record path the backward sweep zero-fills the gradient itself
    // (bandwidth it leaves unused); else one fill kernel first
    const bool fill_in_sweep = f->A > 0 && !fx && !f->rec_off && B > 0 && N > 0 &&
                               ((uintptr_t)grad_arc_score & 15) == 0;
    if (f->A > 0 && !fx && !fill_in_sweep) {
        ProfScope prof(f, s, WFST_KERNEL_GRAD_FILL);
        hipLaunchKernelGGL(fill_f32, dim3(grid_for(f->A, 256, 8192)), dim3(256), 0, s, grad_arc_score, f->A, 0.0f);
    }
    if (B == 0 || N == 0) {
        HIP_OK(hipGetLastError());
        return WFST_OK;
    }
    TapeView tp = tape_view(tape);
    if (into && into->fin) {
        const BatchView v = make_view(f, B, N, tape->offsets, tape->tokens, nullptr, tape->tok_off, nullptr, tape->status);
        hipLaunchKernelGGL(rest_final, dim3(grid_for(B, 1, 1024)), dim3(64), 0, s, v, tp, f->fwd, f->start,
                           (const float *)f->final_score, *into);
    }
    const int32_t K = tape->ck_c > 0 ? tape->ck_K : 1;
    BlockView bk;  // c = 0: the whole tape is resident
    int32_t *counters;
    if (tape->ck_c > 0) {
        bk.c = tape->ck_c;
        bk.base = tape->blk_base;
        const int64_t nb = std::max<int64_t>(tape->blk_total, 1);
        TRY(ensure_t(f->ws[W_ABUF0], nb, s, &bk.abuf[0]));
        TRY(ensure_t(f->ws[W_ABUF1], nb, s, &bk.abuf[1]));
        TRY(ensure_t(f->ws[W_BBUF0], nb, s, &bk.bbuf[0]));
        TRY(ensure_t(f->ws[W_BBUF1], nb, s, &bk.bbuf[1]));
    } else {
        TRY(ensure_t(f->ws[W_BETA], tape->total, s, &tp.beta));
    }
    TRY(ensure_t(f->ws[W_BMAX], N, s, &tp.b_max));
    TRY(ensure_t(f->ws[W_BLOG], N, s, &tp.b_log));
    TRY(ensure_t(f->ws[W_LZB], B, s, &tp.log_z_bwd));
    TRY(ensure_t(f->ws[W_COUNTERS], C_COUNT, s, &counters));
    hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, counters, (int64_t)C_COUNT, 0);
    const BatchView bv = make_view(f, B, N, tape->offsets, tape->tokens, tape->order, tape->tok_off,
                                   counters + C_QUEUE, tape->status);
    int rc;
    // Expected counts as records of the backward pass (sorted and summed per
    // arc) when there are at most rec_max of them; otherwise the grouped count
    // kernel below.  The choice depends only on the number of records; when
    // their slots (records plus unused chunk tails) overflow the buffer, the
    // buffer grows and the pass runs again.
    auto backward_pass = [&](const RecordSink &sink) -> int {
        int r = WFST_OK;
        if (bk.c == 0) {
            DISPATCH_NT(r, f->nt, launch_backward, f, s, bv, tp, bk, sink)
            return r;
        }
        for (int32_t k = K - 1; k >= 0; --k) {  // blocks from the end: recompute alpha~, then beta
            bk.k = k;
            hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, counters + C_QUEUE, (int64_t)1, 0);
            DISPATCH_NT(r, f->nt, launch_forward, f, s, bv, tp, bk, nullptr)
            if (r != WFST_OK) return r;
            hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, counters + C_QUEUE, (int64_t)1, 0);
            RecordSink sk = sink;
            if (k != K - 1) sk.fill = nullptr;  // the first launch zero-fills the gradient
            DISPATCH_NT(r, f->nt, launch_backward, f, s, bv, tp, bk, sk)
            if (r != WFST_OK) return r;
        }
        return WFST_OK;
    };
    // Fixed-point counts: each posterior is added to its arc's 64-bit integer
    // accumulator (indexed by the arc's reverse-layout slot) during the
    // backward sweep; one conversion pass writes the gradient.  Integer sums do
    // not depend on the order of the additions.
    auto fixed_point_counts = [&]() -> int {
        if (into) return slot_counts(f, s, *into, nullptr, backward_pass);
        unsigned long long *acc;
        double *scale;
        const int64_t n_slots = f->rev.n_elem;
        TRY(ensure_t(f->ws[W_FXACC], n_slots, s, &acc));
        TRY(ensure_t(f->ws[W_FXSCALE], 1, s, &scale));
        {
            ProfScope prof(f, s, WFST_KERNEL_GRAD_FILL);
            hipLaunchKernelGGL(fill_i64, dim3(grid_for(n_slots, 256, 8192)), dim3(256), 0, s,
                               reinterpret_cast<int64_t *>(acc), n_slots, (int64_t)0);
        }
        hipLaunchKernelGGL(fx_scale_kernel, dim3(1), dim3(256), 0, s, grad_log_z, B, N, scale);
        hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, counters, (int64_t)C_COUNT, 0);
        RecordSink rs;
        rs.acc = acc;
        rs.fx_scale = scale;
        rs.grad_log_z = grad_log_z;
        TRY(backward_pass(rs));
        {
            ProfScope prof(f, s, WFST_KERNEL_COUNTS);
            hipLaunchKernelGGL(fx_to_grad, dim3(grid_for(n_slots, 256, 8192)), dim3(256), 0, s,
                               (const unsigned long long *)acc, (const int32_t *)f->rev.elem_arc, n_slots,
                               (const double *)scale, grad_arc_score);
        }
        HIP_OK(hipGetLastError());
        return WFST_OK;
    };
    if (fx) return fixed_point_counts();
    bool beta_done = false;  // the beta tape of the resident-tape pass is written
    if (f->A > 0 && !f->rec_off) {
        RecordSink rs;
        rs.count = reinterpret_cast<unsigned long long *>(counters + C_RECS);
        rs.total = reinterpret_cast<unsigned long long *>(counters + C_RTOTAL);
        rs.grad_log_z = grad_log_z;
        if (fill_in_sweep) {
            rs.fill = grad_arc_score;
            rs.fill_n = f->A;
        }
        int64_t cap = std::min(kRecordsMax, f->rec_cap > 0 ? f->rec_cap : 16 * N + 4096);
        for (int attempt = 0; attempt < 2; ++attempt) {
            TRY(ensure_t(f->ws[W_RKEY0], cap, s, &rs.key));
            TRY(ensure_t(f->ws[W_RVAL0], cap, s, &rs.val));
            rs.cap = cap;
            if (attempt > 0) hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, counters, (int64_t)C_COUNT, 0);
            TRY(backward_pass(rs));
            beta_done = true;
            unsigned long long got[2] = {0, 0};  // slots, records
            HIP_OK(hipMemcpyAsync(got, rs.count, sizeof(got), hipMemcpyDeviceToHost, s));
            HIP_OK(hipStreamSynchronize(s));
            if ((int64_t)got[1] > f->rec_max) {  // too many records: grouped count kernel, or fixed point
                if (lds_counts(f) > f->max_lds) return fixed_point_counts();
                break;
            }
            if ((int64_t)got[0] <= cap) {
                ProfScope prof(f, s, WFST_KERNEL_COUNTS);
                uint64_t *k1;
                float *v1;
                TRY(ensure_t(f->ws[W_RKEY1], std::max<int64_t>((int64_t)got[0], 1), s, &k1));
                TRY(ensure_t(f->ws[W_RVAL1], std::max<int64_t>((int64_t)got[0], 1), s, &v1));
                return reduce_records(f, s, (int64_t)got[0], N, rs.key, rs.val, k1, v1, grad_arc_score, grad_log_z, B);
            }
            // slots overflowed: grow to a bound no schedule can pass and run again.  A
            // chunk holds kRecChunk slots and is left with a tail under kRecStage;
            // there are at most records / kRecChunk chunks plus one per workgroup
            // and launch.
            const int64_t launches = bk.c > 0 ? K : 1;
            cap = 3 * (int64_t)got[1] + (int64_t)kRecStage * B * launches + 4096;
            f->rec_cap = std::max<int64_t>(f->rec_cap, std::min(kRecordsMax, (int64_t)got[0] + (int64_t)got[0] / 4));
        }
        // the grouped count kernel needs the beta tape of a pass without records
        hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, counters, (int64_t)C_COUNT, 0);
    }
    if (bk.c == 0 && !beta_done) TRY(backward_pass(RecordSink()));
    RecordSink no_records;

    // group the visits (token positions) by (input label, checkpoint block), stable in position
    const int32_t V = 64;
    const int32_t MK = f->M * K;
    int32_t *tok_sent, *visits, *skeys, *grp_lo, *grp_n, *nip, *item_base, *item_slot;
    TRY(ensure_t(f->ws[W_TOKSENT], N, s, &tok_sent));
    TRY(sort_visits(f, s, N, tape->tokens, tape->offsets, B, tape->ck_c, K, &visits, &skeys, tok_sent));
    TRY(ensure_t(f->ws[W_GRPLO], MK, s, &grp_lo));
    TRY(ensure_t(f->ws[W_GRPN], MK, s, &grp_n));
    TRY(ensure_t(f->ws[W_NIP], MK, s, &nip));
    TRY(ensure_t(f->ws[W_ITEMBASE], MK, s, &item_base));
    const int64_t items_bound = N / V + std::min<int64_t>(MK, N) + 1;
    CountItem *items;
    TRY(ensure_t(f->ws[W_ITEMS], items_bound, s, &items));
    TRY(ensure_t(f->ws[W_ITEMSLOT], items_bound, s, &item_slot));
    const int64_t split_bound = 2 * (N / V) + 2;
    float *partial;
    TRY(ensure_t(f->ws[W_PARTIAL], split_bound * (int64_t)std::max(f->rev.max_elems, 1), s, &partial));
    int64_t *tiles;
    TRY(ensure_t(f->ws[W_TILES], scan_tiles_for(std::max<int64_t>(MK, 256 * ((N + kSortTile - 1) / kSortTile))),
                 s, &tiles));
    hipLaunchKernelGGL(label_groups, dim3(grid_for(MK, 256)), dim3(256), 0, s, (const int32_t *)skeys, N, MK, V,
                       grp_lo, grp_n, nip);
    ScanSource src;
    src.i32 = nip;
    TRY(launch_scan<int32_t>(s, src, MK, tiles, item_base, nullptr));
    hipLaunchKernelGGL(label_items, dim3(grid_for(MK, 256)), dim3(256), 0, s, (const int32_t *)grp_lo,
                       (const int32_t *)grp_n, (const int32_t *)nip, (const int32_t *)item_base, MK, K, V, items,
                       counters + C_NITEMS, (int32_t)items_bound, f->health);
    CountCaps caps;
    caps.items_cap = (int32_t)items_bound;
    caps.slot_cap = (int32_t)split_bound;
    caps.V = V;
    int32_t *list = nullptr, *list_off = nullptr;
    if (bk.c > 0) {
        TRY(ensure_t(f->ws[W_ILIST], items_bound, s, &list));
        TRY(ensure_t(f->ws[W_ILOFF], K + 1, s, &list_off));
        hipLaunchKernelGGL(items_by_block, dim3(1), dim3(1024), 2 * K * sizeof(int32_t), s, (const CountItem *)items,
                           (const int32_t *)(counters + C_NITEMS), K, (int32_t)items_bound, list, list_off,
                           f->health);
    }
    VisitInfo *vinfo;
    TRY(ensure_t(f->ws[W_VINFO], N, s, &vinfo));
    // per-visit records read the backward normalisers: built after the beta sweep (of each block)
    auto build_visits = [&]() {
        hipLaunchKernelGGL(visit_table, dim3(grid_for(N, 256)), dim3(256), 0, s, bv, tp, bk,
                           (const int32_t *)visits, (const int32_t *)tok_sent, grad_log_z, vinfo);
    };
    int32_t *split_e;
    int64_t *se_off;
    TRY(ensure_t(f->ws[W_SPLITE], MK, s, &split_e));
    TRY(ensure_t(f->ws[W_SEOFF], MK, s, &se_off));
    int64_t *se_total = reinterpret_cast<int64_t *>(counters + C_SETOTAL);
    const CountLaunch cl{items, counters + C_NITEMS, list, list_off, counters + C_ITEMQ, items_bound, vinfo,
                         grad_arc_score, partial, item_slot, counters + C_SLOTS, caps};
    // one block of steps (all of them without checkpointing): counts, then the
    // groups split over several items
    auto counts_block = [&](int32_t blk) -> int {
        hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, counters + C_ITEMQ, (int64_t)1, 0);
        TRY(launch_counts(f, s, bv, tp, cl, blk));
        hipLaunchKernelGGL(split_group_elems, dim3(grid_for(MK, 256)), dim3(256), 0, s,
                           (const LabelInfo *)f->rev.label, (const int32_t *)nip, MK, K, bk.c > 0 ? blk : -1,
                           split_e);
        ScanSource ssrc;
        ssrc.i32 = split_e;
        TRY(launch_scan<int64_t>(s, ssrc, MK, tiles, se_off, se_total));
        const int64_t fix_bound = std::min<int64_t>(split_bound, MK) * (int64_t)std::max(f->rev.max_elems, 1);
        hipLaunchKernelGGL((counts_fixup<256>), dim3(grid_for(fix_bound, 256, 16384)), dim3(256), 0, s, f->rev,
                           (const CountItem *)items, (const int32_t *)item_base, (const int32_t *)nip,
                           (const int64_t *)se_off, (const int64_t *)se_total, (const int32_t *)item_slot,
                           (const float *)partial, grad_arc_score, caps, MK, K, f->health);
        return WFST_OK;
    };
    if (bk.c == 0) {
        build_visits();
        TRY(counts_block(0));
    } else {
        for (int32_t k = K - 1; k >= 0; --k) {  // blocks from the end: recompute alpha~, beta sweep, counts
            bk.k = k;
            hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, counters + C_QUEUE, (int64_t)1, 0);
            DISPATCH_NT(rc, f->nt, launch_forward, f, s, bv, tp, bk, nullptr)
            if (rc != WFST_OK) return rc;
            hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, counters + C_QUEUE, (int64_t)1, 0);
            DISPATCH_NT(rc, f->nt, launch_backward, f, s, bv, tp, bk, no_records)
            if (rc != WFST_OK) return rc;
            build_visits();
            TRY(counts_block(k));
        }
    }
    HIP_OK(hipGetLastError());
    return WFST_OK;
}

}  // namespace

extern "C" {

const char *wfst_last_error(void) { return g_err.c_str(); }

int wfst_layout_host(int32_t num_states, int32_t num_ilabels, int64_t num_arcs, const int32_t *src,
                     const int32_t *dst, const int32_t *ilabel, int32_t direction, int32_t chunk_arcs,
                     int64_t *sizes, int32_t *elem_other, int32_t *elem_arc, int32_t *slice_info,
                     int32_t *seg_info, int32_t *label_slice, int32_t *label_seg)
try {
    try {
        if (num_states <= 0 || num_ilabels <= 0 || num_arcs < 0 || num_arcs >= INT32_MAX || !sizes)
            return set_err(WFST_EINVAL, "bad sizes");
        if (num_arcs > 0 && (!src || !dst || !ilabel)) return set_err(WFST_EINVAL, "NULL arc array");
        if (direction != 0 && direction != 1) return set_err(WFST_EINVAL, "direction must be 0 or 1");
        for (int64_t k = 0; k < num_arcs; ++k)
            if (src[k] < 0 || src[k] >= num_states || dst[k] < 0 || dst[k] >= num_states || ilabel[k] < 0 ||
                ilabel[k] >= num_ilabels)
                return set_err(WFST_EINVAL, "arc " + std::to_string(k) + " out of range");
        HostLayout h;
        std::string err;
        const int32_t L = chunk_arcs > 0 ? chunk_arcs : auto_chunk(num_states, num_ilabels, num_arcs);
        int rc = build_layout(num_states, num_ilabels, num_arcs, src, dst, ilabel, nullptr, direction, L, h, err);
        if (rc != WFST_OK) return set_err(rc, err);
        sizes[0] = (int64_t)h.other.size();
        sizes[1] = (int64_t)h.slice.size();
        sizes[2] = (int64_t)h.seg_key.size();
        if (elem_other)
            std::memcpy(elem_other, h.other.data(), h.other.size() * sizeof(int32_t));
        if (elem_arc) std::memcpy(elem_arc, h.elem_arc.data(), h.elem_arc.size() * sizeof(int32_t));
        if (slice_info)
            for (size_t x = 0; x < h.slice.size(); ++x) {
                slice_info[4 * x + 0] = h.slice[x].base;
                slice_info[4 * x + 1] = h.slice[x].height;
                slice_info[4 * x + 2] = h.slice[x].width;
                slice_info[4 * x + 3] = h.slice[x].label;
            }
        if (seg_info || label_slice || label_seg) {
            for (int32_t a = 0; a < num_ilabels; ++a) {
                const LabelInfo &li = h.label[(size_t)a];
                if (label_slice) label_slice[a] = li.slice_first;
                if (label_seg) label_seg[a] = li.seg_first;
                if (seg_info)
                    for (int32_t j = 0; j < li.n_segs; ++j) {
                        const size_t g = (size_t)li.seg_first + j;
                        seg_info[4 * g + 0] = h.seg_key[g];
                        seg_info[4 * g + 1] = h.seg_chunk[g].first;
                        seg_info[4 * g + 2] = h.seg_chunk[g].count;
                        seg_info[4 * g + 3] = a;
                    }
            }
            if (label_slice) label_slice[num_ilabels] = (int32_t)h.slice.size();
            if (label_seg) label_seg[num_ilabels] = (int32_t)h.seg_key.size();
        }
        return WFST_OK;
    } catch (const std::bad_alloc &) {
        return set_err(WFST_ENOMEM, "host allocation failed");
    } catch (const std::exception &e) {
        return set_err(WFST_EINVAL, e.what());
    }
}
C_GUARD

int wfst_fst_create(int32_t num_states, int32_t num_ilabels, int32_t start, int64_t num_arcs,
                    const int32_t *src, const int32_t *dst, const int32_t *ilabel, const int32_t *olabel,
                    const float *arc_score, const float *final_score, const wfst_options *options,
                    void *stream, wfst_fst **out)
try {
    if (!out) return set_err(WFST_EINVAL, "out is NULL");
    *out = nullptr;
    try {
        if (num_states <= 0 || num_states >= INT32_MAX - 1) return set_err(WFST_EINVAL, "num_states out of range");
        if (num_ilabels <= 0) return set_err(WFST_EINVAL, "num_ilabels must be positive");
        if (start < 0 || start >= num_states) return set_err(WFST_EINVAL, "start out of range");
        if (num_arcs < 0 || num_arcs >= INT32_MAX) return set_err(WFST_EUNSUPPORTED, "num_arcs must be < 2^31-1");
        if (num_arcs > 0 && (!src || !dst || !ilabel || !arc_score)) return set_err(WFST_EINVAL, "NULL arc array");
        if (!final_score) return set_err(WFST_EINVAL, "final_score is NULL");
        for (int64_t k = 0; k < num_arcs; ++k) {
            if (src[k] < 0 || src[k] >= num_states || dst[k] < 0 || dst[k] >= num_states)
                return set_err(WFST_EINVAL, "arc " + std::to_string(k) + ": state out of range");
            if (ilabel[k] < 0 || ilabel[k] >= num_ilabels)
                return set_err(WFST_EINVAL, "arc " + std::to_string(k) + ": ilabel out of range");
            if (!std::isfinite(arc_score[k]))
                return set_err(WFST_EINVAL, "arc " + std::to_string(k) + ": score is not finite");
        }
        for (int32_t q = 0; q < num_states; ++q)
            if (std::isnan(final_score[q]) || final_score[q] == INFINITY)
                return set_err(WFST_EINVAL, "final_score[" + std::to_string(q) + "] is NaN or +inf");
        wfst_options opt{};
        if (options) opt = *options;
        int32_t L = opt.chunk_arcs > 0 ? opt.chunk_arcs : auto_chunk(num_states, num_ilabels, num_arcs);
        if (L > 64) return set_err(WFST_EINVAL, "chunk_arcs must be <= 64");
        int nt = opt.threads_per_sentence > 0 ? opt.threads_per_sentence : 256;
        if (nt != 64 && nt != 128 && nt != 256 && nt != 512 && nt != 1024)
            return set_err(WFST_EINVAL, "threads_per_sentence must be 64, 128, 256, 512 or 1024");
        if (opt.checkpoint < -1 || opt.checkpoint > 2) return set_err(WFST_EINVAL, "checkpoint must be -1, 0, 1 or 2");
        if (opt.tape_budget_bytes < 0) return set_err(WFST_EINVAL, "tape_budget_bytes must be >= 0");
        if (opt.count_records < -2) return set_err(WFST_EINVAL, "count_records must be >= -2");
        if (opt.state_memory < 0 || opt.state_memory > 3)
            return set_err(WFST_EINVAL, "state_memory must be 0, 1, 2 or 3");

        hipStream_t s = as_stream(stream);
        wfst_fst *f = new wfst_fst();
        for (Buf &b : f->ws) b.limit = &f->alloc_limit;
        f->Q = num_states;
        f->M = num_ilabels;
        f->start = start;
        f->A = num_arcs;
        f->chunk = L;
        f->nt = nt;
        f->ckpt_mode = opt.checkpoint;
        f->rec_off = opt.count_records < 0;
        f->fx_counts = opt.count_records == -2;
        f->state_mem = opt.state_memory;
        f->rec_max = opt.count_records > 0 ? opt.count_records : kRecordsMax;
        if (opt.tape_budget_bytes > 0) f->tape_budget = opt.tape_budget_bytes;
        if (hipGetDevice(&f->device) != hipSuccess) {
            delete f;
            return set_err(WFST_EHIP, "hipGetDevice failed");
        }
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, f->device) != hipSuccess) {
            delete f;
            return set_err(WFST_EHIP, "hipGetDeviceProperties failed");
        }
        f->cu_count = prop.multiProcessorCount;
        f->max_lds = prop.sharedMemPerBlock;
        f->coop = prop.cooperativeLaunch != 0;
        std::string err;
        int rc;
        {
            HostLayout h;
            rc = build_layout(num_states, num_ilabels, num_arcs, src, dst, ilabel, arc_score, 0, L, h, err);
            if (rc != WFST_OK) rc = set_err(rc, err);
            if (rc == WFST_OK) {
                f->label_arcs.assign((size_t)num_ilabels, 0);
                f->label_fwd_segs.resize((size_t)num_ilabels);
                for (int32_t a = 0; a < num_ilabels; ++a) f->label_fwd_segs[(size_t)a] = h.label[(size_t)a].n_segs;
                for (int64_t k = 0; k < num_arcs; ++k) f->label_arcs[(size_t)ilabel[k]] += 1;
            }
            if (rc == WFST_OK) rc = upload_layout(f, h, f->fwd, s);
            if (rc == WFST_OK && hipStreamSynchronize(s) != hipSuccess) rc = set_err(WFST_EHIP, "upload failed");
        }
        if (rc == WFST_OK) {
            HostLayout h;
            rc = build_layout(num_states, num_ilabels, num_arcs, src, dst, ilabel, arc_score, 1, L, h, err);
            if (rc != WFST_OK) rc = set_err(rc, err);
            if (rc == WFST_OK) {
                f->label_rev_segs.resize((size_t)num_ilabels);
                for (int32_t a = 0; a < num_ilabels; ++a) f->label_rev_segs[(size_t)a] = h.label[(size_t)a].n_segs;
            }
            if (rc == WFST_OK) rc = upload_layout(f, h, f->rev, s);
            if (rc == WFST_OK && hipStreamSynchronize(s) != hipSuccess) rc = set_err(WFST_EHIP, "upload failed");
        }
        if (rc == WFST_OK) rc = dev_upload(f, &f->final_score, final_score, num_states, s);
        if (rc == WFST_OK) rc = dev_upload<float>(f, &f->final_max, nullptr, 1, s);
        if (rc == WFST_OK) rc = dev_upload<uint32_t>(f, &f->health, nullptr, 1, s);
        if (rc == WFST_OK)
            hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, reinterpret_cast<int32_t *>(f->health), (int64_t)1, 0);
        if (rc == WFST_OK && olabel) rc = dev_upload(f, &f->olabel, olabel, num_arcs, s);
        if (rc == WFST_OK) {
            // arc-id range per label; labels with many arcs in a compact range get
            // their score updates staged through LDS
            std::vector<int2> range((size_t)num_ilabels, make_int2(INT32_MAX, -1));
            for (int64_t k = 0; k < num_arcs; ++k) {
                int2 &r = range[(size_t)ilabel[k]];
                r.x = std::min(r.x, (int32_t)k);
                r.y = std::max(r.y, (int32_t)k);
            }
            int64_t staged_arcs = 0;
            for (int32_t a = 0; a < num_ilabels; ++a) {
                const int2 r = range[(size_t)a];
                if (r.y >= r.x && (int64_t)r.y - r.x < kScoreStage) staged_arcs += f->label_arcs[(size_t)a];
            }
            f->stage_scores = num_arcs > 0 && num_arcs / num_ilabels >= 256 && 2 * staged_arcs >= num_arcs;
            rc = dev_upload(f, &f->label_range, range.data(), num_ilabels, s);
            if (rc == WFST_OK) rc = build_elem_locs(f, s);
        }
        if (rc == WFST_OK) {
            hipLaunchKernelGGL(final_max_kernel, dim3(1), dim3(1024), 0, s, (const float *)f->final_score, f->Q,
                               f->final_max);
            if (hipGetLastError() != hipSuccess || hipStreamSynchronize(s) != hipSuccess)
                rc = set_err(WFST_EHIP, "final_max kernel failed");
        }
        if (rc == WFST_OK) rc = build_live(f, s);
        if (rc != WFST_OK) {
            free_fst(f);
            return rc;
        }
        *out = f;
        return WFST_OK;
    } catch (const std::bad_alloc &) {
        return set_err(WFST_ENOMEM, "host allocation failed");
    } catch (const std::exception &e) {
        return set_err(WFST_EINVAL, e.what());
    }
}
C_GUARD

int wfst_fst_set_scores(wfst_fst *f, const float *arc_score_dev, const float *final_score_dev, void *stream)
try {
    if (!f) return set_err(WFST_EINVAL, "fst is NULL");
    hipStream_t s = as_stream(stream);
    if (arc_score_dev || final_score_dev) f->score_version += 1;
    if (arc_score_dev && f->A > 0) {
        ProfScope prof(f, s, WFST_KERNEL_SCORES);
        if (f->live.on) {
            const int32_t wide = (((uintptr_t)arc_score_dev | (uintptr_t)f->live.score) & 15) == 0;
            hipLaunchKernelGGL(live_scores, dim3(grid_for((f->A + 15) / 16, 256, 2048)), dim3(256), 0, s, f->live.score,
                               f->A, arc_score_dev, wide, f->live.stale);
            f->live.dense_stale = true;
            if (f->graph_mode || stream_capturing(s)) f->live.dense_check = true;
        } else {
            TRY(scatter_layouts(f, s, arc_score_dev, ScoreGate()));
        }
    }
    if (final_score_dev) {
        hipLaunchKernelGGL(copy_f32, dim3(grid_for(f->Q, 256)), dim3(256), 0, s, f->final_score, final_score_dev,
                           (int64_t)f->Q);
        hipLaunchKernelGGL(final_max_kernel, dim3(1), dim3(1024), 0, s, (const float *)f->final_score, f->Q,
                           f->final_max);
    }
    HIP_OK(hipGetLastError());
    return WFST_OK;
}
C_GUARD

void wfst_fst_destroy(wfst_fst *f) { free_fst(f); }

int wfst_fst_label_stats(const wfst_fst *f, int32_t *arcs, int32_t *fwd_segments, int32_t *rev_segments)
try {
    if (!f) return set_err(WFST_EINVAL, "fst is NULL");
    const size_t n = (size_t)f->M * sizeof(int32_t);
    if (arcs) std::memcpy(arcs, f->label_arcs.data(), n);
    if (fwd_segments) std::memcpy(fwd_segments, f->label_fwd_segs.data(), n);
    if (rev_segments) std::memcpy(rev_segments, f->label_rev_segs.data(), n);
    return WFST_OK;
}
C_GUARD

int wfst_fst_profile(wfst_fst *f, int32_t enable)
try {
    if (!f) return set_err(WFST_EINVAL, "fst is NULL");
    f->prof = enable != 0;
    return WFST_OK;
}
C_GUARD

int wfst_fst_profile_read(wfst_fst *f, double *ms, int64_t *launches, int32_t reset)
try {
    if (!f || !ms || !launches) return set_err(WFST_EINVAL, "NULL argument");
    for (int k = 0; k < WFST_KERNEL_COUNT; ++k) {
        ms[k] = 0.0;
        launches[k] = 0;
    }
    for (auto &m : f->marks) {
        HIP_OK(hipEventSynchronize(m.b));
        float t = 0.0f;
        HIP_OK(hipEventElapsedTime(&t, m.a, m.b));
        if (m.kind >= 0 && m.kind < WFST_KERNEL_COUNT) {
            ms[m.kind] += t;
            launches[m.kind] += 1;
        }
    }
    if (reset) {
        for (auto &m : f->marks) f->spare.push_back(m);
        f->marks.clear();
    }
    return WFST_OK;
}
C_GUARD

int wfst_fst_debug_team_spin(wfst_fst *f, int32_t polls)
try {
    if (!f) return set_err(WFST_EINVAL, "fst is NULL");
    if (polls < 0) return set_err(WFST_EINVAL, "polls must be >= 0");
    f->team_spin = polls;
    return WFST_OK;
}
C_GUARD

int wfst_fst_debug_alloc_limit(wfst_fst *f, int64_t bytes)
try {
    if (!f) return set_err(WFST_EINVAL, "fst is NULL");
    if (bytes < 0) return set_err(WFST_EINVAL, "bytes must be >= 0");
    f->alloc_limit = bytes;
    return WFST_OK;
}
C_GUARD

int wfst_fst_health(const wfst_fst *f, uint32_t *flags, int32_t clear, void *stream)
try {
    if (!f || !flags) return set_err(WFST_EINVAL, "NULL argument");
    hipStream_t s = as_stream(stream);
    HIP_OK(hipMemcpyAsync(flags, f->health, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    HIP_OK(hipStreamSynchronize(s));
    if (clear) {
        hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, reinterpret_cast<int32_t *>(f->health), (int64_t)1, 0);
        HIP_OK(hipGetLastError());
    }
    return WFST_OK;
}
C_GUARD

int wfst_fst_score_version(const wfst_fst *f, uint64_t *version)
try {
    if (!f || !version) return set_err(WFST_EINVAL, "NULL argument");
    *version = f->score_version;
    return WFST_OK;
}
C_GUARD

int wfst_fst_get_info(const wfst_fst *f, wfst_fst_info *info)
try {
    if (!f || !info) return set_err(WFST_EINVAL, "NULL argument");
    std::memset(info, 0, sizeof(*info));
    info->num_states = f->Q;
    info->num_ilabels = f->M;
    info->start = f->start;
    info->chunk_arcs = f->chunk;
    info->num_arcs = f->A;
    info->fwd_elements = f->fwd.n_elem;
    info->rev_elements = f->rev.n_elem;
    info->fwd_segments = f->fwd.n_seg;
    info->rev_segments = f->rev.n_seg;
    info->fwd_slices = f->fwd.n_slice;
    info->rev_slices = f->rev.n_slice;
    info->max_fwd_segments_per_label = f->fwd.max_segs;
    info->max_rev_segments_per_label = f->rev.max_segs;
    info->max_fwd_slots_per_label = f->fwd.max_slots;
    info->max_rev_slots_per_label = f->rev.max_slots;
    info->device_bytes = f->bytes;
    return WFST_OK;
}
C_GUARD

int wfst_viterbi(const wfst_fst *fc, int32_t batch, int64_t num_tokens, const int32_t *offsets,
                 const int32_t *tokens, float *best_score, int32_t *best_arcs, int32_t *best_olabels,
                 int32_t *status, void *stream)
try {
    TRY(check_batch(fc, batch, num_tokens, offsets, tokens));
    if (batch == 0) return WFST_OK;
    if (!best_score || !status || (num_tokens > 0 && !best_arcs)) return set_err(WFST_EINVAL, "NULL output");
    if (best_olabels && !fc->olabel) return set_err(WFST_EINVAL, "FST was created without olabels");
    wfst_fst *f = const_cast<wfst_fst *>(fc);  // the workspace is mutable state of the FST
    hipStream_t s = as_stream(stream);
    if (live_wanted(f, lds_viterbi(f, false))) {
        if (f->graph_mode) TRY(graph_limits(f, num_tokens, kBoundCapBytes / 8, false));
        const int rc = viterbi_live(f, batch, num_tokens, offsets, tokens, best_score, best_arcs, best_olabels, status, s);
        if (!live_no_room(f, s, rc)) return rc;
    }
    return viterbi_dense(f, batch, num_tokens, offsets, tokens, best_score, best_arcs, best_olabels, status, s);
}
C_GUARD

int wfst_viterbi_noalloc(const wfst_fst *fc, int32_t batch, int64_t num_tokens, const int32_t *offsets,
                         const int32_t *tokens, float *best_score, int32_t *best_arcs, int32_t *best_olabels,
                         int32_t *status, void *stream)
try {
    TRY(check_batch(fc, batch, num_tokens, offsets, tokens));
    if (batch == 0) return WFST_OK;
    if (!best_score || !status || (num_tokens > 0 && !best_arcs)) return set_err(WFST_EINVAL, "NULL output");
    if (best_olabels && !fc->olabel) return set_err(WFST_EINVAL, "FST was created without olabels");
    int dev = -1;
    HIP_OK(hipGetDevice(&dev));
    if (dev != fc->device) return set_err(WFST_EINVAL, "the FST's device must be the current device");
    unsigned char *base = nullptr;
    TRY(static_scratch(dev, &base));
    hipStream_t s = as_stream(stream);
    const int64_t N = num_tokens;
    // carve the scratch: counters | order | tok_off | scan tiles | path | back-pointers (bound: N x max segments)
    const int64_t segs = std::max(fc->fwd.max_segs, 1);
    size_t at = 0;
    auto carve = [&](size_t bytes) {
        const size_t here = at;
        at += (bytes + 255) / 256 * 256;
        return here;
    };
    const size_t o_cnt = carve(C_COUNT * sizeof(int32_t));
    const size_t o_order = carve((size_t)batch * sizeof(int32_t));
    const size_t o_tok = carve((size_t)std::max<int64_t>(N, 1) * sizeof(int64_t));
    const size_t o_tiles = carve((size_t)scan_tiles_for(N) * sizeof(int64_t));
    const size_t o_path = carve((size_t)std::max<int64_t>(N, 1) * sizeof(int32_t));
    if ((double)N * (double)segs * sizeof(int2) > (double)kStaticScratchBytes)
        return set_err(WFST_EUNSUPPORTED, "batch too large for the no-allocation Viterbi: " + std::to_string(N) +
                                              " tokens x " + std::to_string(segs) +
                                              " segments per label need more than its " +
                                              std::to_string(kStaticScratchBytes >> 20) + " MiB of scratch");
    const size_t o_bp = carve((size_t)N * (size_t)segs * sizeof(int2));
    if (at > kStaticScratchBytes)
        return set_err(WFST_EUNSUPPORTED, "batch too large for the no-allocation Viterbi: needs " +
                                              std::to_string(at) + " bytes of its " +
                                              std::to_string(kStaticScratchBytes) + "-byte scratch");
    int32_t *counters = reinterpret_cast<int32_t *>(base + o_cnt);
    int32_t *order = reinterpret_cast<int32_t *>(base + o_order);
    int64_t *tok_off = reinterpret_cast<int64_t *>(base + o_tok);
    int64_t *tiles = reinterpret_cast<int64_t *>(base + o_tiles);
    int32_t *path_tmp = reinterpret_cast<int32_t *>(base + o_path);
    int2 *bp = reinterpret_cast<int2 *>(base + o_bp);
    TRY(refresh_layouts(const_cast<wfst_fst *>(fc), s, nullptr));
    hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, counters, (int64_t)C_COUNT, 0);
    Plan p;
    // the bound N x max segments always fits here, so the plan reads nothing back
    TRY(make_plan(fc, s, batch, N, offsets, tokens, order, tok_off, tiles,
                  reinterpret_cast<int64_t *>(counters + C_TOTAL), INT64_MAX, p));
    const BatchView bv = make_view(fc, batch, N, offsets, tokens, order, tok_off, counters + C_QUEUE, status);
    int rc;
    DISPATCH_NT(rc, fc->nt, launch_viterbi, fc, s, bv, bp, path_tmp, best_score, best_arcs, best_olabels, true)
    return rc;
}
C_GUARD

int wfst_forward(const wfst_fst *fc, int32_t batch, int64_t num_tokens, const int32_t *offsets,
                 const int32_t *tokens, float *log_z, int32_t *status, wfst_tape **tape_out, void *stream)
try {
    TRY(check_batch(fc, batch, num_tokens, offsets, tokens));
    if (!tape_out) return set_err(WFST_EINVAL, "tape_out is NULL");
    *tape_out = nullptr;
    if (batch > 0 && (!log_z || !status)) return set_err(WFST_EINVAL, "NULL output");
    wfst_fst *f = const_cast<wfst_fst *>(fc);
    hipStream_t s = as_stream(stream);
    // the grouped count kernel and a record limit name the streaming sweeps
    const bool counts_ok = !(f->rec_off && !f->fx_counts) && f->rec_max == kRecordsMax;
    const bool fits = !f->live.narrow || narrow_tape_bytes(f, num_tokens) <= live_tape_bytes(f);
    if (batch == 0 || !counts_ok || !fits || !live_wanted(f, lds_lse(f, f->fwd)))
        return forward_dense(f, batch, num_tokens, offsets, tokens, log_z, status, tape_out, s);
    if (f->graph_mode) TRY(graph_limits(f, num_tokens, kBoundCapBytes / 4, true));
    wfst_tape *t = new_tape(f, batch, num_tokens, offsets, tokens, status);
    const int rc = guarded([&] { return forward_live(f, t, log_z, status, s); });
    if (rc != WFST_OK) {
        wfst_tape_free(t);
        if (!live_no_room(f, s, rc)) return rc;
        return forward_dense(f, batch, num_tokens, offsets, tokens, log_z, status, tape_out, s);
    }
    *tape_out = t;
    return WFST_OK;
}
C_GUARD

void wfst_tape_free(wfst_tape *t)
{
    if (!t) return;
    wfst_tape_free(t->rest);
    if (t->fst && t->bufs) const_cast<wfst_fst *>(t->fst)->tape_pool.push_back(t->bufs);
    delete t;
}

int wfst_backward(const wfst_fst *fc, const wfst_tape *tape, const float *grad_log_z, float *grad_arc_score,
                  float *grad_final, void *stream)
try {
    if (!fc || !tape) return set_err(WFST_EINVAL, "NULL fst or tape");
    if (tape->fst != fc) return set_err(WFST_EINVAL, "tape belongs to another FST");
    if (!grad_arc_score && fc->A > 0) return set_err(WFST_EINVAL, "grad_arc_score is NULL");
    if (tape->score_version != fc->score_version)
        return set_err(WFST_EINVAL, "the FST's scores changed after the forward pass of this tape "
                                    "(wfst_fst_set_scores); run the forward pass again");
    wfst_fst *f = const_cast<wfst_fst *>(fc);
    hipStream_t s = as_stream(stream);
    if (tape->live) {
        const int rc = backward_live(f, tape, grad_log_z, grad_arc_score, grad_final, s);
        if (!live_no_room(f, s, rc)) return rc;
        return backward_again(f, tape, grad_log_z, grad_arc_score, grad_final, s);
    }
    return backward_dense(f, tape, grad_log_z, grad_arc_score, grad_final, s);
}
C_GUARD

int wfst_forward_backward(const wfst_fst *f, int32_t batch, int64_t num_tokens, const int32_t *offsets,
                          const int32_t *tokens, float *log_z, float *arc_posterior, float *final_posterior,
                          int32_t *status, void *stream)
try {
    wfst_tape *t = nullptr;
    TRY(wfst_forward(f, batch, num_tokens, offsets, tokens, log_z, status, &t, stream));
    int rc = wfst_backward(f, t, nullptr, arc_posterior, final_posterior, stream);
    wfst_tape_free(t);
    return rc;
}
C_GUARD

int wfst_fst_autotune(wfst_fst *f, int32_t batch, int64_t num_tokens, const int32_t *offsets,
                      const int32_t *tokens, const char *cache_path, int32_t flags, wfst_autotune_result *res,
                      void *stream)
try {
    if (!f) return set_err(WFST_EINVAL, "fst is NULL");
    TRY(check_batch(f, batch, num_tokens, offsets, tokens));
    static const int32_t sizes[5] = {64, 128, 256, 512, 1024};
    static const int32_t modes[3] = {0, -1, -2};
    hipStream_t s = as_stream(stream);
    wfst_autotune_result r;
    std::memset(&r, 0, sizeof(r));
    for (int c = 0; c < 4; ++c)
        for (int k = 0; k < 5; ++k)
            for (int m = 0; m < 3; ++m) r.ms[c][k][m] = -1.0f;
    const int32_t keep_nt = f->nt, keep_mode = count_mode(f), keep_chunk = f->chunk;
    r.threads_per_sentence = keep_nt;
    r.count_records = keep_mode;
    r.chunk_arcs = keep_chunk;
    r.best_ms = -1.0f;
    if (batch == 0) {
        if (res) *res = r;
        return WFST_OK;
    }
    std::string key;
    std::vector<std::pair<std::string, TuneEntry>> cache;
    if (cache_path && *cache_path) {
        TRY(tune_key(f, batch, num_tokens, offsets, tokens, flags, s, key));
        cache = read_tune_cache(cache_path);
        for (auto &e : cache)
            if (e.first == key) {  // known workload: apply without timing
                TRY(rebuild_layouts(f, e.second.chunk, s));
                f->nt = e.second.nt;
                set_count_mode(f, e.second.mode);
                r.threads_per_sentence = f->nt;
                r.count_records = e.second.mode;
                r.chunk_arcs = f->chunk;
                r.best_ms = e.second.ms;
                r.from_cache = 1;
                if (res) *res = r;
                return WFST_OK;
            }
    }
    // scratch outputs of the timed passes
    const int64_t N = num_tokens;
    const size_t bytes = (size_t)batch * (2 * sizeof(float) + sizeof(int32_t)) + (size_t)N * sizeof(int32_t) +
                         (size_t)std::max<int64_t>(f->A, 1) * sizeof(float);
    void *scratch_out = nullptr;
    if (hipMalloc(&scratch_out, bytes) != hipSuccess) return set_err(WFST_ENOMEM, "autotune scratch");
    float *score = static_cast<float *>(scratch_out);
    float *log_z = score + batch;
    int32_t *status = reinterpret_cast<int32_t *>(log_z + batch);
    int32_t *arcs = status + batch;
    float *grad = reinterpret_cast<float *>(arcs + N);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    int rc = WFST_OK;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) rc = set_err(WFST_EHIP, "event");
    // left (nullable): sentences that went to the streaming sweeps, -1 for all of them
    auto pass = [&](int32_t *left = nullptr) -> int {
        auto read = [&](const int32_t *p, int32_t *to) -> int {
            HIP_OK(hipMemcpyAsync(to, p, sizeof(int32_t), hipMemcpyDeviceToHost, s));
            HIP_OK(hipStreamSynchronize(s));
            return WFST_OK;
        };
        int32_t n = 0;
        TRY(wfst_viterbi(f, batch, N, offsets, tokens, score, arcs, nullptr, status, s));
        if (left) {
            *left = live_wanted(f, lds_viterbi(f, false)) ? 0 : -1;
            if (*left == 0 && !f->live.narrow)
                TRY(read(static_cast<int32_t *>(f->ws[W_LCNT].p) + (f->live.wide && !f->live.safe ? L_LEFT2 : L_LEFT), left));
        }
        wfst_tape *t = nullptr;
        TRY(wfst_forward(f, batch, N, offsets, tokens, log_z, status, &t, s));
        int rb = WFST_OK;
        if (left && *left >= 0) {
            if (!t->live) *left = -1;
            else if (t->n_left) rb = read(t->n_left, &n);
            *left += *left < 0 ? 0 : n;
        }
        if (rb == WFST_OK) rb = wfst_backward(f, t, nullptr, grad, nullptr, s);
        wfst_tape_free(t);
        return rb;
    };
    std::vector<int32_t> chunks;
    if (flags & WFST_TUNE_CHUNK) chunks = {4, 8, 16, 32};
    else chunks = {keep_chunk};
    // A batch that runs over lists of live states alone takes the same launches
    // whatever the workgroup size, the chunk length and the choice between
    // records and fixed point: it is timed once, and those candidates share it.
    float shared_ms = -1.0f;
    for (size_t c = 0; c < chunks.size() && rc == WFST_OK; ++c) {
        r.chunks[c] = chunks[c];
        if ((rc = guarded([&] { return rebuild_layouts(f, chunks[c], s); })) != WFST_OK) break;
        for (int k = 0; k < 5 && rc == WFST_OK; ++k) {
            for (int m = 0; m < 3 && rc == WFST_OK; ++m) {
                f->nt = sizes[k];
                // records and the grouped kernel need the on-chip backward sweep, the
                // grouped kernel its own state in LDS too
                if (modes[m] != -2 && backward_in_gmem(f)) continue;
                if (modes[m] == -1 && lds_counts(f) > f->max_lds) continue;
                float ms = shared_ms;
                if (modes[m] == -1 || shared_ms < 0.0f) {
                    set_count_mode(f, modes[m]);
                    int32_t left = -1;
                    int p = pass(&left);  // untimed: grows workspaces, loads code
                    if (p == WFST_EUNSUPPORTED) continue;  // this size does not fit the FST's needs
                    if (p != WFST_OK) {
                        rc = p;
                        break;
                    }
                    if (hipEventRecord(e0, s) != hipSuccess) {
                        rc = set_err(WFST_EHIP, "event");
                        break;
                    }
                    if ((p = pass()) != WFST_OK) {
                        rc = p;
                        break;
                    }
                    if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
                        hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
                        rc = set_err(WFST_EHIP, "event timing");
                        break;
                    }
                    if (modes[m] != -1 && left == 0) shared_ms = ms;
                }
                r.ms[c][k][m] = ms;
                r.tried += 1;
            }
        }
    }
    // the fastest; among equals the FST's own configuration, then the first
    int bc = -1, bk = -1, bm = -1;
    auto own = [&](int c, int k, int m) {
        return (chunks[(size_t)c] == keep_chunk) * 4 + (sizes[k] == keep_nt) * 2 + (modes[m] == keep_mode);
    };
    for (int c = 0; c < (int)chunks.size(); ++c)
        for (int k = 0; k < 5; ++k)
            for (int m = 0; m < 3; ++m) {
                const float ms = r.ms[c][k][m];
                if (ms < 0.0f) continue;
                if (bc < 0 || ms < r.ms[bc][bk][bm] || (ms == r.ms[bc][bk][bm] && own(c, k, m) > own(bc, bk, bm))) {
                    bc = c;
                    bk = k;
                    bm = m;
                }
            }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    (void)hipStreamSynchronize(s);
    (void)hipFree(scratch_out);
    if (rc == WFST_OK && bc < 0) rc = set_err(WFST_EUNSUPPORTED, "no configuration fits this FST");
    const int32_t chunk = rc == WFST_OK ? chunks[(size_t)bc] : keep_chunk;
    const int rr = guarded([&] { return rebuild_layouts(f, chunk, s); });
    if (rc == WFST_OK) rc = rr;
    f->nt = rc == WFST_OK ? sizes[bk] : keep_nt;
    set_count_mode(f, rc == WFST_OK ? modes[bm] : keep_mode);
    if (rc != WFST_OK) return rc;
    r.threads_per_sentence = f->nt;
    r.count_records = modes[bm];
    r.chunk_arcs = f->chunk;
    r.best_ms = r.ms[bc][bk][bm];
    if (!key.empty()) {
        TuneEntry e;
        e.nt = f->nt;
        e.mode = modes[bm];
        e.chunk = f->chunk;
        e.ms = r.best_ms;
        cache.emplace_back(key, e);
        TRY(write_tune_cache(cache_path, cache));
    }
    if (res) *res = r;
    return WFST_OK;
}
C_GUARD

int wfst_forward_scan(const wfst_fst *fc, int32_t batch, int64_t num_tokens, const int32_t *offsets,
                      const int32_t *tokens, float *log_z, float *alpha, int32_t *status, void *stream)
try {
    TRY(check_batch(fc, batch, num_tokens, offsets, tokens));
    if (batch == 0) return WFST_OK;
    if (!log_z || !status) return set_err(WFST_EINVAL, "NULL output");
    wfst_fst *f = const_cast<wfst_fst *>(fc);
    if (f->Q > kScanMaxQ)
        return set_err(WFST_EUNSUPPORTED, "the scan keeps dense state x state matrices: num_states must be <= " +
                                              std::to_string(kScanMaxQ));
    hipStream_t s = as_stream(stream);
    const int64_t N = num_tokens, QQ = (int64_t)f->Q * f->Q;
    if ((double)N * (double)QQ * 2.0 * sizeof(float) > (double)kScanBudgetBytes)
        return set_err(WFST_EUNSUPPORTED, "the scan needs two state x state matrices per token: " +
                                              std::to_string(N) + " tokens exceed its " +
                                              std::to_string(kScanBudgetBytes >> 30) + " GiB");
    // Narrow labels: a chunk's matrix has one row per destination of the token before it, not |Q|, and one launch
    // does the sentence (T = 200 on the 45-tag tagger: matrices of every token and 8 levels 450 us, this
    // 27 us).
    if (f->live.on && f->live.narrow) {
        if (N > 0 && stream_capturing(s))
            return set_err(WFST_EHIP, "the scan cannot be captured");
        BatchView bv;
        bv.B = batch;
        bv.N = N;
        bv.M = f->M;
        bv.offsets = offsets;
        bv.tokens = tokens;
        bv.status = status;
        ProfScope prof(f, s, WFST_KERNEL_SCAN);
        NARROW_LAUNCH(narrow_scan, f->live, (int)std::min<int64_t>(batch, (int64_t)f->cu_count * 8), kNarrowScanThreads,
                      0, s,
                      f->live.ix, narrow_view(f), f->start, (const float *)f->final_score, bv, log_z, alpha, f->Q);
        HIP_OK(hipGetLastError());
        return WFST_OK;
    }
    int32_t *counters = nullptr, *first = nullptr;
    float *p0 = nullptr, *p1 = nullptr;
    TRY(ensure_t(f->ws[W_COUNTERS], C_COUNT, s, &counters));
    int32_t tmax = 0;
    if (N > 0) {
        TRY(ensure_t(f->ws[W_TOKSENT], N, s, &first));
        TRY(ensure_t(f->ws[W_SCAN0], N * QQ, s, &p0));
        TRY(ensure_t(f->ws[W_SCAN1], N * QQ, s, &p1));
        // longest sentence: the number of levels (one read-back; the scan is the latency path)
        hipLaunchKernelGGL(batch_max_len, dim3(1), dim3(1024), 0, s, offsets, batch, counters + C_TOTAL);
        HIP_OK(hipMemcpyAsync(&tmax, counters + C_TOTAL, sizeof(int32_t), hipMemcpyDeviceToHost, s));
        HIP_OK(hipStreamSynchronize(s));
    }
    TRY(refresh_layouts(f, s, nullptr));
    ProfScope prof(f, s, WFST_KERNEL_SCAN);
    if (N > 0) {
        hipLaunchKernelGGL(token_first, dim3(grid_for(N, 256)), dim3(256), 0, s, offsets, batch, N, first);
        const unsigned g = (unsigned)std::min<int64_t>(N, 65535);
        hipLaunchKernelGGL(scan_leaves, dim3(g), dim3(kScanThreadsPerMat), 0, s, f->fwd, f->Q, tokens, N, f->M, p0);
        for (int64_t stride = 1; stride < tmax; stride *= 2) {
            hipLaunchKernelGGL(scan_level, dim3(g), dim3(kScanThreadsPerMat), 0, s, (const float *)p0, p1,
                               (const int32_t *)first, N, f->Q, (int32_t)stride);
            std::swap(p0, p1);
        }
    }
    hipLaunchKernelGGL(scan_finish, dim3(grid_for(batch, 4)), dim3(256), 0, s, (const float *)p0, offsets, tokens,
                       batch, N, f->M, f->Q, f->start, (const float *)f->final_score, log_z, alpha, status);
    HIP_OK(hipGetLastError());
    return WFST_OK;
}
C_GUARD

size_t lds_lattice(const wfst_fst *f)
{
    return ((size_t)f->Q + 1 + (size_t)std::max(f->fwd.max_segs, 1) + (size_t)std::max(f->fwd.max_slots, 1)) *
               sizeof(double) +
           (size_t)std::max(f->fwd.max_segs, 1) * sizeof(int32_t) + ((size_t)f->Q + 1) * sizeof(float);
}

int wfst_lattice_forward(const wfst_fst *fc, int32_t batch, const int32_t *node_offsets, const int32_t *arc_offsets,
                         int64_t num_nodes, int64_t num_arcs, const int32_t *arc_from, const int32_t *arc_to,
                         const int32_t *arc_label, const float *arc_weight, float *log_z, float *node_log_alpha,
                         int32_t *status, void *stream)
try {
    if (!fc) return set_err(WFST_EINVAL, "fst is NULL");
    if (batch < 0 || num_nodes < 0 || num_arcs < 0) return set_err(WFST_EINVAL, "negative size");
    if (num_nodes > INT32_MAX || num_arcs > INT32_MAX) return set_err(WFST_EINVAL, "lattice ids are int32");
    if (batch == 0) return WFST_OK;
    if (!node_offsets || !arc_offsets || !log_z || !status) return set_err(WFST_EINVAL, "NULL offsets or output");
    if (num_arcs > 0 && (!arc_from || !arc_to || !arc_label || !arc_weight))
        return set_err(WFST_EINVAL, "NULL arc array");
    wfst_fst *f = const_cast<wfst_fst *>(fc);
    hipStream_t s = as_stream(stream);
    constexpr int NT = 256;
    const size_t lds = lds_lattice(f);
    int grid = 0;
    TRY(persistent_grid(f, lattice_forward<NT>, NT, lds, batch, &grid));
    int32_t *counters = nullptr;
    float *nodes = nullptr;
    double *scale = nullptr;
    const int64_t Q1 = (int64_t)f->Q + 1, V = std::max<int64_t>(num_nodes, 1);
    TRY(ensure_t(f->ws[W_COUNTERS], C_COUNT, s, &counters));
    TRY(ensure_t(f->ws[W_LATNODE], V * Q1, s, &nodes));
    TRY(ensure_t(f->ws[W_LATSCALE], V, s, &scale));
    int32_t *far = nullptr;
    TRY(ensure_t(f->ws[W_LATFAR], V, s, &far));
    hipLaunchKernelGGL(fill_i32, dim3(1), dim3(64), 0, s, counters, (int64_t)C_COUNT, 0);
    LatticeView lv;
    lv.B = batch;
    lv.n_nodes = num_nodes;
    lv.n_arcs = num_arcs;
    lv.node_off = node_offsets;
    lv.arc_off = arc_offsets;
    lv.from = arc_from;
    lv.to = arc_to;
    lv.label = arc_label;
    lv.weight = arc_weight;
    lv.nodes = nodes;
    lv.scale = scale;
    lv.far = far;
    lv.queue = counters + C_QUEUE;
    lv.offs_bad = counters + C_NITEMS;
    // Live form first (its kept lists: at most 8 GiB); lattices whose nodes outgrow its lists are left to the other.
    LiveLattices w;
    w.keep = std::min(kLatK2, f->Q);
    w.one = std::ldexp(1.0, lat_bits(f->live.per));
    w.unit = 1.0 / w.one;
    bool live = f->live.on && lat_bits(f->live.per) >= kLatBitsMin &&
                V * w.keep * (int64_t)(sizeof(double) + sizeof(int32_t)) <= (int64_t)8 << 30;
    if (live) {
        auto buffers = [&]() -> int {
            TRY(ensure_t(f->ws[W_LLEFT], 2 * (int64_t)batch, s, &w.left));
            TRY(ensure_t(f->ws[W_LATTOK], V, s, &w.count));
            TRY(ensure_t(f->ws[W_LATSTATE], V * w.keep, s, &w.state));
            TRY(ensure_t(f->ws[W_LATVAL], V * w.keep, s, &w.val));
            return live_order(f, s, batch, arc_offsets, f->ws[W_LORDER], f->cu_count, &w.order);
        };
        const int rc = buffers();
        w.n_left = counters + C_SLOTS;
        if (rc != WFST_OK && !live_no_room(f, s, rc)) return rc;
        live = rc == WFST_OK;
    }
    hipLaunchKernelGGL(lattice_offsets_check, dim3(grid_for((int64_t)batch + 1, 256)), dim3(256), 0, s, node_offsets,
                       arc_offsets, batch, num_nodes, num_arcs, counters + C_NITEMS);
    if (live && node_log_alpha)
        hipLaunchKernelGGL(fill_f32, dim3(grid_for(num_nodes * f->Q, 256, 8192)), dim3(256), 0, s, node_log_alpha,
                           num_nodes * (int64_t)f->Q, -INFINITY);
    ProfScope prof(f, s, WFST_KERNEL_LATTICE);
    if (live) {
        constexpr int LT = 256, LT2 = 1024;
        w.lv = lv;
        int lgrid = 0, lgrid2 = 0;
        const int rc = by_listed(f->live, [&](auto listed) -> int {
            constexpr bool L = decltype(listed)::value;
            TRY(persistent_grid(f, live_lattice<LT, kLatK, kLatH, L>, LT, 0, batch, &lgrid));
            TRY(persistent_grid(f, live_lattice<LT2, kLatK2, kLatH2, L>, LT2, 0, batch, &lgrid2));
            hipLaunchKernelGGL((live_lattice<LT, kLatK, kLatH, L>), dim3(lgrid), dim3(LT), 0, s, f->live.ix, f->Q,
                               f->start, f->M, (const float *)f->final_score, w, log_z, node_log_alpha, status);
            w.order = w.left;
            w.n = w.n_left;
            w.left = w.left + batch;
            w.n_left = counters + C_TOTAL;
            w.lv.queue = counters + C_TOTAL + 1;
            hipLaunchKernelGGL((live_lattice<LT2, kLatK2, kLatH2, L>), dim3(lgrid2), dim3(LT2), 0, s, f->live.ix, f->Q,
                               f->start, f->M, (const float *)f->final_score, w, log_z, node_log_alpha, status);
            return WFST_OK;
        });
        if (rc != WFST_OK) return rc;
        lv.order = w.left;
        lv.n = w.n_left;
        lv.queue = counters + C_ITEMQ;
    }
    TRY(refresh_layouts(f, s, lv.n));
    hipLaunchKernelGGL(lattice_far_clear, dim3(grid_for(V, 256, 1024)), dim3(256), 0, s, far, V, lv.n,
                       f->live.stale);
    hipLaunchKernelGGL((lattice_forward<NT>), dim3(grid), dim3(NT), lds, s, f->fwd, f->Q, f->start, f->M,
                       (const float *)f->final_score, lv, log_z, node_log_alpha, status, f->health);
    HIP_OK(hipGetLastError());
    return WFST_OK;
}
C_GUARD

int wfst_em_update(wfst_fst *f, const float *counts, float smoothing, const float *cur_score, float *new_score,
                   void *stream)
try {
    if (!f) return set_err(WFST_EINVAL, "fst is NULL");
    if (f->A > 0 && (!counts || !cur_score || !new_score)) return set_err(WFST_EINVAL, "NULL argument");
    if (!(smoothing >= 0.0f) || std::isinf(smoothing)) return set_err(WFST_EINVAL, "smoothing must be finite and >= 0");
    if (f->A == 0) return WFST_OK;
    hipStream_t s = as_stream(stream);
    TRY(ensure_source_index(f, s));
    double *sums;  // segment sums, then the logs of the totals
    TRY(ensure_t(f->ws[W_EMSUM], f->em_items + f->Q, s, &sums));
    hipLaunchKernelGGL(em_segment_sums, dim3(grid_for(f->em_items * 64, 256, 8192)), dim3(256), 0, s,
                       (const int32_t *)f->em_order, (const EmItem *)f->em_item, f->em_items, counts, smoothing, sums);
    hipLaunchKernelGGL(em_source_sums, dim3(grid_for((int64_t)f->Q * 64, 256, 65535)), dim3(256), 0, s,
                       (const int64_t *)f->em_seg, f->Q, (const double *)sums, sums + f->em_items);
    hipLaunchKernelGGL(em_normalize, dim3(grid_for(f->A, 256, 16384)), dim3(256), 0, s, (const int32_t *)f->em_src,
                       f->A, counts, smoothing, (const double *)(sums + f->em_items), cur_score, new_score);
    HIP_OK(hipGetLastError());
    return WFST_OK;
}
C_GUARD

// One pass sequence of a graph (scores, Viterbi, forward, backward), as the
// eager entry points queue it.
static int graph_sequence(wfst_fst *f, const wfst_graph_args &a, void *stream)
{
    if (a.arc_score) TRY(wfst_fst_set_scores(f, a.arc_score, nullptr, stream));
    if (a.best_score)
        TRY(wfst_viterbi(f, a.batch, a.num_tokens, a.offsets, a.tokens, a.best_score, a.best_arcs, a.best_olabels,
                         a.status, stream));
    if (a.log_z) {
        wfst_tape *t = nullptr;
        TRY(wfst_forward(f, a.batch, a.num_tokens, a.offsets, a.tokens, a.log_z, a.status, &t, stream));
        const int r = a.grad_arc_score ? wfst_backward(f, t, a.grad_log_z, a.grad_arc_score, a.grad_final, stream)
                                       : WFST_OK;
        wfst_tape_free(t);
        TRY(r);
    }
    return WFST_OK;
}

static void graph_free(wfst_graph *g)
{
    if (!g) return;
    if (g->exec) (void)hipGraphExecDestroy(g->exec);
    if (g->graph) (void)hipGraphDestroy(g->graph);
    for (Buf &b : g->ws) free_buf(b);
    for (TapeBufs *t : g->pool) {
        t->free_all();
        delete t;
    }
    delete g;
}

int wfst_graph_create(wfst_fst *f, const wfst_graph_args *args, void *stream, wfst_graph **out)
try {
    if (!out) return set_err(WFST_EINVAL, "out is NULL");
    *out = nullptr;
    if (!f || !args) return set_err(WFST_EINVAL, "NULL fst or args");
    const wfst_graph_args &a = *args;
    TRY(check_batch(f, a.batch, a.num_tokens, a.offsets, a.tokens));
    if (!a.best_score && !a.log_z) return set_err(WFST_EINVAL, "a graph needs Viterbi or forward outputs");
    if (!a.status) return set_err(WFST_EINVAL, "status is NULL");
    if (a.grad_final && !a.grad_arc_score) return set_err(WFST_EINVAL, "grad_final needs grad_arc_score");
    hipStream_t s = as_stream(stream);
    if (s == nullptr) return set_err(WFST_EINVAL, "graphs are captured on a created stream, not the null stream");
    wfst_graph *g = new wfst_graph();
    g->fst = f;
    g->args = a;
    const bool prof = f->prof;
    auto enter = [&]() {
        for (int i = 0; i < W_NUM; ++i) std::swap(f->ws[i], g->ws[i]);
        std::swap(f->tape_pool, g->pool);
        f->prof = false;
        f->graph_mode = true;
        f->live.refused = false;
    };
    auto leave = [&]() {
        for (int i = 0; i < W_NUM; ++i) std::swap(f->ws[i], g->ws[i]);
        std::swap(f->tape_pool, g->pool);
        f->prof = prof;
        f->graph_mode = false;
        f->live.refused = false;
    };
    enter();
    // eager run: sizes the graph's buffers (nothing grows during capture) and checks the arguments
    int rc = graph_sequence(f, a, stream);
    if (rc == WFST_OK && hipStreamSynchronize(s) != hipSuccess) rc = set_err(WFST_EHIP, "eager pass of the graph");
    if (rc == WFST_OK) {
        hipError_t e = hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal);
        if (e != hipSuccess) {
            rc = set_err(WFST_EHIP, std::string("hipStreamBeginCapture: ") + hipGetErrorString(e));
        } else {
            rc = graph_sequence(f, a, stream);
            e = hipStreamEndCapture(s, &g->graph);
            if (rc == WFST_OK && e != hipSuccess)
                rc = set_err(WFST_EHIP, std::string("hipStreamEndCapture: ") + hipGetErrorString(e));
        }
    }
    leave();
    if (rc == WFST_OK) {
        const hipError_t e = hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0);
        if (e != hipSuccess) rc = set_err(WFST_EHIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(e));
    }
    if (rc != WFST_OK) {
        (void)hipStreamSynchronize(s);
        graph_free(g);
        return rc;
    }
    f->live_graphs += 1;
    *out = g;
    return WFST_OK;
}
C_GUARD

int wfst_graph_launch(wfst_graph *g, void *stream)
try {
    if (!g || !g->exec) return set_err(WFST_EINVAL, "graph is NULL");
    HIP_OK(hipGraphLaunch(g->exec, as_stream(stream)));
    if (g->args.arc_score) {  // the replay replaced the scores
        g->fst->score_version += 1;
        g->fst->live.dense_stale = true;
    }
    return WFST_OK;
}
C_GUARD

void wfst_graph_destroy(wfst_graph *g)
{
    if (!g) return;
    int cur = 0;
    const int dev = g->fst->device;
    const bool other = hipGetDevice(&cur) == hipSuccess && cur != dev;
    if (other) (void)hipSetDevice(dev);
    (void)hipDeviceSynchronize();
    g->fst->live_graphs -= 1;
    graph_free(g);
    if (other) (void)hipSetDevice(cur);
}

}  // extern "C"
