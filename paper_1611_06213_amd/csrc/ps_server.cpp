// Host side of the parameter server: the C ABI declared in include/ps.h.
//
// The protocol state of the paper's server (Sec. 2.1, 4.1) -- queues,
// timestamps, pull history, staleness -- lives in gadei::Protocol
// (ps_protocol.h), which does no device work. This file owns the device side:
// w and v in HBM, the server's stream, and the kernel launches. ps_push moves
// no data, an apply launches one kernel per run of equal-dtype gradients, a
// pull launches one fan-out. Every call validates and plans on the host,
// launches, and only then commits the protocol state.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <vector>

#include "ps.h"
#include "ps_kernels.h"
#include "ps_layout.h"
#include "ps_protocol.h"

using gadei::align_up;
using gadei::Batch;
using gadei::fail;
using gadei::kRowAlign;
using gadei::PushDesc;

namespace {

// One device allocation carved into staggered rows (ps_alloc_rows).
struct RowSet {
    void *base;          // what hipMalloc returned
    char *first;         // row 0
    char *end;           // one past the last row's data
};

}  // namespace

// One kernel launch of a call, with every argument it was given: the plan
// that a captured graph (ps_graph_create) replays. Zero-filled before use,
// so two records compare equal byte for byte exactly when the launches are
// the same.
struct LaunchRecord {
    int kind;   // 0 apply, 1 synchronous step, 2 pull fan-out, 3 steps, 4 synchronous steps
    int grad_dtype;
    int pull_dtype;
    int level;
    int blocks_per_cu;
    int group;
    gadei::StepsArgs apply;   // rend: kinds 3 and 4
    gadei::PullArgs pull;
};

// The device work of a script's calls (ps_run) that is planned but not yet
// enqueued: the gradients of one or more applies and the replicas pulled
// between and after them, to go out as one launch. Empty while args.k == 0.
struct StepGroup {
    bool open = false;    // a script is running and its calls may join
    bool failed = false;  // a launch of joined calls failed
    const ps_op *ops = nullptr;   // the script, for a look at the step ahead
    int count = 0;
    int at = 0;           // the call being made
    int first = 0;        // the call whose gradients opened the group
    int pushed = 0;       // pushes since the last apply call
    size_t left = 0;      // gradients that the last apply left queued
    int steps = 0;        // applies whose gradients the group holds
    int covered = 0;      // the call up to which joining has been found worth it
    bool sync = false;    // synchronous steps
    int grad_dtype = PS_F32;
    int pull_dtype = PS_F32;   // of the replicas, once args.r > 0
    gadei::StepsArgs args;
    gadei::Journal journal;   // of the calls from `first` on
};

struct ps_server {
    size_t n = 0;
    float lr = 0.0f;
    float m = 0.0f;
    void *wv_base = nullptr;   // one allocation holding w and v
    float *w = nullptr;
    float *v = nullptr;
    std::vector<RowSet> row_sets;
    int device = 0;
    hipStream_t stream = nullptr;
    hipStream_t pull_stream = nullptr;   // lock-free pulls when pull_lock_free
    bool pull_lock_free = false;
    // recorded on pull_stream so that ps_apply_pull's replica writes follow
    // earlier lock-free pulls into the same buffers
    hipEvent_t pulls_done = nullptr;
    // ps_apply_pull writes up to this many replicas in the apply pass; -1:
    // chosen per call (fuse_replicas)
    int fuse_max_r = -1;
    // ps_set_launch_shape: -1 / 0 = the shape tables' choice
    int force_blocks_per_cu = -1;
    int force_group = 0;
    gadei::Geometry geo;
    gadei::Protocol proto;
    // ps_graph_create / ps_graph_launch: the launches of the calls in
    // progress are recorded here; with plan_only they are not made
    std::vector<LaunchRecord> *record = nullptr;
    bool plan_only = false;
    // with plan_only: the launch that fails (its place in *record) and how;
    // kNone: none
    static constexpr size_t kNone = ~size_t(0);
    size_t plan_fails = kNone;
    hipError_t plan_error = hipSuccess;
    StepGroup group;
    // Every call on the handle holds this lock, so several host threads (a
    // push thread per learner, as in Sec. 4.1) may share one server; device
    // work is enqueued in lock order. Recursive: some calls use others.
    mutable std::recursive_mutex mu;
};

#define PS_LOCK(ps) std::lock_guard<std::recursive_mutex> ps_lock_(ps->mu)

namespace {

int fail_hip(hipError_t e, const char *what) {
    return fail(PS_EHIP, "%s: %s", what, hipGetErrorString(e));
}

bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

size_t elem_bytes(int dtype) { return dtype == PS_BF16 ? 2 : 4; }

// Whether the vector kernels (1) may read this gradient, or the scalar ones
// (0) are to: they take any 4-byte boundary. From the other 2-byte ones, 16-byte
// loads run at half the rate and one coordinate per lane is faster for bf16
// (100M coordinates, K = 32 with momentum: 1361 us scalar, 1506 vector; from
// 4-byte boundaries 1371 vector, 1558 with 8-byte lanes).
int grad_level(const void *p) { return aligned(p, 4) ? 1 : 0; }

// The same for a replica: stores take any element boundary (the fan-outs move
// their chunks to the replica's own line boundaries: 100M coordinates, 16
// replicas at odd offsets: fp32 1.39 ms, 2.12 scalar; bf16 0.86, 1.39 scalar).
int dst_level(const void *p, int dtype) { return aligned(p, elem_bytes(dtype)) ? 1 : 0; }

// Whether [p, p + bytes) shares a byte with w or v.
bool overlaps_state(const ps_server *ps, const void *p, size_t bytes) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(p), b = a + bytes;
    for (const float *x : {static_cast<const float *>(ps->w), static_cast<const float *>(ps->v)}) {
        if (x == nullptr) continue;
        const uintptr_t lo = reinterpret_cast<uintptr_t>(x), hi = lo + ps->n * sizeof(float);
        if (a < hi && lo < b) return true;
    }
    return false;
}

// Replica buffers must not overlap w or v (a bf16 replica written over w
// would corrupt it). Called after plan_pulls has validated the arguments.
int check_dsts(const ps_server *ps, int n, void *const *dsts, int dtype) {
    for (int i = 0; i < n; ++i)
        if (overlaps_state(ps, dsts[i], ps->n * elem_bytes(dtype)))
            return fail(PS_EINVAL, "destination %d overlaps the server's w or v", i);
    return PS_OK;
}

int check(const ps_server *ps) {
    if (ps == nullptr) return fail(PS_EINVAL, "null server handle");
    return PS_OK;
}

int use_device(const ps_server *ps) {
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
    if (cur != ps->device) {
        e = hipSetDevice(ps->device);
        if (e != hipSuccess) return fail_hip(e, "hipSetDevice");
    }
    return PS_OK;
}

// Make the server's stream wait (on the device) for every producer event of
// the batch, each once.
int wait_ready(ps_server *ps, const std::vector<PushDesc> &items) {
    std::vector<void *> seen;
    for (const PushDesc &d : items) {
        if (d.ready == nullptr || std::find(seen.begin(), seen.end(), d.ready) != seen.end())
            continue;
        seen.push_back(d.ready);
        hipError_t e = hipStreamWaitEvent(ps->stream, static_cast<hipEvent_t>(d.ready), 0);
        if (e != hipSuccess) return fail_hip(e, "waiting for a producer event");
    }
    return PS_OK;
}

// Host-side wait for lock-free pulls still reading w (before w is reset,
// saved, loaded or freed).
int drain_pulls(ps_server *ps) {
    if (!ps->pull_lock_free) return PS_OK;
    hipError_t e = hipStreamSynchronize(ps->pull_stream);
    if (e != hipSuccess) return fail_hip(e, "hipStreamSynchronize (pull stream)");
    return PS_OK;
}

// Fronts for an apply or synchronous step over a.g[0..k) of dtype gdt, w and
// v: the server's setting, or chosen from the buffers' offsets and length
// (fronts_log2_for, kFrontsBytes).
int fronts_for(const ps_server *ps, const gadei::ApplyArgs &a, int gdt) {
    if (ps->geo.fronts_log2 >= 0) return ps->geo.fronts_log2;
    if (a.n * elem_bytes(gdt) < gadei::kFrontsBytes) return 0;
    const void *p[PS_MAX_QUEUE_DEPTH + 2];
    int c = 0;
    for (int j = 0; j < a.k; ++j) p[c++] = a.g[j];
    p[c++] = a.w;
    p[c++] = a.v;   // null without momentum: not a stream
    return gadei::fronts_log2_for(p, c);
}

// The launch shape for a table entry, with the caller's overrides.
gadei::Shape shape_for(const ps_server *ps, const gadei::ApplyShape &t) {
    gadei::Shape shape;
    shape.blocks_per_cu = ps->force_blocks_per_cu >= 0 ? ps->force_blocks_per_cu : t.blocks_per_cu;
    shape.group = ps->force_group > 0 ? ps->force_group : t.group;
    return shape;
}

// fuse_replicas for r replicas of an apply of k gradients of this server.
bool fuses(const ps_server *ps, int r, int k, int grad_dtype, int pull_dtype) {
    return gadei::fuse_replicas(r, k, grad_dtype == PS_BF16, pull_dtype == PS_F32, ps->v != nullptr,
                                ps->n);
}

// The launch shape of an apply of a.k gradients that writes a.r replicas.
gadei::Shape shape_of(const ps_server *ps, const gadei::ApplyArgs &a, int grad_dtype,
                      int pull_dtype) {
    const bool bf16 = grad_dtype == PS_BF16;
    return shape_for(ps, gadei::apply_shape(a.k, a.v != nullptr, bf16, a.n,
                                            bf16 && pull_dtype == PS_F32 && a.r > 1));
}

// What a launch that was only planned (and recorded) returns.
hipError_t planned(const ps_server *ps) {
    return ps->record->size() - 1 == ps->plan_fails ? ps->plan_error : hipSuccess;
}

// The kernel launches of the calls, through the recorder.
hipError_t run_apply(ps_server *ps, const gadei::ApplyArgs &a, int gdt, int pdt, int level,
                     const gadei::Shape &shape, bool sync) {
    if (ps->record) {
        LaunchRecord r;
        std::memset(&r, 0, sizeof r);
        r.kind = sync ? 1 : 0;
        r.grad_dtype = gdt;
        r.pull_dtype = pdt;
        r.level = level;
        r.blocks_per_cu = shape.blocks_per_cu;
        r.group = shape.group;
        static_cast<gadei::ApplyArgs &>(r.apply) = a;
        ps->record->push_back(r);
    }
    if (ps->plan_only) return planned(ps);
    return sync ? gadei::launch_sync(a, gdt, level, shape, ps->geo, ps->stream)
                : gadei::launch_apply(a, gdt, pdt, level, shape, ps->geo, ps->stream);
}

hipError_t run_steps(ps_server *ps, const gadei::StepsArgs &a, bool sync, int gdt, int pdt,
                     int blocks_per_cu) {
    if (ps->record) {
        LaunchRecord r;
        std::memset(&r, 0, sizeof r);
        r.kind = sync ? 4 : 3;
        r.grad_dtype = gdt;
        r.pull_dtype = pdt;
        r.blocks_per_cu = blocks_per_cu;
        r.apply = a;
        ps->record->push_back(r);
    }
    if (ps->plan_only) return planned(ps);
    return gadei::launch_steps(a, sync, gdt, pdt, blocks_per_cu, ps->geo, ps->stream);
}

hipError_t run_pull(ps_server *ps, const gadei::PullArgs &a, int dtype, int level, hipStream_t s) {
    if (ps->record) {
        LaunchRecord r;
        std::memset(&r, 0, sizeof r);
        r.kind = 2;
        r.pull_dtype = dtype;
        r.level = level;
        r.pull = a;
        ps->record->push_back(r);
    }
    if (ps->plan_only) return planned(ps);
    return gadei::launch_pull(a, dtype, level, ps->geo, s);
}

// ---------------------------------------------------------------- steps
//
// The steps of a script go out together: the server's loop (Sec. 4.1) applies
// the gradients of one batch, lets learners pull, applies the next, and per
// coordinate the whole sequence needs w and v only at its ends. One launch
// (launch_steps) reads w and v once for several steps, writes the replicas of
// each from the pass, and a replica that the next step writes again is often still
// in cache then. Where that saves enough is steps_join's rule (ps_layout.h); a
// single step's replicas follow fuse_replicas.

int group_mark(const StepGroup &g, int j) {
    return static_cast<int>(g.args.rend[j >> 3] >> (8 * (j & 7))) & 255;
}

int group_end(const StepGroup &g, int j) {   // replicas written up to gradient j
    return group_mark(g, j) & (gadei::kLastOfStep - 1);
}

void set_group_mark(StepGroup &g, int j, int mark) {
    uint64_t &w = g.args.rend[j >> 3];
    w = (w & ~(uint64_t(255) << (8 * (j & 7)))) | static_cast<uint64_t>(mark) << (8 * (j & 7));
}

// Empty the group: nothing of it stays for the next one (a recorded launch
// holds every field).
void clear_group(StepGroup &g) {
    std::memset(&g.args, 0, sizeof g.args);
    g.sync = false;
    g.grad_dtype = g.pull_dtype = PS_F32;
    g.steps = 0;
    g.covered = -1;
}

// Enqueue the joined calls. Asynchronous ones with replicas only after the
// last gradient (or none) make an ordinary apply, a single synchronous step
// without replicas an ordinary one. If the launch fails, those calls are not
// made: the protocol is as the one before g.first left it.
int flush_group(ps_server *ps) {
    StepGroup &g = ps->group;
    if (!g.open || g.args.k == 0) return PS_OK;
    const gadei::StepsArgs a = g.args;
    const bool sync = g.sync;
    const int gdt = g.grad_dtype, pdt = g.pull_dtype;
    int pulls = 0, lasts = 0;   // places where replicas are written; synchronous steps
    for (int j = 0; j < a.k; ++j) {
        pulls += group_end(g, j) != (j > 0 ? group_end(g, j - 1) : 0);
        lasts += (group_mark(g, j) & gadei::kLastOfStep) != 0;
    }
    const bool plain =
        sync ? lasts == 1 && a.r == 0 : a.k == 1 || group_end(g, a.k - 2) == 0;
    clear_group(g);
    hipError_t e;
    if (plain) {
        gadei::ApplyArgs one = a;
        one.fronts_log2 = fronts_for(ps, one, gdt);
        const gadei::Shape shape =
            sync ? shape_for(ps, gadei::sync_shape(one.k, one.v != nullptr, gdt == PS_BF16, one.n))
                 : shape_of(ps, one, gdt, pdt);
        e = run_apply(ps, one, gdt, one.r > 0 ? pdt : -1, 1, shape, sync);
    } else {
        const int blocks =
            ps->force_blocks_per_cu >= 0
                ? ps->force_blocks_per_cu
                : gadei::steps_blocks_per_cu(a.r / std::max(1, pulls), elem_bytes(pdt),
                                             elem_bytes(gdt), a.n);
        gadei::StepsArgs steps = a;
        steps.fronts_log2 = fronts_for(ps, steps, gdt);
        e = run_steps(ps, steps, sync, gdt, pdt, blocks);
    }
    if (e == hipSuccess) {
        ps->proto.forget();
        return PS_OK;
    }
    g.failed = true;
    ps->proto.undo();
    return fail_hip(e, "apply kernel launch");
}

bool share_bytes(const void *a, size_t na, const void *b, size_t nb) {
    const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
    return x < y + nb && y < x + na;
}

bool is_apply(const ps_op &o) {
    return o.kind == PS_OP_APPLY || o.kind == PS_OP_APPLY_PULL || o.kind == PS_OP_APPLY_SYNC;
}

// What the group holds and would hold if the calls ahead join it.
struct Extent {
    int steps = 0, k = 0, r = 0;
    int last = 0;    // the call that its last step ends with
    int stay = 0;    // replicas that no later step writes again
};
struct Prospect : Extent {
    const void *dst[PS_MAX_REPLICAS];   // the `stay` ones

    explicit Prospect(const StepGroup &g) {
        steps = g.steps;
        k = g.args.k;
        last = g.at;
        pull(g.args.dst, g.args.r);
    }
    // Add one call's replicas: false if they do not fit.
    bool pull(const void *const *d, int count) {
        if (count < 0 || r + static_cast<int64_t>(count) > PS_MAX_REPLICAS || (count > 0 && d == nullptr))
            return false;
        for (int i = 0; i < count; ++i)
            if (std::find(dst, dst + stay, d[i]) == dst + stay) dst[stay++] = d[i];
        r += count;
        return true;
    }
};

// `now` with the step that the call being made belongs to (g.at: its apply or a
// pull after it), its further pulls and the steps after it, as far as whole
// steps fit: gradients of one type for the vector kernels, replicas of
// pull_dtype. `before` if that step does not fit itself. The calls ahead have not
// been checked yet.
Extent look_ahead(const StepGroup &g, const Extent &before, Prospect &now, int grad_dtype,
                  int pull_dtype, bool sync) {
    Extent whole = before;   // up to a step's end
    size_t queued = g.left + static_cast<size_t>(g.pushed);
    for (int i = g.at + 1; i < g.count; ++i) {
        const ps_op &o = g.ops[i];
        if (o.kind == PS_OP_PUSH) {
            ++queued;
            // (the next step is none to join; pulls from here on to its apply
            // are left out)
            if (o.dtype != grad_dtype || grad_level(o.grad) == 0) break;
            continue;
        }
        if (is_apply(o)) {
            now.last = i - 1;
            whole = now;
            if ((o.kind == PS_OP_APPLY_SYNC) != sync) return whole;
            if (queued > 0) {   // (with nothing queued it is no step)
                if (now.k + queued > PS_MAX_QUEUE_DEPTH) return whole;
                now.k += static_cast<int>(queued);
                ++now.steps;
                queued = 0;
            }
        }
        if (o.kind == PS_OP_PULL || o.kind == PS_OP_APPLY_PULL) {
            if (o.count != 0 && (o.dtype != pull_dtype || !now.pull(o.dsts, o.count))) return whole;
        } else if (!is_apply(o)) {
            break;   // (an unknown call: the script ends there)
        }
        now.last = i;
    }
    return now;
}

// Whether the steps of the prospect are worth one launch (steps_join,
// ps_layout.h); if so the group need not ask again up to its end.
bool worth_joining(ps_server *ps, const Extent &p, int grad_dtype, int pull_dtype) {
    gadei::StepsSize s;
    s.steps = p.steps;
    s.grad_bytes = p.k * elem_bytes(grad_dtype);
    s.pull_bytes = p.r * elem_bytes(pull_dtype);
    s.final_bytes = p.stay * elem_bytes(pull_dtype);
    if (!gadei::steps_join(s, ps->v != nullptr, ps->n)) return false;
    ps->group.covered = p.last;
    return true;
}

// Whether the step of the call being made, with `count` gradients, joins the
// replicas the group holds.
bool step_joins(ps_server *ps, int count, int gdt, bool sync) {
    StepGroup &g = ps->group;
    if (g.at <= g.covered) return true;
    Prospect now(g);
    const Extent before = now;
    now.k += count;
    ++now.steps;
    const ps_op &o = g.ops[g.at];
    if (o.kind == PS_OP_APPLY_PULL && o.count != 0 &&
        (o.dtype != g.pull_dtype || !now.pull(o.dsts, o.count)))
        return false;
    const Extent p = look_ahead(g, before, now, gdt, g.pull_dtype, sync);
    return p.steps > before.steps && worth_joining(ps, p, gdt, g.pull_dtype);
}

// Whether replicas pulled now, the group's first, are worth writing from it
// because steps ahead will join.
bool pulls_join(ps_server *ps, void *const *dsts, int dtype, const std::vector<int> &write) {
    StepGroup &g = ps->group;
    Prospect now(g);
    const Extent before = now;
    for (int i : write)
        if (!now.pull(&dsts[i], 1)) return false;
    const Extent p = look_ahead(g, before, now, g.grad_dtype, dtype, g.sync);
    return p.steps > before.steps && worth_joining(ps, p, g.grad_dtype, dtype);
}

// Add the gradients of an apply or synchronous step (one dtype, vector level) to the group,
// enqueueing what it holds first if they do not fit. A gradient that shares a
// byte with a replica the group writes must be read after that write, so it
// starts a new group. Nothing the call does after this can throw: its commit
// finds its room (a call that throws is not made, and its gradients must not be in
// the group).
int join_gradients(ps_server *ps, const PushDesc *d, int count, int gdt, bool sync) {
    StepGroup &g = ps->group;
    g.journal.room(PS_MAX_QUEUE_DEPTH + PS_MAX_REPLICAS);
    bool fits = g.args.k == 0 ||
                (g.sync == sync && g.grad_dtype == gdt && g.args.k + count <= PS_MAX_QUEUE_DEPTH);
    if (fits && g.args.r > 0) {
        fits = step_joins(ps, count, gdt, sync);
        const size_t gb = ps->n * elem_bytes(gdt), rb = ps->n * elem_bytes(g.pull_dtype);
        for (int i = 0; fits && i < count; ++i)
            for (int r = 0; fits && r < g.args.r; ++r)
                fits = !share_bytes(d[i].grad, gb, g.args.dst[r], rb);
    }
    if (!fits)
        if (int rc = flush_group(ps)) return rc;
    if (g.args.k == 0) {
        // (the calls of a graph are put back as a whole, but for a replay half made)
        if (ps->record == nullptr || ps->plan_fails != ps_server::kNone) ps->proto.mark(g.journal);
        g.first = g.at;
        g.sync = sync;
        g.grad_dtype = gdt;
        g.args.w = ps->w;
        g.args.v = ps->v;
        g.args.n = ps->n;
        g.args.lr = ps->lr;
        g.args.m = ps->m;
    }
    for (int i = 0; i < count; ++i) {
        g.args.g[g.args.k] = d[i].grad;
        set_group_mark(g, g.args.k,
                       g.args.r | (sync && i == count - 1 ? gadei::kLastOfStep : 0));
        ++g.args.k;
    }
    ++g.steps;
    return PS_OK;
}

// Add replicas pulled now to the group: false if they do not fit, or would
// be a single step's and are better written by the fan-out. A replica may
// repeat one the group already writes (the same lanes write it again, in
// order) but not share bytes with it otherwise, nor with a gradient the group
// reads.
bool join_pulls(ps_server *ps, void *const *dsts, int dtype, const std::vector<int> &write) {
    StepGroup &g = ps->group;
    const int r = static_cast<int>(write.size());
    if (g.args.k == 0 || g.args.r + r > PS_MAX_REPLICAS) return false;
    if (g.args.r > 0 && g.pull_dtype != dtype) return false;
    const bool worth = ps->fuse_max_r >= 0
                           ? r <= ps->fuse_max_r
                           : g.args.r > 0 ||
                                 (!g.sync && fuses(ps, r, g.args.k, g.grad_dtype, dtype)) ||
                                 pulls_join(ps, dsts, dtype, write);
    if (!worth) return false;
    const size_t rb = ps->n * elem_bytes(dtype), gb = ps->n * elem_bytes(g.grad_dtype);
    for (size_t i = 0; i < write.size(); ++i) {
        void *d = dsts[write[i]];
        if (dst_level(d, dtype) == 0) return false;
        for (int j = 0; j < g.args.k; ++j)
            if (share_bytes(d, rb, g.args.g[j], gb)) return false;
        for (int j = 0; j < g.args.r; ++j)
            if (d != g.args.dst[j] && share_bytes(d, rb, g.args.dst[j], rb)) return false;
        for (size_t j = 0; j < i; ++j)
            if (share_bytes(d, rb, dsts[write[j]], rb)) return false;
    }
    g.pull_dtype = dtype;
    const int before = g.args.r;
    for (int i : write) {
        for (int j = before - 1; j >= 0; --j)
            if (g.args.dst[j] == dsts[i]) {
                g.args.again |= uint64_t(1) << j;
                break;
            }
        g.args.dst[g.args.r++] = dsts[i];
    }
    set_group_mark(g, g.args.k - 1,
                   g.args.r | (g.sync ? gadei::kLastOfStep : 0));
    return true;
}

// Launch a batch as runs of equal gradient dtype, in order. The last run
// also writes the replicas listed in `write` when pull_dtype >= 0.
int launch_batch(ps_server *ps, const std::vector<PushDesc> &items, int pull_dtype,
                 void *const *dsts, const std::vector<int> &write) {
    // joined calls go out before the stream waits for a producer
    if (std::any_of(items.begin(), items.end(), [](const PushDesc &d) { return d.ready; }))
        if (int rc = flush_group(ps)) return rc;
    if (int rc = wait_ready(ps, items)) return rc;
    ps->group.left = ps->proto.pending() - items.size();
    gadei::ApplyArgs a;
    std::memset(&a, 0, sizeof a);
    a.w = ps->w;
    a.v = ps->v;
    a.n = ps->n;
    a.lr = ps->lr;
    a.m = ps->m;
    const size_t q = items.size();
    size_t start = 0;
    while (start < q) {
        const int gdt = items[start].dtype;
        size_t end = start;
        int level = 1;
        while (end < q && items[end].dtype == gdt) {
            a.g[end - start] = items[end].grad;
            level = std::min(level, grad_level(items[end].grad));
            ++end;
        }
        if (ps->group.open && level == 1) {
            if (int rc = join_gradients(ps, &items[start], static_cast<int>(end - start), gdt, false))
                return rc;
            start = end;
            continue;
        }
        if (int rc = flush_group(ps)) return rc;
        a.k = static_cast<int>(end - start);
        a.r = 0;
        a.fronts_log2 = fronts_for(ps, a, gdt);
        int pdt = -1;
        if (end == q && pull_dtype >= 0 && !write.empty()) {
            pdt = pull_dtype;
            a.r = static_cast<int>(write.size());
            for (size_t j = 0; j < write.size(); ++j) {
                a.dst[j] = dsts[write[j]];
                level = std::min(level, dst_level(a.dst[j], pull_dtype));
            }
        }
        hipError_t e = run_apply(ps, a, gdt, pdt, level, shape_of(ps, a, gdt, pdt), false);
        if (e != hipSuccess) return fail_hip(e, "apply kernel launch");
        start = end;
    }
    return PS_OK;
}

// Make the server's stream wait (on the device) for every lock-free pull
// enqueued so far. ps_apply_pull marks its replicas current; without this an
// earlier lock-free pull into the same buffer, still running on the pull
// stream, could land after the newer weights.
int order_after_pulls(ps_server *ps) {
    if (!ps->pull_lock_free) return PS_OK;
    hipError_t e = hipEventRecord(ps->pulls_done, ps->pull_stream);
    if (e == hipSuccess) e = hipStreamWaitEvent(ps->stream, ps->pulls_done, 0);
    if (e != hipSuccess) return fail_hip(e, "ordering after lock-free pulls");
    return PS_OK;
}

// `ordered`: on the server's stream, after every earlier apply; otherwise on
// the lock-free pull stream when that mode is on.
int launch_pulls(ps_server *ps, void *const *dsts, int dtype, const std::vector<int> &write,
                 bool ordered) {
    if (write.empty()) return PS_OK;
    if (ps->group.open) {
        if (join_pulls(ps, dsts, dtype, write)) return PS_OK;
        if (int rc = flush_group(ps)) return rc;
    }
    hipStream_t s = (!ordered && ps->pull_lock_free) ? ps->pull_stream : ps->stream;
    gadei::PullArgs a;
    std::memset(&a, 0, sizeof a);
    a.w = ps->w;
    a.n = ps->n;
    a.r = static_cast<int>(write.size());
    int level = 1;
    for (size_t j = 0; j < write.size(); ++j) {
        a.dst[j] = dsts[write[j]];
        level = std::min(level, dst_level(a.dst[j], dtype));
    }
    hipError_t e = run_pull(ps, a, dtype, level, s);
    if (e != hipSuccess) return fail_hip(e, "pull kernel launch");
    return PS_OK;
}

// ---------------------------------------------------------------- checkpoint
//
// File layout (little-endian, as the host writes it):
//   CkptHeader, then learner_ts[n_learner_ts] (uint64), then w[n] (fp32),
//   then v[n] (fp32) when the server has momentum.
// `checksum` is FNV-1a (64-bit) over the header (with `checksum` itself
// zero) and then every byte after it.

struct CkptHeader {
    char magic[8];
    uint32_t version;
    uint32_t has_v;
    uint64_t n;
    float lr;
    float m;
    uint64_t ts;
    int64_t last_served;
    uint64_t n_learner_ts;
    int32_t queue_mode;   // the queue configuration the run was made with:
    int32_t depth;        // a restart under another one would serve the
    int32_t slots;        // gradients in another order
    int32_t reserved;
    uint64_t checksum;
};

constexpr char kMagic[8] = {'G', 'A', 'D', 'E', 'I', 'P', 'S', '1'};
// 2: the checksum covers the header too; 3: the queue configuration is kept
constexpr uint32_t kVersion = 3;
constexpr size_t kChunk = size_t(16) << 20;   // floats per device<->host copy

struct Fnv {
    uint64_t h = 1469598103934665603ull;
    void add(const void *p, size_t bytes) {
        const unsigned char *c = static_cast<const unsigned char *>(p);
        for (size_t i = 0; i < bytes; ++i) {
            h ^= c[i];
            h *= 1099511628211ull;
        }
    }
};

int write_all(FILE *f, const void *p, size_t bytes, Fnv *fnv) {
    if (fnv) fnv->add(p, bytes);
    return std::fwrite(p, 1, bytes, f) == bytes ? PS_OK : fail(PS_EIO, "checkpoint write failed");
}

// Device array -> file, in chunks through a host buffer.
int save_array(FILE *f, const float *dev, size_t n, std::vector<float> &buf, Fnv &fnv) {
    for (size_t off = 0; off < n; off += kChunk) {
        const size_t cnt = std::min(kChunk, n - off);
        hipError_t e = hipMemcpy(buf.data(), dev + off, cnt * sizeof(float), hipMemcpyDeviceToHost);
        if (e != hipSuccess) return fail_hip(e, "checkpoint read-back");
        if (int rc = write_all(f, buf.data(), cnt * sizeof(float), &fnv)) return rc;
    }
    return PS_OK;
}

// Row sets this process mapped with ps_import_rows: first row -> the base
// hipIpcOpenMemHandle returned and the handle it was opened from.
struct Import {
    void *base;
    hipIpcMemHandle_t handle;
};
std::mutex g_import_mu;
std::map<void *, Import> g_imports;

}  // namespace

// A captured script: its device work as one HIP graph, the launches it was
// captured from, and its own copy of the script (ids and buffer lists).
struct ps_graph {
    ps_server *server = nullptr;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    hipEvent_t done = nullptr;   // recorded after each replay
    std::vector<ps_op> ops;
    std::vector<std::vector<int>> ids;
    std::vector<std::vector<void *>> dsts;
    std::vector<LaunchRecord> plan;
};

namespace {

// A plan of at most this many kernels is launched kernel by kernel: the
// runtime takes longer to enqueue a graph than so few launches (1M
// coordinates, us a replay, graph vs launches: 1 kernel 18.5 vs 8.5, 2 kernels
// 16.3 vs 6.5, 4 kernels 15.7 vs 11.9, 6 kernels 16.9 vs 18.3).
constexpr size_t kDirectLaunches = 4;

// Launch a captured plan's kernels as they were captured; `launched` counts
// those before the one that failed.
hipError_t launch_plan(ps_server *ps, const std::vector<LaunchRecord> &plan, size_t &launched) {
    hipError_t e = hipSuccess;
    for (launched = 0; launched < plan.size(); ++launched) {
        const LaunchRecord &r = plan[launched];
        gadei::Shape shape;
        shape.blocks_per_cu = r.blocks_per_cu;
        shape.group = r.group;
        switch (r.kind) {
            case 0:
                e = gadei::launch_apply(r.apply, r.grad_dtype, r.pull_dtype, r.level, shape,
                                        ps->geo, ps->stream);
                break;
            case 1:
                e = gadei::launch_sync(r.apply, r.grad_dtype, r.level, shape, ps->geo, ps->stream);
                break;
            case 2: e = gadei::launch_pull(r.pull, r.pull_dtype, r.level, ps->geo, ps->stream); break;
            default:
                e = gadei::launch_steps(r.apply, r.kind == 4, r.grad_dtype, r.pull_dtype,
                                        r.blocks_per_cu, ps->geo, ps->stream);
        }
        if (e != hipSuccess) break;
    }
    return e;
}

// What a script needs of the server to be captured or replayed: a stream
// other than the legacy null stream (which cannot be captured), ordered
// pulls only (lock-free pulls run on a second stream), and an empty queue
// (so that the script's applies take only its own pushes).
int graph_state(const ps_server *ps) {
    if (ps->stream == nullptr)
        return fail(PS_ESTATE, "graphs need a server stream other than the null stream");
    if (ps->pull_lock_free) return fail(PS_ESTATE, "graphs need ordered pulls");
    if (ps->proto.pending() != 0) return fail(PS_ESTATE, "gradients pending");
    return PS_OK;
}

// The script's calls made for real or, with plan_only, planned and
// committed on the host without launching; the launches land in *rec.
int run_recorded(ps_server *ps, const ps_graph &g, std::vector<LaunchRecord> &rec, bool plan_only) {
    ps->record = &rec;
    ps->plan_only = plan_only;
    int rc;
    try {
        rc = ps_run(ps, g.ops.data(), static_cast<int>(g.ops.size()), nullptr);
    } catch (...) {
        rc = fail(PS_ENOMEM, "host allocation failed");
    }
    ps->record = nullptr;
    ps->plan_only = false;
    return rc;
}

bool same_plan(const std::vector<LaunchRecord> &a, const std::vector<LaunchRecord> &b) {
    return a.size() == b.size() &&
           (a.empty() || std::memcmp(a.data(), b.data(), a.size() * sizeof(LaunchRecord)) == 0);
}

// Waits for the graph's last replay before freeing it.
void free_graph(ps_graph *g) {
    if (g->done) {
        (void)hipEventSynchronize(g->done);
        (void)hipEventDestroy(g->done);
    }
    if (g->exec) (void)hipGraphExecDestroy(g->exec);
    if (g->graph) (void)hipGraphDestroy(g->graph);
    delete g;
}

int run_op(ps_server *ps, const ps_op &o, int index) {
    switch (o.kind) {
        case PS_OP_PUSH: return ps_push_dtype(ps, o.learner_id, o.grad, o.dtype);
        case PS_OP_APPLY: return ps_apply_pending(ps);
        case PS_OP_APPLY_SYNC: return ps_apply_sync(ps);
        case PS_OP_PULL: return ps_pull_many(ps, o.count, o.learner_ids, o.dsts, o.dtype);
        case PS_OP_APPLY_PULL: return ps_apply_pull(ps, o.count, o.learner_ids, o.dsts, o.dtype);
        default: return fail(PS_EINVAL, "op %d: unknown kind %d", index, o.kind);
    }
}

}  // namespace

extern "C" {

const char *ps_last_error(void) { return gadei::last_error(); }

int ps_import_rows(const void *handle, size_t offset, void **first_row) {
    if (handle == nullptr || first_row == nullptr) return fail(PS_EINVAL, "null argument");
    hipIpcMemHandle_t h;
    std::memcpy(&h, handle, sizeof h);
    std::lock_guard<std::mutex> lock(g_import_mu);
    for (const auto &kv : g_imports)
        if (std::memcmp(&kv.second.handle, &h, sizeof h) == 0)
            return fail(PS_EINVAL, "row set already imported in this process");
    void *base = nullptr;
    hipError_t e = hipIpcOpenMemHandle(&base, h, hipIpcMemLazyEnablePeerAccess);
    if (e != hipSuccess) return fail_hip(e, "hipIpcOpenMemHandle");
    // the offset must name a byte of the mapped allocation
    void *range_base = nullptr;
    size_t range_size = 0;
    e = hipMemGetAddressRange(&range_base, &range_size, base);
    if (e != hipSuccess || range_base != base || offset >= range_size) {
        (void)hipIpcCloseMemHandle(base);
        if (e != hipSuccess) return fail_hip(e, "hipMemGetAddressRange");
        return fail(PS_EINVAL, "offset %zu outside the %zu-byte allocation", offset, range_size);
    }
    void *first = static_cast<char *>(base) + offset;
    try {
        g_imports[first] = Import{base, h};
    } catch (...) {
        (void)hipIpcCloseMemHandle(base);
        return fail(PS_ENOMEM, "host allocation failed");
    }
    *first_row = first;
    return PS_OK;
}

int ps_release_rows(void *first_row) {
    void *base = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_import_mu);
        auto it = g_imports.find(first_row);
        if (it == g_imports.end()) return fail(PS_EINVAL, "not a row set imported here");
        base = it->second.base;
        g_imports.erase(it);
    }
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess) e = hipIpcCloseMemHandle(base);
    if (e != hipSuccess) return fail_hip(e, "hipIpcCloseMemHandle");
    return PS_OK;
}

ps_server *ps_create(size_t n_params, float lr, float momentum) {
    if (n_params == 0 || n_params > (size_t(1) << 48)) {
        fail(PS_EINVAL, "n_params must be in [1, 2^48]");
        return nullptr;
    }
    if (!std::isfinite(lr) || !std::isfinite(momentum)) {
        fail(PS_EINVAL, "lr and momentum must be finite");
        return nullptr;
    }
    ps_server *ps = new (std::nothrow) ps_server();
    if (ps == nullptr) {
        fail(PS_ENOMEM, "host allocation failed");
        return nullptr;
    }
    ps->n = n_params;
    ps->lr = lr;
    ps->m = momentum;
    // w and v in one allocation, v one stagger after w's 2 MiB-rounded end
    const size_t bytes = n_params * sizeof(float);
    const size_t v_off = gadei::velocity_offset(bytes);
    hipError_t e = hipGetDevice(&ps->device);
    if (e == hipSuccess)
        e = hipMalloc(&ps->wv_base, (momentum != 0.0f ? v_off + bytes : bytes) + kRowAlign);
    if (e == hipSuccess) {
        char *w = align_up(ps->wv_base, kRowAlign);
        ps->w = reinterpret_cast<float *>(w);
        if (momentum != 0.0f) ps->v = reinterpret_cast<float *>(w + v_off);
        e = hipMemset(ps->w, 0, bytes);
    }
    if (e == hipSuccess && ps->v) e = hipMemset(ps->v, 0, bytes);
    if (e != hipSuccess) {
        fail(e == hipErrorOutOfMemory ? PS_ENOMEM : PS_EHIP, "ps_create: %s", hipGetErrorString(e));
        if (ps->wv_base) (void)hipFree(ps->wv_base);
        delete ps;
        return nullptr;
    }
    for (int b = 1; b <= 4; ++b) ps->geo.lds_for_blocks[b] = gadei::blocks_per_cu_lds(b);
    return ps;
}

void ps_destroy(ps_server *ps) {
    if (ps == nullptr) return;
    {
        PS_LOCK(ps);   // waits for a call still running on another thread
        if (use_device(ps) == PS_OK) {
            (void)hipStreamSynchronize(ps->stream);
            if (ps->pull_lock_free) (void)hipStreamSynchronize(ps->pull_stream);
            for (const RowSet &r : ps->row_sets) (void)hipFree(r.base);
            (void)hipFree(ps->wv_base);
            if (ps->pulls_done) (void)hipEventDestroy(ps->pulls_done);
        }
    }
    delete ps;
}

int ps_alloc_rows(ps_server *ps, int count, int dtype, void **rows) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (count < 1 || count > PS_MAX_ROWS)
        return fail(PS_EINVAL, "row count %d outside [1, %d]", count, PS_MAX_ROWS);
    if (dtype != PS_F32 && dtype != PS_BF16) return fail(PS_EINVAL, "bad row dtype %d", dtype);
    if (rows == nullptr) return fail(PS_EINVAL, "null rows output");
    if (int rc = use_device(ps)) return rc;
    const gadei::RowLayout lay = gadei::row_layout(ps->n * (dtype == PS_BF16 ? 2 : 4), count);
    void *base = nullptr;
    hipError_t e = hipMalloc(&base, lay.span + kRowAlign);
    if (e != hipSuccess)
        return fail(e == hipErrorOutOfMemory ? PS_ENOMEM : PS_EHIP, "ps_alloc_rows: %s",
                    hipGetErrorString(e));
    char *first = align_up(base, kRowAlign) + lay.head;
    try {
        ps->row_sets.push_back(RowSet{base, first, first - lay.head + lay.span});
    } catch (...) {
        (void)hipFree(base);
        return fail(PS_ENOMEM, "host allocation failed");
    }
    for (int i = 0; i < count; ++i) rows[i] = first + static_cast<size_t>(i) * lay.stride;
    return PS_OK;
}

int ps_free_rows(ps_server *ps, void *first_row) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    auto it = std::find_if(ps->row_sets.begin(), ps->row_sets.end(),
                           [&](const RowSet &r) { return r.first == first_row; });
    if (it == ps->row_sets.end()) return fail(PS_EINVAL, "not the first row of a row set");
    if (ps->proto.references(it->first, it->end))
        return fail(PS_ESTATE, "a pending gradient lies in these rows");
    if (int rc = use_device(ps)) return rc;
    if (int rc = drain_pulls(ps)) return rc;
    hipError_t e = hipStreamSynchronize(ps->stream);
    if (e == hipSuccess) e = hipFree(it->base);
    if (e != hipSuccess) return fail_hip(e, "ps_free_rows");
    ps->row_sets.erase(it);
    return PS_OK;
}

int ps_push_async(ps_server *ps, int learner_id, const void *grad, int dtype, void *ready_event) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (grad != nullptr && overlaps_state(ps, grad, ps->n * elem_bytes(dtype)))
        return fail(PS_EINVAL, "gradient buffer overlaps the server's w or v");
    return ps->proto.push(learner_id, dtype, grad, ready_event);
}

int ps_push_dtype(ps_server *ps, int learner_id, const void *grad, int dtype) {
    return ps_push_async(ps, learner_id, grad, dtype, nullptr);
}

int ps_push(ps_server *ps, int learner_id, const void *grad) {
    return ps_push_dtype(ps, learner_id, grad, PS_F32);
}

int ps_apply_pending(ps_server *ps) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (ps->proto.pending() == 0) {
        ps->proto.clear_last();
        return PS_OK;
    }
    if (int rc = use_device(ps)) return rc;
    Batch b;
    ps->proto.plan_async(b);
    static const std::vector<int> none;
    if (int rc = launch_batch(ps, b.items, -1, nullptr, none)) return rc;
    ps->proto.commit_async(b);
    return PS_OK;
}

int ps_apply_sync(ps_server *ps) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (ps->proto.pending() == 0) {
        ps->proto.clear_last();
        return PS_OK;
    }
    Batch b;
    if (int rc = ps->proto.plan_sync(b)) return rc;
    const int gdt = b.items.front().dtype;
    if (int rc = use_device(ps)) return rc;
    ps->group.left = ps->proto.pending() - b.items.size();
    if (ps->group.open &&
        std::all_of(b.items.begin(), b.items.end(), [](const PushDesc &d) {
            return d.ready == nullptr && grad_level(d.grad) == 1;
        })) {
        if (int rc = join_gradients(ps, b.items.data(), static_cast<int>(b.items.size()), gdt, true))
            return rc;
        ps->proto.commit_sync(b);
        return PS_OK;
    }
    if (int rc = flush_group(ps)) return rc;
    if (int rc = wait_ready(ps, b.items)) return rc;
    gadei::ApplyArgs a;
    std::memset(&a, 0, sizeof a);
    a.w = ps->w;
    a.v = ps->v;
    a.n = ps->n;
    a.lr = ps->lr;
    a.m = ps->m;
    a.k = static_cast<int>(b.items.size());
    int level = 1;
    for (size_t j = 0; j < b.items.size(); ++j) {
        a.g[j] = b.items[j].grad;
        level = std::min(level, grad_level(a.g[j]));
    }
    a.fronts_log2 = fronts_for(ps, a, gdt);
    const gadei::Shape shape =
        shape_for(ps, gadei::sync_shape(a.k, a.v != nullptr, gdt == PS_BF16, a.n));
    hipError_t e = run_apply(ps, a, gdt, -1, level, shape, true);
    if (e != hipSuccess) return fail_hip(e, "synchronous step launch");
    ps->proto.commit_sync(b);
    return PS_OK;
}

int ps_pull_many(ps_server *ps, int n, const int *learner_ids, void *const *dsts, int dst_dtype) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    std::vector<int> write;
    if (int rc = ps->proto.plan_pulls(n, learner_ids, dsts, dst_dtype, ps->proto.ts, write))
        return rc;
    if (int rc = check_dsts(ps, n, dsts, dst_dtype)) return rc;
    ps->proto.prepare_pulls(n, learner_ids);
    if (!write.empty()) {
        if (int rc = use_device(ps)) return rc;
        if (int rc = launch_pulls(ps, dsts, dst_dtype, write, false)) return rc;
    }
    ps->proto.commit_pulls(n, learner_ids, dsts, dst_dtype, write, !ps->pull_lock_free);
    return PS_OK;
}

int ps_pull(ps_server *ps, int learner_id, void *dst) {
    return ps_pull_many(ps, 1, &learner_id, &dst, PS_F32);
}

int ps_apply_pull(ps_server *ps, int n, const int *learner_ids, void *const *dsts, int dst_dtype) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (ps->proto.pending() == 0) {
        const int rc = ps_pull_many(ps, n, learner_ids, dsts, dst_dtype);
        if (rc == PS_OK) ps->proto.clear_last();
        return rc;
    }
    Batch b;
    ps->proto.plan_async(b);
    std::vector<int> write;
    const uint64_t ts_after = ps->proto.ts + b.items.size();
    if (int rc = ps->proto.plan_pulls(n, learner_ids, dsts, dst_dtype, ts_after, write))
        return rc;
    if (int rc = check_dsts(ps, n, dsts, dst_dtype)) return rc;
    ps->proto.prepare_pulls(n, learner_ids);
    if (int rc = use_device(ps)) return rc;
    if (!write.empty())
        if (int rc = order_after_pulls(ps)) return rc;
    const int r = static_cast<int>(write.size());
    const bool fuse = ps->fuse_max_r >= 0 ? r <= ps->fuse_max_r
                                           : fuses(ps, r, static_cast<int>(b.items.size()),
                                                   b.items.back().dtype, dst_dtype);
    // Gradients for the scalar kernels join no group: in a script too, their
    // replicas are written by the same rule as outside one.
    const bool joins = ps->group.open &&
                       std::all_of(b.items.begin(), b.items.end(),
                                   [](const PushDesc &d) { return grad_level(d.grad) == 1; });
    if (fuse && !joins) {
        const bool open = ps->group.open;
        if (int rc = flush_group(ps)) return rc;
        ps->group.open = false;
        const int rc = launch_batch(ps, b.items, dst_dtype, dsts, write);
        ps->group.open = open;
        if (rc) return rc;
    } else {
        static const std::vector<int> none;
        if (int rc = launch_batch(ps, b.items, -1, nullptr, none)) return rc;
        if (int rc = launch_pulls(ps, dsts, dst_dtype, write, true)) {
            // the apply is on the stream, its gradients are consumed, unless
            // it was the launch of the joined calls that failed
            if (!ps->group.failed) ps->proto.commit_async(b);
            return rc;
        }
    }
    ps->proto.commit_async(b);
    ps->proto.commit_pulls(n, learner_ids, dsts, dst_dtype, write, true);
    return PS_OK;
}

int ps_drop_learner(ps_server *ps, int learner_id) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    return ps->proto.drop_learner(learner_id);
}

int ps_retire_learner(ps_server *ps, int learner_id) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (int rc = gadei::check_learner(learner_id)) return rc;
    // its gradients stay queued, so they must live in memory the server
    // owns: a borrowed buffer may have gone with the learner
    for (const PushDesc &d : ps->proto.queued_of(learner_id)) {
        const char *g = static_cast<const char *>(d.grad);
        const size_t bytes = ps->n * elem_bytes(d.dtype);
        const bool owned = std::any_of(ps->row_sets.begin(), ps->row_sets.end(), [&](const RowSet &r) {
            return g >= r.first && g <= r.end && bytes <= static_cast<size_t>(r.end - g);
        });
        if (!owned)
            return fail(PS_ESTATE,
                        "learner %d has a queued gradient outside the server's rows; drop it "
                        "(ps_drop_learner) instead",
                        learner_id);
    }
    return ps->proto.retire_learner(learner_id);
}

static_assert(sizeof(hipIpcMemHandle_t) == PS_IPC_HANDLE_BYTES, "IPC handle size");

int ps_export_rows(ps_server *ps, void *first_row, void *handle, size_t *offset) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (handle == nullptr || offset == nullptr) return fail(PS_EINVAL, "null output");
    auto it = std::find_if(ps->row_sets.begin(), ps->row_sets.end(),
                           [&](const RowSet &r) { return r.first == first_row; });
    if (it == ps->row_sets.end()) return fail(PS_EINVAL, "not the first row of a row set");
    if (int rc = use_device(ps)) return rc;
    hipIpcMemHandle_t h;
    hipError_t e = hipIpcGetMemHandle(&h, it->base);
    if (e != hipSuccess) return fail_hip(e, "hipIpcGetMemHandle");
    std::memcpy(handle, &h, sizeof h);
    *offset = static_cast<size_t>(it->first - static_cast<char *>(it->base));
    return PS_OK;
}

int ps_save(ps_server *ps, const char *path) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (path == nullptr) return fail(PS_EINVAL, "null path");
    if (ps->proto.pending() != 0) return fail(PS_ESTATE, "gradients pending");
    if (int rc = use_device(ps)) return rc;
    if (int rc = drain_pulls(ps)) return rc;
    hipError_t e = hipStreamSynchronize(ps->stream);
    if (e != hipSuccess) return fail_hip(e, "hipStreamSynchronize");
    FILE *f = std::fopen(path, "wb");
    if (f == nullptr) return fail(PS_EIO, "cannot open %s for writing", path);
    const gadei::Protocol &pr = ps->proto;
    CkptHeader h;
    std::memset(&h, 0, sizeof h);
    std::memcpy(h.magic, kMagic, sizeof kMagic);
    h.version = kVersion;
    h.has_v = ps->v != nullptr;
    h.n = ps->n;
    h.lr = ps->lr;
    h.m = ps->m;
    h.ts = pr.ts;
    h.last_served = pr.last_served;
    h.n_learner_ts = pr.learner_ts.size();
    h.queue_mode = pr.mode;
    h.depth = pr.depth;
    h.slots = pr.mode == PS_QUEUE_ROUND_ROBIN ? pr.slots : 0;
    Fnv fnv;
    int rc = write_all(f, &h, sizeof h, &fnv);   // checksum still zero here
    std::vector<float> buf;
    if (rc == PS_OK && h.n_learner_ts)
        rc = write_all(f, pr.learner_ts.data(), h.n_learner_ts * sizeof(uint64_t), &fnv);
    if (rc == PS_OK) {
        buf.resize(std::min(kChunk, ps->n));
        rc = save_array(f, ps->w, ps->n, buf, fnv);
    }
    if (rc == PS_OK && ps->v) rc = save_array(f, ps->v, ps->n, buf, fnv);
    if (rc == PS_OK) {
        h.checksum = fnv.h;
        if (std::fseek(f, 0, SEEK_SET) != 0) rc = fail(PS_EIO, "checkpoint seek failed");
        else rc = write_all(f, &h, sizeof h, nullptr);
    }
    if (std::fclose(f) != 0 && rc == PS_OK) rc = fail(PS_EIO, "checkpoint close failed");
    return rc;
}

int ps_load(ps_server *ps, const char *path) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (path == nullptr) return fail(PS_EINVAL, "null path");
    if (ps->proto.pending() != 0) return fail(PS_ESTATE, "gradients pending");
    FILE *f = std::fopen(path, "rb");
    if (f == nullptr) return fail(PS_EIO, "cannot open %s", path);
    CkptHeader h;
    int rc = PS_OK;
    if (std::fread(&h, 1, sizeof h, f) != sizeof h || std::memcmp(h.magic, kMagic, 8) != 0)
        rc = fail(PS_EIO, "%s is not a parameter-server checkpoint", path);
    else if (h.version != kVersion)
        rc = fail(PS_EIO, "checkpoint format version %u; this library reads %u", h.version,
                  kVersion);
    else if (h.n != ps->n || (h.has_v != 0) != (ps->v != nullptr))
        rc = fail(PS_EINVAL, "checkpoint holds %llu params%s; server has %zu%s",
                  static_cast<unsigned long long>(h.n), h.has_v ? " with momentum" : "", ps->n,
                  ps->v ? " with momentum" : "");
    else if (std::memcmp(&h.lr, &ps->lr, sizeof(float)) != 0 ||
             std::memcmp(&h.m, &ps->m, sizeof(float)) != 0)
        rc = fail(PS_EINVAL, "checkpoint lr/momentum differ from the server's");
    else if (h.queue_mode != ps->proto.mode || h.depth != ps->proto.depth ||
             h.slots != (ps->proto.mode == PS_QUEUE_ROUND_ROBIN ? ps->proto.slots : 0))
        rc = fail(PS_EINVAL,
                  "checkpoint queue configuration (mode %d, depth %d, slots %d) differs from "
                  "the server's (mode %d, depth %d, slots %d)",
                  h.queue_mode, h.depth, h.slots, ps->proto.mode, ps->proto.depth,
                  ps->proto.mode == PS_QUEUE_ROUND_ROBIN ? ps->proto.slots : 0);
    else if (h.n_learner_ts > static_cast<uint64_t>(PS_MAX_LEARNERS) || h.last_served < -1 ||
             h.last_served >= PS_MAX_LEARNERS)
        rc = fail(PS_EIO, "corrupt checkpoint (learner table)");
    // read and verify everything before touching the server
    std::vector<uint64_t> lts;
    std::vector<float> w, v;
    Fnv fnv;
    if (rc == PS_OK) {
        CkptHeader z = h;
        z.checksum = 0;
        fnv.add(&z, sizeof z);
        lts.resize(h.n_learner_ts);
        w.resize(h.n);
        if (h.has_v) v.resize(h.n);
        const size_t lb = lts.size() * sizeof(uint64_t), wb = w.size() * sizeof(float);
        if (std::fread(lts.data(), 1, lb, f) != lb || std::fread(w.data(), 1, wb, f) != wb ||
            (h.has_v && std::fread(v.data(), 1, wb, f) != wb))
            rc = fail(PS_EIO, "checkpoint truncated");
        else {
            fnv.add(lts.data(), lb);
            fnv.add(w.data(), wb);
            if (h.has_v) fnv.add(v.data(), wb);
            if (fnv.h != h.checksum) rc = fail(PS_EIO, "checkpoint checksum mismatch");
        }
    }
    std::fclose(f);
    if (rc != PS_OK) return rc;
    if (int rc2 = use_device(ps)) return rc2;
    if (int rc2 = drain_pulls(ps)) return rc2;
    hipError_t e = hipStreamSynchronize(ps->stream);
    if (e == hipSuccess) e = hipMemcpy(ps->w, w.data(), h.n * sizeof(float), hipMemcpyHostToDevice);
    if (e == hipSuccess && ps->v)
        e = hipMemcpy(ps->v, v.data(), h.n * sizeof(float), hipMemcpyHostToDevice);
    if (e != hipSuccess) return fail_hip(e, "checkpoint upload");
    ps->proto.restore(h.ts, static_cast<int>(h.last_served), lts);
    return PS_OK;
}

int ps_set_stream(ps_server *ps, void *hip_stream) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    ps->stream = static_cast<hipStream_t>(hip_stream);
    return PS_OK;
}

int ps_set_queue_depth(ps_server *ps, int depth) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    return ps->proto.set_depth(depth);
}

int ps_set_queue_mode(ps_server *ps, int mode, int slots_per_learner) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    return ps->proto.set_mode(mode, slots_per_learner);
}

int ps_set_pull_fusion(ps_server *ps, int max_replicas) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (max_replicas < -1 || max_replicas > PS_MAX_REPLICAS)
        return fail(PS_EINVAL, "fusion limit %d outside [-1, %d]", max_replicas, PS_MAX_REPLICAS);
    ps->fuse_max_r = max_replicas;
    return PS_OK;
}

int ps_set_fronts(ps_server *ps, int fronts_log2) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (fronts_log2 < -1 || fronts_log2 > 3)
        return fail(PS_EINVAL, "fronts_log2 %d outside [-1, 3]", fronts_log2);
    ps->geo.fronts_log2 = fronts_log2;
    return PS_OK;
}

int ps_set_launch_shape(ps_server *ps, int blocks_per_cu, int group) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (blocks_per_cu < -1 || blocks_per_cu > 4)
        return fail(PS_EINVAL, "blocks_per_cu %d outside [-1, 4]", blocks_per_cu);
    if (group != 0 && group != 4 && group != 8 && group != 12 && group != 16 && group != 24 &&
        group != 32)
        return fail(PS_EINVAL, "group %d is not 0, 4, 8, 12, 16, 24 or 32", group);
    ps->force_blocks_per_cu = blocks_per_cu;
    ps->force_group = group;
    return PS_OK;
}

int ps_set_pull_skip(ps_server *ps, int enabled) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    ps->proto.pull_skip = enabled != 0;
    return PS_OK;
}

int ps_set_weights(ps_server *ps, const float *src) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (src == nullptr) return fail(PS_EINVAL, "null source");
    if (overlaps_state(ps, src, ps->n * sizeof(float)))
        return fail(PS_EINVAL, "source overlaps the server's w or v");
    if (ps->proto.pending() != 0) return fail(PS_ESTATE, "gradients pending");
    if (int rc = use_device(ps)) return rc;
    if (int rc = drain_pulls(ps)) return rc;
    hipError_t e = hipMemcpyAsync(ps->w, src, ps->n * sizeof(float), hipMemcpyDeviceToDevice,
                                  ps->stream);
    if (e != hipSuccess) return fail_hip(e, "weights copy");
    if (ps->v) {
        e = gadei::launch_zero(ps->v, ps->n, ps->stream);
        if (e != hipSuccess) return fail_hip(e, "velocity reset");
    }
    ps->proto.reset();
    return PS_OK;
}

const float *ps_weights(const ps_server *ps) { return ps ? ps->w : nullptr; }
const float *ps_velocity(const ps_server *ps) { return ps ? ps->v : nullptr; }
size_t ps_num_params(const ps_server *ps) { return ps ? ps->n : 0; }
uint64_t ps_timestamp(const ps_server *ps) {
    if (ps == nullptr) return 0;
    PS_LOCK(ps);
    return ps->proto.ts;
}

int ps_pending(const ps_server *ps) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    return static_cast<int>(ps->proto.pending());
}

int ps_last_staleness(const ps_server *ps, int64_t *out, int cap) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (cap < 0 || (cap > 0 && out == nullptr)) return fail(PS_EINVAL, "bad output buffer");
    const std::vector<int64_t> &s = ps->proto.last_staleness;
    const int count = static_cast<int>(s.size());
    for (int i = 0; i < count && i < cap; ++i) out[i] = s[i];
    return count;
}

int ps_last_applied(const ps_server *ps, int *learner_ids, int cap) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (cap < 0 || (cap > 0 && learner_ids == nullptr)) return fail(PS_EINVAL, "bad output buffer");
    const std::vector<int> &a = ps->proto.last_applied;
    const int count = static_cast<int>(a.size());
    for (int i = 0; i < count && i < cap; ++i) learner_ids[i] = a[i];
    return count;
}

int ps_run(ps_server *ps, const ps_op *ops, int count, int *done) {
    if (done) *done = 0;
    if (int rc = check(ps)) return rc;
    if (count < 0 || (count > 0 && ops == nullptr)) return fail(PS_EINVAL, "bad op script");
    PS_LOCK(ps);
    // Calls may go out together as long as they all run on one stream, and the
    // caller has not asked for a gradient group (ps_set_launch_shape), which the
    // kernels of single steps take.
    StepGroup &g = ps->group;
    g.open = !ps->pull_lock_free && ps->force_group == 0;
    g.failed = false;
    g.ops = ops;
    g.count = count;
    g.pushed = 0;
    clear_group(g);
    int rc = PS_OK, completed = 0;
    try {
        for (; completed < count; ++completed) {
            const ps_op &o = ops[completed];
            if (o.kind == PS_OP_PUSH) ++g.pushed;
            else if (is_apply(o)) g.pushed = 0;
            g.at = completed;
            if ((rc = run_op(ps, o, completed)) != PS_OK) break;
        }
    } catch (...) {
        rc = fail(PS_ENOMEM, "host allocation failed");
    }
    // The calls before a refused one are done: they go out now. (fail() is not
    // called on success, so the refusal's message stays.)
    try {
        if (int rc2 = flush_group(ps)) rc = rc2;
    } catch (...) {   // a plan being recorded could not grow: nothing was enqueued
        rc = fail(PS_ENOMEM, "host allocation failed");
        g.failed = true;
    }
    if (done) *done = g.failed ? g.first : completed;
    g.open = g.failed = false;
    ps->proto.forget();
    return rc;
}

int ps_graph_create(ps_server *ps, const ps_op *ops, int count, ps_graph **out) {
    if (out) *out = nullptr;
    if (int rc = check(ps)) return rc;
    if (out == nullptr || count < 1 || ops == nullptr) return fail(PS_EINVAL, "bad graph script");
    PS_LOCK(ps);
    if (int rc = graph_state(ps)) return rc;
    if (int rc = use_device(ps)) return rc;
    ps_graph *g = nullptr;
    try {
        g = new ps_graph;
        g->server = ps;
        g->ops.assign(ops, ops + count);
        g->ids.resize(count);
        g->dsts.resize(count);
        for (int i = 0; i < count; ++i) {
            ps_op &o = g->ops[i];
            if (o.kind == PS_OP_PULL || o.kind == PS_OP_APPLY_PULL) {
                if (o.count < 0 || o.count > PS_MAX_REPLICAS ||
                    (o.count > 0 && (o.learner_ids == nullptr || o.dsts == nullptr))) {
                    free_graph(g);
                    return fail(PS_EINVAL, "op %d: bad pull list", i);
                }
                g->ids[i].assign(o.learner_ids, o.learner_ids + o.count);
                g->dsts[i].assign(o.dsts, o.dsts + o.count);
                o.learner_ids = g->ids[i].data();
                o.dsts = g->dsts[i].data();
            }
        }
    } catch (...) {
        if (g) free_graph(g);
        return fail(PS_ENOMEM, "host allocation failed");
    }
    // Capture: the calls run as usual, their kernels go into the graph
    // instead of running, and the server's host state is put back, since
    // nothing has run yet.
    const gadei::Protocol saved = ps->proto;
    hipError_t e = hipStreamBeginCapture(ps->stream, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) {
        free_graph(g);
        return fail_hip(e, "hipStreamBeginCapture");
    }
    int rc = run_recorded(ps, *g, g->plan, false);
    e = hipStreamEndCapture(ps->stream, &g->graph);
    ps->proto = saved;
    if (rc == PS_OK && e != hipSuccess) rc = fail_hip(e, "hipStreamEndCapture");
    if (rc == PS_OK && g->plan.empty()) rc = fail(PS_EINVAL, "the script launches no kernel");
    if (rc == PS_OK) {
        e = hipGraphInstantiate(&g->exec, g->graph, nullptr, nullptr, 0);
        if (e != hipSuccess) rc = fail_hip(e, "hipGraphInstantiate");
    }
    if (rc == PS_OK) {
        e = hipEventCreateWithFlags(&g->done, hipEventDisableTiming);
        if (e != hipSuccess) rc = fail_hip(e, "hipEventCreateWithFlags");
    }
    if (rc != PS_OK) {
        free_graph(g);
        return rc;
    }
    *out = g;
    return PS_OK;
}

int ps_graph_launch(ps_server *ps, ps_graph *g) {
    if (int rc = check(ps)) return rc;
    if (g == nullptr || g->server != ps) return fail(PS_EINVAL, "not a graph of this server");
    PS_LOCK(ps);
    if (int rc = graph_state(ps)) return rc;
    if (int rc = use_device(ps)) return rc;
    // The calls again, planned and committed on the host only: the replay
    // is valid if they would launch exactly the captured kernels.
    const gadei::Protocol saved = ps->proto;
    std::vector<LaunchRecord> now;
    int rc = run_recorded(ps, *g, now, true);
    if (rc == PS_OK && !same_plan(now, g->plan))
        rc = fail(PS_ESTATE, "the script would now launch other kernels than were captured");
    if (rc == PS_OK) {
        // (a stream that is itself being captured refuses the graph, as ever)
        hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
        const bool direct = g->plan.size() <= kDirectLaunches &&
                            hipStreamIsCapturing(ps->stream, &capturing) == hipSuccess &&
                            capturing == hipStreamCaptureStatusNone;
        size_t launched = 0;
        const hipError_t e =
            direct ? launch_plan(ps, g->plan, launched) : hipGraphLaunch(g->exec, ps->stream);
        if (e == hipSuccess || launched > 0)   // the event only serves destroy
            (void)hipEventRecord(g->done, ps->stream);
        if (e != hipSuccess) {
            ps->proto = saved;
            rc = fail_hip(e, "graph launch");
            if (launched > 0) {
                // kernels that went out before the failing one count: the calls
                // once more, planned as if that launch had failed in ps_run
                now.clear();
                ps->plan_fails = launched;
                ps->plan_error = e;
                rc = run_recorded(ps, *g, now, true);
                ps->plan_fails = ps_server::kNone;
            }
        }
    } else {
        ps->proto = saved;
    }
    return rc;
}

void ps_graph_destroy(ps_graph *g) {
    if (g != nullptr) free_graph(g);
}

int ps_sync(ps_server *ps) {
    if (int rc = check(ps)) return rc;
    hipStream_t s, ps_s;
    bool lock_free;
    {
        // take the streams under the lock, wait without it so that pushes
        // from other threads are not held up by the wait
        PS_LOCK(ps);
        if (int rc = use_device(ps)) return rc;
        s = ps->stream;
        ps_s = ps->pull_stream;
        lock_free = ps->pull_lock_free;
    }
    hipError_t e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail_hip(e, "hipStreamSynchronize");
    if (lock_free) {
        e = hipStreamSynchronize(ps_s);
        if (e != hipSuccess) return fail_hip(e, "hipStreamSynchronize (pull stream)");
    }
    return PS_OK;
}

int ps_record(ps_server *ps, void *event) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (event == nullptr) return fail(PS_EINVAL, "null event");
    if (int rc = use_device(ps)) return rc;
    hipError_t e = hipEventRecord(static_cast<hipEvent_t>(event), ps->stream);
    if (e != hipSuccess) return fail_hip(e, "hipEventRecord");
    return PS_OK;
}

int ps_set_pull_stream(ps_server *ps, void *hip_stream) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (int rc = use_device(ps)) return rc;
    if (int rc = drain_pulls(ps)) return rc;
    if (hip_stream != nullptr && ps->pulls_done == nullptr) {
        hipError_t e = hipEventCreateWithFlags(&ps->pulls_done, hipEventDisableTiming);
        if (e != hipSuccess) {
            ps->pulls_done = nullptr;
            return fail_hip(e, "hipEventCreateWithFlags");
        }
    }
    ps->pull_lock_free = hip_stream != nullptr;
    ps->pull_stream = static_cast<hipStream_t>(hip_stream);
    return PS_OK;
}

int ps_get_stats(const ps_server *ps, ps_stats *out) {
    if (int rc = check(ps)) return rc;
    PS_LOCK(ps);
    if (out == nullptr) return fail(PS_EINVAL, "null stats output");
    *out = ps->proto.stats;
    out->timestamp = ps->proto.ts;
    return PS_OK;
}

}  // extern "C"
