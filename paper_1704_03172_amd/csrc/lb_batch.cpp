// lb_batch.cpp -- batched executor behind the lb_batch_* calls of
// include/lbwave.h: many independent shots of the linear LB scheme advance
// together, in rounds of several steps, each round one launch of the flowing
// kernel over all shots (a shot with fewer steps left takes those), with
// per-shot time and buffer parity kept on the device so that a tick of k steps
// is captured once as a HIP graph and replayed until the set of active shots
// changes.
#include "lbwave.h"
#include "lb_host.h"
#include "lb_internal.h"

#include <algorithm>
#include <cstring>
#include <deque>
#include <new>
#include <vector>

namespace {

constexpr int kGraphRounds = 2;          // rounds of a captured graph
constexpr size_t kStageBytes = 4 << 20;  // pinned staging of the uploads
constexpr size_t kStageFlag = 256;       // its first bytes receive the c^2 check's flag
constexpr int kTickEvents = 64;          // ticks whose completion can be tracked at once

using lbw::align_up;
using lbw::BatchParams;
using lbw::ShotEntry;
using lbw::ShotState;

// Per-set device tables of the active shots (two sets: a rebuild writes the
// set that no tick in flight reads).
struct SetLayout {
    size_t order = 0, prefix = 0;
};

struct BatchLayout {
    size_t table = 0, state = 0, img = 0, scratch = 0, total = 0;
    SetLayout set[2];
};

BatchLayout batch_layout(int32_t max_shots) {
    BatchLayout L;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
    L.table = take((size_t)max_shots * sizeof(ShotEntry));
    L.state = take((size_t)max_shots * sizeof(ShotState));
    for (SetLayout &t : L.set) {
        t.order = take((size_t)max_shots * sizeof(int32_t));
        t.prefix = take(((size_t)max_shots + 1) * sizeof(int32_t));
    }
    L.img = take((size_t)max_shots * sizeof(lbw::FlowParams));
    L.scratch = take(256);
    L.total = off;
    return L;
}

struct ShotLayout {
    int64_t pstride = 0;
    size_t pop0 = 0, pop1 = 0, c2 = 0, wavelet = 0, rrow = 0, rxs = 0, rslot = 0, total = 0;
};

struct DeviceSet {
    int32_t *order = nullptr, *prefix = nullptr;
};

// A tick whose completion is tracked: its event and the host times of every
// slot once it has run (-1: free).
struct TickRecord {
    int64_t id = 0;
    std::vector<int64_t> t;
};

}  // namespace

struct lb_batch {
    lb_grid_desc scheme;
    int q = 5, storage = 0;
    size_t ssize = 4, tsize = 4;
    lbw::Collision coll;
    hipStream_t stream = nullptr;      // ticks
    hipStream_t up = nullptr;          // admission and table uploads
    int use_graph = 0;
    int32_t max_shots = 0;
    ShotEntry *d_table = nullptr;
    ShotState *d_state = nullptr;
    lbw::FlowParams *d_img = nullptr;
    int32_t *d_scratch = nullptr;
    DeviceSet dset[2];
    int set = 0;                       // the set the next ticks read
    hipEvent_t ev_set[2] = {nullptr, nullptr};   // last tick that read each set
    hipEvent_t ev_up = nullptr;        // uploads the next tick must wait for
    bool up_pending = false;
    std::vector<hipEvent_t> ev_slot;   // per slot: work enqueued when it was freed
    char *stage = nullptr;             // pinned staging (reused once `up` is idle)
    std::vector<ShotEntry> table;
    std::vector<char> used;
    std::vector<int64_t> ht, hend;     // host-tracked time and last time per slot
    std::vector<int64_t> admit_tick;   // tick counter when the slot's shot was admitted
    std::vector<int32_t> order;
    std::vector<int32_t> prefix;
    bool small = false;                // shape of the flowing kernel for the active shots
    int steps = 1;                     // steps of a round
    int64_t nodes = 0;                 // of the active shots
    bool dirty = true;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    // tick completion
    hipEvent_t ev_tick[kTickEvents] = {};
    std::deque<TickRecord> pending;    // enqueued ticks, oldest first
    TickRecord done;                   // the newest completed tick
    int64_t ticks = 0;
    int sticky = LB_OK;
};

namespace {

int fail(lb_batch *b, hipError_t e) {
    if (e == hipSuccess) return LB_OK;
    b->sticky = LB_E_HIP;
    return LB_E_HIP;
}

#define BT_TRY(b, expr)                               \
    do {                                              \
        hipError_t e__ = (expr);                      \
        if (e__ != hipSuccess) return fail((b), e__); \
    } while (0)

int check_shot(const lb_shot_desc *s) {
    if (!s) return LB_E_INVALID;
    if (s->nx < 1 || s->ny < 1 || s->ny > 65535 || s->nx > (1 << 24)) return LB_E_RANGE;
    if (s->nsteps < 0 || s->nrec < 0) return LB_E_RANGE;
    if (s->src_x < 0 || s->src_y < 0 || s->src_x >= s->nx || s->src_y >= s->ny) return LB_E_RANGE;
    if (s->sponge_width < 0 || !(s->sponge_sigma_max >= 0.0 && s->sponge_sigma_max <= 1.0)) return LB_E_RANGE;
    return LB_OK;
}

ShotLayout shot_layout(const lb_batch *b, const lb_shot_desc *s) {
    ShotLayout L;
    const int64_t n = (int64_t)s->nx * s->ny;
    L.pstride = lbw::population_stride(n);
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align_up(off + bytes); return o; };
    L.pop0 = take((size_t)b->q * L.pstride * b->ssize);
    L.pop1 = take((size_t)b->q * L.pstride * b->ssize);
    L.c2 = take((size_t)n * b->tsize);
    L.wavelet = take(((size_t)s->nsteps + 1) * sizeof(double));
    L.rrow = take(((size_t)s->ny + 1) * 4);
    L.rxs = take((size_t)std::max(s->nrec, 1) * 4);
    L.rslot = take((size_t)std::max(s->nrec, 1) * 4);
    L.total = off;
    return L;
}

// Staged copy to the device on the upload stream: host bytes go through the
// pinned staging buffer at *off (advanced), so the copy runs without the
// host waiting on it (a pageable source would make the call wait).
int stage_copy(lb_batch *b, void *dst, const void *src, size_t bytes, size_t *off) {
    for (size_t done = 0; done < bytes;) {   // in pieces if it is larger than the buffer
        const size_t n = std::min(bytes - done, kStageBytes - kStageFlag);
        if (*off + n > kStageBytes) {   // full: let the uploads so far finish
            BT_TRY(b, hipStreamSynchronize(b->up));
            *off = kStageFlag;
        }
        std::memcpy(b->stage + *off, (const char *)src + done, n);
        BT_TRY(b, hipMemcpyAsync((char *)dst + done, b->stage + *off, n, hipMemcpyHostToDevice, b->up));
        *off = align_up(*off + n);
        done += n;
    }
    return LB_OK;
}

// Several parts to places that lie within `span` bytes from dst on, at offsets
// from there: one copy for all (the bytes between them are not used), where a
// copy each costs the host 5 us; part by part if they do not fit the staging
// buffer together.
struct Part {
    size_t at;
    const void *src;
    size_t bytes;
};
int stage_parts(lb_batch *b, char *dst, size_t span, const Part *part, int n, size_t *off) {
    if (kStageFlag + span > kStageBytes) {
        for (int i = 0; i < n; ++i) {
            const int rc = stage_copy(b, dst + part[i].at, part[i].src, part[i].bytes, off);
            if (rc) return rc;
        }
        return LB_OK;
    }
    if (*off + span > kStageBytes) {
        BT_TRY(b, hipStreamSynchronize(b->up));
        *off = kStageFlag;
    }
    for (int i = 0; i < n; ++i)
        if (part[i].bytes > 0) std::memcpy(b->stage + *off + part[i].at, part[i].src, part[i].bytes);
    BT_TRY(b, hipMemcpyAsync(dst, b->stage + *off, span, hipMemcpyHostToDevice, b->up));
    *off = align_up(*off + span);
    return LB_OK;
}

// Rebuild the compact list of active shots and their shares of the blocks into
// the set that no tick in flight reads, on the upload stream after the last
// tick that read it; the ticks enqueued from now on read it once the upload
// is done.  *off: staging offset in use.
int rebuild(lb_batch *b, size_t *off) {
    b->order.clear();
    int64_t nodes = 0;
    for (int32_t k = 0; k < b->max_shots; ++k) {
        if (!b->used[(size_t)k]) continue;
        b->order.push_back(k);
        nodes += (int64_t)b->table[(size_t)k].nx * b->table[(size_t)k].ny;
    }
    // one block per CU, shared out by the shots' bundles of rows (each shot
    // at least one block), so that the blocks end at about the same time
    const size_t na = b->order.size();
    const lbw::FlowChoice c = lbw::flow_choose(b->storage, b->q, nodes);
    b->nodes = nodes;
    b->small = c.small;
    b->steps = c.steps;
    if (b->scheme.steps_per_launch > 0) b->steps = std::min(b->steps, (int)b->scheme.steps_per_launch);
    const lbw::FlowInfo f = lbw::flow_info(b->storage, b->q, b->small);
    std::vector<int64_t> bundles(na), blocks(na, 1);
    int64_t all = 0, given = 0;
    for (size_t a = 0; a < na; ++a) {
        const ShotEntry &e = b->table[(size_t)b->order[a]];
        lbw::FlowParams p;
        p.nx = e.nx;
        lbw::flow_strips(f, b->steps, p);
        bundles[a] = (int64_t)p.nstrip * ((e.ny + f.R - 1) / f.R);
        all += bundles[a];
    }
    for (size_t a = 0; a < na; ++a) {
        blocks[a] = std::max<int64_t>(1, std::min(bundles[a], lbw::kFlowBlocks * bundles[a] / all));
        given += blocks[a];
    }
    while (given < lbw::kFlowBlocks) {   // the rest to the longest shares
        size_t best = na;
        for (size_t a = 0; a < na; ++a)
            if (blocks[a] < bundles[a] && (best == na || bundles[a] * blocks[best] > bundles[best] * blocks[a])) best = a;
        if (best == na) break;
        ++blocks[best];
        ++given;
    }
    b->prefix.assign(1, 0);
    for (size_t a = 0; a < na; ++a) b->prefix.push_back(b->prefix.back() + (int32_t)blocks[a]);
    const int ns = 1 - b->set;
    const DeviceSet &d = b->dset[ns];
    BT_TRY(b, hipStreamWaitEvent(b->up, b->ev_set[ns], 0));
    int rc;
    if (!b->order.empty()) {
        const size_t at = (size_t)((char *)d.prefix - (char *)d.order), bytes = b->prefix.size() * 4;
        const Part part[2] = {{0, b->order.data(), b->order.size() * 4}, {at, b->prefix.data(), bytes}};
        if ((rc = stage_parts(b, (char *)d.order, at + bytes, part, 2, off))) return rc;
    }
    BT_TRY(b, hipEventRecord(b->ev_up, b->up));
    b->up_pending = true;
    b->set = ns;
    b->dirty = true;
    return LB_OK;
}

BatchParams params(const lb_batch *b) {
    const DeviceSet &d = b->dset[b->set];
    BatchParams p;
    p.table = b->d_table;
    p.state = b->d_state;
    p.prefix = d.prefix;
    p.order = d.order;
    p.img = b->d_img;
    p.nact = (int32_t)b->order.size();
    p.coll = b->coll;
    return p;
}

// k steps of every active shot (a shot stops at its last step), in rounds of
// b->steps steps; a round of one step goes through the one-step kernel.
int enqueue_steps(lb_batch *b, int64_t k) {
    const BatchParams p = params(b);
    const lbw::FlowInfo f = lbw::flow_info(b->storage, b->q, b->small);
    while (k > 0) {
        const int run = (int)std::min<int64_t>(b->steps, k);
        BT_TRY(b, lbw::launch_batch_prep(p, run, b->steps, f, b->stream));
        if (run > 1) BT_TRY(b, lbw::launch_flow_batch(b->storage, b->q, b->small, p, b->prefix.back(), b->stream));
        else BT_TRY(b, lbw::launch_step_batch(b->storage, b->q, p, b->prefix.back(), b->nodes, b->stream));
        k -= run;
    }
    return LB_OK;
}

// Most steps any active shot has left (host times).
int64_t steps_left(const lb_batch *b) {
    int64_t left = 0;
    for (int32_t s : b->order) left = std::max(left, b->hend[(size_t)s] - b->ht[(size_t)s]);
    return left;
}

void drop_graph(lb_batch *b) {
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    b->exec = nullptr;
    b->graph = nullptr;
}

int capture(lb_batch *b) {
    drop_graph(b);
    BT_TRY(b, hipStreamBeginCapture(b->stream, hipStreamCaptureModeThreadLocal));
    int rc = enqueue_steps(b, kGraphRounds * b->steps);
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(b->stream, &g);
    if (rc) {
        if (g) (void)hipGraphDestroy(g);
        return rc;
    }
    BT_TRY(b, e);
    b->graph = g;
    BT_TRY(b, hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0));
    b->dirty = false;
    return LB_OK;
}

// Host times after k more steps of every active shot.
void advance_host(lb_batch *b, int64_t k) {
    for (int32_t s : b->order) {
        int64_t &t = b->ht[(size_t)s];
        t = std::min(t + k, b->hend[(size_t)s]);
    }
}

// Retire the records of the ticks that have completed (non-blocking).
int collect(lb_batch *b) {
    while (!b->pending.empty()) {
        const hipError_t e = hipEventQuery(b->ev_tick[b->pending.front().id % kTickEvents]);
        if (e == hipErrorNotReady) break;
        BT_TRY(b, e);
        b->done = std::move(b->pending.front());
        b->pending.pop_front();
    }
    return LB_OK;
}

}  // namespace

extern "C" {

size_t lb_batch_workspace_bytes(int32_t max_shots) {
    if (max_shots < 1 || max_shots > (1 << 16)) return 0;
    return batch_layout(max_shots).total;
}

int lb_batch_create(const lb_grid_desc *scheme, int32_t max_shots, void *d_workspace, size_t ws_bytes,
                    void *stream, int use_graph, lb_batch **out) {
    if (!out || !scheme) return LB_E_INVALID;
    *out = nullptr;
    int rc = lbw::validate_scheme(scheme);
    if (rc) return rc;
    if (max_shots < 1 || max_shots > (1 << 16)) return LB_E_RANGE;
    BatchLayout L = batch_layout(max_shots);
    if (!d_workspace || ws_bytes < L.total || ((uintptr_t)d_workspace & 255u)) return LB_E_WORKSPACE;
    lb_batch *b = new (std::nothrow) lb_batch();
    if (!b) return LB_E_INVALID;
    b->scheme = *scheme;
    b->q = scheme->lattice;
    b->storage = lbw::storage_kind(scheme->precision);
    b->ssize = lbw::storage_bytes(scheme->precision);
    b->tsize = lbw::compute_bytes(scheme->precision);
    b->coll = lbw::make_collision(scheme);
    if (scheme->precision == LB_F32) b->coll.written = 0;   // each shot's own
    b->stream = (hipStream_t)stream;
    b->use_graph = use_graph ? 1 : 0;
    b->max_shots = max_shots;
    char *ws = (char *)d_workspace;
    b->d_table = (ShotEntry *)(ws + L.table);
    b->d_state = (ShotState *)(ws + L.state);
    b->d_img = (lbw::FlowParams *)(ws + L.img);
    b->d_scratch = (int32_t *)(ws + L.scratch);
    for (int i = 0; i < 2; ++i) {
        b->dset[i].order = (int32_t *)(ws + L.set[i].order);
        b->dset[i].prefix = (int32_t *)(ws + L.set[i].prefix);
    }
    b->table.assign((size_t)max_shots, ShotEntry());
    b->used.assign((size_t)max_shots, 0);
    b->ht.assign((size_t)max_shots, 0);
    b->hend.assign((size_t)max_shots, 0);
    b->admit_tick.assign((size_t)max_shots, 0);
    b->ev_slot.assign((size_t)max_shots, nullptr);
    bool ok = hipStreamCreateWithFlags(&b->up, hipStreamNonBlocking) == hipSuccess &&
              hipHostMalloc((void **)&b->stage, kStageBytes, hipHostMallocDefault) == hipSuccess &&
              hipEventCreateWithFlags(&b->ev_up, hipEventDisableTiming) == hipSuccess;
    for (int i = 0; ok && i < 2; ++i) ok = hipEventCreateWithFlags(&b->ev_set[i], hipEventDisableTiming) == hipSuccess;
    for (int i = 0; ok && i < kTickEvents; ++i)
        ok = hipEventCreateWithFlags(&b->ev_tick[i], hipEventDisableTiming) == hipSuccess;
    for (int32_t i = 0; ok && i < max_shots; ++i)
        ok = hipEventCreateWithFlags(&b->ev_slot[(size_t)i], hipEventDisableTiming) == hipSuccess;
    // zeroed slot states; the set events mark that nothing reads either set
    ok = ok && lbw::launch_fill_zero(ws + L.state, (int64_t)((size_t)max_shots * sizeof(ShotState)), b->stream) ==
                   hipSuccess;
    for (int i = 0; ok && i < 2; ++i) ok = hipEventRecord(b->ev_set[i], b->stream) == hipSuccess;
    for (int32_t i = 0; ok && i < max_shots; ++i) ok = hipEventRecord(b->ev_slot[(size_t)i], b->stream) == hipSuccess;
    ok = ok && hipStreamSynchronize(b->stream) == hipSuccess;
    b->done.t.assign((size_t)max_shots, -1);
    if (!ok) {
        lb_batch_destroy(b);
        return LB_E_HIP;
    }
    *out = b;
    return LB_OK;
}

size_t lb_shot_workspace_bytes(const lb_batch *b, const lb_shot_desc *s) {
    if (!b || check_shot(s) != LB_OK) return 0;
    return shot_layout(b, s).total;
}

int lb_batch_add_shot(lb_batch *b, const lb_shot_desc *s, void *d_ws, size_t ws_bytes, const void *c2, lb_dtype t,
                      int on_device, const double *wavelet, int64_t nt, const int32_t *rxy, void *d_traces,
                      int32_t *slot) {
    if (!b || !slot || !c2) return LB_E_INVALID;
    *slot = -1;
    if (b->sticky) return b->sticky;
    int rc = check_shot(s);
    if (rc) return rc;
    if (t != LB_F32 && t != LB_F64) return LB_E_INVALID;
    if (nt < 0 || (nt > 0 && !wavelet)) return LB_E_INVALID;
    if (s->nrec > 0 && (!rxy || !d_traces)) return LB_E_INVALID;
    ShotLayout L = shot_layout(b, s);
    if (!d_ws || ws_bytes < L.total || ((uintptr_t)d_ws & 255u)) return LB_E_WORKSPACE;
    for (int32_t r = 0; r < s->nrec; ++r)
        if (rxy[2 * r] < 0 || rxy[2 * r + 1] < 0 || rxy[2 * r] >= s->nx || rxy[2 * r + 1] >= s->ny) return LB_E_RANGE;
    // a free slot, preferring one whose last ticks have run
    int32_t k = -1;
    for (int32_t i = 0; i < b->max_shots; ++i) {
        if (b->used[(size_t)i]) continue;
        if (k < 0) k = i;
        if (hipEventQuery(b->ev_slot[(size_t)i]) == hipSuccess) {
            k = i;
            break;
        }
    }
    if (k < 0) return LB_E_RANGE;

    // everything below runs on the upload stream, so the ticks in flight
    // keep the GPU busy; the host waits only for this shot's uploads (the
    // range check of c^2)
    BT_TRY(b, hipStreamSynchronize(b->up));   // the staging buffer is free
    size_t off = kStageFlag;
    char *ws = (char *)d_ws;
    const int64_t n = (int64_t)s->nx * s->ny;
    if ((rc = lbw::upload_c2(b->up, b->scheme.precision, b->q, b->scheme.d2q9_ratio, ws + L.c2, c2, t, on_device,
                             n, b->d_scratch, (int32_t *)b->stage))) {
        if (rc == LB_E_HIP) b->sticky = LB_E_HIP;
        return rc;
    }
    BT_TRY(b, lbw::launch_fill_zero(ws + L.pop0, (int64_t)(L.c2 - L.pop0), b->up));
    const int64_t nw = std::min<int64_t>(nt, s->nsteps + 1);

    // receiver tables: CSR over rows, x ascending
    struct R { int32_t x, y, slot; };
    std::vector<R> v((size_t)s->nrec);
    for (int32_t r = 0; r < s->nrec; ++r) v[(size_t)r] = {rxy[2 * r], rxy[2 * r + 1], r};
    std::sort(v.begin(), v.end(), [](const R &a, const R &c) {
        return a.y != c.y ? a.y < c.y : (a.x != c.x ? a.x < c.x : a.slot < c.slot);
    });
    std::vector<int32_t> row((size_t)s->ny + 1, 0), xs(v.size()), sl(v.size());
    for (const R &r : v) row[(size_t)r.y + 1]++;
    for (int32_t y = 0; y < s->ny; ++y) row[(size_t)y + 1] += row[(size_t)y];
    for (size_t i = 0; i < v.size(); ++i) {
        xs[i] = v[i].x;
        sl[i] = v[i].slot;
    }
    {   // the wavelet and the tables lie one after the other
        const size_t tables = s->nrec > 0 ? 1 : 0;
        const Part part[4] = {{0, wavelet, (size_t)nw * 8},
                              {L.rrow - L.wavelet, row.data(), tables * row.size() * 4},
                              {L.rxs - L.wavelet, xs.data(), xs.size() * 4},
                              {L.rslot - L.wavelet, sl.data(), sl.size() * 4}};
        const size_t span = tables ? L.rslot - L.wavelet + sl.size() * 4 : (size_t)nw * 8;
        if (span > 0 && (rc = stage_parts(b, ws + L.wavelet, span, part, 4, &off))) return rc;
    }

    ShotEntry e;
    e.pop0 = ws + L.pop0;
    e.pop1 = ws + L.pop1;
    e.c2 = ws + L.c2;
    e.wavelet = (const double *)(ws + L.wavelet);
    e.wavelet_len = nw;
    if (s->nrec > 0) {
        e.rec.row_ptr = (const int32_t *)(ws + L.rrow);
        e.rec.xs = (const int32_t *)(ws + L.rxs);
        e.rec.slot = (const int32_t *)(ws + L.rslot);
        e.rec.traces = d_traces;
        e.rec.nslots = s->nrec;
        e.rec.what = LB_FIELD_P;
        e.rec.cap = s->nsteps + 1;
    }
    e.nx = s->nx;
    e.ny = s->ny;
    e.pstride = L.pstride;
    e.sponge_width = s->sponge_width;
    e.sponge_smax = s->sponge_sigma_max;
    e.src_x = s->src_x;
    e.src_y = s->src_y;
    e.written = b->scheme.precision == LB_F32 && lbw::has_two_forms(&b->scheme) && n <= lbw::kWrittenNodes;

    // collision of time 0 (records time 0): pop0 (at rest) -> pop1
    lbw::StepParams p;
    p.src = e.pop0;
    p.dst = e.pop1;
    p.c2 = e.c2;
    p.nx = e.nx;
    p.ny = e.ny;
    p.pstride = e.pstride;
    p.q = b->q;
    p.coll = b->coll;
    if (e.written) p.coll.written = 1;
    p.sponge_width = e.sponge_width;
    p.sponge_smax = e.sponge_smax;
    p.src_x = e.src_x;
    p.src_y = e.src_y;
    p.s_n = nw > 0 ? wavelet[0] : 0.0;
    p.rec = e.rec;
    p.rec.col = 0;
    BT_TRY(b, lbw::launch_step(b->storage, p, false, b->up));

    // the slot's table entry and state, once no tick in flight can read the
    // slot's previous shot
    ShotState st;
    st.t = 0;
    st.t_end = s->nsteps;
    st.cur = 1;
    st.active = 1;
    BT_TRY(b, hipStreamWaitEvent(b->up, b->ev_slot[(size_t)k], 0));
    if ((rc = stage_copy(b, b->d_table + k, &e, sizeof(e), &off))) return rc;
    if ((rc = stage_copy(b, b->d_state + k, &st, sizeof(st), &off))) return rc;
    b->table[(size_t)k] = e;
    b->used[(size_t)k] = 1;
    b->ht[(size_t)k] = 0;
    b->hend[(size_t)k] = s->nsteps;
    b->admit_tick[(size_t)k] = b->ticks;
    if ((rc = rebuild(b, &off))) return rc;
    *slot = k;
    return LB_OK;
}

int lb_batch_remove_shot(lb_batch *b, int32_t slot) {
    if (!b) return LB_E_INVALID;
    if (b->sticky) return b->sticky;
    if (slot < 0 || slot >= b->max_shots || !b->used[(size_t)slot]) return LB_E_RANGE;
    // an unfinished shot stops in stream order; the slot stays reserved until
    // the work enqueued so far (which may still read it) has run
    if (b->ht[(size_t)slot] < b->hend[(size_t)slot])
        BT_TRY(b, lbw::launch_fill_zero(&b->d_state[slot].active, 4, b->stream));
    BT_TRY(b, hipEventRecord(b->ev_slot[(size_t)slot], b->stream));
    b->used[(size_t)slot] = 0;
    b->table[(size_t)slot] = ShotEntry();
    BT_TRY(b, hipStreamSynchronize(b->up));   // the staging buffer is free
    size_t off = kStageFlag;
    return rebuild(b, &off);
}

int lb_batch_tick(lb_batch *b, int64_t k) {
    if (!b) return LB_E_INVALID;
    if (b->sticky) return b->sticky;
    if (k < 0) return LB_E_RANGE;
    if (k == 0 || b->order.empty()) return LB_OK;
    if ((int64_t)b->pending.size() >= kTickEvents) {   // the oldest tracked tick must have run
        BT_TRY(b, hipEventSynchronize(b->ev_tick[b->pending.front().id % kTickEvents]));
        int rc = collect(b);
        if (rc) return rc;
    }
    if (b->up_pending) {   // the tables and shots uploaded since the last tick
        BT_TRY(b, hipStreamWaitEvent(b->stream, b->ev_up, 0));
        b->up_pending = false;
    }
    int rc;
    const int64_t left = std::min(k, steps_left(b));   // nothing to launch once every shot is at its end
    if (!b->use_graph) {
        if ((rc = enqueue_steps(b, left))) return rc;
    } else {
        // graphs of kGraphRounds rounds, captured again when the set of active
        // shots changes, and replayed; the remainder runs as direct launches
        const int64_t gs = (int64_t)kGraphRounds * b->steps;
        for (int64_t i = 0; i < left / gs; ++i) {
            if (b->dirty || !b->exec)
                if ((rc = capture(b))) return rc;
            BT_TRY(b, hipGraphLaunch(b->exec, b->stream));
        }
        if ((rc = enqueue_steps(b, left % gs))) return rc;
    }
    advance_host(b, k);
    BT_TRY(b, hipEventRecord(b->ev_set[b->set], b->stream));
    TickRecord rec;
    rec.id = ++b->ticks;
    rec.t.assign((size_t)b->max_shots, -1);
    for (int32_t s : b->order) rec.t[(size_t)s] = b->ht[(size_t)s];
    BT_TRY(b, hipEventRecord(b->ev_tick[rec.id % kTickEvents], b->stream));
    b->pending.push_back(std::move(rec));
    return LB_OK;
}

int lb_batch_times(lb_batch *b, int64_t *t_out) {
    if (!b || !t_out) return LB_E_INVALID;
    if (b->sticky) return b->sticky;
    for (int32_t k = 0; k < b->max_shots; ++k) t_out[k] = b->used[(size_t)k] ? b->ht[(size_t)k] : -1;
    return LB_OK;
}

int lb_batch_completed(lb_batch *b, int64_t *t_out) {
    if (!b || !t_out) return LB_E_INVALID;
    if (b->sticky) return b->sticky;
    int rc = collect(b);
    if (rc) return rc;
    for (int32_t k = 0; k < b->max_shots; ++k) {
        const bool valid = b->used[(size_t)k] && b->done.id > b->admit_tick[(size_t)k] && !b->done.t.empty();
        t_out[k] = valid ? b->done.t[(size_t)k] : -1;
    }
    return LB_OK;
}

int lb_batch_sync(lb_batch *b) {
    if (!b) return LB_E_INVALID;
    if (hipStreamSynchronize(b->up) != hipSuccess || hipStreamSynchronize(b->stream) != hipSuccess)
        b->sticky = LB_E_HIP;
    if (!b->sticky) (void)collect(b);
    return b->sticky;
}

int lb_batch_destroy(lb_batch *b) {
    if (!b) return LB_OK;
    hipError_t e = hipSuccess;
    if (b->stream || b->up) {
        const hipError_t e1 = b->up ? hipStreamSynchronize(b->up) : hipSuccess;
        const hipError_t e2 = hipStreamSynchronize(b->stream);
        e = e1 != hipSuccess ? e1 : e2;
    }
    drop_graph(b);
    for (hipEvent_t &ev : b->ev_tick)
        if (ev) (void)hipEventDestroy(ev);
    for (hipEvent_t ev : b->ev_slot)
        if (ev) (void)hipEventDestroy(ev);
    for (hipEvent_t ev : b->ev_set)
        if (ev) (void)hipEventDestroy(ev);
    if (b->ev_up) (void)hipEventDestroy(b->ev_up);
    if (b->stage) (void)hipHostFree(b->stage);
    if (b->up) (void)hipStreamDestroy(b->up);
    int rc = b->sticky ? b->sticky : (e == hipSuccess ? LB_OK : LB_E_HIP);
    delete b;
    return rc;
}

}  // extern "C"
