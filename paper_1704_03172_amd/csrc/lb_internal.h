// lb_internal.h -- kernel parameter blocks and launchers shared by the
// runtime (lb_runtime.cpp) and the kernels (lb_kernels.hip).  Not part of
// the public interface.
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>
#include <type_traits>

namespace lbw {

// Storage formats of the population arrays.
enum Storage : int { ST_F32 = 0, ST_F64 = 1, ST_F16 = 2 };

// Receivers of one grid: a CSR table over rows.  Within row y the entries
// row_ptr[y] .. row_ptr[y+1]-1 hold the receiver x positions in ascending
// order (xs) and the output slot of each (slot).
struct Receivers {
    const int32_t *row_ptr = nullptr;  // [ny + 1]; nullptr: nothing recorded
    const int32_t *xs = nullptr;
    const int32_t *slot = nullptr;
    void *traces = nullptr;            // [nfields][nslots][cap], compute type
    int32_t nslots = 0;                // receivers registered on the handle
    uint32_t what = 0;                 // LB_FIELD_* mask
    int64_t cap = 0;                   // columns per trace
    int64_t col = 0;                   // column written by this launch
};

// Relaxation constants.  For MRT only the non-conserved moments matter:
// srate[k] is s_k / |M_k|^2 for moment k (zero for conserved ones).
struct Collision {
    int32_t kind = 0;                  // LB_BGK or LB_MRT
    double omega = 2.0;                // BGK 1/tau
    double srate[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    double kax = 0.5, kdg = 0.0;       // w_i / c^2 for axis / diagonal movers in the
                                       // equilibrium's J term (2 kax + 4 kdg = 1 exactly
                                       // in the arithmetic type)
    double kw = 0.5;                   // D2Q9 weights: w1 = c^2 kw, kw = 1 / (2 + 4r)
    double ratio = 0.0;                // D2Q9 w5 / w1
    int32_t written = 0;               // the collision's older form (step_kind)
};

// Collision kind the forward kernels are instantiated for: 0 BGK, 1 MRT,
// 2 BGK with omega = 2 (tau = 1/2), whose collision is written as
// 2 g^eq - g.  With `written` 3 more: the same collision with the equilibrium
// of each mover and, for MRT, each moment written out.  Half storage has it (the
// storage turns a last bit into 2^-11 of a value at every step), and so have
// FP32 runs recorded for a gradient and FP32 grids of up to kWrittenNodes: what
// they hold in FP64 (the gradient, the sum of rho) keeps its values, which the
// shorter form moves by 1e-6 and 4e-7, and a small grid has the same bits
// whatever it records.  Larger grids have the shorter form, which is nearer to
// 64 bits (4096^2, 400 steps: 1.1e-6 against 1.6e-6; MRT with a patch on 2048^2
// 3.7e-7 against 1.5e-6).  D2Q9 BGK has one form only.  With 6 more the form is
// each grid's own (batched launches of FP32 shots of all sizes).
// The adjoint keeps Collision::kind.
inline int step_kind(const Collision &c) {
    return (c.kind == 1 ? 1 : c.omega == 2.0 ? 2 : 0) + (c.written ? 3 : 0);
}

// Where the line lies (us per step, written out / shorter): BGK 256^2 1.75 / 1.71,
// 512^2 1.91 / 1.87, 1024^2 2.94 / 2.71, 2048^2 6.4 / 5.7, 4096^2 16.6 / 14.3; MRT
// 256^2 1.95 / 1.78, 512^2 2.18 / 1.96, 1024^2 4.11 / 3.04; D2Q9 MRT 256^2 3.29 /
// 2.75, 512^2 4.14 / 3.53: below it BGK, the usual collision, gains 2 %.
constexpr int64_t kWrittenNodes = 1 << 18;

// f(std::integral_constant<int, KIND>) for the kind of a launch over storage S
// and lattice Q.
template <typename S, int Q, typename F>
hipError_t for_kind(int kind, F &&f) {
    constexpr bool half = sizeof(S) == 2, f32 = sizeof(S) == 4;
    if constexpr (Q == 5 && (half || f32)) {
        if (kind == 3) return f(std::integral_constant<int, 3>());
        if (kind == 5) return f(std::integral_constant<int, 5>());
    }
    if constexpr (half || f32)
        if (kind == 4) return f(std::integral_constant<int, 4>());
    if constexpr (Q != 5 || !half) {
        if (kind == 0) return f(std::integral_constant<int, 0>());
        if (kind == 2) return f(std::integral_constant<int, 2>());
    }
    if constexpr (!half)
        if (kind == 1) return f(std::integral_constant<int, 1>());
    return hipErrorInvalidValue;
}

// The kind of a batched launch: FP32 shots of schemes with two forms have each
// its own.
inline int batch_kind(int storage, int q, const Collision &c) {
    return storage == ST_F32 && (q == 5 || c.kind == 1) ? step_kind(c) % 3 + 6 : step_kind(c);
}
template <typename S, int Q, typename F>
hipError_t for_batch_kind(int kind, F &&f) {
    if constexpr (sizeof(S) == 4) {
        if (kind == 7) return f(std::integral_constant<int, 7>());
        if constexpr (Q == 5) {
            if (kind == 6) return f(std::integral_constant<int, 6>());
            if (kind == 8) return f(std::integral_constant<int, 8>());
        }
    }
    return for_kind<S, Q>(kind, f);
}

// Interface geometry of a factor-2 refinement patch (coarse units).
struct PatchGeom {
    int32_t X0 = 0, Y0 = 0;            // fine node (0, 0) at coarse (X0, Y0)
    int32_t W = 0, H = 0;              // fine grid spans W x H coarse cells
    int32_t nxf = 0, nyf = 0;          // 2W + 1, 2H + 1
    int32_t xa = 0, xb = 0, ya = 0, yb = 0;   // coarse inner ring rectangle
    int32_t nring = 0;                 // fine outer ring nodes
    int32_t ninner = 0;                // coarse inner ring nodes
    int32_t nsnap = 0;                 // coarse ring-line snapshot nodes
};

// A grid as seen by the interface kernels.
struct GridRef {
    const void *pop = nullptr;         // populations to read
    int32_t pre = 0;                   // 1: pop holds the pre-collision state
    const void *c2 = nullptr;
    int32_t nx = 0, ny = 0;
    int64_t pstride = 0;
};

struct InterfaceParams {
    PatchGeom g;
    GridRef coarse;                    // coarse state read
    GridRef fine;                      // fine state read (restriction)
    void *snap = nullptr;              // [5][nsnap] ring-line snapshot of time T
    double a_snap = 0.0, a_now = 1.0;  // prolongation: a_snap*snap + a_now*coarse
    void *dst = nullptr;               // populations written (fine or coarse)
    const void *dst_c2 = nullptr;      // c^2 of the written grid
    int32_t dst_nx = 0, dst_ny = 0;
    int64_t dst_pstride = 0;
    double f = 1.0;                    // non-equilibrium rescaling factor
    Collision coll;                    // collision of the written grid
    int32_t sponge_width = 0;          // sponge of the written grid
    double sponge_smax = 0.0;
    uint32_t field = 0;                // nonzero: write this LB_FIELD_* of the
    void *field_out = nullptr;         // interface state instead of populations
    void *ring_out = nullptr;          // prolongation pair: [2][5][nring] post-collision
                                       // ring states of fine times T+1 (mid), T+2 (end)
};

// Times of the launches of a captured graph that lb_step_n replays: the
// launches carry times relative to the first time t0 of the replayed chunk,
// and t0 and the chunk's source amplitudes s[k] = S(t0 + 1 + k) sit here, in
// device memory that the host fills (one small launch) before each replay.
constexpr int kGraphMaxSteps = 256;
struct GraphTab {
    int64_t t0 = 0;
    int64_t pad = 0;
    double s[kGraphMaxSteps] = {};
};

// One launch of the fused step (or of the collide-only variant).
struct StepParams {
    const void *src = nullptr;         // populations read
    void *dst = nullptr;               // populations written
    const void *c2 = nullptr;          // c^2 per node, compute type
    int32_t nx = 0, ny = 0;
    int64_t pstride = 0;               // elements between populations
    int32_t q = 5;
    Collision coll;
    int32_t sponge_width = 0;
    double sponge_smax = 0.0;
    int32_t src_x = -1, src_y = -1;    // source node
    double s_n = 0.0;                  // source amplitude of this time
    Receivers rec;
    double *sum = nullptr;             // partial sums of rho, one per row and strip of the flowing
    int32_t sum_v = 1, sum_hx = 0;     // kernel (nullptr: off): its columns per lane, halo columns
    int32_t sum_nstrip = 0;            // and strips
    void *rho_out = nullptr;           // [ny][nx] pre-collision rho (nullptr: off)
    void *snap = nullptr;              // refinement ring-line snapshot [5][snap_n]
    int32_t snap_x0 = 0, snap_y0 = 0;  // ring line: rows Y0, Y0+H over x in
    int32_t snap_w = 0, snap_h = 0;    // [X0-1, X0+W+1]; columns X0, X0+W over
    int32_t snap_n = 0;                // y in [Y0-1, Y0+H+1]
    const void *ring_buf = nullptr;    // fine grid of a patch: post-collision outer-ring
    int32_t ring_n = 0;                // states [5][ring_n] taken from the coarse grid
    int32_t restrict_on = 0;           // fine grid of a patch: also write the coarse
                                       // inner ring from this launch's pre-collision
                                       // state (iface: as for launch_restrict)
    int32_t prolong_on = 0;            // coarse grid of a patch: also compute the fine
                                       // outer-ring pair (iface: as launch_prolong_pair)
    InterfaceParams iface;
    int32_t pre_rows = 0;              // set by launch_step: leading block rows that
                                       // do the prolong_on work
    int32_t x0 = 0, x1 = 0;            // region updated, [x0, x1) x [y0, y1) (x1 = 0: the whole
    int32_t y0 = 0, y1 = 0;            // grid), of a destination with a population stride of its
    int64_t dst_pstride = 0;           // own; the region's neighbours are read from src
    const GraphTab *gtab = nullptr;    // graph replay: rec.col is relative to gtab->t0 and
    int32_t goff = 0;                  // the source amplitude is gtab->s[goff]
};

// One launch of the flowing kernel (lb_flow.h): nrun steps h(n) -> h(n + nrun)
// of one grid.  Kernels read it with scalar loads, from their arguments or
// from a batch's params images.
constexpr int kFlowSteps = 16;             // most steps of a launch
constexpr int kFlowPlain = 4;              // weights of a bundle of rows in a block's share: away from
constexpr int kFlowSponge = 5;             // the side edges, and in a strip that meets a side edge's sponge
constexpr int kFlowBlocks = 256;           // one block per CU
struct FlowParams {
    const void *src = nullptr;         // h(n)
    void *dst = nullptr;               // h(n + nrun): another buffer
    const void *c2 = nullptr;
    int32_t nx = 0, ny = 0;
    int64_t pstride = 0;
    int32_t nrun = 0;
    int32_t hx = 0;                    // halo columns on each side of a strip (a multiple of the
                                       // lane's columns, at least nrun)
    int32_t nstrip = 0;                // strips, the first nl and the last nr of which
    int32_t nl = 0, nr = 0;            // meet the sponge of a side edge
    int32_t nblk = 0;                  // blocks of the grid
    int32_t sponge_width = 0;
    int32_t src_x = -1, src_y = -1;
    int32_t goff = 0;                  // graph replay, as in StepParams
    double sponge_smax = 0.0;
    Collision coll;
    Receivers rec;                     // col: the column of time n + 1
    void *rho_out = nullptr;           // pre-collision rho of time n + s at rho_out + (s - 1) *
    int64_t rho_stride = 0;            // rho_stride (nullptr: off)
    double *sum = nullptr;             // partial sums of rho of time n + s, one per row and strip,
    int64_t sum_stride = 0;            // at sum + (s - 1) * sum_stride (nullptr: off)
    const GraphTab *gtab = nullptr;
    double s[kFlowSteps] = {};         // source amplitudes of times n + 1 ..
};

// The fine steps of one coarse step of a refined grid in one launch of the
// flowing kernel: f is the fine grid's (f.nrun = 2, receivers recorded at the
// last step only, into column f.rec.col + nrun - 1); after each step the outer
// ring takes its states from ring ([nrun][5][ring_n]); the last step writes
// the coarse inner ring from its pre-collision state (iface, as for
// launch_restrict).
struct FlowPatchParams {
    FlowParams f;
    const void *ring = nullptr;
    int32_t ring_n = 0;
    InterfaceParams iface;
};
hipError_t launch_flow_patch(int storage, const FlowPatchParams &p, hipStream_t s);
// Its strips and blocks.
void flow_patch_geometry(int storage, FlowParams &p);

// The active shots of a batched launch.
struct FlowBatch {
    const FlowParams *img = nullptr;   // [max_shots] params of the round (nullptr: a single grid)
    const int32_t *order = nullptr;    // [nact] slot of each active shot
    const int32_t *prefix = nullptr;   // [nact + 1] first block of each active shot
    int32_t nact = 0;
};

// Shape of the flowing kernel for a storage format and lattice (small: the
// one for grids too small to give every CU rows enough of the wide strips).
struct FlowInfo {
    int32_t V = 1, R = 1;              // columns per lane, rows per bundle
    int32_t steps = 1;                 // most steps per launch
};
FlowInfo flow_info(int storage, int q, bool small);
// The shape and the steps per launch for `nodes` lattice nodes advanced
// together (a grid, or all shots of a batch).
struct FlowChoice {
    bool small = false;
    int32_t steps = 1;
};
FlowChoice flow_choose(int storage, int q, int64_t nodes);
// Halo and strips of a grid for launches of up to `steps` steps: fills hx,
// nstrip, nl and nr of p from its nx and sponge_width.  The halo is rounded up
// to 8 columns: the strips' stored columns then start on 32-byte boundaries
// (FP32 storage) or better (4096^2, D2Q5 FP32: 14 steps per launch with 16
// halo columns 17.3 us per step, with 14 18.2; 10 steps 20.0 against 22.4).
__host__ __device__ inline void flow_strips(const FlowInfo &f, int steps, FlowParams &p) {
    p.hx = (steps + 7) / 8 * 8;
    const int ow = 64 * f.V - 2 * p.hx, L = p.sponge_width;
    p.nstrip = (p.nx + ow - 1) / ow;
    p.nl = p.nr = 0;
    if (L > 0) {
        const int64_t nl = ((int64_t)L + p.hx + ow - 1) / ow;                      // strips with sx ow - hx < L
        const int64_t r0 = (int64_t)p.nx - L + p.hx - 64 * f.V + 1;                // and with sx ow >= r0
        p.nl = (int32_t)(nl < p.nstrip ? nl : p.nstrip);
        const int64_t first = r0 > 0 ? (r0 + ow - 1) / ow : 0;
        if (first < p.nstrip) p.nr = p.nstrip - (int32_t)(first > p.nl ? first : p.nl);
    }
}
// The same, and the number of blocks (at most `blocks`).
void flow_geometry(const FlowInfo &f, int steps, int blocks, FlowParams &p);

// One backward step of the discrete adjoint (misfit gradient w.r.t. c^2):
// lambda(n) = K^T (1 - sigma) P^T lambda(n+1) + r(n), with the gradient
// terms of time n accumulated into grad (FP64).
struct AdjointParams {
    const void *lam_next = nullptr;    // lambda(n+1) [q][pstride], compute type
    void *lam = nullptr;               // lambda(n) written
    const void *rho = nullptr;         // forward pre-collision rho(n) [ny][nx]
    const void *c2 = nullptr;
    double *grad = nullptr;            // [ny][nx]
    int32_t nx = 0, ny = 0;
    int64_t pstride = 0;
    int32_t q = 5;
    Collision coll;
    double dw[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};   // d w_i / d c^2
    int32_t sponge_width = 0;
    double sponge_smax = 0.0;
    int32_t src_x = -1, src_y = -1;
    double s_n = 0.0;                  // S(n)
    Receivers rec;                     // tables + residual array in `traces`
    int32_t terminal = 0;              // 1: n = N (no step, lambda(N+1) = 0)
    int32_t initial = 0;               // 1: n = 0, add the initial-state term
};

// One launch of the backward flowing kernel (lb_flow_adjoint.hip): the nrun
// backward steps of times n, n - 1, .., n - nrun + 1, none of them the
// terminal one.  f: src lambda(n + 1), dst lambda(n - nrun + 1), s[k] = S(n - k),
// rec the receivers with the residuals as traces and col = n; rho_out,
// rho_stride, sum, sum_stride and gtab are not used.
struct AdjointFlowParams {
    FlowParams f;
    const void *rho = nullptr;         // forward pre-collision rho(n) [ny][nx]; that of time
    int64_t rho_back = 0;              // n - k at rho - k * rho_back elements
    double *grad = nullptr;            // [ny][nx]
    double dw[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    int32_t initial_stage = 0;         // k + 1 where time n - k is 0 (0: none)
};

// Field extraction: one field of the state at the current time.
struct FieldParams {
    const void *pop = nullptr;
    int32_t pre = 0;                   // 1: direct read; 0: pull from post-collision
    const void *c2 = nullptr;
    int32_t nx = 0, ny = 0;
    int64_t pstride = 0;
    int32_t q = 5;
    uint32_t what = 0;
    void *out = nullptr;
};

// One shot of the batched executor (serving).  Static description, written
// by the host when the shot is admitted.
struct ShotEntry {
    void *pop0 = nullptr, *pop1 = nullptr;   // population buffers A / B
    const void *c2 = nullptr;
    const double *wavelet = nullptr;         // S(n), n < wavelet_len
    int64_t wavelet_len = 0;
    Receivers rec;                           // col is set per launch
    int32_t nx = 0, ny = 0;
    int64_t pstride = 0;
    int32_t sponge_width = 0;
    double sponge_smax = 0.0;
    int32_t src_x = -1, src_y = -1;
    int32_t written = 0;                     // the collision's older form (FP32 schemes with two)
};

// Dynamic state of a shot, advanced on the device.
struct ShotState {
    int64_t t = 0;                           // time of the newest state
    int64_t t_end = 0;                       // last time to compute
    int32_t cur = 0;                         // buffer holding h(t): 0 = A
    int32_t active = 0;
};

struct BatchParams {
    const ShotEntry *table = nullptr;        // [max_shots]
    ShotState *state = nullptr;              // [max_shots]
    const int32_t *prefix = nullptr;         // [nact + 1] first block of each active shot
    const int32_t *order = nullptr;          // [nact] slot of each active shot
    FlowParams *img = nullptr;               // [max_shots] params images of the round
    int32_t nact = 0;
    Collision coll;
};

inline FlowBatch flow_batch(const BatchParams &bp) {
    FlowBatch fb;
    fb.img = bp.img;
    fb.order = bp.order;
    fb.prefix = bp.prefix;
    fb.nact = bp.nact;
    return fb;
}

// Launchers (lb_kernels.hip).  All return the launch status.
hipError_t launch_adjoint(int storage, const AdjointParams &p, hipStream_t s);
// The shape and the steps per launch of the backward flowing kernel; its
// launch: 2 <= f.nrun <= flow_adjoint_info().steps.
FlowInfo flow_adjoint_info(int storage, int q, bool small);
FlowChoice flow_adjoint_choose(int storage, int q, int64_t nodes);
hipError_t launch_flow_adjoint(int storage, int q, bool small, const AdjointFlowParams &p, hipStream_t s);
// Trace misfit: res = traces - obs over columns 0 .. ncols-1 of nrec rows of
// cap columns, and phi = 1/2 sum res^2 (FP64) through misfit_blocks(nrec,
// ncols) block partials in `partial` (at most kMisfitMaxBlocks doubles), then
// one finalize block; the result depends only on the inputs (fixed order).
constexpr int kMisfitMaxBlocks = 2048;
int misfit_blocks(int32_t nrec, int64_t ncols);
hipError_t launch_misfit(int storage, const void *traces, const void *obs, void *res, int32_t nrec,
                         int64_t cap, int64_t ncols, double *phi, double *partial, hipStream_t s);
hipError_t launch_step(int storage, const StepParams &p, bool pull,
                       hipStream_t s);
// p.nrun steps of one grid in one launch of the flowing kernel, geometry as
// flow_geometry() filled it for the same shape.  1 <= p.nrun <=
// flow_info().steps, p.hx >= p.nrun.
hipError_t launch_flow(int storage, int q, bool small, const FlowParams &p, hipStream_t s);
// One round of a batch: prep writes the params image of every active shot for
// min(run, steps left) steps (nrun = 0: none) with halos for `steps` steps and
// moves the shot's state past them; the launch takes nblk blocks over the
// images.
hipError_t launch_batch_prep(const BatchParams &bp, int run, int steps, const FlowInfo &f, hipStream_t s);
hipError_t launch_flow_batch(int storage, int q, bool small, const BatchParams &bp, int64_t nblk, hipStream_t s);
// The same for a round of one step, through the one-step kernel; nodes: of the
// active shots together.
hipError_t launch_step_batch(int storage, int q, const BatchParams &bp, int64_t nblk, int64_t nodes, hipStream_t s);
// Sums of `times` (at most kFlowSteps) consecutive groups of n partials to out[0 ..], or
// (gtab set: a replayed graph) to out[gtab->t0 ..].
// fold: kFlowSteps * kSumFolds doubles of scratch.
constexpr int kSumFolds = 64;
hipError_t launch_sum_finalize(const double *partial, int64_t n, int times, double *fold,
                               double *out, const GraphTab *gtab, hipStream_t s);
// *dst = val on the device, in stream order (before a graph replay).
hipError_t launch_graph_prime(GraphTab *dst, const GraphTab &val, hipStream_t s);
hipError_t launch_equilibrium(int storage, int32_t q, void *pop,
                              int64_t pstride, const void *c2,
                              const void *rho, const void *jx, const void *jy,
                              int in_f64, int32_t nx, int32_t ny,
                              const Collision &coll, hipStream_t s);
hipError_t launch_convert_c2(int storage, const void *in, int in_f64,
                             void *out, int64_t n, double c2max,
                             int32_t *bad_count, hipStream_t s);
hipError_t launch_fill_zero(void *p, int64_t bytes, hipStream_t s);
hipError_t launch_field(int storage, const FieldParams &p, hipStream_t s);
hipError_t launch_prolong(int storage, const InterfaceParams &p,
                          hipStream_t s);
hipError_t launch_restrict(int storage, const InterfaceParams &p,
                           hipStream_t s);
// The fine outer-ring states of one coarse step (p.ring_out), see
// InterfaceParams::ring_out.
hipError_t launch_prolong_pair(int storage, const InterfaceParams &p, hipStream_t s);
// The ring-line snapshot (p.snap) of the time of p.coarse.
hipError_t launch_ring_line(int storage, const InterfaceParams &p, hipStream_t s);
hipError_t launch_copy(void *dst, const void *src, size_t bytes,
                       hipStream_t s);

}  // namespace lbw
