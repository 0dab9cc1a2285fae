// lb_flow.hip -- host side of the flowing kernels (lb_flow.h, instantiated per
// storage format and lattice in lb_flow_{f32,f64,f16}_*.hip, and backwards
// lb_flow_adjoint.h, lb_flow_adjoint_*.hip): shapes, geometry, argument
// checks and dispatch, and the batched executor's per-shot params and advance.
#include "lb_flow_adjoint.h"

#include <algorithm>

namespace lbw {
namespace {

constexpr int kAdvBlock = 256;

// Params images of a batched round (see launch_batch_prep).
__global__ __launch_bounds__(kAdvBlock) void k_batch_prep(BatchParams bp, int run, int steps, FlowInfo f) {
    const int a = blockIdx.x * kAdvBlock + threadIdx.x;
    if (a >= bp.nact) return;
    const int slot = bp.order[a];
    const ShotState ss = bp.state[slot];
    const ShotEntry &e = bp.table[slot];
    FlowParams p;
    p.src = ss.cur ? e.pop1 : e.pop0;
    p.dst = ss.cur ? e.pop0 : e.pop1;
    p.c2 = e.c2;
    p.nx = e.nx;
    p.ny = e.ny;
    p.pstride = e.pstride;
    p.sponge_width = e.sponge_width;
    p.sponge_smax = e.sponge_smax;
    flow_strips(f, steps, p);
    p.nblk = bp.prefix[a + 1] - bp.prefix[a];
    p.src_x = e.src_x;
    p.src_y = e.src_y;
    p.coll = bp.coll;
    if (e.written) p.coll.written = 1;
    p.rec = e.rec;
    const int64_t tn = ss.t + 1;
    p.rec.col = tn;
    for (int k = 0; k < kFlowSteps; ++k) p.s[k] = tn + k < e.wavelet_len ? e.wavelet[tn + k] : 0.0;
    p.nrun = ss.active && ss.t < ss.t_end ? (int)min<int64_t>(run, ss.t_end - ss.t) : 0;
    bp.img[slot] = p;
    if (p.nrun > 0) {   // the state after the round
        bp.state[slot].t = ss.t + p.nrun;
        bp.state[slot].cur = ss.cur ^ 1;
    }
}

hipError_t dispatch(int storage, int q, bool small, const FlowParams &p, const FlowBatch &fb, int64_t nblk,
                    int kind, hipStream_t s) {
    if (storage == ST_F32) return q == 5 ? launch_flow_f32_q5(small, p, fb, nblk, kind, s) : launch_flow_f32_q9(small, p, fb, nblk, kind, s);
    if (storage == ST_F64) return q == 5 ? launch_flow_f64_q5(small, p, fb, nblk, kind, s) : launch_flow_f64_q9(small, p, fb, nblk, kind, s);
    return q == 5 ? launch_flow_f16_q5(small, p, fb, nblk, kind, s) : launch_flow_f16_q9(small, p, fb, nblk, kind, s);
}

// What the kernels take for granted: halos of whole lanes, wide enough, and
// every column and bundle in some strip and block.
bool flow_fits(const FlowInfo &f, const FlowParams &p) {
    return p.nx >= 1 && p.ny >= 1 && p.nrun >= 1 && p.nrun <= f.steps && p.hx >= p.nrun && p.hx % f.V == 0 &&
           2 * p.hx < 64 * f.V && p.nblk >= 1 && p.nl >= 0 && p.nr >= 0 && p.nl + p.nr <= p.nstrip &&
           (int64_t)p.nstrip * (64 * f.V - 2 * p.hx) >= p.nx;
}

}  // namespace

FlowInfo flow_info(int storage, int q, bool small) {
    if (storage == ST_F32) return q == 5 ? flow_info_f32_q5(small) : flow_info_f32_q9(small);
    if (storage == ST_F64) return q == 5 ? flow_info_f64_q5(small) : flow_info_f64_q9(small);
    return q == 5 ? flow_info_f16_q5(small) : flow_info_f16_q9(small);
}

// Measured with a 64-node sponge and 64 receivers on square grids (us per step
// in calls of 97 steps; small shape / wide one, each at its best step count):
//   FP32 D2Q5   512^2 1.84 (8 steps) / 2.20 (16)    768^2 2.48 (8) / 2.50 (12)
//               1024^2 3.29 (8) / 2.84 (12)
//   FP64 D2Q5   768^2 2.99 (8) / 2.92 (8)           1024^2 4.40 (8) / 3.70 (8)
//   FP32 D2Q9   2048^2 14.6 (8) / 15.3 (8)          2400^2 19.1 (8) / 19.2 (8)
//               2700^2 30.9 (8) / 24.8 (8)
//   FP64 D2Q9   512^2 3.85 (6) / 4.08 (8)           600^2 4.71 (6) / 4.62 (8)
//               800^2 6.88 (6) / 6.57 (8)
// More steps per launch cost halo rows and columns computed twice, fewer cost
// launches and passes over memory.  Small shape: 16 steps pay while the GPU is
// not filled by the rows a block stores (FP32 D2Q5 128^2 1.41 at 16 steps,
// 1.61 at 8; 256^2 1.67 at 8, 1.78 at 12), after that the narrow strips' halo
// columns of 8 steps do.  Wide shape: 16 steps need grids whose blocks have
// many more rows than the 2 x 16 at their head (FP32 D2Q5 1024^2 2.84 at 12
// steps, 3.19 at 16; 1600^2 4.23 and 4.57; 1700^2 4.95 and 4.75; 4096^2 17.3
// and 14.1; half storage 2048^2 7.50 and 7.69; FP64 D2Q5 1024^2 3.70 at 8, 4.36
// at 16; 1448^2 6.68 and 6.40).  D2Q9's and FP64's larger states leave fewer
// waves per CU, which then wait for each other beyond 8 steps (FP32 D2Q9
// 4096^2 43.9 at 8 steps, 53.1 at 12).
FlowChoice flow_choose(int storage, int q, int64_t nodes) {
    FlowChoice c;
    const bool f64 = storage == ST_F64;
    c.small = nodes < (q == 5 ? 800000 : f64 ? 320000 : 5500000);
    if (q == 9) c.steps = !c.small ? 8 : f64 ? 6 : nodes <= 32768 ? 12 : 8;
    else if (c.small) c.steps = nodes <= 32768 ? 16 : 8;
    else if (f64) c.steps = nodes < 1600000 ? 8 : 16;
    else c.steps = nodes < (storage == ST_F16 ? 4500000 : 2700000) ? 12 : 16;
    return c;
}

void flow_geometry(const FlowInfo &f, int steps, int blocks, FlowParams &p) {
    flow_strips(f, steps, p);
    const int64_t bundles = (int64_t)p.nstrip * ((p.ny + f.R - 1) / f.R);
    p.nblk = (int32_t)std::max<int64_t>(1, std::min<int64_t>(blocks, bundles));
}

hipError_t launch_flow(int storage, int q, bool small, const FlowParams &p, hipStream_t s) {
    if ((q != 5 && q != 9) || !flow_fits(flow_info(storage, q, small), p)) return hipErrorInvalidValue;
    return dispatch(storage, q, small, p, FlowBatch(), p.nblk, step_kind(p.coll), s);
}

namespace {
template <typename S>
FlowInfo patch_info() {
    static_assert(flow_steps_ok(2, PatchShape<S>::R, PatchShape<S>::W, PatchShape<S>::E));
    FlowInfo f;
    f.V = PatchShape<S>::V;
    f.R = PatchShape<S>::R;
    f.steps = 2;
    return f;
}
FlowInfo patch_info(int storage) {
    return storage == ST_F64 ? patch_info<double>() : storage == ST_F32 ? patch_info<float>() : patch_info<_Float16>();
}
}  // namespace

// Halos of exactly two columns (the odd rows of a fine grid start anywhere) and
// as many blocks as run at once.
void flow_patch_geometry(int storage, FlowParams &p) {
    const FlowInfo f = patch_info(storage);
    p.hx = 2;
    const int ow = 64 * f.V - 2 * p.hx;
    p.nstrip = (p.nx + ow - 1) / ow;
    p.nl = p.nr = 0;
    const int64_t bundles = (int64_t)p.nstrip * ((p.ny + f.R - 1) / f.R);
    p.nblk = (int32_t)std::max<int64_t>(1, std::min<int64_t>((storage == ST_F64 ? 1 : 2) * kFlowBlocks, bundles));
}

hipError_t launch_flow_patch(int storage, const FlowPatchParams &p, hipStream_t s) {
    if (p.ring == nullptr || p.f.nrun != 2 || p.f.nx < 16 || p.f.ny < 16 || !flow_fits(patch_info(storage), p.f)) return hipErrorInvalidValue;
    if (storage == ST_F32) return launch_flow_patch_f32(p, s);
    if (storage == ST_F64) return launch_flow_patch_f64(p, s);
    return launch_flow_patch_f16(p, s);
}

FlowInfo flow_adjoint_info(int storage, int q, bool small) {
    if (storage == ST_F64) return q == 5 ? flow_adjoint_info_f64_q5(small) : flow_adjoint_info_f64_q9(small);
    return q == 5 ? flow_adjoint_info_f32_q5(small) : flow_adjoint_info_f32_q9(small);
}

// Measured as above, with a tape (us per backward step at 8 / 16 steps per
// launch, the best shape): FP32 D2Q5 128^2 4.39 / 4.24, 256^2 3.44 / 3.16,
// 512^2 3.27 / 3.73, 1024^2 5.43 / 6.78 (small shape; the wide one 7.07 / 6.72),
// 2048^2 13.3 / 12.4; FP64 D2Q5 256^2 3.73 / 3.43, 1024^2 7.00 / 7.69, 2048^2
// 23.7 / 22.7; FP32 D2Q9 (8 / 12 steps) 1024^2 8.38 / 10.8, 2048^2 23.7 / 27.2;
// FP64 D2Q9 (6 / 8) 1024^2 12.2 / 12.1, 2048^2 42.4 / 36.3.
FlowChoice flow_adjoint_choose(int storage, int q, int64_t nodes) {
    FlowChoice c;
    c.small = storage != ST_F64 && nodes < 2000000;
    c.steps = q == 5 && (nodes <= 100000 || nodes >= 2000000) ? 16 : 8;
    return c;
}

hipError_t launch_flow_adjoint(int storage, int q, bool small, const AdjointFlowParams &p, hipStream_t s) {
    if ((q != 5 && q != 9) || p.f.nrun < 2 || p.f.rec.col < p.f.nrun - 1 || p.rho_back <= 0 ||
        p.f.nx < 2 || !flow_fits(flow_adjoint_info(storage, q, small), p.f))
        return hipErrorInvalidValue;
    if (storage == ST_F64) return q == 5 ? launch_flow_adjoint_f64_q5(small, p, s) : launch_flow_adjoint_f64_q9(small, p, s);
    return q == 5 ? launch_flow_adjoint_f32_q5(small, p, s) : launch_flow_adjoint_f32_q9(small, p, s);
}

hipError_t launch_batch_prep(const BatchParams &bp, int run, int steps, const FlowInfo &f, hipStream_t s) {
    if (bp.nact <= 0) return hipSuccess;
    if (bp.img == nullptr || run < 1 || run > steps || steps > f.steps) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_batch_prep, dim3((unsigned)((bp.nact + kAdvBlock - 1) / kAdvBlock)), dim3(kAdvBlock), 0, s, bp,
                       run, steps, f);
    return hipGetLastError();
}

hipError_t launch_flow_batch(int storage, int q, bool small, const BatchParams &bp, int64_t nblk, hipStream_t s) {
    if (nblk <= 0 || bp.nact <= 0) return hipSuccess;
    if (bp.img == nullptr || (q != 5 && q != 9)) return hipErrorInvalidValue;
    return dispatch(storage, q, small, FlowParams(), flow_batch(bp), nblk, batch_kind(storage, q, bp.coll), s);
}

}  // namespace lbw
