// lb_flow.h -- many time steps per launch: the flowing kernel of the linear LB
// scheme, for single grids, replayed graphs and the batched executor.  The
// per-node arithmetic is that of the one-step kernel (lb_node.h), so both give
// the same bits.  Included by one source per storage format and lattice
// (lb_flow_*.hip, compiled in parallel) and by the dispatcher lb_flow.hip.
// Device code only; not part of the public interface.
//
// One pass reads h(n) and writes h(n + ns).  A strip is 64 lanes of V columns
// (hx >= ns of them halo columns on each side, recomputed and not stored); a
// bundle is R consecutive rows of a strip, and one wavefront carries a bundle
// through all ns steps with its whole state in registers.  Bundles of a strip
// follow each other downwards: bundle q belongs to wave q mod W of the block.
// At step s a bundle's slot r holds row Y + r - s, one row further up at every
// step, so a row's sources at the step before (the rows above, at and below
// it) are slots r - 2, r - 1 and r: a step rewrites the slots from the last to
// the first in place, and all a bundle needs from outside are the last two
// rows of the bundle above it, one step back.  Those go through LDS (two
// buffers per wave).  No row is computed twice except the 2 ns rows at the
// head of a block's run of bundles.
//
// Waves are ordered by counters in LDS, not by barriers: pub[w] counts the
// steps whose boundary wave w has put into its buffers, con[w] what wave w has
// taken from the wave before it, fin[w] the bundles wave w has finished.  So
// some waves load or store while the others compute, and the memory pipe and
// the vector units work at the same time.  DS operations of one wave execute
// in order, so a counter written after the data is seen after the data.  Every
// wait ends: a bundle waits only for earlier bundles, or (before it overwrites
// a buffer) for the next bundle, whose wave is free because the bundle it
// carried before was an earlier one; flow_steps_ok() is the condition under
// which a wave cannot be kept from its next bundle by bundles that wait for it.
//
// What bounds it: a launch of 16 steps of D2Q5 FP32 BGK at tau = 1/2 over
// 4096^2 needs 92 us at the HBM peak and 68 us of the vector units (10
// operations per update); it takes 205 us, 12.8 per step (30.5 with the
// marching kernel it replaced, whose waves recomputed 65 % of their updates and
// waited on their own dependency chains).  It issues 21 vector instructions per
// stored update: a third more updates than stored ones (128 columns per strip
// for 96), 11 instructions each, and 4 for a step's hand-over and a bundle's
// loads and stores.  At the 2.26 GHz that the chip then runs at they fill 73 %
// of the launch, whose 1050 MB (halo columns read twice) are 78 % of the rate
// of a plain copy.  In calls of 97 steps, the last one alone:
// 2048^2 5.5 us per step (13.5), 1024^2 2.9 (6.5), 256^2 1.7 (5.9).
#pragma once

#include "lb_iface.h"
#include "lb_internal.h"
#include "lb_rows.h"

namespace lbw {
namespace {

// Shape of the kernel: V columns per lane, R rows per bundle, W waves per
// block, EU waves per SIMD (the register budget), E further bundles whose c^2
// the ring keeps.  Wide shapes fill a CU with one block (LDS: two boundaries
// per wave and the c^2 of W + E bundles); the small one has short bundles, so
// that a small grid gives every CU some.  Measured (us per step, best step
// count of each), at 4096^2 / 2048^2 / 1024^2 where no size is given:
//   FP32 D2Q5   V2 R7 W16 14.0 / 5.5 / 2.9, V2 R8 W16 (10 registers spilled)
//               15.0 / 6.0 / 3.0, V2 R6 W16 with E = 3 14.5 / 5.4 / 2.7
//   FP32 D2Q5 with the collision written out (step_kind), 16 operations for 10
//               V2 R7 W16 16.8 / 5.8 / 2.8, V2 R10 W12 18.7 / 6.8 / 3.1,
//               V2 R16 W8 24.8 / 9.3 / 3.8
//   FP32 D2Q9   V2 R10 W8 44.0 / 15.2, V2 R6 W12 46.5 / 13.2, V2 R5 W12 46.7 /
//               13.7, V1 R7 W16 48.8 / 13.8; small V1 R4 W16 - / - / 5.4
//   FP64 D2Q5   V1 R7 W16 31.5 / 10.1 / 3.7, with E = 2 31.6 / 9.8 / 3.7
//   FP64 D2Q5 with the collision written out, as no FP64 grid has it now
//               V1 R7 W16 36.7 / 11.5 / 4.1, V2 R6 W8 36.5 / 13.0 / 5.5,
//               V1 R12 W12 38.9 / 12.2 / 5.1
//   FP64 D2Q9 (MRT)  V1 R5 W12 132 / 40.6 / 14.9, V1 R7 W8 136 / 42.6 / 15.8,
//               V1 R9 W8 134 / 42.7 / 16.1
//   small FP32 D2Q5 at 512^2 / 256^2 / 128^2
//               V1 R4 W16 1.84 / 1.69 / 1.43, V1 R5 W16 1.86 / 1.82 / 1.49
//   the same with the collision written out (128^2 without receivers)
//               V1 R4 W16 1.92 / 1.69 / 1.12, V1 R3 W16 2.18 / 1.93 / 1.13, the
//               wide shape 2.36 / 2.25 / 1.91
template <typename S, int Q, bool SMALL> struct FlowShape {
    static constexpr int V = 2, R = 7, W = 16, EU = 4, E = 0;
};
template <typename S, int Q> struct FlowShape<S, Q, true> {
    static constexpr int V = 1, R = 4, W = 16, EU = 4, E = 0;
};
template <typename S> struct FlowShape<S, 9, false> {
    static constexpr int V = 2, R = 10, W = 8, EU = 2, E = 2;
};
template <> struct FlowShape<double, 5, false> {
    static constexpr int V = 1, R = 7, W = 16, EU = 4, E = 0;
};
template <> struct FlowShape<double, 9, false> {
    static constexpr int V = 1, R = 5, W = 12, EU = 3, E = 2;
};
template <> struct FlowShape<double, 9, true> {
    static constexpr int V = 1, R = 3, W = 12, EU = 3, E = 2;
};

// Whether a launch of ns steps is free of circular waits (R, W, E as in
// FlowShape).  A bundle cannot be more than two steps ahead of the one below
// it, so while the bundle q + W of some wave has not started, bundle q + W - j
// gets to the start of its step 2 j + 1.  Bundle q + W starts when wave w is
// done with bundle q and the bundles up to q - E + m (m = ceil((ns - 1) / R),
// which read the c^2 rows that it overwrites) are done, and publishes its
// first rows when bundle q + 1 has taken all but the last of bundle q's.
constexpr bool flow_steps_ok(int ns, int R, int W, int E) {
    const int mlast = (R + ns - 1) / R, m = mlast - E;
    return ns >= 1 && ns <= kFlowSteps && R + ns <= 32 && mlast < W && ns <= 2 * W - 1 && (m <= 0 || ns <= 2 * (W - m));
}

typedef const __attribute__((address_space(4))) FlowParams *KernFlow;
typedef const __attribute__((address_space(4))) FlowPatchParams *KernPatch;
typedef const __attribute__((address_space(4))) int32_t *ConstInt;

// A pointer whose value the compiler cannot follow: fields read through it are
// loaded where they are used (scalar loads) instead of being kept in scalar
// registers across the whole kernel.
__device__ inline KernFlow rare(KernFlow q) {
    asm volatile("" : "+s"(q));
    return q;
}

// Counters in LDS; order() keeps the compiler from moving memory operations
// across it (the hardware executes a wave's DS operations in order).
__device__ inline int count_of(int *f) {
    return __builtin_amdgcn_readfirstlane(__hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
}
__device__ inline void set_count(int *f, int v) {
    if ((threadIdx.x & 63) == 0) __hip_atomic_store(f, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ inline void order() { asm volatile("" ::: "memory"); }
__device__ inline void wait_count(int *f, int v) {
    while (count_of(f) < v) __builtin_amdgcn_s_sleep(1);
    order();
}

__device__ inline float uniform(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ inline double uniform(double v) { return v; }

__device__ inline float lane_of(float v, int k) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), k));
}
__device__ inline double lane_of(double v, int k) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, k);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), k);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Block k's share of the strips' bundles of rows starts at share_start(k) and
// ends at share_start(k + 1): equal weights, where a bundle of the strips that
// lie in the sponge of a side edge counts more (kFlowSponge against
// kFlowPlain).  nbs: bundles of a strip.
__device__ inline int share_start(KernFlow p, int nbs, int k) {
    const int64_t wl = (int64_t)p->nl * nbs, wm = (int64_t)(p->nstrip - p->nl - p->nr) * nbs, wr = (int64_t)p->nr * nbs;
    const int64_t all = (wl + wr) * kFlowSponge + wm * kFlowPlain, t = all * k / p->nblk;
    if (t < wl * kFlowSponge) return (int)(t / kFlowSponge);
    if (t < wl * kFlowSponge + wm * kFlowPlain) return (int)(wl + (t - wl * kFlowSponge) / kFlowPlain);
    return (int)(wl + wm + (t - wl * kFlowSponge - wm * kFlowPlain) / kFlowSponge);
}

// Bundles that carry the share [b0, b1): each run of rows within a strip has
// 2 ns more rows at its head.
__device__ inline int share_bundles(int R, int ny, int ns, int nbs, int b0, int b1) {
    int total = 0;
    for (int b = b0; b < b1;) {
        const int j0 = b % nbs, j1 = min(nbs, j0 + (b1 - b));
        total += (min(j1 * R, ny) - j0 * R + 2 * ns + R - 1) / R;
        b += j1 - j0;
    }
    return total;
}

// MODE 1: the launch writes rho or its sums; 2: the fine steps of a patch (p is
// the f of a FlowPatchParams).  Kernels of their own: the code costs the
// others scalar registers, 2 % of a 4096^2 shot.
template <typename S, int Q, int KIND, int V, int R, int W, int E, int MODE>
__device__ __attribute__((always_inline)) inline void flow_body(KernFlow p, int blk) {
    using T = typename Tr<S>::T;
    typedef typename LaneVec<V, T>::type ct;
    typedef typename LaneVec<V, S>::type vt;
    constexpr int RING = (W + E) * R;   // rows of the c^2 ring
    static_assert(R >= 3 && R <= 16 && V * 64 <= 256, "row masks and the receiver table");
    constexpr bool OUT = MODE == 1, PATCH = MODE == 2;
    static_assert(!PATCH || (V == 1 && Q == 5), "one ring node per lane and row");
    __shared__ ct c2s[(RING + R) * 64];           // c^2 of the bundles' rows (the first R repeated at the end)
    __shared__ ct edge[2][W][Q][64];              // last two rows of each wave's bundle, one step back
    __shared__ uint32_t rtab[W][64 * V];              // receivers of each wave's bundle
    __shared__ T sfys[RING + R];                  // sponge factor of each ring row by its distance to the top or bottom
    __shared__ int pub[W], con[W], fin[W];
    __shared__ T ringsd[PATCH ? W : 1][PATCH ? 20 * R : 1];
    const int nx = p->nx, ny = p->ny, ns = p->nrun, hx = p->hx, ow = 64 * V - 2 * hx;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x < W) {
        pub[threadIdx.x] = 0;
        con[threadIdx.x] = 0;
        fin[threadIdx.x] = 0;
    }
    __syncthreads();
    const bool frho = OUT && p->rho_out != nullptr, fsum = OUT && p->sum != nullptr;
    const int wp = w > 0 ? w - 1 : W - 1, wc = w < W - 1 ? w + 1 : 0;
    const int L = p->sponge_width;
    const bool written = KIND >= 6 && p->coll.written != 0;
    CollisionT<T> coll;
    if constexpr (KIND % 3 == 0) coll.omega = uniform(T(p->coll.omega));
    if constexpr (KIND % 3 == 1)
        for (int k = 3; k < Q; ++k) coll.srate[k] = uniform(T(p->coll.srate[k]));
    if constexpr (Q == 9) {
        coll.kax = uniform(T(p->coll.kax));
        coll.kdg = uniform(T(p->coll.kdg));
        coll.kw = uniform(T(p->coll.kw));
        coll.ratio = uniform(T(p->coll.ratio));
    }

    const int nbs = (ny + R - 1) / R;
    const int b0 = share_start(p, nbs, blk), b1 = share_start(p, nbs, blk + 1);
    const int total = share_bundles(R, ny, ns, nbs, b0, b1);
    const int mlast = (R + ns - 1) / R;   // bundles q .. q + mlast read the c^2 rows of bundle q
    int b = b0, base = 0, it = 0, ring = w * R;
    for (int q = w; q < total; q += W, ++it) {
        int sx, ya, yb;   // strip, and the rows this run stores
        for (;;) {
            const int j0 = b % nbs, j1 = min(nbs, j0 + (b1 - b));
            sx = b / nbs;
            ya = j0 * R;
            yb = min(j1 * R, ny);
            const int nbr = (yb - ya + 2 * ns + R - 1) / R;
            if (q < base + nbr) break;
            base += nbr;
            b += j1 - j0;
        }
        const int Y = ya - ns + (q - base) * R;   // row of slot 0 before the first step (not wrapped)
        const int xa = sx * ow - hx;              // first column of the strip (not wrapped)
        T h[R][Q][V], fx[V];
        // bit k, row Y - ns + k: what to do with its pre-collision state (rho,
        // its sum, receivers), the source, the sponge
        uint32_t mpre = 0, mrec = 0, msrc = 0, mspo = 0;
        // PATCH: rows of the coarse inner ring and their coarse c^2; rows with
        // nodes of the outer ring, those that are its top or bottom row, and
        // its states at that row after either step (the sides' are in LDS).
        // All are read with the rows themselves: read where they are used they
        // were a chain of a microsecond per row (a 1033 x 521 patch 15.5 us,
        // 8.1 without any interface)
        uint32_t mres = 0, mring = 0, mtb = 0;
        T ringtb[2][PATCH ? 5 : 1], ringc[PATCH ? R : 1];
        int nrec = 0;
        // OUT: rows that this run stores, and whether the lane stores some or
        // all of its columns (the others find out where they need it)
        uint32_t mown = 0;
        auto stores = [&](int n) { return lane * V >= hx && lane * V < hx + ow && xa + lane * V + n <= nx; };
        const bool some = OUT && stores(1), whole = OUT && stores(V), ragged = OUT && V > 1 && __ballot(some && !whole) != 0;
        {
            const int xl = xa + lane * V;
            int xw[V];
#pragma unroll
            for (int j = 0; j < V; ++j) xw[j] = wrapi(xl + j, nx);
            const int row_l = Y - ns + lane, rowi = wrapi(row_l, ny);   // lane k: row Y - ns + k
            T cl[R][V];
            // the lanes' columns are contiguous in memory if nx is a multiple
            // of V or the strip does not cross the periodic seam
            const bool vec = V == 1 || nx % V == 0 || (xa >= 0 && xa + 64 * V <= nx);
            auto load = [&](auto vc) __attribute__((always_inline)) {
                constexpr bool VEC = decltype(vc)::value;
                const S *src = reinterpret_cast<const S *>(p->src);
                const T *c2 = reinterpret_cast<const T *>(p->c2);
                static_for<0, R>([&](auto rc) __attribute__((always_inline)) {
                    constexpr int r = decltype(rc)::value;
                    const int64_t ro = (int64_t)__builtin_amdgcn_readlane(rowi, ns + r) * nx;
                    load_row2<VEC, 0, true, S, T, Q, V>(src, p->pstride, ro, xw[0], xw, h[r]);
                    load_c2row<VEC, true, T, V>(c2, ro, xw[0], xw, cl[r]);
                });
            };
            if (vec) load(std::true_type()); else load(std::false_type());
            const bool mine = lane < R + ns, owned = mine && row_l >= ya && row_l < yb;
            const int dyl = min(rowi, ny - 1 - rowi);
            msrc = (uint32_t)__ballot(mine && rowi == p->src_y);
#pragma unroll
            for (int j = 0; j < V; ++j) fx[j] = T(1);
            T sfy = T(1);
            if (L > 0) {
                const bool side = xa < L || xa + 64 * V - 1 >= nx - L;
                mspo = side ? ~0u : (uint32_t)__ballot(mine && dyl < L);
                if (mspo) {
                    const double smax = rare(p)->sponge_smax;
#pragma unroll
                    for (int j = 0; j < V; ++j) fx[j] = sponge_at<T>(min(xw[j], nx - 1 - xw[j]), L, smax);
                    sfy = sponge_at<T>(dyl, L, smax);
                }
            }
            if constexpr (PATCH) {
                const KernPatch pp = (KernPatch)p;
                const int cy = pp->iface.g.Y0 + (row_l >> 1);
                mres = (uint32_t)__ballot(owned && !(row_l & 1) && cy >= pp->iface.g.ya && cy <= pp->iface.g.yb);
                // only nodes of the grid itself count: what lies beyond the
                // ring does not reach the nodes within
                const bool side = xa <= 0 || xa + 64 > nx - 1;
                mtb = (uint32_t)__ballot(mine && (row_l == 0 || row_l == ny - 1));
                mring = side ? ~0u : mtb;
                const GlobalPtr<const T> rb = (GlobalPtr<const T>)pp->ring, cc = (GlobalPtr<const T>)pp->iface.dst_c2;
                const int rn = pp->ring_n;
                if (mtb) {
                    const int k = (Y <= 2 ? 0 : nx) + min(max(xl, 0), nx - 1);
#pragma unroll
                    for (int i = 0; i < 10; ++i) ringtb[i / 5][i % 5] = rb[i * rn + k];
                }
                if (side) {   // [step][side][population][slot]
                    for (int e = lane; e < 20 * R; e += 64) {
                        const int st = e / (10 * R), sd = e / (5 * R) % 2, i = e / R % 5, y = Y + e % R - st - 1;
                        ringsd[w][e] = y >= 1 && y <= ny - 2 ? rb[(st * 5 + i) * rn + 2 * nx + sd * (ny - 2) + y - 1] : T(0);
                    }
                }
                const int cx = min(max(pp->iface.g.X0 + (xl >> 1), 0), pp->iface.dst_nx - 1);
                static_for<0, R>([&](auto rc) __attribute__((always_inline)) {
                    constexpr int r = decltype(rc)::value;
                    const int y = min(max(pp->iface.g.Y0 + ((Y + r - 2) >> 1), 0), pp->iface.dst_ny - 1);
                    ringc[r] = (mres >> r) & 1 ? cc[(int64_t)y * pp->iface.dst_nx + cx] : T(0);
                });
            }
            if (p->rec.row_ptr != nullptr) {
                // receivers among the rows and columns this bundle stores go
                // into the wave's table (row, column of the strip, slot).  The
                // lanes look at 64 entries of a row's list at a time: the
                // searches of a lane of its own were a chain of a dozen loads,
                // 10 us of a launch over a small grid
                const GlobalPtr<const int32_t> rp = (GlobalPtr<const int32_t>)p->rec.row_ptr,
                                               xs = (GlobalPtr<const int32_t>)p->rec.xs,
                                               sl = (GlobalPtr<const int32_t>)p->rec.slot;
                int rb_l = 0, re_l = 0;
                if (owned) {
                    rb_l = rp[row_l];
                    re_l = rp[row_l + 1];
                }
                const int x0 = xa + hx, x1 = x0 + ow;
                for (uint32_t m = (uint32_t)__ballot(rb_l < re_l); m; m &= m - 1) {
                    const int k = __builtin_ctz(m);
                    const int re = __builtin_amdgcn_readlane(re_l, k);
                    int l = __builtin_amdgcn_readlane(rb_l, k), u = re;   // the first entry with x >= x0 is in [l, u]
                    while (u - l > 64) {
                        const int st = (u - l + 63) / 64, e = l + lane * st;
                        const int c = __builtin_popcountll(__ballot(e < u && xs[min(e, u - 1)] < x0));
                        u = min(u, l + c * st);
                        l = c > 0 ? l + (c - 1) * st + 1 : l;
                    }
                    for (bool more = true; more && l < re; l += 64) {
                        const int e = min(l + lane, re - 1), x = xs[e], slot = sl[e];
                        const bool in = l + lane < re && x >= x0 && x < x1;
                        const uint64_t hits = __ballot(in);
                        const int n = __builtin_popcountll(hits);
                        if (n > 0) mrec |= 1u << k;
                        if (in && nrec + n <= 64 * V)
                            rtab[w][nrec + __builtin_popcountll(hits & ((1ull << lane) - 1))] =
                                (uint32_t)k << 27 | (uint32_t)(x - xa) << 19 | (uint32_t)(slot & 0x7ffff);
                        nrec += n;
                        more = __builtin_amdgcn_readlane(x, 63) < x1;
                    }
                }
                if (p->rec.nslots > 0x80000) nrec = 64 * V + 1;   // slots too large for the table
            }
            mpre = mrec | mres;
            if constexpr (OUT) {
                mown = (uint32_t)__ballot(owned);
                mpre |= mown;
            }
            // the ring slot is free once the bundles that read its rows are done
            for (int m = 0; m <= mlast; ++m) {
                const int qq = q - W - E + m;
                if (qq >= 0 && qq != q - W) wait_count(&fin[qq % W], qq / W + 1);
            }
            order();
            static_for<0, R>([&](auto rc) __attribute__((always_inline)) {
                constexpr int r = decltype(rc)::value;
                ct t;
#pragma unroll
                for (int j = 0; j < V; ++j) t[j] = cl[r][j];
                c2s[(ring + r) * 64 + lane] = t;
                if (ring == 0) c2s[(RING + r) * 64 + lane] = t;
            });
            if (L > 0 && lane >= ns && lane < ns + R) {
                sfys[ring + lane - ns] = sfy;
                if (ring == 0) sfys[RING + lane - ns] = sfy;
            }
            order();
        }
        const int itp = w > 0 ? it : it - 1;
        for (int s = 1; s <= ns; ++s) {
            const int n = it * ns + s, np = itp * ns + s;   // counts of this step in pub[w] and pub[wp]
            if (q + 1 < total) {   // for the bundle below
                wait_count(&con[wc], n - 2);
                int k = 0;
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    ct t;
#pragma unroll
                    for (int j = 0; j < V; ++j) t[j] = h[R - 1][i][j];
                    if (cyv<Q>(i) >= 0) edge[n & 1][w][k++][lane] = t;
                    if (cyv<Q>(i) > 0) {
#pragma unroll
                        for (int j = 0; j < V; ++j) t[j] = h[R - 2][i][j];
                        edge[n & 1][w][k++][lane] = t;
                    }
                }
                order();
                set_count(&pub[w], n);
            }
            order();
            const int rs = ring - s + (ring < s ? RING : 0);   // ring row of slot 0
            const ct *cb = c2s + rs * 64 + lane;
            const T *sb = sfys + rs + min(lane, R - 1);
            const int sh = ns - s;
            const uint32_t bpre = PATCH && s < ns ? 0 : mpre >> sh, bpost = (msrc | mspo | mring) >> sh;
            T fyl = T(1);
            if (mspo) fyl = *sb;
            // where slot 0's row of rho and of its sums goes
            T *const rho_s = frho ? reinterpret_cast<T *>(p->rho_out) + (int64_t)(s - 1) * p->rho_stride + (int64_t)(Y - s) * nx : nullptr;
            double *const sum_s = fsum ? p->sum + (int64_t)(s - 1) * p->sum_stride + (int64_t)(Y - s) * p->nstrip + sx : nullptr;
            ct cn = cb[(R - 1) * 64];
            auto row = [&](auto rc, const T (&U)[Q][V], const T (&C)[Q][V], const T (&D)[Q][V]) __attribute__((always_inline)) {
                constexpr int r = decltype(rc)::value;
                T cm[V];
#pragma unroll
                for (int j = 0; j < V; ++j) cm[j] = cn[j];
                if constexpr (r > 0) cn = cb[(r - 1) * 64];
                T g[Q][V];
                pull_row2<T, Q, V>(U, C, D, g);
                if (__builtin_expect((bpre >> r) & 1, OUT)) {
                    const int gy = Y + r - s, xl = xa + lane * V;
                    const bool own0 = OUT ? some : stores(1);
                    if (OUT) {   // rho with the bits that the one-step kernel gives it
                        T rv[V];
#pragma unroll
                        for (int j = 0; j < V; ++j) {
                            rv[j] = g[0][j];
#pragma unroll
                            for (int i = 1; i < Q; ++i) rv[j] += g[i][j];
                        }
                        if (frho && ((mown >> (sh + r)) & 1)) {
                            T *rr = rho_s + (int64_t)r * nx;
                            if (whole) {
                                ct t;
#pragma unroll
                                for (int j = 0; j < V; ++j) t[j] = rv[j];
                                st_nt(t, at_lane<ct>(rr, xl));
                            }
                            if (ragged) {
#pragma unroll
                                for (int j = 0; j < V - 1; ++j)
                                    if (own0 && !whole && xl + j < nx) st_nt(rv[j], rr + xl + j);
                            }
                        }
                        if (fsum && ((mown >> (sh + r)) & 1)) {   // one partial per row and strip
                            double a = 0.0;
#pragma unroll
                            for (int j = 0; j < V; ++j)
                                if (own0 && xl + j < nx) a += double(rv[j]);
                            a = wave_total(a);
                            if (lane == 63) st_nt(a, sum_s + r * p->nstrip);
                        }
                    }
                    if constexpr (PATCH) {
                        if ((mres >> (sh + r)) & 1) {
                            // fine nodes that coincide with a coarse node of
                            // the inner ring replace its state
                            const auto &ip = ((KernPatch)rare(p))->iface;
                            const int cy = ip.g.Y0 + (gy >> 1);
#pragma unroll
                            for (int j = 0; j < V; ++j) {
                                const int x = xl + j, cx = ip.g.X0 + (x >> 1);
                                if (own0 && x < nx && !(x & 1) && cx >= ip.g.xa && cx <= ip.g.xb &&
                                    (cx == ip.g.xa || cx == ip.g.xb || cy == ip.g.ya || cy == ip.g.yb)) {
                                    T gj[5], out[5];
#pragma unroll
                                    for (int i = 0; i < 5; ++i) gj[i] = g[i][j];
                                    rescale_collide<S, KIND>(ip, gj, cx, cy, ringc[r], out);
                                    S *d = reinterpret_cast<S *>(ip.dst) + (int64_t)cy * ip.dst_nx + cx;
#pragma unroll
                                    for (int i = 0; i < 5; ++i) *(GlobalPtr<S>)(d + i * ip.dst_pstride) = to_store<S>(out[i]);
                                }
                            }
                        }
                    }
                    if ((mrec >> (sh + r)) & 1) {
                        const KernFlow z = rare(p);
                        Receivers rx;
                        rx.row_ptr = z->rec.row_ptr;
                        rx.xs = z->rec.xs;
                        rx.slot = z->rec.slot;
                        rx.traces = z->rec.traces;
                        rx.nslots = z->rec.nslots;
                        rx.what = z->rec.what;
                        rx.cap = z->rec.cap;
                        rx.col = z->rec.col + s - 1;
                        if (z->gtab != nullptr) rx.col += z->gtab->t0;
                        if (nrec <= 64 * V) {
                            // each lane takes an entry of the table and its
                            // value from the lane that holds the column
                            const int64_t plane = (int64_t)rx.nslots * rx.cap;
                            for (int e0 = 0; e0 < nrec; e0 += 64) {
                                const uint32_t t0 = rtab[w][min(e0 + lane, 64 * V - 1)];
                                const bool hit = e0 + lane < nrec && (int)(t0 >> 27) == r + sh;
                                const int c = (t0 >> 19) & 0xff, from = c / V, jj = c % V;
                                GlobalPtr<T> tr = (GlobalPtr<T>)rx.traces + (int64_t)(t0 & 0x7ffff) * rx.cap + rx.col;
                                for (int f = 0; f < 4; ++f) {
                                    if (!((rx.what >> f) & 1)) continue;
                                    T out = T(0);
#pragma unroll
                                    for (int j = 0; j < V; ++j) {
                                        T rho = T(0), jx = T(0), jy = T(0);
#pragma unroll
                                        for (int i = 0; i < Q; ++i) {
                                            rho += g[i][j];
                                            jx += T(cxv<Q>(i)) * g[i][j];
                                            jy += T(cyv<Q>(i)) * g[i][j];
                                        }
                                        const T v = f == 0 ? cm[j] * rho : f == 1 ? rho : f == 2 ? jx : jy;
                                        const T vs = __shfl(v, from);
                                        if (jj == j) out = vs;
                                    }
                                    if (hit) *tr = out;
                                    tr += plane;
                                }
                            }
                        } else {
                            const ConstInt rp = (ConstInt)rx.row_ptr;
                            const int rb = rp[gy], re = rp[gy + 1];
#pragma unroll
                            for (int j = 0; j < V; ++j) {
                                T gj[Q];
#pragma unroll
                                for (int i = 0; i < Q; ++i) gj[i] = g[i][j];
                                if (own0 && xl + j < nx) record_node<T, Q>(rx, rb, re, xl + j, gj, cm[j]);
                            }
                        }
                    }
                }
                T pj[V][Q];
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    T gj[Q], wt[Q];
#pragma unroll
                    for (int i = 0; i < Q; ++i) gj[i] = g[i][j];
                    if constexpr (KIND < 6) collide<T, Q, KIND>(gj, cm[j], coll, pj[j], wt);
                    else if (written) collide<T, Q, KIND - 3>(gj, cm[j], coll, pj[j], wt);
                    else collide<T, Q, KIND - 6>(gj, cm[j], coll, pj[j], wt);
                }
                if (__builtin_expect((bpost >> r) & 1, 0)) {
                    if ((msrc >> (sh + r)) & 1) {
                        const KernFlow z = rare(p);
                        const double snv = z->gtab != nullptr ? z->gtab->s[z->goff + s - 1] : z->s[s - 1];
                        const int sxs = z->src_x, xl = xa + lane * V;
#pragma unroll
                        for (int j = 0; j < V; ++j) {
                            if (wrapi(xl + j, nx) == sxs) {
                                T wt[Q];
                                weights<T, Q>(cm[j], coll, wt);
                                add_source<T, Q>(wt, snv, pj[j]);
                            }
                        }
                    }
                    // the factor falls with the distance to the nearest edge,
                    // so it is the smaller one of the two directions'
                    const T fy = lane_of(fyl, r);
#pragma unroll
                    for (int j = 0; j < V; ++j) {
                        const T sf = min(fx[j], fy);
#pragma unroll
                        for (int i = 0; i < Q; ++i) pj[j][i] = pj[j][i] * sf;
                    }
                    if constexpr (PATCH) {   // the outer ring's states come from the coarse grid
                        const int x = xa + lane;
                        if ((mtb >> (sh + r)) & 1) {
#pragma unroll
                            for (int i = 0; i < 5; ++i) pj[0][i] = s == 1 ? ringtb[0][i] : ringtb[1][i];
                        } else if ((mring >> (sh + r)) & 1) {
                            if (x == 0 || x == nx - 1) {
#pragma unroll
                                for (int i = 0; i < 5; ++i) pj[0][i] = ringsd[w][((s - 1) * 10 + (x == 0 ? 0 : 5) + i) * R + r];
                            }
                        }
                    }
                }
                // rounded to the storage format, as a stored state would be
#pragma unroll
                for (int j = 0; j < V; ++j)
#pragma unroll
                    for (int i = 0; i < Q; ++i) h[r][i][j] = T(to_store<S>(pj[j][i]));
                __builtin_amdgcn_sched_barrier(0);   // one row after the other: bounds the registers
            };
            static_for<0, R - 2>([&](auto mc) __attribute__((always_inline)) {
                constexpr int r = R - 1 - decltype(mc)::value;
                row(std::integral_constant<int, r>{}, h[r - 2], h[r - 1], h[r]);
            });
            // the last two rows above, one step back; with them the c^2 and
            // sponge factors of the rows that came from that bundle
            if (q > 0) wait_count(&pub[wp], np);
            T e1[Q][V], e2[Q][V];   // its last row (c_y >= 0) and the one above (c_y > 0)
            {
                int k = 0;
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    if (cyv<Q>(i) >= 0) {
                        const ct t = edge[np & 1][wp][k++][lane];
#pragma unroll
                        for (int j = 0; j < V; ++j) e1[i][j] = t[j];
                    }
                    if (cyv<Q>(i) > 0) {
                        const ct t = edge[np & 1][wp][k++][lane];
#pragma unroll
                        for (int j = 0; j < V; ++j) e2[i][j] = t[j];
                    }
                }
            }
            cn = cb[64];
            if (mspo) fyl = *sb;
            order();
            if (q > 0) set_count(&con[w], np);
            order();
            row(std::integral_constant<int, 1>{}, e1, h[0], h[1]);
            row(std::integral_constant<int, 0>{}, e2, e1, h[0]);
        }
        order();
        set_count(&fin[w], it + 1);
        order();
        ring += W * R;
        if (ring >= RING) ring -= RING;
        const int xl = xa + lane * V;
        if (stores(1)) {
            const bool all = xl + V <= nx;
            static_for<0, R>([&](auto rc) __attribute__((always_inline)) {
                constexpr int r = decltype(rc)::value;
                const int gy = Y + r - ns;
                if (gy >= ya && gy < yb) {
                    S *d = reinterpret_cast<S *>(p->dst) + (int64_t)gy * nx;
#pragma unroll
                    for (int i = 0; i < Q; ++i, d += p->pstride) {
                        if (all) {
                            vt t;
#pragma unroll
                            for (int j = 0; j < V; ++j) t[j] = S(h[r][i][j]);
                            st_nt(t, at_lane<vt>(d, xl));
                        } else {
#pragma unroll
                            for (int j = 0; j < V - 1; ++j)
                                if (xl + j < nx) st_nt(S(h[r][i][j]), d + xl + j);
                        }
                    }
                }
            });
        }
    }
}

// Single grid (fb.img == nullptr: the parameters are the kernel arguments) or
// every active shot of a batch (block k belongs to the shot a with prefix[a]
// <= k < prefix[a + 1] and takes its params image of the round).
template <typename S, int Q, int KIND, bool SMALL, bool OUT>
__global__ __launch_bounds__((FlowShape<S, Q, SMALL>::W * 64))
__attribute__((amdgpu_waves_per_eu(FlowShape<S, Q, SMALL>::EU, FlowShape<S, Q, SMALL>::EU)))
void k_flow(FlowParams, FlowBatch fb) {
    using F = FlowShape<S, Q, SMALL>;
    int blk = xcd_block();
    KernFlow p = (KernFlow)__builtin_amdgcn_kernarg_segment_ptr();
    if (fb.img != nullptr) {
        int lo = 0, hi = fb.nact - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (fb.prefix[mid] <= blk) lo = mid; else hi = mid - 1;
        }
        blk -= __builtin_amdgcn_readfirstlane(fb.prefix[lo]);
        p = (KernFlow)(fb.img + __builtin_amdgcn_readfirstlane(fb.order[lo]));
        if (p->nrun < 1) return;
    }
    flow_body<S, Q, KIND, F::V, F::R, F::W, F::E, OUT ? 1 : 0>(p, blk);
}

// The two fine steps of a coarse step of a refined grid, 10.9 us for a
// 1033 x 521 patch (10.1 and 10.6 as two one-step launches).  Two steps are a
// latency more than a throughput: blocks of 8 waves, two per CU (FP64: one,
// with twice the registers), so that a share is one bundle per wave.
template <typename S> struct PatchShape {
    static constexpr int V = 1, R = 4, W = 8, EU = sizeof(S) == 8 ? 2 : 4, E = 0;
};

template <typename S, int KIND>
__global__ __launch_bounds__(PatchShape<S>::W * 64)
__attribute__((amdgpu_waves_per_eu(PatchShape<S>::EU, PatchShape<S>::EU)))
void k_flow_patch(FlowPatchParams) {
    using F = PatchShape<S>;
    flow_body<S, 5, KIND, F::V, F::R, F::W, F::E, 2>((KernFlow)__builtin_amdgcn_kernarg_segment_ptr(), xcd_block());
}

template <typename S>
hipError_t flow_patch_launch(const FlowPatchParams &p, hipStream_t s) {
    return for_kind<S, 5>(step_kind(p.f.coll), [&](auto kc) {
        hipLaunchKernelGGL((k_flow_patch<S, decltype(kc)::value>), dim3((unsigned)p.f.nblk),
                           dim3(PatchShape<S>::W * 64), 0, s, p);
        return hipGetLastError();
    });
}

template <typename S, int Q, bool SMALL, bool OUT>
hipError_t flow_launch(const FlowParams &p, const FlowBatch &fb, int64_t nblk, int kind, hipStream_t s) {
    using F = FlowShape<S, Q, SMALL>;
    if (nblk < 1 || nblk > (1 << 30)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nblk), block(F::W * 64);
    auto go = [&](auto kc) {
        hipLaunchKernelGGL((k_flow<S, Q, decltype(kc)::value, SMALL, OUT>), grid, block, 0, s, p, fb);
        return hipGetLastError();
    };
    if constexpr (OUT) return for_kind<S, Q>(kind, go);
    else return for_batch_kind<S, Q>(kind, go);
}

template <typename S, int Q, bool SMALL>
FlowInfo flow_info() {
    using F = FlowShape<S, Q, SMALL>;
    FlowInfo f;
    f.V = F::V;
    f.R = F::R;
    f.steps = 1;
    for (int ns = 2; ns <= kFlowSteps; ++ns)
        if (flow_steps_ok(ns, F::R, F::W, F::E)) f.steps = ns;
    return f;
}

}  // namespace

// One source per storage format and lattice instantiates the kernels with
// LBW_FLOW_UNIT; lb_flow.hip dispatches to them.
#define LBW_FLOW_UNIT(SS, QQ, NAME)                                                                                 \
    hipError_t launch_flow_##NAME(bool small, const FlowParams &p, const FlowBatch &fb, int64_t nblk, int kind,      \
                                  hipStream_t s) {                                                                  \
        const bool out = p.rho_out != nullptr || p.sum != nullptr;                                                  \
        if (out) return small ? flow_launch<SS, QQ, true, true>(p, fb, nblk, kind, s)                               \
                              : flow_launch<SS, QQ, false, true>(p, fb, nblk, kind, s);                             \
        return small ? flow_launch<SS, QQ, true, false>(p, fb, nblk, kind, s)                                       \
                     : flow_launch<SS, QQ, false, false>(p, fb, nblk, kind, s);                                     \
    }                                                                                                               \
    FlowInfo flow_info_##NAME(bool small) { return small ? flow_info<SS, QQ, true>() : flow_info<SS, QQ, false>(); }

#define LBW_FLOW_PATCH_UNIT(SS, NAME) \
    hipError_t launch_flow_patch_##NAME(const FlowPatchParams &p, hipStream_t s) { return flow_patch_launch<SS>(p, s); }
hipError_t launch_flow_patch_f32(const FlowPatchParams &p, hipStream_t s);
hipError_t launch_flow_patch_f64(const FlowPatchParams &p, hipStream_t s);
hipError_t launch_flow_patch_f16(const FlowPatchParams &p, hipStream_t s);

#define LBW_FLOW_DECL(NAME)                                                                                         \
    hipError_t launch_flow_##NAME(bool small, const FlowParams &p, const FlowBatch &fb, int64_t nblk, int kind,      \
                                  hipStream_t s);                                                                   \
    FlowInfo flow_info_##NAME(bool small);
LBW_FLOW_DECL(f32_q5)
LBW_FLOW_DECL(f32_q9)
LBW_FLOW_DECL(f64_q5)
LBW_FLOW_DECL(f64_q9)
LBW_FLOW_DECL(f16_q5)
LBW_FLOW_DECL(f16_q9)
#undef LBW_FLOW_DECL

}  // namespace lbw
