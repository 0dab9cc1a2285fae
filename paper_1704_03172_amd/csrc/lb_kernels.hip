// lb_kernels.hip -- gfx950 kernels of the linear lattice Boltzmann scheme
// (arXiv:1704.03172).
//
// Storage: populations structure-of-arrays, pop[i][y][x], x fastest, with a
// stride of pstride elements between populations.  The step kernel keeps the
// post-collision state: launch n reads h(n-1) = post-collision populations of
// time n-1, pulls g_i(x, n) = h_i(x - c_i, n-1) (streaming, eq. BGK-LB lhs,
// periodic wrap), records time n, collides (eq. BGK-LB / eq. MRT-LB around
// eq. linear eqm dist), adds w_i S(n) at the source node (eq. MRT-LB linear
// acoustic), damps in the sponge (Sec. IV) and writes h(n) at the node it
// owns.  Every element of every array is read once and written once per
// step: the kernel is HBM-bound (no data reuse to stage in LDS), so it is
// written as a pure streaming pass with 16-byte vector accesses.
//
// Each thread owns V consecutive x-nodes of one row (V * sizeof(storage) =
// 16 bytes).  Pulls along x are offset by one element; gfx950 accepts
// 4-byte-aligned dwordx4 loads, so the shifted pulls are single vector loads
// except at the periodic seam, which takes an element-wise path.  Population
// and c^2 traffic is single-use, so loads and stores carry the nontemporal
// hint (measured on MI355X: +8-11 % HBM throughput over cached accesses for
// this 11-stream pattern, and +7 % for a plain copy).
//
// This one-step kernel serves single steps (the last of a call, checkpoint
// boundaries), the refinement patch, whose interface work is fused into it,
// and the collide-only launch of time 0; runs of steps (the adjoint's
// recompute included) go to the flowing kernel of lb_flow.h.  Both take their
// per-node arithmetic from lb_node.h.
#include "lb_iface.h"
#include "lb_internal.h"
#include "lb_node.h"
#include "lb_rows.h"

#include <algorithm>

namespace lbw {
namespace {

constexpr int kBlock = 256;       // set-up, field and interface kernels
constexpr int kStepBlock = 128;   // fused step (best of a block-size sweep)

// ---- refinement interface (D2Q5, factor 2) -------------------------------------
template <typename S, typename T>
__device__ inline void pre_at(const GridRef &r, int x, int y, T (&g)[5]) {
    const S *pop = reinterpret_cast<const S *>(r.pop);
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        int xs = r.pre ? x : wrapi(x - cxv<5>(i), r.nx);
        int ys = r.pre ? y : wrapi(y - cyv<5>(i), r.ny);
        g[i] = T(pop[i * r.pstride + (int64_t)ys * r.nx + xs]);
    }
}

// Snapshot layout (written by the coarse step, see update_tile): top row
// (y = Y0, x = X0-1 .. X0+W+1), bottom row (y = Y0+H), left column (x = X0,
// y = Y0-1 .. Y0+H+1), right column (x = X0+W).

// Interpolation stencil of fine outer-ring node (i, j): coincident nodes
// copy the coarse node (weight 1 on entry 1, the other entries repeat it with
// weight 0), mid-edge nodes take the cubic (-1, 9, 9, -1)/16 along their
// edge.  nodes_*: coarse nodes; sidx: their ring-line snapshot entries.
template <typename T>
__device__ inline void ring_stencil(const PatchGeom &g, int i, int j, int (&nodes_x)[4], int (&nodes_y)[4],
                                    int (&sidx)[4], T (&wt)[4]) {
    const int nh = g.W + 3, nv = g.H + 3;
    const bool horiz = (j == 0 || j == g.nyf - 1);
    const int hbase = (j == 0) ? 0 : nh;                 // top / bottom arrays
    const int vbase = 2 * nh + ((i == 0) ? 0 : nv);      // left / right arrays
    if ((i & 1) == 0 && (j & 1) == 0) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            nodes_x[s] = g.X0 + i / 2;
            nodes_y[s] = g.Y0 + j / 2;
            wt[s] = s == 1 ? T(1) : T(0);
            sidx[s] = horiz ? hbase + i / 2 + 1 : vbase + j / 2 + 1;
        }
    } else if (i & 1) {
        const int a = g.X0 + (i - 1) / 2;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            nodes_x[s] = a - 1 + s;
            nodes_y[s] = g.Y0 + j / 2;
            sidx[s] = hbase + (i - 1) / 2 + s;
        }
        wt[0] = wt[3] = T(-1) / T(16);
        wt[1] = wt[2] = T(9) / T(16);
    } else {
        const int b = g.Y0 + (j - 1) / 2;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            nodes_x[s] = g.X0 + i / 2;
            nodes_y[s] = b - 1 + s;
            sidx[s] = vbase + (j - 1) / 2 + s;
        }
        wt[0] = wt[3] = T(-1) / T(16);
        wt[1] = wt[2] = T(9) / T(16);
    }
}

// Coarse state interpolated to fine outer-ring node (i, j) along the edge;
// in time a_snap * (snapshot of T) + a_now * (coarse now).
template <typename S>
__device__ inline void ring_interp(const InterfaceParams &p, int i, int j, typename Tr<S>::T (&gh)[5]) {
    using T = typename Tr<S>::T;
    const PatchGeom &g = p.g;
    int nodes_x[4], nodes_y[4], sidx[4];
    T wt[4];
    ring_stencil<T>(g, i, j, nodes_x, nodes_y, sidx, wt);
#pragma unroll
    for (int q = 0; q < 5; ++q) gh[q] = T(0);
    const T *snap = reinterpret_cast<const T *>(p.snap);
    const T an = T(p.a_now), as = T(p.a_snap);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        if (wt[s] == T(0)) continue;
        T gn[5];
        pre_at<S, T>(p.coarse, nodes_x[s], nodes_y[s], gn);
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            T v = an * gn[q];
            if (p.a_snap != 0.0) v += as * snap[q * g.nsnap + sidx[s]];
            gh[q] += wt[s] * v;
        }
    }
}

// Blocks of NT fine outer-ring nodes: each side of the ring (top, bottom,
// left, right, in the ring's order) in runs of NT, so that no block spans a
// corner.
template <int NT>
__host__ __device__ inline int ring_tile_blocks(const PatchGeom &g) {
    return 2 * ((g.nxf + NT - 1) / NT) + 2 * ((g.nyf - 2 + NT - 1) / NT);
}

// The outer-ring states of the two fine steps of one coarse step T -> T+2:
// R_{1/2} of the coarse state interpolated to each fine ring node, at T+1
// (mean of the ring-line snapshot of T and the coarse state of T+2) and at
// T+2, each followed by the fine collision.  Block b (of ring_tile_blocks)
// takes NT consecutive nodes of one side.  Their stencils (the copy of a
// coincident coarse node, or the cubic (-1, 9, 9, -1)/16 along the side; see
// ring_stencil) cover at most NT/2 + 5 consecutive nodes of that side's
// ring line, which the block first pulls from the coarse state and reads
// from the snapshot into an LDS tile, once each instead of once per stencil
// that reaches them (up to three).  The stencil arithmetic then reads the
// tile.  All NT threads of the block must call this (it synchronises).
template <typename S, int KIND, int NT>
__device__ inline void prolong_pair_tile(const InterfaceParams &p, int b) {
    using T = typename Tr<S>::T;
    constexpr int NE = NT / 2 + 5;
    __shared__ T tn[5][NE], ts[5][NE];
    const PatchGeom &g = p.g;
    const int bh = (g.nxf + NT - 1) / NT, bv = (g.nyf - 2 + NT - 1) / NT;
    int side, c;
    if (b < bh) { side = 0; c = b; }
    else if (b < 2 * bh) { side = 1; c = b - bh; }
    else if (b < 2 * bh + bv) { side = 2; c = b - 2 * bh; }
    else if (b < 2 * bh + 2 * bv) { side = 3; c = b - 2 * bh - bv; }
    else return;   // the whole block
    const bool horiz = side < 2;
    const int nh = g.W + 3, nv = g.H + 3;
    const int nline = horiz ? nh : nv;   // ring-line nodes of the side
    const int lbase = side == 0 ? 0 : side == 1 ? nh : side == 2 ? 2 * nh : 2 * nh + nv;
    // along-side fine index u of thread 0 (i on the top and bottom rows, j
    // on the left and right columns); line node e is coarse node
    // (X0 - 1 + e, row) or (column, Y0 - 1 + e)
    const int u0 = (horiz ? 0 : 1) + c * NT;
    const int e_lo = u0 > 0 ? (u0 - 1) / 2 : 0;
    const int crow = g.Y0 + (side == 1 ? g.H : 0), ccol = g.X0 + (side == 3 ? g.W : 0);
    const T *snap = reinterpret_cast<const T *>(p.snap);
    for (int k = threadIdx.x; k < NE; k += NT) {
        const int e = e_lo + k;
        if (e < nline) {
            T gn[5];
            pre_at<S, T>(p.coarse, horiz ? g.X0 - 1 + e : ccol, horiz ? crow : g.Y0 - 1 + e, gn);
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                tn[q][k] = gn[q];
                ts[q][k] = snap[q * g.nsnap + lbase + e];
            }
        }
    }
    __syncthreads();
    const int u = u0 + (int)threadIdx.x;
    if (c * NT + (int)threadIdx.x >= (horiz ? g.nxf : g.nyf - 2)) return;
    const int i = horiz ? u : (side == 2 ? 0 : g.nxf - 1);
    const int j = horiz ? (side == 0 ? 0 : g.nyf - 1) : u;
    const int r = (side == 0 ? 0 : side == 1 ? g.nxf : side == 2 ? 2 * g.nxf : 2 * g.nxf + g.nyf - 2) + c * NT +
                  (int)threadIdx.x;
    // the stencil of ring_stencil, as tile entries; the weight-0 entries of
    // a coincident node repeat it
    int ek[4];
    T wt[4];
    if ((u & 1) == 0) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            ek[s] = u / 2 + 1 - e_lo;
            wt[s] = s == 1 ? T(1) : T(0);
        }
    } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) ek[s] = (u - 1) / 2 + s - e_lo;
        wt[0] = wt[3] = T(-1) / T(16);
        wt[1] = wt[2] = T(9) / T(16);
    }
    T gn[4][5], gs[4][5];
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            gn[s][q] = tn[q][ek[s]];
            gs[s][q] = ts[q][ek[s]];
        }
    T mid[5], end[5];
#pragma unroll
    for (int q = 0; q < 5; ++q) mid[q] = end[q] = T(0);
    const T half = T(0.5);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            mid[q] += wt[s] * (half * gn[s][q] + half * gs[s][q]);
            end[q] += wt[s] * gn[s][q];
        }
    }
    T *ro = reinterpret_cast<T *>(p.ring_out);
    T out0[5], out1[5];
    rescale_collide<S, KIND>(p, mid, i, j, out0);
    rescale_collide<S, KIND>(p, end, i, j, out1);
#pragma unroll
    for (int k = 0; k < 5; ++k) {
        ro[k * g.nring + r] = out0[k];
        ro[(5 + k) * g.nring + r] = out1[k];
    }
}

// ---- fused step -------------------------------------------------------------
template <typename S>
constexpr bool kIsF64 = sizeof(S) == 8;

// The receivers of a row, entries [rb, re), among the wave's columns: lane l of
// the m active ones (the first m) holds columns x0 .. x0 + V - 1 with their
// pre-collision state g; x1 ends the row.  The lanes look at m entries at a
// time, and each writes the fields of its entry, taken from the lane that
// holds the column.  (A search by each lane was a chain of loads: 8.5 us for a
// step of 256^2 with 64 receivers in a row, 5.1 so; of 300^2, whose rows end
// with 11 lanes, 8.7 and 6.3.)
template <typename T, int Q, int V>
__device__ inline void record_wave(const Receivers &rc, int rb, int re, int x0, int x1, const T (&g)[Q][V], const T (&c2)[V]) {
    const int lane = threadIdx.x & 63, m = __builtin_popcountll(__ballot(true));
    const int xa = __builtin_amdgcn_readfirstlane(x0), xe = min(xa + m * V, x1);
    if (m < 4) {   // a short end of a row
#pragma unroll
        for (int j = 0; j < V; ++j) {
            T gj[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i) gj[i] = g[i][j];
            if (x0 + j < x1) record_node<T, Q>(rc, rb, re, x0 + j, gj, c2[j]);
        }
        return;
    }
    int l = rb, u = re;   // the first entry with x >= xa is in [l, u]
    while (u - l > m) {
        const int st = (u - l + m - 1) / m, e = l + lane * st;
        const int c = __builtin_popcountll(__ballot(e < u && rc.xs[min(e, u - 1)] < xa));
        u = min(u, l + c * st);
        l = c > 0 ? l + (c - 1) * st + 1 : l;
    }
    const int64_t plane = (int64_t)rc.nslots * rc.cap;
    for (bool more = true; more && l < re; l += m) {
        const int e = min(l + lane, re - 1), x = rc.xs[e], slot = rc.slot[e];
        const bool hit = l + lane < re && x >= xa && x < xe;
        more = __builtin_amdgcn_readlane(x, m - 1) < xe;
        if (__ballot(hit) == 0) continue;
        const int c = min(max(x - xa, 0), m * V - 1), from = c / V, jj = c % V;
        T *tr = reinterpret_cast<T *>(rc.traces) + (int64_t)slot * rc.cap + rc.col;
        for (int f = 0; f < 4; ++f) {
            if (!((rc.what >> f) & 1)) continue;
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
                const T v = f == 0 ? c2[j] * rho : f == 1 ? rho : f == 2 ? jx : jy;
                const T vs = __shfl(v, from);
                if (jj == j) out = vs;
            }
            if (hit) *tr = out;
            tr += plane;
        }
    }
}

// One thread's share of the update: V consecutive nodes (x0 .. x0+V-1) of row
// y, of which those from x1 on are another block's.  SUM: their rho goes to
// rho_row.
template <typename S, int Q, int KIND, bool PULL, bool SUM>
__device__ inline void update_tile(const StepParams &p, int x0, int x1, int y, typename Tr<S>::T *rho_row) {
    using T = typename Tr<S>::T;
    constexpr int V = PULL ? Tr<S>::V : 1;
    const int nx = p.nx, ny = p.ny;
    if (x0 >= x1) return;

    const S *src = reinterpret_cast<const S *>(p.src);
    T g[Q][V];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const int ys = PULL ? wrapi(y - cyv<Q>(i), ny) : y;
        const S *row = src + i * p.pstride + (int64_t)ys * nx;
        S t[V];
        load_x<S, V>(row, PULL ? x0 - cxv<Q>(i) : x0, nx, t);
#pragma unroll
        for (int j = 0; j < V; ++j) g[i][j] = T(t[j]);
    }
    T c2v[V];
    {
        const T *c2row = reinterpret_cast<const T *>(p.c2) + (int64_t)y * nx;
        if (V > 1 && x0 + V <= nx) {
            typedef T ct __attribute__((ext_vector_type(V), aligned(sizeof(T))));
            ct t = __builtin_nontemporal_load(reinterpret_cast<const ct *>(c2row + x0));
#pragma unroll
            for (int j = 0; j < V; ++j) c2v[j] = t[j];
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j) c2v[j] = c2row[min(x0 + j, nx - 1)];
        }
    }

    // refinement: the pre-collision state of this time on the coarse ring
    // line feeds the temporal interpolation of the next coarse step
    if (Q == 5 && p.snap) {
        T *snap = reinterpret_cast<T *>(p.snap);
        const int X0 = p.snap_x0, Y0 = p.snap_y0, W = p.snap_w, H = p.snap_h;
        const int nh = W + 3, nv = H + 3;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const int x = x0 + j;
            if (x >= x1) break;
            if ((y == Y0 || y == Y0 + H) && x >= X0 - 1 && x <= X0 + W + 1) {
                const int t = (y == Y0 ? 0 : nh) + (x - (X0 - 1));
#pragma unroll
                for (int i = 0; i < Q; ++i) snap[i * p.snap_n + t] = g[i][j];
            }
            if ((x == X0 || x == X0 + W) && y >= Y0 - 1 && y <= Y0 + H + 1) {
                const int t = 2 * nh + (x == X0 ? 0 : nv) + (y - (Y0 - 1));
#pragma unroll
                for (int i = 0; i < Q; ++i) snap[i * p.snap_n + t] = g[i][j];
            }
        }
    }

    // receivers of this row (CSR lookup; rows without receivers cost one
    // uniform pair of loads)
    int rb = 0, re = 0;
    if (p.rec.row_ptr) {
        rb = p.rec.row_ptr[y];
        re = p.rec.row_ptr[y + 1];
    }
    // Registers are short for the 8 x 9 populations of D2Q9 with half storage:
    // its nodes search for themselves as they are updated (2300^2: 57 us per
    // step, 62 with a search before the updates)
    constexpr bool by_node = V * Q > 64;
    if constexpr (!by_node)
        if (rb < re) record_wave<T, Q, V>(p.rec, rb, re, x0, x1, g, c2v);

    S outv[Q][V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        T gj[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) gj[i] = g[i][j];
        const int x = x0 + j;
        if constexpr (by_node)
            if (rb < re && x < x1) record_node<T, Q>(p.rec, rb, re, x, gj, c2v[j]);
        if ((SUM || p.rho_out) && x < x1) {
            T rho = T(0);
#pragma unroll
            for (int i = 0; i < Q; ++i) rho += gj[i];
            if constexpr (SUM) rho_row[j] = rho;
            if (p.rho_out) reinterpret_cast<T *>(p.rho_out)[(int64_t)y * nx + x] = rho;
        }
        T po[Q];
        post_node<T, Q, KIND>(p, gj, c2v[j], x, y, edge_dist(min(x, nx - 1), y, nx, ny), p.s_n, po);
#pragma unroll
        for (int i = 0; i < Q; ++i) outv[i][j] = to_store<S>(po[i]);
        if constexpr (Q == 5) {
            if (p.restrict_on && x < nx && !((x | y) & 1)) {
                // this fine node coincides with a coarse node: on the coarse
                // inner ring, its state (R_2, then the coarse collision)
                // replaces the coarse grid's own
                const PatchGeom &pg = p.iface.g;
                const int X = pg.X0 + (x >> 1), Y = pg.Y0 + (y >> 1);
                if (X >= pg.xa && X <= pg.xb && Y >= pg.ya && Y <= pg.yb &&
                    (X == pg.xa || X == pg.xb || Y == pg.ya || Y == pg.yb))
                    rescale_collide_store_impl<S, KIND>(p.iface, gj, X, Y);
            }
            if (p.ring_buf && x < nx && (y == 0 || y == ny - 1 || x == 0 || x == nx - 1)) {
                // outer ring of a fine grid: the state comes from the coarse
                // grid, not from streaming
                const int r = y == 0 ? x : y == ny - 1 ? nx + x : x == 0 ? 2 * nx + y - 1 : 2 * nx + ny - 2 + y - 1;
                const T *rb = reinterpret_cast<const T *>(p.ring_buf);
#pragma unroll
                for (int i = 0; i < 5; ++i) outv[i][j] = to_store<S>(rb[i * p.ring_n + r]);
            }
        }
    }
    S *dst = reinterpret_cast<S *>(p.dst);
#pragma unroll
    for (int i = 0; i < Q; ++i)
        store_x<S, V>(dst + i * p.dst_pstride + (int64_t)y * nx, x0, x1, outv[i]);
}

// Columns of a block that takes the sum of rho: whole strips of `ow` columns.
__host__ __device__ inline int sum_columns(int columns, int ow) { return columns / ow * ow; }


template <typename S, int Q, int KIND, bool PULL, bool SUM>
__device__ __attribute__((always_inline)) inline void step_body(const StepParams &p) {
    constexpr int V = PULL ? Tr<S>::V : 1;
    if constexpr (Q == 5 && !kIsF64<S> && !SUM) {
        // leading block rows of a coarse launch: the fine outer-ring states
        // of this coarse step (they read only what this launch reads; FP64
        // runs them as a launch of their own, whose registers would lower
        // this kernel's occupancy)
        if ((int)blockIdx.y < p.pre_rows) {
            prolong_pair_tile<S, KIND, kStepBlock>(p.iface, (int)blockIdx.y * gridDim.x + blockIdx.x);
            return;
        }
    }
    const int y = blockIdx.y - p.pre_rows + p.y0;
    if constexpr (!SUM) {
        update_tile<S, Q, KIND, PULL, false>(p, p.x0 + (blockIdx.x * kStepBlock + threadIdx.x) * V, p.x1, y, nullptr);
    } else {
        // The sum of rho by row and strip, added as the flowing kernel adds it,
        // so that a time's sum does not depend on the launch that records it.
        // (A single step of 4096^2 and its sum: 131 us in FP32 and 254 in FP64;
        // through the flowing kernel, whose blocks read a third more columns,
        // 206 and 399.)
        using T = typename Tr<S>::T;
        __shared__ T rho_row[V * kStepBlock];
        const int ow = 64 * p.sum_v - 2 * p.sum_hx, n = sum_columns(V * kStepBlock, ow);
        const int xb = (int)blockIdx.x * n, x1 = min(xb + n, p.nx), own = (int)threadIdx.x * V;
        update_tile<S, Q, KIND, PULL, true>(p, xb + own, x1, y, rho_row + own);
        __syncthreads();
        const int lane = threadIdx.x & 63;
        for (int k = threadIdx.x >> 6; k * ow < x1 - xb; k += kStepBlock / 64) {
            double a = 0.0;
            for (int j = 0; j < p.sum_v; ++j) {
                const int c = lane * p.sum_v + j - p.sum_hx;
                if (c >= 0 && c < ow && k * ow + c < x1 - xb) a += double(rho_row[k * ow + c]);
            }
            a = wave_total(a);
            if (lane == 63) p.sum[(int64_t)y * p.sum_nstrip + xb / ow + k] = a;
        }
    }
}

template <typename S, int Q, int KIND, bool PULL, bool SUM>
__global__ __launch_bounds__(kStepBlock) void k_step(StepParams p) {
    step_body<S, Q, KIND, PULL, SUM>(p);
}

// A one-step launch of a replayed graph (pull-stream, no interface work).
template <typename S, int Q, int KIND, bool SUM>
__global__ __launch_bounds__(kStepBlock) void k_step_graph(StepParams p) {
    const StepParams q = graph_params(p);
    step_body<S, Q, KIND, true, SUM>(q);
}

// One step of every active shot of a batch, from its params image of the round.
// `per` blocks stand for each of the flowing kernel's shares, and go through the
// shot's tiles in turn.  (Two shots of 4096^2: 263 us a step with a tile per
// block, 283 and 304 with 4 and 16; 370 through the flowing kernel, whose blocks
// read a third more columns.)
template <typename S, int Q, int KIND>
__global__ __launch_bounds__(kStepBlock) void k_step_batch(FlowBatch fb, int per) {
    constexpr int V = Tr<S>::V;
    const int share = blockIdx.x / per;
    int lo = 0, hi = fb.nact - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (fb.prefix[mid] <= share) lo = mid; else hi = mid - 1;
    }
    lo = __builtin_amdgcn_readfirstlane(lo);
    const auto &f = *(const __attribute__((address_space(4))) FlowParams *)(fb.img + __builtin_amdgcn_readfirstlane(fb.order[lo]));
    if (f.nrun < 1) return;
    StepParams p;
    p.src = f.src;
    p.dst = f.dst;
    p.c2 = f.c2;
    p.nx = f.nx;
    p.ny = f.ny;
    p.pstride = p.dst_pstride = f.pstride;
    p.coll.omega = f.coll.omega;
    for (int k = 3; k < Q; ++k) p.coll.srate[k] = f.coll.srate[k];
    p.coll.kax = f.coll.kax;
    p.coll.kdg = f.coll.kdg;
    p.coll.kw = f.coll.kw;
    p.coll.ratio = f.coll.ratio;
    p.sponge_width = f.sponge_width;
    p.sponge_smax = f.sponge_smax;
    p.src_x = f.src_x;
    p.src_y = f.src_y;
    p.s_n = f.s[0];
    p.rec.row_ptr = f.rec.row_ptr;
    p.rec.xs = f.rec.xs;
    p.rec.slot = f.rec.slot;
    p.rec.traces = f.rec.traces;
    p.rec.nslots = f.rec.nslots;
    p.rec.what = f.rec.what;
    p.rec.cap = f.rec.cap;
    p.rec.col = f.rec.col;
    const int bx = (f.nx + V * kStepBlock - 1) / (V * kStepBlock), first = __builtin_amdgcn_readfirstlane(fb.prefix[lo]) * per;
    const int64_t tiles = (int64_t)bx * f.ny, blocks = (int64_t)__builtin_amdgcn_readfirstlane(fb.prefix[lo + 1]) * per - first;
    for (int64_t t = blockIdx.x - first; t < tiles; t += blocks) {
        const int y = (int)(t / bx), x0 = ((int)(t - (int64_t)y * bx) * kStepBlock + (int)threadIdx.x) * V;
        if constexpr (KIND < 6) update_tile<S, Q, KIND, true, false>(p, x0, f.nx, y, nullptr);
        else if (f.coll.written) update_tile<S, Q, KIND - 3, true, false>(p, x0, f.nx, y, nullptr);
        else update_tile<S, Q, KIND - 6, true, false>(p, x0, f.nx, y, nullptr);
    }
}

// ---- discrete adjoint (gradient of the trace misfit w.r.t. c^2) -----------------
// Backward step n: mu(x) = (1 - sigma(x)) lambda(n+1)(x + c_i) (transpose of
// the pull), nu = C mu (C symmetric; its conserved rows drop out of every
// term below), lambda(n) = mu - nu + E^T nu with
// (E^T nu)_j = sum_i w_i nu_i + c_j . sum_i (w_i / c^2) c_i nu_i, plus the
// receiver residuals c^2(x_r) r_r(n) on every population.  Gradient terms of
// time n: rho(n) dw . nu, S(n) dw . mu at the source node, r_r(n) rho(n) at
// receivers, and at n = 0 rho(0) dw . lambda(0) (g(0) is an equilibrium).
// lambda is single-use per step, so it streams like the forward populations.
template <typename T, int Q, int KIND>
__global__ __launch_bounds__(kStepBlock) void k_adjoint(AdjointParams p) {
    constexpr int V = Tr<T>::V;
    const int y = blockIdx.y;
    const int x0 = (blockIdx.x * kStepBlock + threadIdx.x) * V;
    const int nx = p.nx, ny = p.ny;
    if (x0 >= nx) return;
    T mu[Q][V];
    if (p.terminal) {
#pragma unroll
        for (int i = 0; i < Q; ++i)
#pragma unroll
            for (int j = 0; j < V; ++j) mu[i][j] = T(0);
    } else {
        const T *ln = reinterpret_cast<const T *>(p.lam_next);
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const int ys = wrapi(y + cyv<Q>(i), ny);
            T t[V];
            load_x<T, V>(ln + i * p.pstride + (int64_t)ys * nx, x0 + cxv<Q>(i), nx, t);
#pragma unroll
            for (int j = 0; j < V; ++j) mu[i][j] = t[j];
        }
    }
    T c2v[V], rhov[V];
    {
        const T *c2row = reinterpret_cast<const T *>(p.c2) + (int64_t)y * nx;
        const T *rrow = reinterpret_cast<const T *>(p.rho) + (int64_t)y * nx;
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const int x = min(x0 + j, nx - 1);
            c2v[j] = c2row[x];
            rhov[j] = rrow[x];
        }
    }
    // the FP64 gradient of these nodes, read before the arithmetic (16-byte
    // accesses where the row and nx allow) and written back after it
    double gv[V];
    double *grow = p.grad + (int64_t)y * nx;
    const bool gvec = x0 + V <= nx && (((int64_t)y * nx + x0) & 1) == 0;
    if (gvec) {
#pragma unroll
        for (int j = 0; j < V; j += 2) {
            const double2 t = *reinterpret_cast<const double2 *>(grow + x0 + j);
            gv[j] = t.x;
            gv[j + 1] = t.y;
        }
    } else {
#pragma unroll
        for (int j = 0; j < V; ++j) gv[j] = x0 + j < nx ? grow[x0 + j] : 0.0;
    }
    int rb = 0, re = 0;
    if (p.rec.row_ptr) {
        rb = p.rec.row_ptr[y];
        re = p.rec.row_ptr[y + 1];
    }
    T outv[Q][V];
#pragma unroll
    for (int j = 0; j < V; ++j) {
        const int x = x0 + j;
        T muj[Q], lam[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) muj[i] = mu[i][j];
        const double gacc = adjoint_node<T, Q, KIND>(p, muj, c2v[j], rhov[j], x, y, edge_dist(min(x, nx - 1), y, nx, ny),
                                                     x < nx ? rb : 0, x < nx ? re : 0, p.rec.col, p.s_n, p.initial != 0,
                                                     lam);
        gv[j] += gacc;
#pragma unroll
        for (int i = 0; i < Q; ++i) outv[i][j] = lam[i];
    }
    if (gvec) {
#pragma unroll
        for (int j = 0; j < V; j += 2) *reinterpret_cast<double2 *>(grow + x0 + j) = make_double2(gv[j], gv[j + 1]);
    } else {
#pragma unroll
        for (int j = 0; j < V; ++j)
            if (x0 + j < nx) grow[x0 + j] = gv[j];
    }
    T *lo = reinterpret_cast<T *>(p.lam);
#pragma unroll
    for (int i = 0; i < Q; ++i) store_x<T, V>(lo + i * p.pstride + (int64_t)y * nx, x0, nx, outv[i]);
}

// Sum of a value over the 64 lanes of a wavefront by shuffles (lane 0 gets
// it); the order of the additions is fixed, so the result is reproducible.
__device__ inline double wave_sum(double v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
    return v;
}

// Sum over a block of kBlock threads: wave sums, then the wave partials in
// wave order (thread 0 gets it).
__device__ inline double block_sum(double v) {
    __shared__ double sh[kBlock / 64];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) s += sh[w];
    }
    return s;
}

// Residual r = p - d over columns 0 .. ncols-1 of every receiver (written
// to res) and the per-block partial sums of r^2 in FP64 (partial[b], one per
// block of a grid-stride loop over the nrec x ncols elements).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_misfit_partial(const T *traces, const T *obs, T *res, int32_t nrec,
                                                           int64_t cap, int64_t ncols, double *partial) {
    double s = 0.0;
    const int64_t n = (int64_t)nrec * ncols;
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < n; k += (int64_t)gridDim.x * kBlock) {
        const int64_t r = k / ncols, c = k - r * ncols;
        const int64_t idx = r * cap + c;
        const T d = traces[idx] - obs[idx];
        res[idx] = d;
        s += double(d) * double(d);
    }
    s = block_sum(s);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// phi = 1/2 (sum of the nb block partials), one block, fixed order.
__global__ __launch_bounds__(kBlock) void k_misfit_finalize(const double *partial, int32_t nb, double *phi) {
    double s = 0.0;
    for (int i = threadIdx.x; i < nb; i += kBlock) s += partial[i];
    s = block_sum(s);
    if (threadIdx.x == 0) *phi = 0.5 * s;
}

// A thread's share of n partials, U loads in flight together.
template <int U>
__device__ inline double sum_groups(const double *p, int64_t n) {
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += U * kBlock) {
        double a[U];
#pragma unroll
        for (int k = 0; k < U; ++k) a[k] = p[min(i + k * kBlock, n - 1)];
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (i + k * kBlock < n) s += a[k];
    }
    return s;
}

// Sum of n partials over a block, in thread 0.  (One load at a time was a chain
// of 340 us for the 176 k of a time on 4096^2.)
__device__ inline double sum_partials(const double *p, int64_t n) {
    const double s = n <= kBlock ? sum_groups<1>(p, n) : n <= 4 * kBlock ? sum_groups<4>(p, n) : sum_groups<16>(p, n);
    __shared__ double sh[kBlock];
    sh[threadIdx.x] = s;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    return sh[0];
}

// Many partials per time: kSumFolds sums of equal shares first (block x of
// time y).  One CU reads the 4 MB of a time on 4096^2 in FP64 in 80 us.
__global__ __launch_bounds__(kBlock) void k_sum_fold(const double *partial, int64_t n, double *fold) {
    const int64_t share = (n + kSumFolds - 1) / kSumFolds, b = share * blockIdx.x;
    const double s = b < n ? sum_partials(partial + n * blockIdx.y + b, min(share, n - b)) : 0.0;
    if (threadIdx.x == 0) fold[blockIdx.y * kSumFolds + blockIdx.x] = s;
}

__global__ __launch_bounds__(kBlock) void k_sum_finalize(const double *partial, int64_t n, double *out,
                                                          const GraphTab *gtab) {
    const double s = sum_partials(partial + n * blockIdx.x, n);   // one time per block
    if (threadIdx.x == 0) out[(gtab ? gtab->t0 : 0) + blockIdx.x] = s;
}

// The chunk table of a graph replay, copied from the kernel arguments.
__global__ __launch_bounds__(kBlock) void k_graph_prime(GraphTab *dst, GraphTab val) {
    double *d = reinterpret_cast<double *>(dst);
    const double *v = reinterpret_cast<const double *>(&val);
    for (int i = threadIdx.x; i < (int)(sizeof(GraphTab) / 8); i += kBlock) d[i] = v[i];
}

// ---- set-up kernels --------------------------------------------------------
template <typename S, int Q>
__global__ __launch_bounds__(kBlock) void k_equilibrium(S *pop, int64_t pstride, const void *c2v,
                                                        const void *rho, const void *jx, const void *jy,
                                                        int in_f64, int64_t n, Collision c) {
    using T = typename Tr<S>::T;
    int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= n) return;
    auto rd = [&](const void *a) -> double {
        if (!a) return 0.0;
        return in_f64 ? reinterpret_cast<const double *>(a)[k] : double(reinterpret_cast<const float *>(a)[k]);
    };
    T r = T(rd(rho)), x = T(rd(jx)), y = T(rd(jy));
    T c2 = reinterpret_cast<const T *>(c2v)[k];
    T w[Q];
    weights<T, Q>(c2, c, w);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        T kj = Q == 5 ? T(0.5) : (i <= 4 ? T(c.kax) : T(c.kdg));
        T cj = T(cxv<Q>(i)) * x + T(cyv<Q>(i)) * y;
        pop[i * pstride + k] = to_store<S>(w[i] * r + (i == 0 ? T(0) : kj * cj));
    }
}

template <typename T>
__global__ __launch_bounds__(kBlock) void k_convert_c2(const void *in, int in_f64, T *out, int64_t n,
                                                       double c2max, int32_t *bad) {
    int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= n) return;
    double v = in_f64 ? reinterpret_cast<const double *>(in)[k] : double(reinterpret_cast<const float *>(in)[k]);
    if (!(v > 0.0 && v <= c2max)) atomicAdd(bad, 1);
    out[k] = T(v);
}

__global__ __launch_bounds__(kBlock) void k_fill_zero(uint32_t *p, int64_t nwords) {
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < nwords; k += (int64_t)gridDim.x * kBlock)
        p[k] = 0u;
}

typedef float f4a __attribute__((ext_vector_type(4)));
// Reference copy: 16-byte nontemporal loads and stores, the access pattern of
// the fused step reduced to one read and one write stream.
__global__ __launch_bounds__(kBlock) void k_copy(f4a *__restrict__ dst, const f4a *__restrict__ src, int64_t n) {
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < n; k += (int64_t)gridDim.x * kBlock)
        __builtin_nontemporal_store(__builtin_nontemporal_load(src + k), dst + k);
}

// ---- fields of the current state ----------------------------------------------
template <typename S, int Q>
__global__ __launch_bounds__(kBlock) void k_field(FieldParams p) {
    using T = typename Tr<S>::T;
    int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k >= (int64_t)p.nx * p.ny) return;
    const int x = int(k % p.nx), y = int(k / p.nx);
    const S *pop = reinterpret_cast<const S *>(p.pop);
    T rho = T(0), jx = T(0), jy = T(0);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        int xs = p.pre ? x : wrapi(x - cxv<Q>(i), p.nx);
        int ys = p.pre ? y : wrapi(y - cyv<Q>(i), p.ny);
        T gi = T(pop[i * p.pstride + (int64_t)ys * p.nx + xs]);
        rho += gi;
        jx += T(cxv<Q>(i)) * gi;
        jy += T(cyv<Q>(i)) * gi;
    }
    T v = rho;
    if (p.what == 1u) v = reinterpret_cast<const T *>(p.c2)[k] * rho;
    else if (p.what == 4u) v = jx;
    else if (p.what == 8u) v = jy;
    reinterpret_cast<T *>(p.out)[k] = v;
}

// Fine outer ring layout: top row (j = 0), bottom row (j = nyf-1), left
// column (i = 0, j = 1 .. nyf-2), right column (i = nxf-1).
template <typename S, int KIND>
__global__ __launch_bounds__(kBlock) void k_prolong(InterfaceParams p) {
    using T = typename Tr<S>::T;
    int r = blockIdx.x * kBlock + threadIdx.x;
    if (r >= p.g.nring) return;
    const PatchGeom &g = p.g;
    int i, j;
    if (r < g.nxf) { i = r; j = 0; }
    else if (r < 2 * g.nxf) { i = r - g.nxf; j = g.nyf - 1; }
    else if (r < 2 * g.nxf + g.nyf - 2) { i = 0; j = 1 + r - 2 * g.nxf; }
    else { i = g.nxf - 1; j = 1 + r - 2 * g.nxf - (g.nyf - 2); }
    T gh[5];
    ring_interp<S>(p, i, j, gh);
    rescale_collide_store_impl<S, KIND>(p, gh, i, j);
}

template <typename S, int KIND>
__global__ __launch_bounds__(kBlock) void k_restrict(InterfaceParams p) {
    using T = typename Tr<S>::T;
    int t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= p.g.ninner) return;
    const PatchGeom &g = p.g;
    const int nxr = g.xb - g.xa + 1;
    const int nyr = g.yb - g.ya - 1;
    int x, y;
    if (t < nxr) { x = g.xa + t; y = g.ya; }
    else if (t < 2 * nxr) { x = g.xa + t - nxr; y = g.yb; }
    else if (t < 2 * nxr + nyr) { x = g.xa; y = g.ya + 1 + t - 2 * nxr; }
    else { x = g.xb; y = g.ya + 1 + t - 2 * nxr - nyr; }
    T gf[5];
    pre_at<S, T>(p.fine, 2 * (x - g.X0), 2 * (y - g.Y0), gf);
    rescale_collide_store_impl<S, KIND>(p, gf, x, y);
}

// The ring-line snapshot of p.coarse's time, where no coarse launch has kept it.
template <typename S>
__global__ __launch_bounds__(kBlock) void k_ring_line(InterfaceParams p) {
    using T = typename Tr<S>::T;
    const PatchGeom &g = p.g;
    const int nh = g.W + 3, nv = g.H + 3;
    const int t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= g.nsnap) return;
    int x, y;
    if (t < 2 * nh) { x = g.X0 - 1 + t % nh; y = g.Y0 + (t < nh ? 0 : g.H); }
    else { x = g.X0 + (t - 2 * nh < nv ? 0 : g.W); y = g.Y0 - 1 + (t - 2 * nh) % nv; }
    T gn[5];
    pre_at<S, T>(p.coarse, x, y, gn);
#pragma unroll
    for (int i = 0; i < 5; ++i) reinterpret_cast<T *>(p.snap)[i * g.nsnap + t] = gn[i];
}

template <typename S, int KIND>
__global__ __launch_bounds__(kBlock) void k_prolong_pair(InterfaceParams p) {
    prolong_pair_tile<S, KIND, kBlock>(p, blockIdx.x);
}

// ---- dispatch helpers ----------------------------------------------------------
inline unsigned blocks_for(int64_t n) { return unsigned((n + kBlock - 1) / kBlock); }

template <typename S>
int vwidth(bool pull) { return pull ? Tr<S>::V : 1; }

// f(lattice, kind), both as integral constants.
template <typename S, typename F>
hipError_t step_by_lattice(int q, int kind, F &&f) {
    if (q == 5) return for_kind<S, 5>(kind, [&](auto kc) { return f(std::integral_constant<int, 5>(), kc); });
    return for_kind<S, 9>(kind, [&](auto kc) { return f(std::integral_constant<int, 9>(), kc); });
}

template <typename S>
hipError_t step_dispatch(const StepParams &p0, bool pull, hipStream_t s) {
    const int V = vwidth<S>(pull);
    const int kind = step_kind(p0.coll);
    StepParams p = p0;
    p.pre_rows = 0;
    if (p.x1 <= 0) {   // the whole grid
        p.x0 = p.y0 = 0;
        p.x1 = p.nx;
        p.y1 = p.ny;
        p.dst_pstride = p.pstride;
    }
    if (p.x0 < 0 || p.y0 < 0 || p.x0 >= p.x1 || p.y0 >= p.y1 || p.x1 > p.nx || p.y1 > p.ny) return hipErrorInvalidValue;
    int cols = V * kStepBlock;   // of a block
    if (p.sum) {   // the whole grid, in strips of whole vectors
        const int ow = 64 * p.sum_v - 2 * p.sum_hx;
        if (ow < V || ow % V || ow > cols || p.x1 != p.nx || p.y1 != p.ny || p.x0 || p.y0 || p.prolong_on ||
            (int64_t)p.sum_nstrip * ow < p.nx)
            return hipErrorInvalidValue;
        cols = sum_columns(cols, ow);
    }
    dim3 grid((unsigned)(((int64_t)p.x1 - p.x0 + cols - 1) / cols), (unsigned)(p.y1 - p.y0));
    if (p0.prolong_on) {
        const int rows = (int)((ring_tile_blocks<kStepBlock>(p0.iface.g) + grid.x - 1) / grid.x);
        if (!kIsF64<S> && (int64_t)grid.y + rows <= 65535) {
            p.pre_rows = rows;
            grid.y += (unsigned)rows;
        } else {   // a launch of its own first
            dim3 pg((unsigned)ring_tile_blocks<kBlock>(p0.iface.g));
            const hipError_t e = for_kind<S, 5>(kind, [&](auto kc) {
                hipLaunchKernelGGL((k_prolong_pair<S, decltype(kc)::value>), pg, dim3(kBlock), 0, s, p0.iface);
                return hipGetLastError();
            });
            if (e != hipSuccess) return e;
        }
    }
    // a launch of a captured chunk has its own entry kernel
    if (p.gtab && (!pull || p.prolong_on || p.restrict_on || p.snap || p.ring_buf)) return hipErrorInvalidValue;
    auto launch = [&](auto sc) {
        constexpr bool SUM = decltype(sc)::value;
        return step_by_lattice<S>(p.q, kind, [&](auto qc, auto kc) {
            constexpr int Q = decltype(qc)::value, KIND = decltype(kc)::value;
            if (p.gtab) hipLaunchKernelGGL((k_step_graph<S, Q, KIND, SUM>), grid, dim3(kStepBlock), 0, s, p);
            else if (pull) hipLaunchKernelGGL((k_step<S, Q, KIND, true, SUM>), grid, dim3(kStepBlock), 0, s, p);
            else hipLaunchKernelGGL((k_step<S, Q, KIND, false, SUM>), grid, dim3(kStepBlock), 0, s, p);
            return hipGetLastError();
        });
    };
    return p.sum ? launch(std::true_type()) : launch(std::false_type());
}

}  // namespace

// ---- launchers -------------------------------------------------------------------

hipError_t launch_step(int storage, const StepParams &p, bool pull, hipStream_t s) {
    switch (storage) {
    case ST_F32: return step_dispatch<float>(p, pull, s);
    case ST_F64: return step_dispatch<double>(p, pull, s);
    case ST_F16: return step_dispatch<_Float16>(p, pull, s);
    }
    return hipErrorInvalidValue;
}

template <typename S, int Q>
static hipError_t step_batch(const FlowBatch &fb, int64_t nblk, int64_t nodes, int kind, hipStream_t s) {
    const int64_t tile = Tr<S>::V * kStepBlock;   // about a tile per block
    const int per = (int)std::max<int64_t>(1, std::min<int64_t>(256, (nodes / tile + nblk - 1) / nblk));
    return for_batch_kind<S, Q>(kind, [&](auto kc) {
        hipLaunchKernelGGL((k_step_batch<S, Q, decltype(kc)::value>), dim3((unsigned)(nblk * per)), dim3(kStepBlock), 0, s, fb,
                           per);
        return hipGetLastError();
    });
}

hipError_t launch_step_batch(int storage, int q, const BatchParams &bp, int64_t nblk, int64_t nodes, hipStream_t s) {
    if (nblk <= 0 || bp.nact <= 0) return hipSuccess;
    if (bp.img == nullptr || (q != 5 && q != 9) || nblk > (1 << 22)) return hipErrorInvalidValue;
    const FlowBatch fb = flow_batch(bp);
    const int kind = batch_kind(storage, q, bp.coll);
    if (storage == ST_F32) return q == 5 ? step_batch<float, 5>(fb, nblk, nodes, kind, s) : step_batch<float, 9>(fb, nblk, nodes, kind, s);
    if (storage == ST_F64) return q == 5 ? step_batch<double, 5>(fb, nblk, nodes, kind, s) : step_batch<double, 9>(fb, nblk, nodes, kind, s);
    return q == 5 ? step_batch<_Float16, 5>(fb, nblk, nodes, kind, s) : step_batch<_Float16, 9>(fb, nblk, nodes, kind, s);
}

hipError_t launch_adjoint(int storage, const AdjointParams &p, hipStream_t s) {
    const bool f64 = storage == ST_F64;
    const int V = f64 ? Tr<double>::V : Tr<float>::V;
    dim3 grid((unsigned)(((int64_t)p.nx + (int64_t)V * kStepBlock - 1) / ((int64_t)V * kStepBlock)), (unsigned)p.ny);
    const bool mrt = p.coll.kind == 1;
#define LBW_A(TT, QQ)                                                                             \
    do {                                                                                          \
        if (mrt) hipLaunchKernelGGL((k_adjoint<TT, QQ, 1>), grid, dim3(kStepBlock), 0, s, p);     \
        else hipLaunchKernelGGL((k_adjoint<TT, QQ, 0>), grid, dim3(kStepBlock), 0, s, p);         \
    } while (0)
    if (f64) { if (p.q == 5) LBW_A(double, 5); else LBW_A(double, 9); }
    else { if (p.q == 5) LBW_A(float, 5); else LBW_A(float, 9); }
#undef LBW_A
    return hipGetLastError();
}

int misfit_blocks(int32_t nrec, int64_t ncols) {
    const int64_t n = (int64_t)nrec * ncols;
    return (int)std::max<int64_t>(1, std::min<int64_t>((n + kBlock - 1) / kBlock, kMisfitMaxBlocks));
}

hipError_t launch_misfit(int storage, const void *traces, const void *obs, void *res, int32_t nrec, int64_t cap,
                         int64_t ncols, double *phi, double *partial, hipStream_t s) {
    const int nb = misfit_blocks(nrec, ncols);
    if (storage == ST_F64)
        hipLaunchKernelGGL(k_misfit_partial<double>, dim3(nb), dim3(kBlock), 0, s,
                           reinterpret_cast<const double *>(traces), reinterpret_cast<const double *>(obs),
                           reinterpret_cast<double *>(res), nrec, cap, ncols, partial);
    else
        hipLaunchKernelGGL(k_misfit_partial<float>, dim3(nb), dim3(kBlock), 0, s,
                           reinterpret_cast<const float *>(traces), reinterpret_cast<const float *>(obs),
                           reinterpret_cast<float *>(res), nrec, cap, ncols, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_misfit_finalize, dim3(1), dim3(kBlock), 0, s, partial, nb, phi);
    return hipGetLastError();
}

// The shares are a launch more: a single step and its sum take 15.1 us with
// them and 14.5 without on 700^2 (10.5 k partials), 25.0 and 27.0 on 1024^2 in
// FP64 (22.5 k).
hipError_t launch_sum_finalize(const double *partial, int64_t n, int times, double *fold, double *out, const GraphTab *gtab,
                               hipStream_t s) {
    if (n > 16384) {
        hipLaunchKernelGGL(k_sum_fold, dim3(kSumFolds, (unsigned)times), dim3(kBlock), 0, s, partial, n, fold);
        partial = fold;
        n = kSumFolds;
    }
    hipLaunchKernelGGL(k_sum_finalize, dim3((unsigned)times), dim3(kBlock), 0, s, partial, n, out, gtab);
    return hipGetLastError();
}

hipError_t launch_graph_prime(GraphTab *dst, const GraphTab &val, hipStream_t s) {
    static_assert(sizeof(GraphTab) % 8 == 0 && sizeof(GraphTab) <= 4096, "the table travels as a kernel argument");
    hipLaunchKernelGGL(k_graph_prime, dim3(1), dim3(kBlock), 0, s, dst, val);
    return hipGetLastError();
}

hipError_t launch_equilibrium(int storage, int32_t q, void *pop, int64_t pstride, const void *c2,
                              const void *rho, const void *jx, const void *jy, int in_f64,
                              int32_t nx, int32_t ny, const Collision &coll, hipStream_t s) {
    const int64_t n = (int64_t)nx * ny;
    dim3 grid(blocks_for(n));
#define LBW_EQ(SS, QQ) hipLaunchKernelGGL((k_equilibrium<SS, QQ>), grid, dim3(kBlock), 0, s, \
                                          reinterpret_cast<SS *>(pop), pstride, c2, rho, jx, jy, in_f64, n, coll)
    if (storage == ST_F32) { if (q == 5) LBW_EQ(float, 5); else LBW_EQ(float, 9); }
    else if (storage == ST_F64) { if (q == 5) LBW_EQ(double, 5); else LBW_EQ(double, 9); }
    else { if (q == 5) LBW_EQ(_Float16, 5); else LBW_EQ(_Float16, 9); }
#undef LBW_EQ
    return hipGetLastError();
}

hipError_t launch_convert_c2(int storage, const void *in, int in_f64, void *out, int64_t n, double c2max,
                             int32_t *bad, hipStream_t s) {
    dim3 grid(blocks_for(n));
    if (storage == ST_F64)
        hipLaunchKernelGGL(k_convert_c2<double>, grid, dim3(kBlock), 0, s, in, in_f64,
                           reinterpret_cast<double *>(out), n, c2max, bad);
    else
        hipLaunchKernelGGL(k_convert_c2<float>, grid, dim3(kBlock), 0, s, in, in_f64,
                           reinterpret_cast<float *>(out), n, c2max, bad);
    return hipGetLastError();
}

hipError_t launch_fill_zero(void *p, int64_t bytes, hipStream_t s) {
    int64_t words = bytes / 4;
    if (words <= 0) return hipSuccess;
    unsigned nb = (unsigned)std::min<int64_t>((words + kBlock - 1) / kBlock, 65536);
    hipLaunchKernelGGL(k_fill_zero, dim3(nb), dim3(kBlock), 0, s, reinterpret_cast<uint32_t *>(p), words);
    return hipGetLastError();
}

hipError_t launch_copy(void *dst, const void *src, size_t bytes, hipStream_t s) {
    int64_t n = (int64_t)(bytes / 16);
    unsigned nb = (unsigned)std::min<int64_t>((n + kBlock - 1) / kBlock, 1 << 20);
    if (nb == 0) return hipSuccess;
    hipLaunchKernelGGL(k_copy, dim3(nb), dim3(kBlock), 0, s, reinterpret_cast<f4a *>(dst),
                       reinterpret_cast<const f4a *>(src), n);
    return hipGetLastError();
}

hipError_t launch_field(int storage, const FieldParams &p, hipStream_t s) {
    dim3 grid(blocks_for((int64_t)p.nx * p.ny));
#define LBW_F(SS, QQ) hipLaunchKernelGGL((k_field<SS, QQ>), grid, dim3(kBlock), 0, s, p)
    if (storage == ST_F32) { if (p.q == 5) LBW_F(float, 5); else LBW_F(float, 9); }
    else if (storage == ST_F64) { if (p.q == 5) LBW_F(double, 5); else LBW_F(double, 9); }
    else { if (p.q == 5) LBW_F(_Float16, 5); else LBW_F(_Float16, 9); }
#undef LBW_F
    return hipGetLastError();
}

#define LBW_IFACE_KIND(KERNEL, SS)                                                                 \
    return for_kind<SS, 5>(step_kind(p.coll), [&](auto kc) {                                       \
        hipLaunchKernelGGL((KERNEL<SS, decltype(kc)::value>), grid, dim3(kBlock), 0, s, p);        \
        return hipGetLastError();                                                                  \
    })
#define LBW_IFACE(KERNEL, GRID)                                                                    \
    const dim3 grid(GRID);                                                                         \
    if (storage == ST_F32) LBW_IFACE_KIND(KERNEL, float);                                          \
    if (storage == ST_F64) LBW_IFACE_KIND(KERNEL, double);                                         \
    LBW_IFACE_KIND(KERNEL, _Float16);

hipError_t launch_prolong(int storage, const InterfaceParams &p, hipStream_t s) { LBW_IFACE(k_prolong, blocks_for(p.g.nring)) }

hipError_t launch_prolong_pair(int storage, const InterfaceParams &p, hipStream_t s) {
    LBW_IFACE(k_prolong_pair, (unsigned)ring_tile_blocks<kBlock>(p.g))   // one side's nodes per block
}

hipError_t launch_ring_line(int storage, const InterfaceParams &p, hipStream_t s) {
    const dim3 grid(blocks_for(p.g.nsnap));
    if (storage == ST_F32) hipLaunchKernelGGL((k_ring_line<float>), grid, dim3(kBlock), 0, s, p);
    else if (storage == ST_F64) hipLaunchKernelGGL((k_ring_line<double>), grid, dim3(kBlock), 0, s, p);
    else hipLaunchKernelGGL((k_ring_line<_Float16>), grid, dim3(kBlock), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_restrict(int storage, const InterfaceParams &p, hipStream_t s) { LBW_IFACE(k_restrict, blocks_for(p.g.ninner)) }

}  // namespace lbw
