// lb_flow_adjoint.h -- many backward steps of the discrete adjoint per launch:
// the flowing kernel (lb_flow.h) run back in time.  Strips, bundles, the c^2
// ring, the counters and the conditions under which every wait ends are the
// forward kernel's.  Included by one source per compute type and by the
// dispatcher lb_flow.hip.  Device code only; not part of the public interface.
//
// One pass reads lambda(n + 1) and writes lambda(n - ns + 1).  At step s a
// bundle's slot r holds row Y + r - s of lambda(n - s + 1); its sources at the
// step before are again slots r - 2, r - 1 and r, only that the populations
// that move up come from the row below and those that move down from the row
// above (the transpose of the pull).  The FP64 gradient of a row travels with
// it: it is read once, takes the terms of times n, n - 1, .. in that order (as
// one-step launches add them) and is written once; the last row's goes to the
// bundle below with its lambda.  The forward rho of the row a slot holds next
// is read a step ahead.  The residuals of the receivers are added on halo rows
// and columns too, since later steps read them there.
//
// What bounds it: a step of FP32 D2Q5 at tau = 1/2 takes 45 vector operations
// a node (13 of them the FP64 gradient's), 73 with the nodes of halo columns
// and head rows; at 2048^2 and 16 steps the vector units are busy for 107 us
// of a launch's 163, which moves 740 MB.  12.4 us per step, where the kernel
// it replaced (three steps a launch, every wave with halo rows of its own)
// took 24.8; FP64 39.5 and 22.7, D2Q9 FP32 46.1 and 23.7, FP64 87 and 36;
// 256^2 FP32 6.8 and 3.2.
#pragma once

#include "lb_flow.h"

namespace lbw {
namespace {

// V, R, W, EU and E as in FlowShape; FP64 has one shape for all sizes.
// Measured (us per backward step at 2048^2 / 1024^2 / 512^2, best step count
// of each, tape, 64 receivers, 64-node sponge):
//   FP32 D2Q5   V2 R4 W16 12.4 / 6.7 / 5.5, V2 R5 W12 12.7 / 5.6 / 4.4,
//               V2 R9 W8 14.3 / 6.9 / 5.1, V1 R10 W12 15.6 / 5.7 / 3.7,
//               V1 R7 W16 15.0 / 5.0 / 3.2; small V1 R4 W16 - / 5.4 / 3.3
//   FP32 D2Q9   V2 R6 W8 23.7 / 11.4 / 6.9, V1 R6 W12 24.1 / 9.3 / 4.8;
//               small V1 R4 W16 - / 8.4 / 4.5
//   FP64 D2Q5   V1 R4 W16 22.7 / 7.0 / 3.7, V1 R6 W12 23.7 / 7.3 / 3.9
//   FP64 D2Q9   V1 R4 W12 36.3 / 12.1, V1 R6 W8 36.5 / 13.3
// A shape whose rows do not fit the registers loses more than a row less
// costs (FP32 D2Q5 V2 R6 W12, 40 registers spilled: 21.6 at 2048^2).
template <typename T, int Q, bool SMALL> struct AdjointShape {   // D2Q5, FP32
    static constexpr int V = SMALL ? 1 : 2, R = 4, W = 16, EU = 4, E = 0;
};
template <bool SMALL> struct AdjointShape<float, 9, SMALL> {
    static constexpr int V = SMALL ? 1 : 2, R = SMALL ? 4 : 6, W = SMALL ? 16 : 8, EU = SMALL ? 4 : 2, E = SMALL ? 0 : 2;
};
template <> struct AdjointShape<double, 5, false> {
    static constexpr int V = 1, R = 4, W = 16, EU = 4, E = 0;
};
template <> struct AdjointShape<double, 9, false> {
    static constexpr int V = 1, R = 4, W = 12, EU = 3, E = 0;
};

typedef const __attribute__((address_space(4))) AdjointFlowParams *KernAdjoint;

template <typename T, int Q, int KIND, int V, int R, int W, int E>
__device__ __attribute__((always_inline)) inline void flow_adjoint_body(KernAdjoint pa, int blk) {
    typedef typename LaneVec<V, T>::type ct;
    typedef typename LaneVec<V, double>::type gt;
    constexpr int RING = (W + E) * R;
    static_assert(R >= 3 && R <= 16 && V <= 2, "row masks and the receiver table");
    __shared__ ct c2s[(RING + R) * 64];   // as in flow_body
    __shared__ ct edge[2][W][Q][64];
    __shared__ gt gedge[2][W][64];        // gradient of each wave's last row, one step back
    __shared__ uint32_t rtab[W][64 * V];
    __shared__ T sfys[RING + R];
    __shared__ int pub[W], con[W], fin[W];
    const KernFlow p = &pa->f;
    const int nx = p->nx, ny = p->ny, ns = p->nrun, hx = p->hx, ow = 64 * V - 2 * hx;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (threadIdx.x < W) {
        pub[threadIdx.x] = 0;
        con[threadIdx.x] = 0;
        fin[threadIdx.x] = 0;
    }
    __syncthreads();
    const int wp = w > 0 ? w - 1 : W - 1, wc = w < W - 1 ? w + 1 : 0;
    const int L = p->sponge_width;
    CollisionT<T> coll;
    if constexpr (KIND == 0) coll.omega = uniform(T(p->coll.omega));
    if constexpr (KIND == 1)
        for (int k = 3; k < Q; ++k) coll.srate[k] = uniform(T(p->coll.srate[k]));
    if constexpr (Q == 9) {
        coll.kax = uniform(T(p->coll.kax));
        coll.kdg = uniform(T(p->coll.kdg));
        coll.kw = uniform(T(p->coll.kw));
        coll.ratio = uniform(T(p->coll.ratio));
    }
    // kind 2 takes dw . nu as (2 dw) . m
    double dw[9];
    for (int k = 0; k < 9; ++k) dw[k] = KIND == 2 ? 2.0 * pa->dw[k] : pa->dw[k];

    const int nbs = (ny + R - 1) / R;
    const int b0 = share_start(p, nbs, blk), b1 = share_start(p, nbs, blk + 1);
    const int total = share_bundles(R, ny, ns, nbs, b0, b1);
    const int mlast = (R + ns - 1) / R;
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
        const int xl = xa + lane * V, c0 = lane * V;
        const bool own0 = c0 >= hx && c0 < hx + ow && xl < nx;
        // lambda, gradient and next rho of each slot's row
        T h[R][Q][V], rho[R][V], fx[V];
        double G[R][V];
        // bit k, row Y - ns + k: has receivers, the source, the sponge
        uint32_t mrec = 0, msrc, mspo = 0;
        uint32_t ent[V];   // the lane's entries of the receiver table, and their residuals
        T rv[V];
        int nrec = 0, xw[V];
#pragma unroll
        for (int j = 0; j < V; ++j) xw[j] = wrapi(xl + j, nx);
        const bool vec = V == 1 || nx % V == 0 || (xa >= 0 && xa + 64 * V <= nx);
        // Rho of row gy at the stored columns (others: any value), without a
        // branch: with loads under one, the compiler cannot tell how many are
        // in flight and has each step wait for the last one (V2 R5 W12 at
        // 2048^2: 13.9 us per step, 12.9 so).  A lane whose columns reach beyond the last
        // one reads the last V, of which the later ones are its own (rho_off).
        const int xr = min(max(xl, 0), nx - V);
        const bool rho_off = V > 1 && xl < nx && xl > xr;
        auto load_rho = [&](const T *field, int gy, T (&out)[V]) __attribute__((always_inline)) {
            const ct t = ld_hint(at_lane<const ct>(field + (int64_t)min(max(gy, ya), yb - 1) * nx, xr), false);
#pragma unroll
            for (int j = 0; j < V; ++j) out[j] = t[j];
        };
        {
            const int row_l = Y - ns + lane, rowi = wrapi(row_l, ny);   // lane k: row Y - ns + k
            T cl[R][V];
            auto load = [&](auto vc) __attribute__((always_inline)) {
                constexpr bool VEC = decltype(vc)::value;
                const T *src = reinterpret_cast<const T *>(p->src);
                const T *c2 = reinterpret_cast<const T *>(p->c2);
                static_for<0, R>([&](auto rc) __attribute__((always_inline)) {
                    constexpr int r = decltype(rc)::value;
                    const int64_t ro = (int64_t)__builtin_amdgcn_readlane(rowi, ns + r) * nx;
                    load_row2<VEC, 0, true, T, T, Q, V>(src, p->pstride, ro, xw[0], xw, h[r]);
                    load_c2row<VEC, true, T, V>(c2, ro, xw[0], xw, cl[r]);
                });
            };
            if (vec) load(std::true_type()); else load(std::false_type());
            // slot r's row of the first step is the one above
            static_for<0, R>([&](auto rc) __attribute__((always_inline)) {
                constexpr int r = decltype(rc)::value;
                load_rho(reinterpret_cast<const T *>(pa->rho), Y + r - 1, rho[r]);
            });
            static_for<0, R>([&](auto rc) __attribute__((always_inline)) {
                constexpr int r = decltype(rc)::value;
                const int gy = Y + r;
#pragma unroll
                for (int j = 0; j < V; ++j) G[r][j] = 0.0;
                if (gy >= ya && gy < yb && own0) {
                    const GlobalPtr<const double> gr = (GlobalPtr<const double>)(pa->grad + (int64_t)gy * nx);
#pragma unroll
                    for (int j = 0; j < V; ++j)
                        if (xl + j < nx) G[r][j] = gr[xl + j];
                }
            });
            const bool mine = lane < R + ns;
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
            // receivers on any row and column of the bundle, by row and then
            // in the list's order, where the columns wrap once per image
            {
                const GlobalPtr<const int32_t> rp = (GlobalPtr<const int32_t>)p->rec.row_ptr,
                                               xs = (GlobalPtr<const int32_t>)p->rec.xs,
                                               sl = (GlobalPtr<const int32_t>)p->rec.slot;
                int rb_l = 0, re_l = 0;
                if (mine && p->rec.row_ptr != nullptr) {
                    rb_l = rp[rowi];
                    re_l = rp[rowi + 1];
                }
                for (uint32_t m = (uint32_t)__ballot(rb_l < re_l); m; m &= m - 1) {
                    const int k = __builtin_ctz(m);
                    const int rb = __builtin_amdgcn_readlane(rb_l, k), re = __builtin_amdgcn_readlane(re_l, k);
                    for (int xo = xa - wrapi(xa, nx); xo < xa + 64 * V; xo += nx) {
                        const int x0 = xa - xo, x1 = x0 + 64 * V;   // the image's columns of the strip
                        int l = rb, u = re;   // the first entry with x >= x0 is in [l, u]
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
                                    (uint32_t)k << 27 | (uint32_t)(x - x0) << 19 | (uint32_t)(slot & 0x7ffff);
                            nrec += n;
                            more = __builtin_amdgcn_readlane(x, 63) < x1;
                        }
                    }
                }
                if (p->rec.nslots > 0x80000) nrec = 64 * V + 1;   // slots too large for the table
            }
            order();
#pragma unroll
            for (int j = 0; j < V; ++j) {
                ent[j] = 0xffffffffu;
                rv[j] = T(0);
                if (nrec <= 64 * V && lane + 64 * j < nrec) {
                    ent[j] = rtab[w][lane + 64 * j];
                    rv[j] = ((GlobalPtr<const T>)p->rec.traces)[(int64_t)(ent[j] & 0x7ffff) * p->rec.cap + p->rec.col];
                }
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
                    if (cyv<Q>(i) <= 0) edge[n & 1][w][k++][lane] = t;
                    if (cyv<Q>(i) < 0) {
#pragma unroll
                        for (int j = 0; j < V; ++j) t[j] = h[R - 2][i][j];
                        edge[n & 1][w][k++][lane] = t;
                    }
                }
                gt g;
#pragma unroll
                for (int j = 0; j < V; ++j) g[j] = G[R - 1][j];
                gedge[n & 1][w][lane] = g;
                order();
                set_count(&pub[w], n);
            }
            order();
            // the residuals of the next step
            T rvn[V];
#pragma unroll
            for (int j = 0; j < V; ++j) rvn[j] = T(0);
            if (nrec > 0 && s < ns) {
                const KernFlow z = rare(p);
#pragma unroll
                for (int j = 0; j < V; ++j)
                    if (ent[j] != 0xffffffffu)
                        rvn[j] = ((GlobalPtr<const T>)z->rec.traces)[(int64_t)(ent[j] & 0x7ffff) * z->rec.cap + z->rec.col - s];
            }
            const int rs = ring - s + (ring < s ? RING : 0);   // ring row of slot 0
            const ct *cb = c2s + rs * 64 + lane;
            const T *sb = sfys + rs + min(lane, R - 1);
            const int sh = ns - s;
            const bool initial = pa->initial_stage == s;
            const uint32_t bspo = mspo >> sh, bpost = initial ? ~0u : (msrc | mrec) >> sh;
            const T *rho_s = reinterpret_cast<const T *>(pa->rho) - (int64_t)min(s, ns - 1) * pa->rho_back;   // the next step's
            T fyl = T(1);
            if (mspo) fyl = *sb;
            ct cn = cb[(R - 1) * 64];
            // gin: the gradient of the slot's row before this step
            auto row = [&](auto rc, const T (&U)[Q][V], const T (&C)[Q][V], const T (&D)[Q][V],
                           const double (&gin)[V]) __attribute__((always_inline)) {
                constexpr int r = decltype(rc)::value;
                T cm[V];
#pragma unroll
                for (int j = 0; j < V; ++j) cm[j] = cn[j];
                if constexpr (r > 0) cn = cb[(r - 1) * 64];
                T mu[Q][V];
                pull_back_row<T, Q, V>(U, C, D, mu);
                if (__builtin_expect((bspo >> r) & 1, 0)) {
                    const T fy = lane_of(fyl, r);
#pragma unroll
                    for (int j = 0; j < V; ++j) {
                        const T sf = min(fx[j], fy);
#pragma unroll
                        for (int i = 0; i < Q; ++i) mu[i][j] = mu[i][j] * sf;
                    }
                }
                T lam[V][Q], ro[V];
                double ga[V];
#pragma unroll
                for (int j = 0; j < V; ++j) ro[j] = j + 1 < V && rho_off ? rho[r][V - 1] : rho[r][j];
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    T m[Q], nu[Q];
#pragma unroll
                    for (int i = 0; i < Q; ++i) m[i] = mu[i][j];
                    adjoint_relax<T, Q, KIND>(m, coll, nu);
                    ga[j] = double(ro[j]) * dw_dot<T, Q>(dw, KIND == 2 ? m : nu);
                    adjoint_lambda<T, Q, KIND>(m, nu, cm[j], coll, lam[j]);
                }
                if (__builtin_expect((bpost >> r) & 1, 0)) {
                    if ((msrc >> (sh + r)) & 1) {
                        const KernFlow z = rare(p);
                        const double snv = z->s[s - 1];
                        const int sxs = z->src_x;
#pragma unroll
                        for (int j = 0; j < V; ++j) {
                            if (xw[j] == sxs) {
                                T m[Q];
#pragma unroll
                                for (int i = 0; i < Q; ++i) m[i] = mu[i][j];
                                ga[j] += (KIND == 2 ? 0.5 : 1.0) * (snv * dw_dot<T, Q>(dw, m));
                            }
                        }
                    }
                    if ((mrec >> (sh + r)) & 1) {
                        auto add = [&](auto jc, T rr) __attribute__((always_inline)) {
                            constexpr int j = decltype(jc)::value;
#pragma unroll
                            for (int i = 0; i < Q; ++i) lam[j][i] += cm[j] * rr;
                            ga[j] += double(rr) * double(ro[j]);
                        };
                        if (nrec <= 64 * V) {
#pragma unroll
                            for (int jj = 0; jj < V; ++jj) {
                                for (uint64_t hits = __ballot(ent[jj] != 0xffffffffu && (int)(ent[jj] >> 27) == sh + r); hits;
                                     hits &= hits - 1) {
                                    const int k = __builtin_ctzll(hits);
                                    const int c = (__builtin_amdgcn_readlane((int)ent[jj], k) >> 19) & 0xff;
                                    const T rr = lane_of(rv[jj], k);
                                    static_for<0, V>([&](auto jc) __attribute__((always_inline)) {
                                        if (c0 + decltype(jc)::value == c) add(jc, rr);
                                    });
                                }
                            }
                        } else {   // each lane searches the row's list
                            const KernFlow z = rare(p);
                            const int gy = wrapi(Y + r - s, ny);
                            const GlobalPtr<const int32_t> xs = (GlobalPtr<const int32_t>)z->rec.xs;
                            const int rb = ((ConstInt)z->rec.row_ptr)[gy], re = ((ConstInt)z->rec.row_ptr)[gy + 1];
                            static_for<0, V>([&](auto jc) __attribute__((always_inline)) {
                                const int x = xw[decltype(jc)::value];
                                int lo = rb, hi = re;
                                while (lo < hi) {
                                    const int mid = (lo + hi) >> 1;
                                    if (xs[mid] < x) lo = mid + 1; else hi = mid;
                                }
                                for (; lo < re && xs[lo] == x; ++lo)
                                    add(jc, ((GlobalPtr<const T>)z->rec.traces)[(int64_t)((GlobalPtr<const int32_t>)z->rec.slot)[lo] *
                                                                                    z->rec.cap + z->rec.col - (s - 1)]);
                            });
                        }
                    }
                    if (initial) {
#pragma unroll
                        for (int j = 0; j < V; ++j) ga[j] += (KIND == 2 ? 0.5 : 1.0) * (double(ro[j]) * dw_dot<T, Q>(dw, lam[j]));
                    }
                }
#pragma unroll
                for (int j = 0; j < V; ++j) {
                    G[r][j] = gin[j] + ga[j];
#pragma unroll
                    for (int i = 0; i < Q; ++i) h[r][i][j] = lam[j][i];
                }
                load_rho(rho_s, Y + r - s - 1, rho[r]);
                __builtin_amdgcn_sched_barrier(0);   // one row after the other: bounds the registers
            };
            static_for<0, R - 2>([&](auto mc) __attribute__((always_inline)) {
                constexpr int r = R - 1 - decltype(mc)::value;
                row(std::integral_constant<int, r>{}, h[r - 2], h[r - 1], h[r], G[r - 1]);
            });
            // the last two rows above, one step back; with them the c^2 and
            // sponge factors of the rows that came from that bundle
            if (q > 0) wait_count(&pub[wp], np);
            T e1[Q][V], e2[Q][V];   // its last row (c_y <= 0) and the one above (c_y < 0)
            double eg[V];
            {
                int k = 0;
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    if (cyv<Q>(i) <= 0) {
                        const ct t = edge[np & 1][wp][k++][lane];
#pragma unroll
                        for (int j = 0; j < V; ++j) e1[i][j] = t[j];
                    }
                    if (cyv<Q>(i) < 0) {
                        const ct t = edge[np & 1][wp][k++][lane];
#pragma unroll
                        for (int j = 0; j < V; ++j) e2[i][j] = t[j];
                    }
                }
                const gt g = gedge[np & 1][wp][lane];
#pragma unroll
                for (int j = 0; j < V; ++j) eg[j] = g[j];
            }
            cn = cb[64];
            if (mspo) fyl = *sb;
            order();
            if (q > 0) set_count(&con[w], np);
            order();
            row(std::integral_constant<int, 1>{}, e1, h[0], h[1], G[0]);
            row(std::integral_constant<int, 0>{}, e2, e1, h[0], eg);
#pragma unroll
            for (int j = 0; j < V; ++j) rv[j] = rvn[j];
        }
        order();
        set_count(&fin[w], it + 1);
        order();
        ring += W * R;
        if (ring >= RING) ring -= RING;
        if (own0) {
            const bool whole = xl + V <= nx;
            static_for<0, R>([&](auto rc) __attribute__((always_inline)) {
                constexpr int r = decltype(rc)::value;
                const int gy = Y + r - ns;
                if (gy >= ya && gy < yb) {
                    T *d = reinterpret_cast<T *>(p->dst) + (int64_t)gy * nx;
                    const GlobalPtr<double> gr = (GlobalPtr<double>)(pa->grad + (int64_t)gy * nx);
#pragma unroll
                    for (int i = 0; i < Q; ++i, d += p->pstride) {
                        if (whole) {
                            ct t;
#pragma unroll
                            for (int j = 0; j < V; ++j) t[j] = h[r][i][j];
                            st_nt(t, at_lane<ct>(d, xl));
                        } else {
#pragma unroll
                            for (int j = 0; j < V - 1; ++j)
                                if (xl + j < nx) st_nt(h[r][i][j], d + xl + j);
                        }
                    }
#pragma unroll
                    for (int j = 0; j < V; ++j)
                        if (xl + j < nx) gr[xl + j] = G[r][j];
                }
            });
        }
    }
}

template <typename T, int Q, int KIND, bool SMALL>
__global__ __launch_bounds__((AdjointShape<T, Q, SMALL>::W * 64))
__attribute__((amdgpu_waves_per_eu(AdjointShape<T, Q, SMALL>::EU, AdjointShape<T, Q, SMALL>::EU)))
void k_flow_adjoint(AdjointFlowParams) {
    using F = AdjointShape<T, Q, SMALL>;
    flow_adjoint_body<T, Q, KIND, F::V, F::R, F::W, F::E>((KernAdjoint)__builtin_amdgcn_kernarg_segment_ptr(), xcd_block());
}

template <typename T, int Q, bool SMALL>
hipError_t flow_adjoint_launch(const AdjointFlowParams &p, hipStream_t s) {
    using F = AdjointShape<T, Q, SMALL>;
    const dim3 grid((unsigned)p.f.nblk), block(F::W * 64);
    switch (step_kind(p.f.coll) % 3) {
    case 0: hipLaunchKernelGGL((k_flow_adjoint<T, Q, 0, SMALL>), grid, block, 0, s, p); break;
    case 1: hipLaunchKernelGGL((k_flow_adjoint<T, Q, 1, SMALL>), grid, block, 0, s, p); break;
    default: hipLaunchKernelGGL((k_flow_adjoint<T, Q, 2, SMALL>), grid, block, 0, s, p);
    }
    return hipGetLastError();
}

template <typename T, int Q, bool SMALL>
FlowInfo flow_adjoint_shape() {
    using F = AdjointShape<T, Q, SMALL>;
    FlowInfo f;
    f.V = F::V;
    f.R = F::R;
    for (int ns = 2; ns <= kFlowSteps; ++ns)
        if (flow_steps_ok(ns, F::R, F::W, F::E)) f.steps = ns;
    return f;
}

template <typename T, typename F>
auto for_shape(bool small, F &&f) {
    if constexpr (sizeof(T) == 4)
        if (small) return f(std::true_type());
    return f(std::false_type());
}

}  // namespace

#define LBW_FLOW_ADJOINT_UNIT(TT, QQ, NAME)                                                                         \
    hipError_t launch_flow_adjoint_##NAME(bool small, const AdjointFlowParams &p, hipStream_t s) {                  \
        return for_shape<TT>(small, [&](auto sc) { return flow_adjoint_launch<TT, QQ, decltype(sc)::value>(p, s); }); \
    }                                                                                                               \
    FlowInfo flow_adjoint_info_##NAME(bool small) {                                                                 \
        return for_shape<TT>(small, [](auto sc) { return flow_adjoint_shape<TT, QQ, decltype(sc)::value>(); });     \
    }

#define LBW_FLOW_ADJOINT_DECL(NAME)                                                                                 \
    hipError_t launch_flow_adjoint_##NAME(bool small, const AdjointFlowParams &p, hipStream_t s);                   \
    FlowInfo flow_adjoint_info_##NAME(bool small);
LBW_FLOW_ADJOINT_DECL(f32_q5)
LBW_FLOW_ADJOINT_DECL(f32_q9)
LBW_FLOW_ADJOINT_DECL(f64_q5)
LBW_FLOW_ADJOINT_DECL(f64_q9)
#undef LBW_FLOW_ADJOINT_DECL

}  // namespace lbw
