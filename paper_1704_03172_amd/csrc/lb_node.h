// lb_node.h -- the per-node arithmetic of the linear LB step shared by every
// step kernel (one step per launch, several steps per launch, the batched
// executor, the refinement interface): lattice tables, storage traits, the
// collision, source, sponge and receiver recording of one node.  Device
// code only; included by the kernel sources (not part of the public
// interface).
#pragma once

#include "lb_internal.h"

#include <hip/hip_fp16.h>

// No automatic a*b+c contraction in this file: where the compiler forms fused
// multiply-adds depends on the surrounding code, so the same per-node
// arithmetic inlined into different kernels (one step per launch, several
// steps per launch, the batched executor) could round differently.  The fused
// multiply-adds of the collision are written out (fmaT) instead.
#pragma clang fp contract(off)

namespace lbw {
namespace {

// ---- lattice tables (velocity order of Appendix A) -----------------------
template <int Q>
__host__ __device__ constexpr int cxv(int i) {
    return Q == 5 ? (i == 1 ? 1 : i == 3 ? -1 : 0)
                  : (i == 1 || i == 5 || i == 8 ? 1 : i == 3 || i == 6 || i == 7 ? -1 : 0);
}
template <int Q>
__host__ __device__ constexpr int cyv(int i) {
    return Q == 5 ? (i == 2 ? 1 : i == 4 ? -1 : 0)
                  : (i == 2 || i == 5 || i == 6 ? 1 : i == 4 || i == 7 || i == 8 ? -1 : 0);
}

// Rows of the moment matrix of Appendix A (non-conserved rows only are
// used: D2Q5 k = 3 (e), 4 (pxx); D2Q9 k = 3 (e), 4 (pxx), 5 (eps),
// 6 (qx), 7 (qy), 8 (pxy)); mrt_apply() has D2Q9's factored.
template <int Q>
__host__ __device__ constexpr int mrow(int k, int i) {
    if (Q == 5) {
        if (k == 3) return i == 0 ? -4 : 1;
        if (k == 4) return i == 1 || i == 3 ? 1 : (i == 2 || i == 4 ? -1 : 0);
        return 0;
    }
    switch (k) {
    case 3: return i == 0 ? -4 : (i <= 4 ? -1 : 2);
    case 4: return i == 1 || i == 3 ? 1 : (i == 2 || i == 4 ? -1 : 0);
    case 5: return i == 0 ? 4 : (i <= 4 ? -2 : 1);
    case 6: return i == 1 ? -2 : i == 3 ? 2 : (i == 5 || i == 8 ? 1 : (i == 6 || i == 7 ? -1 : 0));
    case 7: return i == 2 ? -2 : i == 4 ? 2 : (i == 5 || i == 6 ? 1 : (i == 7 || i == 8 ? -1 : 0));
    case 8: return i == 5 || i == 7 ? 1 : (i == 6 || i == 8 ? -1 : 0);
    default: return 0;
    }
}

// ---- storage traits -------------------------------------------------------
template <typename S> struct Tr;
template <> struct Tr<float> {
    using T = float;
    static constexpr int V = 4;
    typedef float vec __attribute__((ext_vector_type(4), aligned(4)));
};
template <> struct Tr<double> {
    using T = double;
    static constexpr int V = 2;
    typedef double vec __attribute__((ext_vector_type(2), aligned(8)));
};
template <> struct Tr<_Float16> {
    using T = float;
    static constexpr int V = 8;
    typedef _Float16 vec __attribute__((ext_vector_type(8), aligned(2)));
};

// Conversion of a computed value to the storage format.  For FP16 storage
// the value is first materialised in FP32 (the empty asm is a value barrier):
// otherwise the compiler may fold the last multiply and the conversion into
// one mixed-precision FMA (a single rounding) in some kernels and not in
// others, and a state stored by different kernels would differ in its bits.
template <typename S, typename T>
__device__ inline S to_store(T v) {
    if constexpr (sizeof(S) < sizeof(T)) asm volatile("" : "+v"(v));
    return S(v);
}

template <typename T>
__device__ inline T fmaT(T a, T b, T c) {
    if constexpr (sizeof(T) == 8) return __builtin_fma(a, b, c);
    else return __builtin_fmaf(a, b, c);
}

__device__ inline int wrapi(int v, int n) {
    v %= n;
    return v < 0 ? v + n : v;
}

// V consecutive elements starting at x = xs of one row, periodic in x.
template <typename S, int V>
__device__ inline void load_x(const S *__restrict__ row, int xs, int nx, S (&v)[V]) {
    if (V > 1 && xs >= 0 && xs + V <= nx) {
        typedef typename Tr<S>::vec vt;
        vt t = __builtin_nontemporal_load(reinterpret_cast<const vt *>(row + xs));
#pragma unroll
        for (int j = 0; j < V; ++j) v[j] = t[j];
    } else {
#pragma unroll
        for (int j = 0; j < V; ++j) v[j] = row[wrapi(xs + j, nx)];
    }
}

template <typename S, int V>
__device__ inline void store_x(S *__restrict__ row, int x0, int nx, const S (&v)[V]) {
    if (V > 1 && x0 + V <= nx) {
        typedef typename Tr<S>::vec vt;
        vt t;
#pragma unroll
        for (int j = 0; j < V; ++j) t[j] = v[j];
        __builtin_nontemporal_store(t, reinterpret_cast<vt *>(row + x0));
    } else {
#pragma unroll
        for (int j = 0; j < V; ++j)
            if (x0 + j < nx) row[x0 + j] = v[j];
    }
}

// The constants of a Collision in the arithmetic type.
template <typename T> struct CollisionT {
    T omega, srate[9], kax, kdg, kw, ratio;
};

// ---- the per-node update ---------------------------------------------------
// Lattice weights from c^2 (Sec. II C): D2Q5 w_i = c^2/2 for movers,
// w0 = 1 - 2 c^2; D2Q9 w1 = c^2 kw (kw = 1 / (2 + 4r)), w5 = r w1,
// w0 = 1 - 4 w1 - 4 w5.
// (1 - 4 w1 as one fused multiply-add: 4 w1 is exact, so this is the
// rounding of 1 - 4 w1 either way.)
// (C: Collision, or CollisionT<T> with its constants in the arithmetic type.)
template <typename T, int Q, typename C>
__device__ inline void weights(T c2, const C &c, T (&w)[Q]) {
    if (Q == 5) {
        T w1 = T(0.5) * c2;
        w[0] = fmaT(T(-4), w1, T(1));
#pragma unroll
        for (int i = 1; i < Q; ++i) w[i] = w1;
    } else {
        T w1 = c2 * T(c.kw);
        T w5 = w1 * T(c.ratio);
        w[0] = fmaT(T(-4), w5, fmaT(T(-4), w1, T(1)));
#pragma unroll
        for (int i = 1; i < Q; ++i) w[i] = i <= 4 ? w1 : w5;
    }
}

// c . J for the velocity (cx, cy) with components 0, +-1 resolved at compile
// time (no multiplications by 0 or 1).
template <typename T>
__device__ inline T cdot(int cx, int cy, T jx, T jy) {
    const T ax = cx > 0 ? jx : -jx, ay = cy > 0 ? jy : -jy;
    return cx != 0 ? (cy != 0 ? ax + ay : ax) : (cy != 0 ? ay : T(0));
}

// D2Q9: the rest population's equilibrium w0 rho written as rho minus the
// movers' rounded rho-parts, rho - 4 (w1 rho) - 4 (w5 rho), so that the
// equilibrium holds the mass rho up to roundings that change with rho.  With
// w0 rho, the rounding of the per-node constant w0 = 1 - 4 w1 - 4 w5 is a
// fixed per-node mass source proportional to rho, the same every step, and
// the error it leaves in FP32 grows with the run (an FP32 emulation of the
// 256^2 layered workload: 3.7e-5 of rho after 1000 steps of D2Q9 BGK,
// 6.8e-6 with this form and the momentum-exact kax, kdg; MRT 6.4e-6 ->
// 4.1e-6).  The value is the same real number.
// D2Q5 keeps w0 rho (its movers' weight c^2 / 2 is exact).
template <typename T, int Q>
__device__ inline T geq_rest(const T (&w)[Q], T rho) {
    if constexpr (Q == 9) return fmaT(T(-4), w[5] * rho, fmaT(T(-4), w[1] * rho, rho));
    else return w[0] * rho;
}

// acc = C d with C = M^-1 S M (symmetric) through the non-conserved moments
// only, row by row.
template <typename T, int Q, typename C>
__device__ inline void mrt_rows(const T (&d)[Q], const C &c, T (&acc)[Q]) {
    T r[9];
#pragma unroll
    for (int k = 3; k < Q; ++k) {
        T a = T(0);
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            const int m = mrow<Q>(k, i);
            if (m != 0) a += T(m) * d[i];
        }
        r[k] = T(c.srate[k]) * a;
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        T a = T(0);
#pragma unroll
        for (int k = 3; k < Q; ++k) {
            const int m = mrow<Q>(k, i);
            if (m != 0) a += T(m) * r[k];
        }
        acc[i] = a;
    }
}

// The same for D2Q9 through the sums and differences of opposite populations:
// 45 operations instead of 130 (FP64 MRT on 701 x 899: 8.6 us per step before,
// 7.6 after).
template <typename T, typename C>
__device__ inline void mrt_apply(const T (&d)[9], const C &c, T (&acc)[9]) {
    const T s1 = d[1] + d[3], s2 = d[2] + d[4], s5 = d[5] + d[7], s6 = d[6] + d[8];
    const T a1 = d[1] - d[3], a2 = d[2] - d[4], a5 = d[5] - d[7], a6 = d[6] - d[8];
    const T sx = s1 + s2, sd = s5 + s6;
    const T re = T(c.srate[3]) * fmaT(T(2), sd, fmaT(T(-4), d[0], -sx));
    const T rp = T(c.srate[4]) * (s1 - s2);
    const T rs = T(c.srate[5]) * fmaT(T(-2), sx, fmaT(T(4), d[0], sd));
    const T rx = T(c.srate[6]) * fmaT(T(-2), a1, a5 - a6);
    const T ry = T(c.srate[7]) * fmaT(T(-2), a2, a5 + a6);
    const T rxy = T(c.srate[8]) * (s5 - s6);
    // axis movers: -re - 2 rs +- rp -+ 2 rx (or ry); diagonal ones:
    // 2 re + rs +- (rx +- ry) +- rxy
    const T ba = fmaT(T(-2), rs, -re), bd = fmaT(T(2), re, rs);
    const T bx = ba + rp, by = ba - rp, b5 = bd + rxy, b6 = bd - rxy, p = rx + ry, m = rx - ry;
    acc[0] = T(4) * (rs - re);
    acc[1] = fmaT(T(-2), rx, bx);
    acc[2] = fmaT(T(-2), ry, by);
    acc[3] = fmaT(T(2), rx, bx);
    acc[4] = fmaT(T(2), ry, by);
    acc[5] = b5 + p;
    acc[6] = b6 - m;
    acc[7] = b5 - p;
    acc[8] = b6 + m;
}

// Collision of one node: out = g - C (g - g^eq) with the linear equilibrium
// g^eq_i = w_i rho + (w_i / c^2)(c_i . J); BGK C = omega I (KIND 0), MRT
// C = M^-1 S M applied through the non-conserved moments only (KIND 1).
// KIND 2 is BGK at omega = 2 (tau = 1/2, the non-dissipative case), where
// g - 2 (g - g^eq) is 2 g^eq - g: one rounding less and fewer operations.
// D2Q5, kinds 0 to 2: the equilibria of opposite movers differ by their own
// difference (2 w_i / c^2 = 1), so g_i - g^eq_i is e / 2 for both, e = g_i +
// g_-i - c^2 rho, and needs no momentum; tau = 1/2 comes to out_i = c^2 rho -
// g_-i.  12, 16 and 10 operations where the equilibrium written out mover by
// mover (kinds 3 to 5) has 23, 30 and 16, and fewer roundings (4096^2 FP32,
// tau = 1/2: 16.2 us per step before, 14.2 after; its error 2.2e-6 and 2.0e-6).
template <typename T, int Q, int KIND, typename C>
__device__ inline void collide(const T (&g)[Q], T c2, const C &c, T (&out)[Q], T (&w)[Q]) {
    static_assert(KIND < 3 || Q == 5 || KIND == 4, "see step_kind");
    if constexpr (Q == 5 && KIND < 3) {
        weights<T, Q>(c2, c, w);
        const T s1 = g[1] + g[3], s2 = g[2] + g[4], rho = g[0] + (s1 + s2);
        if constexpr (KIND == 2) {
            out[0] = fmaT(fmaT(T(-4), c2, T(2)), rho, -g[0]);
            out[1] = fmaT(c2, rho, -g[3]);
            out[2] = fmaT(c2, rho, -g[4]);
            out[3] = fmaT(c2, rho, -g[1]);
            out[4] = fmaT(c2, rho, -g[2]);
            return;
        }
        const T e1 = fmaT(-c2, rho, s1), e2 = fmaT(-c2, rho, s2), e = e1 + e2;   // g_0 - g^eq_0 = -e
        if constexpr (KIND == 0) {
            const T h = T(-0.5) * T(c.omega);
            out[0] = fmaT(T(c.omega), e, g[0]);
            out[1] = fmaT(h, e1, g[1]);
            out[2] = fmaT(h, e2, g[2]);
            out[3] = fmaT(h, e1, g[3]);
            out[4] = fmaT(h, e2, g[4]);
        } else {   // C through the two non-conserved moments: 5 e and e1 - e2
            const T re = (T(5) * T(c.srate[3])) * e, rp = T(c.srate[4]) * (e1 - e2), a1 = re + rp, a2 = re - rp;
            out[0] = fmaT(T(4), re, g[0]);
            out[1] = g[1] - a1;
            out[2] = g[2] - a2;
            out[3] = g[3] - a1;
            out[4] = g[4] - a2;
        }
        return;
    }
    // moments, each sum started from its first term (0 + x is not x for
    // x = -0, so a 0 start would cost an addition the compiler must keep)
    T rho = g[0], jx = T(0), jy = T(0);
    bool hx = false, hy = false;
#pragma unroll
    for (int i = 1; i < Q; ++i) rho += g[i];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        if (cxv<Q>(i) != 0) {
            const T v = cxv<Q>(i) > 0 ? g[i] : -g[i];
            jx = hx ? jx + v : v;
            hx = true;
        }
        if (cyv<Q>(i) != 0) {
            const T v = cyv<Q>(i) > 0 ? g[i] : -g[i];
            jy = hy ? jy + v : v;
            hy = true;
        }
    }
    weights<T, Q>(c2, c, w);
    if constexpr (KIND % 3 == 2) {
        if constexpr (Q == 5) {
            // D2Q5: 2 w_i = c^2 and 2 (w_i / c^2)(c_i . J) = c_i . J for the
            // movers (both exact), 2 w_0 = 2 - 4 c^2
            out[0] = fmaT(fmaT(T(-4), c2, T(2)), rho, -g[0]);
#pragma unroll
            for (int i = 1; i < Q; ++i) out[i] = fmaT(c2, rho, cdot<T>(cxv<Q>(i), cyv<Q>(i), jx, jy)) - g[i];
        } else {
            out[0] = fmaT(T(2), geq_rest<T, Q>(w, rho), -g[0]);
#pragma unroll
            for (int i = 1; i < Q; ++i) {
                const int cx = cxv<Q>(i), cy = cyv<Q>(i);
                const bool pos = cx > 0 || (cx == 0 && cy > 0);
                const T kj = i <= 4 ? T(c.kax) : T(c.kdg);
                const T kc = kj * cdot<T>(pos ? cx : -cx, pos ? cy : -cy, jx, jy);
                out[i] = fmaT(T(2), fmaT(w[i], rho, pos ? kc : -kc), -g[i]);
            }
        }
        return;
    }
    T d[Q];
    d[0] = g[0] - geq_rest<T, Q>(w, rho);
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        // (w_i / c^2)(c_i . J): opposite velocities share one product
        // (k (-a) is -(k a) exactly), taken for the one whose first nonzero
        // component is positive
        const int cx = cxv<Q>(i), cy = cyv<Q>(i);
        const bool pos = cx > 0 || (cx == 0 && cy > 0);
        const T kj = Q == 5 ? T(0.5) : (i <= 4 ? T(c.kax) : T(c.kdg));
        const T kc = kj * cdot<T>(pos ? cx : -cx, pos ? cy : -cy, jx, jy);
        const T geq = fmaT(w[i], rho, pos ? kc : -kc);
        d[i] = g[i] - geq;
    }
    if (KIND % 3 == 0) {
        const T om = T(c.omega);
#pragma unroll
        for (int i = 0; i < Q; ++i) out[i] = fmaT(-om, d[i], g[i]);
    } else {
        T acc[Q];
        if constexpr (Q == 9 && KIND < 3) mrt_apply<T>(d, c, acc);
        else mrt_rows<T, Q>(d, c, acc);
#pragma unroll
        for (int i = 0; i < Q; ++i) out[i] = g[i] - acc[i];
    }
}

// Sponge factor of a node at distance d (in nodes) from the nearest edge.
template <typename T>
__device__ inline T sponge_at(int d, int L, double smax) {
    if (L <= 0 || d >= L) return T(1);
    T f = T(L - d) / T(L);
    return T(1) - T(smax) * f * f;
}

__device__ inline int edge_dist(int x, int y, int nx, int ny) { return min(min(x, y), min(nx - 1 - x, ny - 1 - y)); }

template <typename T>
__device__ inline T sponge_factor(int x, int y, int nx, int ny, int L, double smax) {
    return sponge_at<T>(edge_dist(x, y, nx, ny), L, smax);
}

template <typename T>
__device__ inline void write_fields(const Receivers &rc, int slot, T rho, T jx, T jy, T c2) {
    T *tr = reinterpret_cast<T *>(rc.traces);
    int f = 0;
    const int64_t plane = (int64_t)rc.nslots * rc.cap;
    const int64_t base = (int64_t)slot * rc.cap + rc.col;
    if (rc.what & 1u) { tr[f * plane + base] = c2 * rho; ++f; }
    if (rc.what & 2u) { tr[f * plane + base] = rho; ++f; }
    if (rc.what & 4u) { tr[f * plane + base] = jx; ++f; }
    if (rc.what & 8u) { tr[f * plane + base] = jy; ++f; }
}

// The params of a launch replayed from a captured graph with its times made
// absolute: the launch holds them relative to the chunk's first time, which
// with the chunk's source amplitudes sits in the chunk table (GraphTab).
// The graph entry kernels run the ordinary bodies on this copy, so the
// kernels of eager launches carry nothing of it.
__device__ inline StepParams graph_params(const StepParams &p) {
    StepParams q = p;
    const GraphTab *g = p.gtab;
    q.s_n = g->s[p.goff];
    q.rec.col += g->t0;
    q.gtab = nullptr;
    return q;
}

// Receivers at node x of a row whose CSR entries are [rb, re): record the
// fields of the pre-collision state g.
template <typename T, int Q>
__device__ inline void record_node(const Receivers &rc, int rb, int re, int x, const T (&g)[Q], T c2) {
    T rho = T(0), jx = T(0), jy = T(0);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        rho += g[i];
        jx += T(cxv<Q>(i)) * g[i];
        jy += T(cyv<Q>(i)) * g[i];
    }
    int lo = rb, hi = re;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (rc.xs[mid] < x) lo = mid + 1; else hi = mid;
    }
    for (; lo < re && rc.xs[lo] == x; ++lo)
        write_fields<T>(rc, rc.slot[lo], rho, jx, jy, c2);
}

// The point source w_i S added to a post-collision state (Sec. II D).
template <typename T, int Q>
__device__ inline void add_source(const T (&w)[Q], double s_n, T (&gs)[Q]) {
    const T sn = T(s_n);
#pragma unroll
    for (int i = 0; i < Q; ++i) gs[i] += w[i] * sn;
}

// The sponge factor of a node at distance d < L from the nearest edge
// applied to its post-collision state.
template <typename T, int Q>
__device__ inline void apply_sponge(int d, int L, double smax, T (&gs)[Q]) {
    const T sf = sponge_at<T>(d, L, smax);
#pragma unroll
    for (int i = 0; i < Q; ++i) gs[i] = gs[i] * sf;
}

// Post-collision state of node (x, y): collision, source w_i S at the source
// node, sponge (dedge: the node's distance to the nearest grid edge).
// maybe_sponge: wave-uniform; false when no node of the wave's current row
// lies in the sponge (dedge is then not looked at).
template <typename T, int Q, int KIND>
__device__ inline void post_node(const StepParams &p, const T (&g)[Q], T c2, int x, int y, int dedge, double s_n,
                                 T (&out)[Q], bool maybe_sponge = true) {
    T gs[Q], w[Q];
    collide<T, Q, KIND>(g, c2, p.coll, gs, w);
    if (y == p.src_y) {   // uniform over a row: only the source row tests x
        // (the empty asm keeps this a branch: otherwise the compiler turns
        // the injection into selects evaluated at every node)
        asm volatile("");
        if (x == p.src_x) add_source<T, Q>(w, s_n, gs);
    }
    // sponge: outside it the factor is 1 and g * 1 = g, so only nodes inside
    // multiply (a branch, kept by the empty asm, rather than selects at
    // every node)
    if (maybe_sponge && dedge < p.sponge_width) {
        asm volatile("");
        apply_sponge<T, Q>(dedge, p.sponge_width, p.sponge_smax, gs);
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) out[i] = gs[i];
}

// The backward step of a node at time n (the discrete adjoint; see k_adjoint),
// shared by the one-step and the many-step kernel, so that both give the same
// bits: mu = lambda(n+1) pulled back to the node, m = (1 - sigma) mu, nu = C^T m
// (C is symmetric), then lambda(n) without the residuals.  Kinds as in
// collide(); the form of kind 2 has the values of kind 0 (products by 2 are
// exact).
template <typename T, int Q, int KIND, typename C>
__device__ inline void adjoint_relax(const T (&m)[Q], const C &coll, T (&nu)[Q]) {
    if constexpr (KIND != 1) {
#pragma unroll
        for (int i = 0; i < Q; ++i) nu[i] = KIND == 2 ? T(2) * m[i] : T(coll.omega) * m[i];
    } else {
        mrt_rows<T, Q>(m, coll, nu);
    }
}

template <typename T, int Q, int KIND, typename C>
__device__ inline void adjoint_lambda(const T (&m)[Q], const T (&nu)[Q], T c2, const C &coll, T (&lam)[Q]) {
    T s0, sx = T(0), sy = T(0);
    if constexpr (Q == 5 && KIND == 2) {
        s0 = fmaT(T(-4), c2, T(2)) * m[0];
#pragma unroll
        for (int i = 1; i < Q; ++i) s0 += c2 * m[i];
        sx = m[1] - m[3];
        sy = m[2] - m[4];
        lam[0] = s0 - m[0];
#pragma unroll
        for (int i = 1; i < Q; ++i) lam[i] = (s0 - m[i]) + cdot<T>(cxv<Q>(i), cyv<Q>(i), sx, sy);
        return;
    }
    T w[Q];
    weights<T, Q>(c2, coll, w);
    s0 = w[0] * nu[0];
    bool hx = false, hy = false;
#pragma unroll
    for (int i = 1; i < Q; ++i) {
        s0 += w[i] * nu[i];
        const T kn = (Q == 5 ? T(0.5) : (i <= 4 ? T(coll.kax) : T(coll.kdg))) * nu[i];
        if (cxv<Q>(i) != 0) {
            const T v = cxv<Q>(i) > 0 ? kn : -kn;
            sx = hx ? sx + v : v;
            hx = true;
        }
        if (cyv<Q>(i) != 0) {
            const T v = cyv<Q>(i) > 0 ? kn : -kn;
            sy = hy ? sy + v : v;
            hy = true;
        }
    }
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        T l = m[i] - nu[i] + s0;
        if (cxv<Q>(i) != 0) l += cxv<Q>(i) > 0 ? sx : -sx;
        if (cyv<Q>(i) != 0) l += cyv<Q>(i) > 0 ? sy : -sy;
        lam[i] = l;
    }
}

// dw . v in FP64, the derivatives dw of the weights by c^2 being alike for the
// axis and for the diagonal movers.
template <typename T, int Q, typename P>
__device__ inline double dw_dot(const P &dw, const T (&v)[Q]) {
    double d = fmaT(double(dw[1]), (double(v[1]) + double(v[3])) + (double(v[2]) + double(v[4])), double(dw[0]) * double(v[0]));
    if constexpr (Q == 9)
        d = fmaT(double(dw[5]), (double(v[5]) + double(v[7])) + (double(v[6]) + double(v[8])), d);
    return d;
}

// One node of the one-step kernel: dedge is the node's distance to the nearest
// edge, [rb, re) its row's receiver entries (empty: none), col = n for the
// residuals, s_n = S(n), initial: n = 0.  Writes lambda(n) and returns the
// node's gradient term of time n (FP64).
template <typename T, int Q, int KIND>
__device__ inline double adjoint_node(const AdjointParams &p, const T (&mu)[Q], T c2, T rho, int x, int y, int dedge,
                                      int rb, int re, int64_t col, double s_n, bool initial, T (&lam)[Q]) {
    const T *res = reinterpret_cast<const T *>(p.rec.traces);
    T m[Q], nu[Q];
    // (1 - sigma) P^T lambda: outside the sponge the factor is 1 and
    // mu * 1 = mu, so only nodes inside it multiply
    if (dedge < p.sponge_width) {
        asm volatile("");
        const T sf = sponge_at<T>(dedge, p.sponge_width, p.sponge_smax);
#pragma unroll
        for (int i = 0; i < Q; ++i) m[i] = mu[i] * sf;
    } else {
#pragma unroll
        for (int i = 0; i < Q; ++i) m[i] = mu[i];
    }
    adjoint_relax<T, Q, KIND>(m, p.coll, nu);
    double gacc = double(rho) * dw_dot<T, Q>(p.dw, nu);
    if (y == p.src_y) {   // uniform over a row: only the source row tests x
        asm volatile("");
        if (x == p.src_x) gacc += s_n * dw_dot<T, Q>(p.dw, m);
    }
    adjoint_lambda<T, Q, KIND>(m, nu, c2, p.coll, lam);
    if (rb < re) {
        int lo = rb, hi = re;
        while (lo < hi) {
            int mid = (lo + hi) >> 1;
            if (p.rec.xs[mid] < x) lo = mid + 1; else hi = mid;
        }
        for (; lo < re && p.rec.xs[lo] == x; ++lo) {
            const T rr = res[(int64_t)p.rec.slot[lo] * p.rec.cap + col];
#pragma unroll
            for (int i = 0; i < Q; ++i) lam[i] += c2 * rr;
            gacc += double(rr) * double(rho);
        }
    }
    if (initial) gacc += double(rho) * dw_dot<T, Q>(p.dw, lam);
    return gacc;
}

}  // namespace
}  // namespace lbw
