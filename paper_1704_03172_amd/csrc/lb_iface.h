// lb_iface.h -- a node's passage through the refinement interface, shared by
// the one-step kernels (lb_kernels.hip) and the flowing kernel (lb_flow.h).
// Device code only; not part of the public interface.
#pragma once

#include "lb_internal.h"
#include "lb_node.h"

namespace lbw {
namespace {

// R_f(g) = g^eq(rho(g), J(g)) + f (g - g^eq) with the weights of the
// receiving node's c^2 (eq. coarse-fine dist connect), then the collision
// (and sponge) of the receiving grid; written as the post-collision state at
// node (x, y) of dst.
template <typename S, int KIND, typename P>   // P: InterfaceParams, in any address space
__device__ inline void rescale_collide(P &p, const typename Tr<S>::T (&gh)[5], int x, int y, typename Tr<S>::T c2, typename Tr<S>::T (&out)[5]) {
    using T = typename Tr<S>::T;
    T rho = T(0), jx = T(0), jy = T(0);
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        rho += gh[i];
        jx += T(cxv<5>(i)) * gh[i];
        jy += T(cyv<5>(i)) * gh[i];
    }
    T w[5];
    weights<T, 5>(c2, p.coll, w);
    T gr[5];
    const T f = T(p.f);
#pragma unroll
    for (int i = 0; i < 5; ++i) {
        T geq = w[i] * rho + (i == 0 ? T(0) : T(0.5) * (T(cxv<5>(i)) * jx + T(cyv<5>(i)) * jy));
        gr[i] = geq + f * (gh[i] - geq);
    }
    collide<T, 5, KIND>(gr, c2, p.coll, out, w);
    const T sf = sponge_factor<T>(x, y, p.dst_nx, p.dst_ny, p.sponge_width, p.sponge_smax);
#pragma unroll
    for (int i = 0; i < 5; ++i) out[i] *= sf;
}

template <typename S, int KIND>
__device__ inline void rescale_collide(const InterfaceParams &p, const typename Tr<S>::T (&gh)[5], int x, int y,
                                       typename Tr<S>::T (&out)[5]) {
    using T = typename Tr<S>::T;
    rescale_collide<S, KIND, const InterfaceParams>(p, gh, x, y, reinterpret_cast<const T *>(p.dst_c2)[(int64_t)y * p.dst_nx + x], out);
}

template <typename S, int KIND>
__device__ inline void rescale_collide_store_impl(const InterfaceParams &p, typename Tr<S>::T (&gh)[5], int x, int y) {
    using T = typename Tr<S>::T;
    const int64_t k = (int64_t)y * p.dst_nx + x;
    if (p.field) {   // R_f keeps rho and J: the node's fields are those of gh
        T rho = T(0), jx = T(0), jy = T(0);
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            rho += gh[i];
            jx += T(cxv<5>(i)) * gh[i];
            jy += T(cyv<5>(i)) * gh[i];
        }
        const T c2 = reinterpret_cast<const T *>(p.dst_c2)[k];
        T v = p.field == 1u ? c2 * rho : p.field == 2u ? rho : p.field == 4u ? jx : jy;
        reinterpret_cast<T *>(p.field_out)[k] = v;
        return;
    }
    T out[5];
    rescale_collide<S, KIND>(p, gh, x, y, out);
    S *dst = reinterpret_cast<S *>(p.dst);
#pragma unroll
    for (int i = 0; i < 5; ++i) dst[i * p.dst_pstride + k] = to_store<S>(out[i]);
}

}  // namespace
}  // namespace lbw
