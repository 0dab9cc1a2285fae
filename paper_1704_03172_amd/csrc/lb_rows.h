// lb_rows.h -- row-wise building blocks of the kernels that hold several rows
// of a strip of columns in registers (one wavefront per strip; the lane's
// columns are consecutive): row loads, lane shifts along x, the pull of a row
// from its neighbours, block renumbering over the XCDs and compile-time loops.
// Device code only; not part of the public interface.
#pragma once

#include "lb_internal.h"
#include "lb_node.h"

#include <type_traits>
#include <utility>

namespace lbw {
namespace {

template <int V, typename S> struct LaneVec { typedef S type __attribute__((ext_vector_type(V), aligned(sizeof(S)))); };

// The populations and c^2 live in global memory.  The walks' accesses say
// so: a batched launch reads the arrays' addresses from memory as generic
// pointers, whose accesses would otherwise take the flat path.
template <typename U>
using GlobalPtr = __attribute__((address_space(1))) U *;

// Load with the ordinary cache policy (keep) or nontemporal.
template <typename U>
__device__ inline U ld_hint(const U *p, bool keep) {
    const GlobalPtr<const U> g = (GlobalPtr<const U>)p;
    return keep ? *g : __builtin_nontemporal_load(g);
}

// Nontemporal store to global memory.
template <typename U>
__device__ inline void st_nt(U v, U *p) {
    __builtin_nontemporal_store(v, (GlobalPtr<U>)p);
}

// Element x of a row as a wave-uniform row pointer plus an unsigned 32-bit
// byte offset per lane, so that the access takes the scalar-base form
// (no per-lane 64-bit address arithmetic).  x >= 0 and x * sizeof(U) < 2^32.
template <typename U, typename E>
__device__ inline U *at_lane(E *row, int x) {
    return reinterpret_cast<U *>(reinterpret_cast<
        std::conditional_t<std::is_const_v<E>, const char, char> *>(row) + (uint32_t)x * (uint32_t)sizeof(E));
}

// One row (all populations) of the lane's V columns, converted to T.  VEC:
// one vector access at the lane's wrapped first column xv (the lane's
// columns are contiguous after the wrap when nx is a multiple of V);
// otherwise element accesses at the wrapped columns xw.  SEL > 0 / < 0:
// only the populations that move toward +y / -y (c_y = +1 / -1).
template <bool VEC, int SEL, bool KEEP, typename S, typename T, int Q, int V>
__device__ inline void load_row2(const S *__restrict__ base, int64_t pstride, int64_t rowoff, int xv,
                                 const int (&xw)[V], T (&out)[Q][V]) {
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        if ((SEL > 0 && cyv<Q>(i) <= 0) || (SEL < 0 && cyv<Q>(i) >= 0)) {   // not needed from this row
#pragma unroll
            for (int j = 0; j < V; ++j) out[i][j] = T(0);
            continue;
        }
        const S *r = base + i * pstride + rowoff;
        if constexpr (VEC && V > 1) {
            typedef typename LaneVec<V, S>::type vt;
            vt t = ld_hint(at_lane<const vt>(r, xv), KEEP);
#pragma unroll
            for (int j = 0; j < V; ++j) out[i][j] = T(t[j]);
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j) out[i][j] = T(ld_hint(r + xw[j], KEEP));
        }
    }
}

template <bool VEC, bool KEEP, typename T, int V>
__device__ inline void load_c2row(const T *__restrict__ c2, int64_t rowoff, int xv, const int (&xw)[V], T (&out)[V]) {
    if constexpr (VEC && V > 1) {
        typedef typename LaneVec<V, T>::type vt;
        vt t = ld_hint(at_lane<const vt>(c2 + rowoff, xv), KEEP);
#pragma unroll
        for (int j = 0; j < V; ++j) out[j] = t[j];
    } else {
#pragma unroll
        for (int j = 0; j < V; ++j) out[j] = ld_hint(c2 + rowoff + xw[j], KEEP);
    }
}

// Whole-wave lane shifts by one lane (DPP wave_shr:1 / wave_shl:1, GFX9
// encodings 0x138 / 0x130): from_lower(v) in lane l is v of lane l - 1,
// from_upper(v) is v of lane l + 1 (0 in the end lanes, which are halo
// lanes; with the bound control the shift is one instruction, which the
// compiler may fold into the first use).
template <int CTRL>
__device__ inline uint32_t dpp_u32(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}
template <int CTRL, typename T>
__device__ inline T dpp_shift(T v) {
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, dpp_u32<CTRL>(__builtin_bit_cast(uint32_t, v)));
    } else {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = dpp_u32<CTRL>((uint32_t)u), hi = dpp_u32<CTRL>((uint32_t)(u >> 32));
        return __builtin_bit_cast(T, ((uint64_t)hi << 32) | lo);
    }
}
template <typename T> __device__ inline T from_lower(T v) { return dpp_shift<0x138>(v); }
template <typename T> __device__ inline T from_upper(T v) { return dpp_shift<0x130>(v); }

// Sum over the lanes, in lane 63: DPP row rotations by 8, 4, 2, 1 (every lane
// of a row of 16 then holds that row's sum), then row_bcast:15 into rows 1 and
// 3 and row_bcast:31 into rows 2 and 3.
template <int CTRL, int ROWS>
__device__ inline double dpp_add(double a) {
    const uint64_t u = __builtin_bit_cast(uint64_t, a);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)u, CTRL, ROWS, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(u >> 32), CTRL, ROWS, 0xF, false);
    return a + __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ inline double wave_total(double a) {
    a = dpp_add<0x128, 0xF>(a);
    a = dpp_add<0x124, 0xF>(a);
    a = dpp_add<0x122, 0xF>(a);
    a = dpp_add<0x121, 0xF>(a);
    a = dpp_add<0x142, 0xA>(a);
    return dpp_add<0x143, 0xC>(a);
}

// Pulled (pre-collision) state of one row from the rows above (U, y - 1),
// at (C) and below (D, y + 1) it: g_i(x) = h_i(x - c_i).
template <typename T, int Q, int V>
__device__ inline void pull_row2(const T (&U)[Q][V], const T (&C)[Q][V], const T (&D)[Q][V], T (&g)[Q][V]) {
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        T r[V];
#pragma unroll
        for (int j = 0; j < V; ++j) r[j] = cyv<Q>(i) > 0 ? U[i][j] : cyv<Q>(i) < 0 ? D[i][j] : C[i][j];
        if (cxv<Q>(i) > 0) {          // from x - 1
            const T l = from_lower(r[V - 1]);
#pragma unroll
            for (int j = V - 1; j > 0; --j) g[i][j] = r[j - 1];
            g[i][0] = l;
        } else if (cxv<Q>(i) < 0) {   // from x + 1
            const T rr = from_upper(r[0]);
#pragma unroll
            for (int j = 0; j < V - 1; ++j) g[i][j] = r[j + 1];
            g[i][V - 1] = rr;
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j) g[i][j] = r[j];
        }
    }
}

// mu_i(x) = lambda_i(n+1)(x + c_i): the transpose of the pull, from the row
// below for c_y = +1 (D), above for c_y = -1 (U), and the lane to the right
// (x + 1) or left (x - 1) along x.
template <typename T, int Q, int V>
__device__ inline void pull_back_row(const T (&U)[Q][V], const T (&C)[Q][V], const T (&D)[Q][V], T (&g)[Q][V]) {
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        T r[V];
#pragma unroll
        for (int j = 0; j < V; ++j) r[j] = cyv<Q>(i) > 0 ? D[i][j] : cyv<Q>(i) < 0 ? U[i][j] : C[i][j];
        if (cxv<Q>(i) > 0) {          // from x + 1
            const T rr = from_upper(r[0]);
#pragma unroll
            for (int j = 0; j < V - 1; ++j) g[i][j] = r[j + 1];
            g[i][V - 1] = rr;
        } else if (cxv<Q>(i) < 0) {   // from x - 1
            const T l = from_lower(r[V - 1]);
#pragma unroll
            for (int j = V - 1; j > 0; --j) g[i][j] = r[j - 1];
            g[i][0] = l;
        } else {
#pragma unroll
            for (int j = 0; j < V; ++j) g[i][j] = r[j];
        }
    }
}

// Blocks are dealt to the 8 XCDs round-robin (block b on XCD b mod 8);
// renumbered, each XCD takes a contiguous range of strips and segments, whose
// shared halo rows then meet in that XCD's L2.
__device__ inline int xcd_block() {
    const int nb = gridDim.x, q8 = nb / 8, r8 = nb % 8, b = blockIdx.x, x8 = b % 8;
    return x8 * q8 + min(x8, r8) + b / 8;
}

// f(integral_constant<int, i>) for i = B .. E-1, unrolled at compile time (a
// loop this large is beyond the unroller's size limit, and runtime row
// indices would put the row arrays in scratch memory).
template <int B, typename F, int... I>
__device__ inline void static_for_impl(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, B + I>{}), ...);
}
template <int B, int E, typename F>
__device__ inline void static_for(F &&f) {
    static_for_impl<B>(f, std::make_integer_sequence<int, E - B>{});
}

}  // namespace
}  // namespace lbw
