// Staged transforms (staged.h) of a tile of columns, one element of all its
// columns `stride` bytes from the next: the y and z passes.
#pragma once

#include "staged.h"

namespace kw {

struct ColPlan {
    StageAxis ax;            // at least two stages (the first of radix 1 for short lengths)
    int S0;                  // n / R0
    int ltb;                 // log2 of the tile's columns
};

struct ColTile {
    float2 *sh;              // [position][tb]
    const float2 *tws;       // twiddles of length n
    int n, tb, ltb;
    uint32_t stride;         // bytes between elements of a column (n stride / R0 below 4 GiB)
};

// first forward stage: global points j + r S0 -> LDS run of j
template <RadixSet RS>
__device__ __forceinline__ void col_load(const ColPlan &a, const ColTile &T, const float2 *src,
                                        const float2 *add0, const float2 *add1, int cols, float2 *sh) {
    const int S0 = a.S0;
    with_radix<RS | radix_bit(1)>(a.ax.r[0], [&](auto RC) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        const int nt = S0 << T.ltb;
        for (int i = threadIdx.x; i < nt; i += blockDim.x) {
            const int j = i >> T.ltb, c = i & (T.tb - 1);
            int hi = j;
            if (a.ax.np == 3) {
                const int q1 = a.ax.d2.div(j);
                hi = q1 + a.ax.r[1] * (j - q1 * a.ax.r[2]);
            }
            float2 v[R];
            const uint32_t lane = (uint32_t)j * T.stride + (uint32_t)c * 8u;
            const size_t step = (size_t)S0 * T.stride / 8;
            if (c < cols) {
#pragma unroll
                for (int r = 0; r < R; ++r) v[r] = ld_at(src + r * step, lane);
                if (add0) {                                  // block-uniform
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        v[r] = c_add(v[r], ld_at(add0 + r * step, lane));
                    __builtin_amdgcn_sched_barrier(0);       // (two arrays in flight, not three)
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        v[r] = c_add(v[r], ld_at(add1 + r * step, lane));
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) v[r] = make_float2(0.0f, 0.0f);
            }
            Dft<R, false>::template run<1, 0>(v);
            twiddle<R, false>(v, T.tws, j);
            float2 *const e = sh + ((hi * R) << T.ltb) + c;
#pragma unroll
            for (int d = 0; d < R; ++d) e[d << T.ltb] = v[d];
        }
    });
}

// first inverse stage: LDS run -> global points
template <RadixSet RS>
__device__ __forceinline__ void col_store(const ColPlan &a, const ColTile &T, float2 *dst, int cols,
                                         const float2 *sh) {
    const int S0 = a.S0;
    with_radix<RS | radix_bit(1)>(a.ax.r[0], [&](auto RC) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        const int nt = S0 << T.ltb;
        for (int i = threadIdx.x; i < nt; i += blockDim.x) {
            const int j = i >> T.ltb, c = i & (T.tb - 1);
            int hi = j;
            if (a.ax.np == 3) {
                const int q1 = a.ax.d2.div(j);
                hi = q1 + a.ax.r[1] * (j - q1 * a.ax.r[2]);
            }
            float2 v[R];
            const float2 *const e = sh + ((hi * R) << T.ltb) + c;
#pragma unroll
            for (int d = 0; d < R; ++d) v[d] = e[d << T.ltb];
            twiddle<R, true>(v, T.tws, j);
            Dft<R, true>::template run<1, 0>(v);
            const uint32_t lane = (uint32_t)j * T.stride + (uint32_t)c * 8u;
            const size_t step = (size_t)S0 * T.stride / 8;
            if (c < cols) {
#pragma unroll
                for (int r = 0; r < R; ++r) st_at(dst + r * step, lane, v[r]);
            }
        }
    });
}

// middle stage of a three-stage length
template <RadixSet RS, bool INV>
__device__ __forceinline__ void col_middle(const ColPlan &a, const ColTile &T, float2 *sh) {
    const int w = a.ax.w[1];
    with_radix<RS>(a.ax.r[1], [&](auto RC) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        const int nt = (T.n / R) << T.ltb;
        for (int i = threadIdx.x; i < nt; i += blockDim.x) {
            const int t = i >> T.ltb, c = i & (T.tb - 1);
            const int hi = a.ax.dw1.div(t), lo = t - hi * w;
            float2 *const e = sh + ((lo + w * R * hi) << T.ltb) + c;
            const int step = w << T.ltb;
            float2 v[R];
#pragma unroll
            for (int d = 0; d < R; ++d) v[d] = e[d * step];
            if (INV) twiddle<R, true>(v, T.tws, w * hi);
            Dft<R, INV>::template run<1, 0>(v);
            if (!INV) twiddle<R, false>(v, T.tws, w * hi);
#pragma unroll
            for (int d = 0; d < R; ++d) e[d * step] = v[d];
        }
    });
}

// last inverse stage read from global memory (the first one of an inverse
// transform to run): rows b + w q -> LDS.  join0: column 0 holds the unpacked
// spectrum of the y pass (see col0_type) and is repacked
template <RadixSet RS>
__device__ __forceinline__ void col_load_last(const ColPlan &a, const ColTile &T, const float2 *src,
                                              int cols, float2 *sh, bool join0) {
    const int w = a.ax.wl;
    with_radix<RS>(a.ax.rl, [&](auto RC) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        const int nt = w << T.ltb, step = w << T.ltb;
        for (int i = threadIdx.x; i < nt; i += blockDim.x) {
            const int b = i >> T.ltb, c = i & (T.tb - 1);
            const uint32_t lane = (uint32_t)b * T.stride + (uint32_t)c * 8u;
            const size_t gstep = (size_t)w * T.stride / 8;
            float2 v[R];
            if (c < cols) {
#pragma unroll
                for (int q = 0; q < R; ++q) v[q] = ld_at(src + q * gstep, lane);
                if (join0 && c == 0) {
                    // (every load before the first use, each row's two in one go)
                    float2 A[R], B[R];
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const Col0Rows o = col0_rows(b + w * q, T.n);
                        A[q] = ld_at(src, (uint32_t)o.a * T.stride);
                        B[q] = ld_at(src, (uint32_t)o.b * T.stride);
                    }
#pragma unroll
                    for (int q = 0; q < R; ++q) v[q] = col0_join(col0_rows(b + w * q, T.n), A[q], B[q]);
                }
            } else {
#pragma unroll
                for (int q = 0; q < R; ++q) v[q] = make_float2(0.0f, 0.0f);
            }
            Dft<R, true>::template run<1, 0>(v);
            float2 *const e = sh + (b << T.ltb) + c;
#pragma unroll
            for (int q = 0; q < R; ++q) e[q * step] = v[q];
        }
    });
}

// last forward stage written to global memory; column 0 stays in LDS where
// keep0 is set
template <RadixSet RS>
__device__ __forceinline__ void col_store_last(const ColPlan &a, const ColTile &T, float2 *dst,
                                               int cols, float2 *sh, bool keep0) {
    const int w = a.ax.wl;
    with_radix<RS>(a.ax.rl, [&](auto RC) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        const int nt = w << T.ltb, step = w << T.ltb;
        for (int i = threadIdx.x; i < nt; i += blockDim.x) {
            const int b = i >> T.ltb, c = i & (T.tb - 1);
            float2 *const e = sh + (b << T.ltb) + c;
            float2 v[R];
#pragma unroll
            for (int q = 0; q < R; ++q) v[q] = e[q * step];
            Dft<R, false>::template run<1, 0>(v);
            const uint32_t lane = (uint32_t)b * T.stride + (uint32_t)c * 8u;
            const size_t gstep = (size_t)w * T.stride / 8;
            if (keep0 && c == 0) {
#pragma unroll
                for (int q = 0; q < R; ++q) e[q * step] = v[q];
            } else if (c < cols) {
#pragma unroll
                for (int q = 0; q < R; ++q) st_at(dst + q * gstep, lane, v[q]);
            }
        }
    });
}

}  // namespace kw
