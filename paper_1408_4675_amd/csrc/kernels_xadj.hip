// The x passes of a reverse step (the updates of kernels_adj.hip) on the staged
// transforms of xstaged_impl.h: the velocity pass on z planes with the y transforms
// around it or on rows, as in the forward step, and the other three on rows (which
// of them: LaunchCfg::xs_adj).
//
// What bounds them is what bounds the forward passes, and the density pass the loads of
// its three components one after the other (twelve wavefronts a CU; registers: 72 bytes
// a lane go to scratch with absorption, 20 in the equation of state).  us a
// launch, the engines of kernels_adj.hip and these, 250 x 135 x 90: density 357 -> 143
// (19 fields, 1.6 TB/s), equation of state 155 -> 41 (3.2 TB/s), sum 112 -> 21, velocity
// with its y passes 245 -> 90; 128^3 velocity with its y passes 52 -> 36.
#include "xstaged_impl.h"

namespace kw {

namespace {

// vel: u = ub + T, T <- -q dt/rho0 u, ub <- q^2 u; blockIdx.y: the component
KW_XS_TEMPLATE>
__global__ void KW_XS_BOUNDS(1024, 4) kw_adjx_vel_s(XSArgs a, AdjDev ad) {
    KW_XS_BEGIN(pml_sy, pml_sz)
    const int xi = blockIdx.y;
    to_points<RSY, RSM, RSP, PLANES, 1>(a, P, [&](int) __attribute__((always_inline)) { return pick3(x.Sin, xi) + soff; });
    float *const ub = pick3(ad.ub, xi);
    const Coef dtr = xi == 0 ? x.m.dtr[0] : xi == 1 ? x.m.dtr[1] : x.m.dtr[2];
    const float *const q_rows = xi == 1 ? P.qy : P.qz;
    x_middle<RSM>(a, P, roff, [&](auto RC, const XTask &T, int off, int j) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        float2 u[R], d[R], v[R];
        ld_run<R>(ub, T, u);
        ld_run<R>(dtr, T, d);
        run_inverse<R>(P, P.sh + off, j, v);
        const float q1 = q_rows[T.y];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float2 q = xi == 0 ? *reinterpret_cast<const float2 *>(x.t.pml_sx + T.x + 2 * r * T.S0)
                                     : make_float2(q1, q1);
            const float2 w = c_add(u[r], v[r]);
            u[r] = make_float2(q.x * q.x * w.x, q.y * q.y * w.y);
            v[r] = make_float2(-q.x * d[r].x * w.x, -q.y * d[r].y * w.y);
        }
        st_run<R>(ub, T, u);
        run_forward<R>(P, P.sh + off, j, v);
    });
    to_spectra<RSY, RSM, RSP, PLANES, true, 1>(a, P, 1, [&](int) __attribute__((always_inline)) { return pick3(x.Sout, xi) + soff; });
}

// sum: pb = T0 + T1 + T2
KW_XS_TEMPLATE>
__global__ void KW_XS_BOUNDS(512, 4) kw_adjx_sum_s(XSArgs a, AdjDev ad) {
    KW_XS_BEGIN(pml_y, pml_z)
    to_points<RSY, RSM, RSP, PLANES, 3>(a, P, [&](int g) __attribute__((always_inline)) { return pick3(x.Sin, g) + soff; });
    x_middle<RSM>(a, P, roff, [&](auto RC, const XTask &T, int off, int j) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        float2 acc[R];
        run_inverse<R>(P, P.sh + off, j, acc);
#pragma unroll 1
        for (int g = 1; g < 3; ++g) {
            float2 v[R];
            run_inverse<R>(P, P.set(g) + off, j, v);
#pragma unroll
            for (int r = 0; r < R; ++r) acc[r] = c_add(acc[r], v[r]);
        }
        st_run<R>(ad.pb, T, acc);
    });
}

// pbar = pb + w p' (p' from its spectrum in set 0 when loss) and c = c0^2 + 2 nl rho
template <int R>
__device__ __forceinline__ void pbar_run(const XSArgs &a, const AdjDev &ad, const Rows &P, int loss, const XTask &T,
                                         int off, int j, float2 (&pbar)[R], float2 (&c)[R]) {
    const Medium &m = a.x.m;
    ld_run<R>(ad.pb, T, pbar);
    if (loss) {
        float2 v[R], w[R];
        ld_run<R>(ad.w, T, w);
        run_inverse<R>(P, P.sh + off, j, v);
        const float inx = 1.0f / (float)a.x.g.nx;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            pbar[r].x += w[r].x * (v[r].x * inx);
            pbar[r].y += w[r].y * (v[r].y * inx);
        }
    }
    ld_run<R>(m.c0sq, T, c);
    if (m.nonlinear) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const XPos i = T.at(r);
            const float2 nl = coef2_at(m.nl, i);
            const float2 r0 = ld2(ad.rho[0], i), r1 = ld2(ad.rho[1], i), r2 = ld2(ad.rho[2], i);
            c[r].x += 2.0f * nl.x * (r0.x + r1.x + r2.x);
            c[r].y += 2.0f * nl.y * (r0.y + r1.y + r2.y);
        }
    }
}

// eos: rbt = c pbar stored, ta pbar and tb pbar transformed
KW_XS_TEMPLATE>
__global__ void KW_XS_BOUNDS(512, 4) kw_adjx_eos_s(XSArgs a, AdjDev ad, const float2 *p_spec, int loss) {
    KW_XS_BEGIN(pml_y, pml_z)
    if (loss) to_points<RSY, RSM, RSP, PLANES, 1>(a, P, [&](int) __attribute__((always_inline)) { return p_spec + soff; });
    else __syncthreads();
    x_middle<RSM>(a, P, roff, [&](auto RC, const XTask &T, int off, int j) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        float2 pbar[R], c[R], t[R];
        pbar_run<R>(a, ad, P, loss, T, off, j, pbar, c);
#pragma unroll
        for (int r = 0; r < R; ++r) c[r] = make_float2(c[r].x * pbar[r].x, c[r].y * pbar[r].y);
        st_run<R>(ad.rbt, T, c);
        ld_run<R>(x.m.ta, T, c);
        ld_run<R>(x.m.tb, T, t);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            c[r] = make_float2(c[r].x * pbar[r].x, c[r].y * pbar[r].y);
            t[r] = make_float2(t[r].x * pbar[r].x, t[r].y * pbar[r].y);
        }
        run_forward<R>(P, P.sh + off, j, c);
        run_forward<R>(P, P.set(1) + off, j, t);
    });
    to_spectra<RSY, RSM, RSP, PLANES, false, 2>(a, P, 2, [&](int s) __attribute__((always_inline)) { return (s ? x.Sout[1] : x.Sout[0]) + soff; });
}

// The source points among x = xp, xp + 1 of a row: R (the old rb and base) stored for
// the points, their terms 2 dt R src / den (nonlinear) returned
__device__ __forceinline__ float2 source_terms(const XArgs &x, const AdjDev &ad, const float *rb, const float *dfw,
                                               XPos i, float2 base, int row, int xp, int g) {
    const SourceDev &src = x.src;
    const float dt = x.g.dt;
    const float2 Rv = c_add(ld2(rb, i), base), d = x.m.nonlinear ? ld2(dfw, i) : make_float2(0.0f, 0.0f);
    float2 t = make_float2(0.0f, 0.0f);
    for (int e = src.row_ptr[row]; e < src.row_ptr[row + 1]; ++e) {
        const int o = src.pos[e] - row * x.g.nx - xp;
        if (o != 0 && o != 1) continue;
        const float R = o ? Rv.y : Rv.x, den = 1.0f + 2.0f * dt * (o ? d.y : d.x);
        ad.rsrc[(size_t)g * ad.n_src + e] = R;
        if (x.m.nonlinear) (o ? t.y : t.x) += R * 2.0f * dt * ad.add[e] / den;
    }
    return t;
}

// den (kw_adjx_den): the three divergence adjoints.  The source points of the block's
// rows are bits of an LDS mask; only at a set bit its row's list is searched.
KW_XS_TEMPLATE, bool ABS>
__global__ void KW_XS_BOUNDS(512, 3) kw_adjx_den_s(XSArgs a, AdjDev ad, const float2 *p_spec, int loss) {
    KW_XS_BEGIN(pml_y, pml_z)
    const SourceDev &src = x.src;
    const bool any_src = rows_have_points(src.row_ptr, row0, P.rows);      // block-uniform
    const int words = (x.g.nx + 31) / 32;
    uint32_t *const mask = reinterpret_cast<uint32_t *>(P.set(3));
    if (any_src) {
        for (int i = threadIdx.x; i < P.rows * words; i += blockDim.x) mask[i] = 0;
        __syncthreads();
        for_points(src.row_ptr, row0, P.rows, [&](const int (&e)[kPoints], const bool (&ok)[kPoints]) __attribute__((always_inline)) {
#pragma unroll
            for (int k = 0; k < kPoints; ++k) {
                const int i = src.pos[e[k]] - row0 * x.g.nx, row = i / x.g.nx, xp = i - row * x.g.nx;
                if (ok[k]) atomicOr(mask + row * words + xp / 32, 1u << (xp % 32));
            }
        });
    }
    if constexpr (ABS) {
        to_points<RSY, RSM, RSP, PLANES, 2>(a, P, [&](int s) __attribute__((always_inline)) { return (s ? x.Sin[1] : x.Sin[0]) + soff; });
    } else {
        if (loss) to_points<RSY, RSM, RSP, PLANES, 1>(a, P, [&](int) __attribute__((always_inline)) { return p_spec + soff; });
        else __syncthreads();
    }
    const float dt = x.g.dt;
    x_middle<RSM>(a, P, roff, [&](auto RC, const XTask &T, int off, int j) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        float2 r0[R], base[R], dcom[ABS ? R : 1];      // rbt (+ T1'), rho0 T0' (ABS)
        ld_run<R>(x.m.rho0, T, r0);
        if constexpr (ABS) {
            float2 rbt[R];
            ld_run<R>(ad.rbt, T, rbt);
            run_inverse<R>(P, P.sh + off, j, dcom);
            run_inverse<R>(P, P.set(1) + off, j, base);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                base[r] = c_add(rbt[r], base[r]);
                dcom[r] = make_float2(r0[r].x * dcom[r].x, r0[r].y * dcom[r].y);
            }
        } else {
            float2 c[R];
            pbar_run<R>(a, ad, P, loss, T, off, j, base, c);
#pragma unroll
            for (int r = 0; r < R; ++r) base[r] = make_float2(c[r].x * base[r].x, c[r].y * base[r].y);
        }
#pragma unroll 1
        for (int g = 0; g < 3; ++g) {
            float *const rb = pick3(ad.rb, g);
            const float *const dfw = pick3(ad.dfw, g), *const rho = pick3(ad.rho, g);
            const float q1 = (g == 1 ? P.qy : P.qz)[T.y];
            float2 v[R], nb[R];
            ld_run<R>(rb, T, nb);
            if (x.m.nonlinear) {
                float2 d[R], rn[R];
                ld_run<R>(dfw, T, d);
                ld_run<R>(rho, T, rn);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float2 q = g == 0 ? *reinterpret_cast<const float2 *>(x.t.pml_x + T.x + 2 * r * T.S0)
                                            : make_float2(q1, q1);
                    const float2 Rv = c_add(nb[r], base[r]);
                    const float2 den = make_float2(1.0f + 2.0f * dt * d[r].x, 1.0f + 2.0f * dt * d[r].y);
                    v[r].x = -Rv.x * (q.x * dt * r0[r].x + 2.0f * dt * rn[r].x) / den.x;
                    v[r].y = -Rv.y * (q.y * dt * r0[r].y + 2.0f * dt * rn[r].y) / den.y;
                    nb[r] = make_float2(Rv.x * q.x * q.x / den.x, Rv.y * q.y * q.y / den.y);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const float2 q = g == 0 ? *reinterpret_cast<const float2 *>(x.t.pml_x + T.x + 2 * r * T.S0)
                                            : make_float2(q1, q1);
                    const float2 Rv = c_add(nb[r], base[r]);
                    v[r] = make_float2(-Rv.x * q.x * dt * r0[r].x, -Rv.y * q.y * dt * r0[r].y);
                    nb[r] = make_float2(Rv.x * q.x * q.x, Rv.y * q.y * q.y);
                }
            }
            if constexpr (ABS) {
#pragma unroll
                for (int r = 0; r < R; ++r) v[r] = c_add(v[r], dcom[r]);
            }
            if (any_src) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const int xp = T.x + 2 * r * T.S0;               // (even: both bits in one word)
                    const uint32_t bits = mask[T.y * words + xp / 32] >> (xp % 32) & 3u;
                    if (bits) v[r] = c_add(v[r], source_terms(x, ad, rb, dfw, T.at(r), base[r], row0 + T.y, xp, g));
                }
            }
            st_run<R>(rb, T, nb);
            run_forward<R>(P, P.set(g) + off, j, v);
        }
    });
    to_spectra<RSY, RSM, RSP, PLANES, false, 3>(a, P, 3, [&](int s) __attribute__((always_inline)) { return pick3(x.Sout, s) + soff; });
}

template <RadixSet RSY, RadixSet RSM, RadixSet RSP>
hipError_t launch_vel(hipStream_t s, const LaunchCfg &c, const XArgs &x, const AdjDev &ad) {
    auto q = XStagedLaunch<RSY, RSM, RSP>::shape(c, x, XS_VEL, 1, nullptr);
    q.grid.y = 3;
    if (c.planes >> XS_VEL & 1)
        hipLaunchKernelGGL((kw_adjx_vel_s<RSY, RSM, RSP, true>), q.grid, q.block, q.lds, s, q.a, ad);
    else
        hipLaunchKernelGGL((kw_adjx_vel_s<RSY, RSM, RSP, false>), q.grid, q.block, q.lds, s, q.a, ad);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_xs_adj(hipStream_t s, int pass, const LaunchCfg &c, const XArgs &x, const AdjDev &ad,
                         const float2 *p_spec, bool loss) {
    if (pass == ADJX_VEL)
        return c.xs == 1 ? launch_vel<kPow2Y, kPow2M, kPow2P>(s, c, x, ad)
                         : launch_vel<kAnyY, kAnyM, kAnyP>(s, c, x, ad);
    const int L = loss ? 1 : 0;
    auto q = XStagedLaunch<kAnyY, kAnyM, kAnyP>::shape(c, x, pass == ADJX_EOS ? XS_EOS : XS_DEN,
                                                       pass == ADJX_EOS ? 2 : 3, nullptr);
    switch (pass) {
    case ADJX_EOS:
        hipLaunchKernelGGL((kw_adjx_eos_s<kAnyY, kAnyM, kAnyP, false>), q.grid, q.block, q.lds, s, q.a, ad, p_spec, L);
        break;
    case ADJX_DEN:
        q.lds += xs_mask_bytes(x.g.nx, q.a.rows);
        hipLaunchKernelGGL((kw_adjx_den_s<kAnyY, kAnyM, kAnyP, false, false>), q.grid, q.block, q.lds, s, q.a, ad, p_spec, L);
        break;
    case ADJX_DEN_ABS:
        q.lds += xs_mask_bytes(x.g.nx, q.a.rows);
        hipLaunchKernelGGL((kw_adjx_den_s<kAnyY, kAnyM, kAnyP, false, true>), q.grid, q.block, q.lds, s, q.a, ad, p_spec, L);
        break;
    default:
        hipLaunchKernelGGL((kw_adjx_sum_s<kAnyY, kAnyM, kAnyP, false>), q.grid, q.block, q.lds, s, q.a, ad);
        break;
    }
    return hipGetLastError();
}

}  // namespace kw
