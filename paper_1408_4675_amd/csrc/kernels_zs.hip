// The fused z pass on in-place staged transforms (staged.h): forward z FFT ->
// k-space operator(s) -> inverse z FFT of column tiles, every length but 625.
//
// A block holds a tile of tb columns in LDS.  The first stage reads global
// memory, the last forward stage, the operator and the last inverse stage run in
// registers one after the other (the butterfly of both has the same elements),
// and the first inverse stage writes global memory: two barriers for the two
// transforms of a two-stage length.  kappa is evaluated once a point for the
// gradient's three outputs, which leave through three tiles.
//
// What bounds it: vector instructions and the latency of a block's few phases
// (4 to 6 wavefronts a SIMD), then the strided 128-byte rows of a tile.  Before
// (one-butterfly-a-thread or fixed-width engines) and now, us a launch of
// gradient / divergence / absorption: 250 x 135 x 90 46 / 55 / 40 -> 27 / 35 / 24;
// 160^3 41 / 45 / 35 -> 30 / 34 / 23 (2.2 / 2.9 / 2.8 TB/s); 128^3 22 / 23 / 17 ->
// 15 / 17 / 13; 64^3 15.5 / 8.5 / 9.3 -> 9.2 / 7.6 / 8.9; 256^3 divergence 103 -> 96
// (4.2 TB/s), absorption 58 -> 59.
#include "staged_cols.h"
#include "zstaged.h"

namespace kw {

namespace {

struct ZSArgs {
    ZArgs z;
    ColPlan p;
};

// a column's wavenumbers and x, y factors
struct ZCol {
    float kxy2;
    float2 dx, dy;
};

template <int MODE>
__device__ __forceinline__ ZCol z_col(const ZArgs &a, int ix, int iy) {
    ZCol c;
    const float kx = a.t.kx[ix], ky = a.t.ky[iy];
    c.kxy2 = kx * kx + ky * ky;
    if constexpr (MODE != ZM_ABS && MODE != ZM_ABSM) {
        constexpr bool plus = MODE == ZM_GRAD || MODE == ZM_GRADT;
        c.dx = plus ? a.t.dpx[ix] : a.t.dmx[ix];
        c.dy = plus ? a.t.dpy[iy] : a.t.dmy[iy];
    }
    return c;
}

// what the operators of a point share: kappa / N (gradient, divergence; the
// host takes this pass only where the polynomial holds at every k, so that no
// call sits in the unrolled loops) or k^2 (absorption)
template <int MODE>
__device__ __forceinline__ float z_base(const ZArgs &a, const ZCol &c, int iz) {
    const float kz = kz_of(a.g, iz);
    const float k2 = c.kxy2 + kz * kz;
    if constexpr (MODE == ZM_ABS || MODE == ZM_ABSM) return k2;
    else return kappa_poly(a.g.half_cdt * a.g.half_cdt * k2) * a.g.inv_n;
}

// v times the operator of output o
template <int MODE>
__device__ __forceinline__ float2 z_mul(const ZArgs &a, const ZCol &c, int o, int iz, float base,
                                        float scale, const float2 *dzl, float2 v) {
    if constexpr (MODE == ZM_ABS || MODE == ZM_ABSM) {
        // (the hardware's log2 and exp2, see z_operator)
        const float e = (o == 0) ? a.g.y_tau : a.g.y_eta;
        const float s = base > 0.0f
            ? __builtin_amdgcn_exp2f(e * __builtin_amdgcn_logf(base)) * a.g.inv_n * scale : 0.0f;
        return c_scale(v, s);
    } else {
        // (by value: a choice between addresses would put the struct in memory)
        float2 d = o == 2 ? dzl[iz] : make_float2(0.0f, 0.0f);
        d.x = o == 0 ? c.dx.x : o == 1 ? c.dy.x : d.x;
        d.y = o == 0 ? c.dx.y : o == 1 ? c.dy.y : d.y;
        d = c_scale(d, base);
        return (MODE == ZM_DIVT || MODE == ZM_GRADT) ? c_mulc(v, d) : c_mul(v, d);
    }
}

// Column 0 of a double row holds A + i B (kx = 0 and the Nyquist kx), whose raw
// z spectrum lies in LDS column 0: A and B separate with the partner at -kz,
// each gets its own operator, and A' + i B' of every output goes back.  A thread
// reads and writes a pair (kz, -kz).
template <int MODE, int NOUT>
__device__ __forceinline__ void zs_pairs(const ZArgs &z, const ColTile &T, const float2 *sh2,
                                         const float2 *dzl, int iy, int o, float s0) {
    const ZCol ca = z_col<MODE>(z, 0, iy), cb = z_col<MODE>(z, z.g.M, iy);
    constexpr int NIN = MODE == ZM_ABSM ? 2 : 1;
    __syncthreads();
    for (int k = threadIdx.x; k <= T.n / 2; k += blockDim.x) {
        const int mk = k == 0 ? 0 : T.n - k;
        float2 A[NIN], B[NIN];
#pragma unroll
        for (int in = 0; in < NIN; ++in) {
            const float2 *const raw = in ? sh2 : T.sh;
            const float2 c1 = raw[k << T.ltb], c2 = raw[mk << T.ltb];
            // (C(k) + conj C(-k)) / 2 and (C(k) - conj C(-k)) / 2i
            A[in] = make_float2(0.5f * (c1.x + c2.x), 0.5f * (c1.y - c2.y));
            B[in] = make_float2(0.5f * (c1.y + c2.y), 0.5f * (c2.x - c1.x));
        }
#pragma unroll 1
        for (int side = 0; side < 2; ++side) {
            // A(-kz) = conj A(kz), B(-kz) = conj B(kz)
            const int kk = side ? mk : k;
            if (side && mk == k) break;
            const float ba = z_base<MODE>(z, ca, kk), bb = z_base<MODE>(z, cb, kk);
#pragma unroll
            for (int oo = 0; oo < NOUT; ++oo) {
                float2 sum = make_float2(0.0f, 0.0f);
#pragma unroll
                for (int in = 0; in < NIN; ++in) {
                    const int op = NOUT == 3 ? oo : MODE == ZM_ABSM ? in : o;
                    const float sc = MODE == ZM_ABSM ? (in ? z.sb : z.sa) : s0;
                    const float2 a = side ? c_conj(A[in]) : A[in], b = side ? c_conj(B[in]) : B[in];
                    const float2 ya = z_mul<MODE>(z, ca, op, kk, ba, sc, dzl, a);
                    const float2 yb = z_mul<MODE>(z, cb, op, kk, bb, sc, dzl, b);
                    sum = c_add(sum, make_float2(ya.x - yb.y, ya.y + yb.x));      // ya + i yb
                }
                T.sh[((size_t)oo * T.n + kk) << T.ltb] = sum;
            }
        }
    }
    __syncthreads();
}

// (The operator of one element at a time, sched_barrier: interleaved over the R
// elements of a butterfly it takes up to 100 registers more.)
// MODE as in kw_zfused; NOUT 3: the gradient's outputs from one block, else one
// output a block
template <RadixSet RS, int MODE, int NOUT>
__global__ void __launch_bounds__(512) kw_zstaged(ZSArgs a) {
    extern __shared__ float2 lds_all[];
    const ZArgs &z = a.z;
    const int n = z.g.nz, tb = z.tb, M = z.g.M, ny = z.g.ny;
    constexpr bool split = MODE == ZM_GRAD && NOUT == 1;
    int blk, o;
    if (!xcd_order(blockIdx.x, line_group(tb), split ? 3 : 1, z.ntiles * ny, blk, o)) return;
    if constexpr (MODE != ZM_GRAD) o = blockIdx.y;
    float2 *const tws = lds_all, *const dzl = lds_all + n;
    const ColPlan &p = a.p;
    const ColTile T{lds_all + 2 * n, tws, n, tb, p.ltb, (uint32_t)M * ny * 8u};
    float2 *const sh = T.sh;
    const int iy = uniform(blk / z.ntiles), tile = uniform(blk - iy * z.ntiles);
    const size_t off = (size_t)iy * M + (size_t)tile * tb;
    const int cols = min(tb, M - tile * tb);
    const int c0type = col0_type(iy, ny);
    const bool pairing = tile == 0 && c0type == C0_DOUBLE;

    stage_table(tws, z.t.tw_z, n);
    if constexpr (MODE != ZM_ABS && MODE != ZM_ABSM)
        stage_table(dzl, (MODE == ZM_GRAD || MODE == ZM_GRADT) ? z.t.dpz : z.t.dmz, n);
    __syncthreads();
    float2 *const sh2 = sh + ((size_t)n << T.ltb);     // ABSM: tile of the second input
    const int f = (MODE == ZM_GRAD || MODE == ZM_ABSM) ? 0 : o;
    const bool sum = (MODE == ZM_ABS || MODE == ZM_ABSM) && f == 0 && z.add0[0];
    constexpr int NIN = MODE == ZM_ABSM ? 2 : 1;
#pragma unroll 1
    for (int in = 0; in < NIN; ++in) {
        const bool add = sum && in == 0;
        col_load<RS>(p, T, (in ? z.in[1] : pick3(z.in, f)) + off, add ? z.add0[0] + off : nullptr,
                     add ? z.add0[1] + off : nullptr, cols, in ? sh2 : sh);
    }
    __syncthreads();
    if (p.ax.np == 3) {
#pragma unroll 1
        for (int in = 0; in < NIN; ++in) col_middle<RS, false>(p, T, in ? sh2 : sh);
        __syncthreads();
    }
    // last forward stage, operator, last inverse stage
    const int w = p.ax.wl;
    const float s0 = (MODE == ZM_ABSM || (MODE == ZM_ABS && o == 0)) ? z.sa : 1.0f;
    with_radix<RS>(p.ax.rl, [&](auto RC) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        const int nt = w << T.ltb, step = w << T.ltb;
        for (int i = threadIdx.x; i < nt; i += blockDim.x) {
            const int b = i >> T.ltb, c = i & (tb - 1);
            if (c >= cols) continue;
            int ix = tile * tb + c, iyk = iy;
            if (ix == 0) {                                   // column 0, see kw_zfused
                ix = (c0type == C0_A) ? 0 : M;
                iyk = col0_ky(iy, ny);
            }
            const ZCol col = z_col<MODE>(z, ix, iyk);
            float2 *const e = sh + (b << T.ltb) + c, *const e2 = sh2 + (b << T.ltb) + c;
            float2 X[R], v[NOUT == 3 ? R : 1];
            if constexpr (MODE == ZM_ABSM) {
                // the first input's term waits in its tile while the second is formed
#pragma unroll
                for (int q = 0; q < R; ++q) X[q] = e[q * step];
                Dft<R, false>::template run<1, 0>(X);
                if (!(pairing && c == 0)) {
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const int k = b + w * q;
                        X[q] = z_mul<MODE>(z, col, 0, k, z_base<MODE>(z, col, k), z.sa, dzl, X[q]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
#pragma unroll
                for (int q = 0; q < R; ++q) e[q * step] = X[q];
            }
#pragma unroll
            for (int q = 0; q < R; ++q) X[q] = (MODE == ZM_ABSM ? e2 : e)[q * step];
            Dft<R, false>::template run<1, 0>(X);
            if (pairing && c == 0) {
                // the raw spectrum, for the pairs below
#pragma unroll
                for (int q = 0; q < R; ++q) (MODE == ZM_ABSM ? e2 : e)[q * step] = X[q];
                continue;
            }
            if constexpr (MODE == ZM_ABSM) {
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const int k = b + w * q;
                    X[q] = c_add(e[q * step],
                                 z_mul<MODE>(z, col, 1, k, z_base<MODE>(z, col, k), z.sb, dzl, X[q]));
                    __builtin_amdgcn_sched_barrier(0);
                }
                Dft<R, true>::template run<1, 0>(X);
#pragma unroll
                for (int q = 0; q < R; ++q) e[q * step] = X[q];
            } else if constexpr (NOUT == 3) {
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    X[q] = c_scale(X[q], z_base<MODE>(z, col, b + w * q));
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int oo = 0; oo < 3; ++oo) {
                    float2 *const eo = e + oo * ((size_t)n << T.ltb);
#pragma unroll
                    for (int q = 0; q < R; ++q)
                        v[q] = c_mul(X[q], oo == 2 ? dzl[b + w * q] : make_float2(oo == 0 ? col.dx.x : col.dy.x,
                                                                                  oo == 0 ? col.dx.y : col.dy.y));
                    Dft<R, true>::template run<1, 0>(v);
#pragma unroll
                    for (int q = 0; q < R; ++q) eo[q * step] = v[q];
                }
            } else {
                if (MODE == ZM_ABS || o < 2) {               // block-uniform
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const int k = b + w * q;
                        X[q] = z_mul<MODE>(z, col, o == 0 ? 0 : 1, k, z_base<MODE>(z, col, k), s0, dzl, X[q]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < R; ++q) {
                        const int k = b + w * q;
                        X[q] = z_mul<MODE>(z, col, 2, k, z_base<MODE>(z, col, k), s0, dzl, X[q]);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                Dft<R, true>::template run<1, 0>(X);
#pragma unroll
                for (int q = 0; q < R; ++q) e[q * step] = X[q];
            }
        }
    });
    if (pairing) {                                           // block-uniform
        zs_pairs<MODE, NOUT>(z, T, sh2, dzl, iy, o, s0);
        with_radix<RS>(p.ax.rl, [&](auto RC) __attribute__((always_inline)) {
            constexpr int R = decltype(RC)::value;
            const int step = w << T.ltb;
            for (int b = threadIdx.x; b < w * NOUT; b += blockDim.x) {
                const int oo = b / w;
                float2 *const e = sh + oo * ((size_t)n << T.ltb) + ((b - oo * w) << T.ltb);
                float2 v[R];
#pragma unroll
                for (int q = 0; q < R; ++q) v[q] = e[q * step];
                Dft<R, true>::template run<1, 0>(v);
#pragma unroll
                for (int q = 0; q < R; ++q) e[q * step] = v[q];
            }
        });
    }
    __syncthreads();
    if (p.ax.np == 3) {
#pragma unroll 1
        for (int oo = 0; oo < NOUT; ++oo) col_middle<RS, true>(p, T, sh + oo * ((size_t)n << T.ltb));
        __syncthreads();
    }
#pragma unroll 1
    for (int oo = 0; oo < NOUT; ++oo)
        col_store<RS>(p, T, pick3(z.out, NOUT == 3 ? oo : o) + off, cols, sh + oo * ((size_t)n << T.ltb));
}

template <RadixSet RS>
hipError_t launch_set(hipStream_t s, const LaunchCfg &c, int mode, ZSArgs a, int nout, dim3 grid,
                      size_t lds) {
    const dim3 block(c.zs_threads);
    switch (mode) {
    case ZM_GRAD:
        if (nout == 3) hipLaunchKernelGGL((kw_zstaged<RS, ZM_GRAD, 3>), grid, block, lds, s, a);
        else hipLaunchKernelGGL((kw_zstaged<RS, ZM_GRAD, 1>), grid, block, lds, s, a);
        break;
    case ZM_DIV: hipLaunchKernelGGL((kw_zstaged<RS, ZM_DIV, 1>), grid, block, lds, s, a); break;
    case ZM_ABS: hipLaunchKernelGGL((kw_zstaged<RS, ZM_ABS, 1>), grid, block, lds, s, a); break;
    case ZM_DIVT: hipLaunchKernelGGL((kw_zstaged<RS, ZM_DIVT, 1>), grid, block, lds, s, a); break;
    case ZM_GRADT: hipLaunchKernelGGL((kw_zstaged<RS, ZM_GRADT, 1>), grid, block, lds, s, a); break;
    default: hipLaunchKernelGGL((kw_zstaged<RS, ZM_ABSM, 1>), grid, block, lds, s, a); break;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_zstaged(hipStream_t s, const LaunchCfg &c, int mode, const ZArgs &z, int n_out) {
    ZSArgs a{};
    a.z = z;
    a.p.ax = c.zs_axis;
    const int n = z.g.nz;
    a.p.S0 = n / a.p.ax.r[0];
    // the gradient's three outputs from one block where their tiles leave room
    // for a second block on the CU, else one block an output
    int tb = mode == ZM_GRAD ? c.zs_tb_grad : mode == ZM_ABSM ? c.zs_tb_absm : c.zs_tb;
    const int nout = mode == ZM_GRAD && c.zs_grad3 ? 3 : 1;
    a.z.tb = tb;
    a.z.ntiles = (z.g.M + tb - 1) / tb;
    a.p.ltb = 0;
    while ((1 << a.p.ltb) < tb) ++a.p.ltb;
    const int tiles = mode == ZM_ABSM ? 2 : nout;
    const size_t lds = 8 * ((size_t)2 * n + (size_t)tiles * n * tb);
    const int nblk = a.z.ntiles * z.g.ny;
    const dim3 grid(xcd_grid(nblk, line_group(tb), mode == ZM_GRAD && nout == 1 ? 3 : 1),
                    mode == ZM_GRAD ? 1 : n_out);
    return c.zs == 1 ? launch_set<kPow2Y>(s, c, mode, a, nout, grid, lds)
                     : launch_set<kAnyY>(s, c, mode, a, nout, grid, lds);
}

}  // namespace kw
