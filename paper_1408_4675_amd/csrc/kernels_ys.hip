// The y pass on in-place staged transforms (staged.h), every length but 625.
//
// A block reads its tile's columns into the first stage's registers, exchanges
// through LDS once (twice for three stages) and writes the last stage's results:
// HBM traffic is the field in and out, and what bounds the pass is that copy and,
// on small grids, the latency of the two or three phases.  Before (one butterfly
// a thread: 135 = 3 3 15 leaves four threads of five idle in its radix-15 pass)
// and now, us of a step's forward / inverse passes (6 / 8 fields, none of them part of an
// x pass):
// 250 x 135 x 90 192 / 221 -> 73 / 85; 160^3 70 / 85 -> 54 / 68 (3.6 / 3.9 TB/s);
// 360 x 270 x 120 480 / 557 -> 164 / 206; 450 x 480 x 324 1360 / 1851 -> 799 / 1208
// (4.2 / 3.7 TB/s); 48 x 20 x 18 42 / 40 -> 20 / 20.
#include "staged_cols.h"
#include "ystaged.h"

namespace kw {

namespace {

struct YSArgs {
    YArgs y;
    ColPlan p;
};

template <bool INV>
__global__ void __launch_bounds__(512) kw_ystaged(YSArgs a) {
    extern __shared__ float2 lds_all[];
    constexpr RadixSet RS = kAnyY;
    const YArgs &y = a.y;
    const ColPlan &p = a.p;
    const int ny = y.ny, M = y.M;
    int blk, rep_;
    if (!xcd_order(blockIdx.x, line_group(y.tb), 1, y.ntiles * y.nz, blk, rep_)) return;
    const int iz = uniform(blk / y.ntiles), tile = uniform(blk - iz * y.ntiles);
    const int cols = min(y.tb, M - tile * y.tb);
    const size_t off = (size_t)iz * ny * M + (size_t)tile * y.tb;
    const float2 *const src = pick3(y.f, (int)blockIdx.z) + off;
    float2 *const dst = pick3(y.o, (int)blockIdx.z) + off;
    const ColTile T{lds_all + ny, lds_all, ny, y.tb, p.ltb, (uint32_t)M * 8u};
    if constexpr (!INV) y_prologue(y, blk == 0 && blockIdx.z == 0);
    stage_table(lds_all, y.tw, ny);
    const bool tile0 = tile == 0;                            // block-uniform
    if constexpr (INV) {
        // (an in-place pass reads column 0 before the barrier, writes it after)
        col_load_last<RS>(p, T, src, cols, T.sh, tile0);
        __syncthreads();
        if (p.ax.np == 3) {
            col_middle<RS, true>(p, T, T.sh);
            __syncthreads();
        }
        col_store<RS>(p, T, dst, cols, T.sh);
    } else {
        __syncthreads();
        col_load<RS>(p, T, src, nullptr, nullptr, cols, T.sh);
        __syncthreads();
        if (p.ax.np == 3) {
            col_middle<RS, false>(p, T, T.sh);
            __syncthreads();
        }
        col_store_last<RS>(p, T, dst, cols, T.sh, tile0);
        if (tile0) {
            // unpack column 0 into A (rows 1..h) and B (rows ny-h..ny-1)
            __syncthreads();
            for (int r = threadIdx.x; r < ny; r += blockDim.x) {
                const int type = col0_type(r, ny), j = col0_ky(r, ny);
                float2 v = T.sh[j << T.ltb];
                if (type != C0_DOUBLE) {
                    const float2 pc = c_conj(T.sh[(ny - j) << T.ltb]);
                    if (type == C0_A) {
                        v = c_scale(c_add(v, pc), 0.5f);             // (C + conj C(-ky)) / 2
                    } else {
                        const float2 d = c_sub(v, pc);
                        v = make_float2(0.5f * d.y, -0.5f * d.x);    // (C - conj C(-ky)) / 2i
                    }
                }
                dst[(size_t)r * M] = v;
            }
        }
    }
}

}  // namespace

hipError_t launch_ystaged(hipStream_t s, const LaunchCfg &c, const YArgs &y, bool inverse, int nfields) {
    YSArgs a{};
    a.y = y;
    a.p.ax = c.ys_axis;
    a.p.S0 = y.ny / a.p.ax.r[0];
    a.y.tb = c.ys_tb;
    a.y.ntiles = (y.M + c.ys_tb - 1) / c.ys_tb;
    while ((1 << a.p.ltb) < c.ys_tb) ++a.p.ltb;
    const dim3 grid(xcd_grid(a.y.ntiles * y.nz, line_group(c.ys_tb), 1), 1, nfields);
    const size_t lds = 8 * ((size_t)y.ny + (size_t)y.ny * c.ys_tb);
    const dim3 block(c.ys_threads);
    if (inverse) hipLaunchKernelGGL((kw_ystaged<true>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((kw_ystaged<false>), grid, block, lds, s, a);
    return hipGetLastError();
}

}  // namespace kw
