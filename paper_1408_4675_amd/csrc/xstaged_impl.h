// The x passes of a step on in-place staged transforms (staged.h), for the row
// lengths that have stages (stage_axis), and with the y transforms around them where a z
// plane fits LDS.
//
// A block holds `rows` rows of every field that its update couples: one set of
// rows for a velocity component, three for the density (the three divergence
// components), two for the equation of state (the two absorption terms).  Rows
// are loaded as they lie in memory, transformed in place, updated in the middle
// sweep -- first stage of the inverse transform, point-wise update, first stage of the
// forward transform, all in registers -- and leave through the first sets again.
//
// PLANES: the rows are those of one z plane, and the block runs the inverse y
// transform before and the forward y transform after the x pass too: the
// spectrum moves through HBM once instead of three times, in one launch instead of
// three.
//
// What bounds them: on rows vector instructions and barriers (three to four
// wavefronts a SIMD, five phases a block), on planes the phases of the one or two
// blocks that a CU holds, which a barrier each keeps in step.  us a launch on the engines
// (one butterfly a thread; density with its three components exchanged through LDS) and
// here, kernel trace: 250 x 135 x 90 maps, velocity with its y passes 323 -> 90 (planes;
// 3.0 M points, 15 fields in and out), density 235 -> 54 (2.9 TB/s), pressure 147 -> 42
// (3.5 TB/s); 160^3 velocity with its y passes 138 -> 83 (3.0 TB/s), density 88 -> 71,
// pressure 58 -> 53; 450 x 480 x 324 water, velocity 1055 -> 856, density 1550 -> 966,
// lossless density with the equation of state 2354 -> 1191; 128^3 velocity with its y
// passes 54 -> 34.
// Registers: the bounds below keep four wavefronts a SIMD (density three).  Scratch that
// this costs, bytes a lane: rows, velocity 8, pressure 16 merged and 12-24 unmerged;
// planes none.
#pragma once

#include "staged.h"
#include "xstaged.h"

namespace kw {

namespace {

struct XSArgs {
    XArgs x;
    StageAxis ax, ay;
    FastDiv dM, drows, dS0;  // by M, the rows of a set and the runs of an x row (M / R0)
    int pitch, pad;          // LDS distance of rows; padding slots per x run
    int rows;                // rows of a set
    float *scr;              // scratch: a real field
};

// LDS column of x index k: `pad` slots after each run of R0 (the radix of the
// first x stage).  The lanes of that stage are R0 + pad apart, an odd distance,
// which meets every bank; and the elements of a butterfly stay equidistant in
// every stage (one addition an element; a slot per 16 columns cost three).
__device__ __forceinline__ int pcol(const XSArgs &a, int k) { return k + a.pad * a.ax.dw1.div(k); }

// The rows of one block: LDS and tables
struct Rows {
    float2 *sh;              // [set][row][pitch]
    const float2 *twx, *twp, *twy;
    const int *ypos;         // LDS row of row y between the y transforms
    const float *qy, *qz;    // PML factors of the rows along y and z
    int M, ny, pitch;        // ny: rows of a set in LDS
    int rows;                // rows in the grid (fewer in the last block)
    __device__ __forceinline__ float2 *set(int s) const { return sh + s * ny * pitch; }
};

// The threads at one set: number first of count
struct Lanes {
    int first, count;
};
// f(set, its threads) for NS sets (0: ns of them): on planes the sets side by side,
// whole wavefronts each; on rows one after the other (there a set has a task for every
// thread).  us on planes, one after the other and side by side: density 48 x 20 x 18
// 30 -> 20, 64^3 36 -> 29, absorption terms 18 -> 14, 23 -> 18
template <bool PLANES, int NS, class F>
__device__ __forceinline__ void for_sets(int ns, F f) {
    const int t = threadIdx.x, n = blockDim.x;
    if constexpr (NS == 1) {
#pragma unroll 1
        for (int s = 0; s < 1; ++s) f(s, Lanes{t, n});     // (without the loop a variant spilled)
    } else if constexpr (PLANES) {
        const int per = n / warpSize / ns * warpSize;
        const int s = uniform(t / per);
        if (s < ns) f(s, Lanes{t - s * per, per});
    } else {
#pragma unroll 1
        for (int s = 0; s < ns; ++s) f(s, Lanes{t, n});
    }
}

// ---- y stages: lanes along the columns -----------------------------------------

// inverse, last stage: rows of the global spectrum -> LDS (column 0 repacked:
// C(ky) = A(ky) + i B(ky) with A(-ky) = conj A(ky), see col0_type)
template <RadixSet RSY>
__device__ __forceinline__ void y_load_inv(const XSArgs &a, const Rows &P, Lanes L, float2 *sh, const float2 *S) {
    const int w = a.ay.wl, ny = P.ny;
    with_radix<RSY>(a.ay.rl, [&](auto RC) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        const int nt = P.M * w;
        for (int i = L.first; i < nt; i += L.count) {
            const int b = a.dM.div(i), c = i - b * P.M;
            float2 v[R];
#pragma unroll
            for (int q = 0; q < R; ++q) v[q] = ld_at(S + (size_t)q * nt, (uint32_t)i * 8u);
            if (c == 0) {
                float2 A[R], B[R];
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const Col0Rows o = col0_rows(b + w * q, ny);
                    A[q] = S[(size_t)o.a * P.M];
                    B[q] = S[(size_t)o.b * P.M];
                }
#pragma unroll
                for (int q = 0; q < R; ++q) v[q] = col0_join(col0_rows(b + w * q, ny), A[q], B[q]);
            }
            Dft<R, true>::template run<1, 0>(v);
            float2 *const dst = sh + b * P.pitch + pcol(a, c);
#pragma unroll
            for (int r = 0; r < R; ++r) dst[r * w * P.pitch] = v[r];
        }
    });
}

// stage p in LDS (not the last one)
template <RadixSet RSY, bool INV>
__device__ __forceinline__ void y_stage(const XSArgs &a, const Rows &P, Lanes L, float2 *sh, int p) {
    const int w = pick3(a.ay.w, p);
    with_radix<RSY>(pick3(a.ay.r, p), [&](auto RC) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        const int nt = P.M * (P.ny / R);
        for (int i = L.first; i < nt; i += L.count) {
            const int t = a.dM.div(i), c = i - t * P.M;
            const int hi = p == 0 ? t : a.ay.dw1.div(t), lo = t - hi * w;
            const int ts = w * digit_index(a.ay, p, hi);
            float2 *const e = sh + (lo + w * R * hi) * P.pitch + pcol(a, c);
            const int step = w * P.pitch;
            float2 v[R];
#pragma unroll
            for (int d = 0; d < R; ++d) v[d] = e[d * step];
            if (INV) twiddle<R, true>(v, P.twy, ts);
            Dft<R, INV>::template run<1, 0>(v);
            if (!INV) twiddle<R, false>(v, P.twy, ts);
#pragma unroll
            for (int d = 0; d < R; ++d) e[d * step] = v[d];
        }
    });
}

// last forward stage, to the rows of the global spectrum; column 0 stays in LDS
template <RadixSet RSY>
__device__ __forceinline__ void y_store(const XSArgs &a, const Rows &P, Lanes L, float2 *sh, float2 *S) {
    const int w = a.ay.wl;
    with_radix<RSY>(a.ay.rl, [&](auto RC) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        const int nt = P.M * w;
        for (int i = L.first; i < nt; i += L.count) {
            const int b = a.dM.div(i), c = i - b * P.M;
            float2 *const e = sh + b * P.pitch + pcol(a, c);
            const int step = w * P.pitch;
            float2 v[R];
#pragma unroll
            for (int d = 0; d < R; ++d) v[d] = e[d * step];
            Dft<R, false>::template run<1, 0>(v);
            if (c == 0) {
#pragma unroll
                for (int d = 0; d < R; ++d) e[d * step] = v[d];
            } else {
#pragma unroll
                for (int d = 0; d < R; ++d) st_at(S + (size_t)d * nt, (uint32_t)i * 8u, v[d]);
            }
        }
    });
}
// column 0 unpacked into A (rows 1..h) and B (rows ny-h..ny-1), see col0_type
__device__ __forceinline__ void y_store_col0(const Rows &P, Lanes L, const float2 *sh, float2 *S) {
    const int ny = P.ny;
    for (int r = L.first; r < ny; r += L.count) {
        const int type = col0_type(r, ny);
        const int j = col0_ky(r, ny);
        float2 v = sh[j * P.pitch];
        if (type != C0_DOUBLE) {
            const float2 pc = c_conj(sh[(ny - j) * P.pitch]);
            if (type == C0_A) {
                v = c_scale(c_add(v, pc), 0.5f);                 // (C + conj C(-ky)) / 2
            } else {
                const float2 d = c_sub(v, pc);
                v = make_float2(0.5f * d.y, -0.5f * d.x);        // (C - conj C(-ky)) / 2i
            }
        }
        S[(size_t)r * P.M] = v;
    }
}

// ---- x stages --------------------------------------------------------------------

// The last x stage with the real-transform split.  Elements k and M - k share
// the split, and the butterflies of lo = b and lo = w - b hold each other's
// partners, so one task runs both (lanes along the rows).  b = 0 and 2 b = w
// are their own partners: they run one butterfly's worth of stores.
// w - b + w q wraps only for b = 0: element q of the partner list is then
// element q + 1 of the butterfly itself.
template <RadixSet RSP, bool INV>
__device__ __forceinline__ void x_pair(const XSArgs &a, const Rows &P, Lanes L, float2 *sh) {
    const int w = a.ax.wl, cw = pcol(a, w);
    with_radix<RSP>(a.ax.rl, [&](auto RC) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        const int nt = P.ny * (w / 2 + 1);
        for (int i = L.first; i < nt; i += L.count) {
            const int b = a.drows.div(i), row = i - b * P.ny;
            const bool self = b == 0 || 2 * b == w;
            float2 *const e = sh + row * P.pitch;
            const int cb = pcol(a, b), cz = pcol(a, w - b);
            const int z0 = !INV && self ? cb : cz;
            float2 X[R], Z[R];
#pragma unroll
            for (int q = 0; q < R; ++q) X[q] = e[cb + q * cw];
#pragma unroll
            for (int q = 0; q < R; ++q) {
                int o = z0 + q * cw;
                if (INV && q == R - 1 && b == 0) o = 0;
                Z[q] = e[o];
            }
            if constexpr (INV) {
                // packed spectrum -> x[2n] + i x[2n+1] (before the transform):
                // A + i B, A = X_k + conj X_{M-k}, B = (X_k - conj X_{M-k}) w^-k
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const float2 xk = X[q], xm = Z[R - 1 - q];
                    const float2 A = make_float2(xk.x + xm.x, xk.y - xm.y);
                    const float2 D = make_float2(xk.x - xm.x, xk.y + xm.y);
                    const float2 B = c_mulc(D, P.twp[b + w * q]);
                    X[q] = make_float2(A.x - B.y, A.y + B.x);
                    Z[R - 1 - q] = make_float2(A.x + B.y, B.x - A.y);     // conj A + i conj B
                    if (q == 0 && b == 0) X[0] = make_float2(xk.x + xk.y, xk.x - xk.y);
                }
                Dft<R, true>::template run<1, 0>(X);
                Dft<R, true>::template run<1, 0>(Z);
            } else {
                Dft<R, false>::template run<1, 0>(X);
                Dft<R, false>::template run<1, 0>(Z);
                // A - i w^k B, A = (Z_k + conj Z_{M-k}) / 2, B = (Z_k - conj Z_{M-k}) / 2
                float2 O[R];
#pragma unroll
                for (int q = 0; q < R; ++q) {
                    const float2 zk = X[q];
                    const float2 zs = X[(R - q) % R], zp = Z[R - 1 - q];
                    const float2 zm = b == 0 ? zs : zp;
                    const float2 A = make_float2(0.5f * (zk.x + zm.x), 0.5f * (zk.y - zm.y));
                    const float2 B = make_float2(0.5f * (zk.x - zm.x), 0.5f * (zk.y + zm.y));
                    const float2 c = c_mul(P.twp[b + w * q], B);
                    O[q] = make_float2(A.x + c.y, A.y - c.x);
                    Z[R - 1 - q] = make_float2(A.x - c.y, -A.y - c.x);    // conj A - i conj c
                    if (q == 0 && b == 0) O[0] = make_float2(zk.x + zk.y, zk.x - zk.y);
                }
#pragma unroll
                for (int q = 0; q < R; ++q) X[q] = O[q];
            }
#pragma unroll
            for (int q = 0; q < R; ++q) e[cb + q * cw] = X[q];
            if (!self) {
#pragma unroll
                for (int q = 0; q < R; ++q) e[cz + q * cw] = Z[q];
            }
        }
    });
}

// middle stage of a three-stage x axis (p = 1)
template <RadixSet RSM, bool INV>
__device__ __forceinline__ void x_stage1(const XSArgs &a, const Rows &P, Lanes L, float2 *sh) {
    const int w = a.ax.w[1];
    with_radix<RSM>(a.ax.r[1], [&](auto RC) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        const int nt = P.ny * (P.M / R);
        for (int i = L.first; i < nt; i += L.count) {
            const int t = a.drows.div(i), row = i - t * P.ny;
            const int hi = a.ax.dw1.div(t), lo = t - hi * w;
            const int ts = w * hi;
            const int step = w + a.pad;
            float2 *const e = sh + row * P.pitch + lo + hi * R * step;
            float2 v[R];
#pragma unroll
            for (int d = 0; d < R; ++d) v[d] = e[d * step];
            if (INV) twiddle<R, true>(v, P.twx, ts);
            Dft<R, INV>::template run<1, 0>(v);
            if (!INV) twiddle<R, false>(v, P.twx, ts);
#pragma unroll
            for (int d = 0; d < R; ++d) e[d * step] = v[d];
        }
    });
}

// A task of the middle sweep: the R points n = j + r S0 (r < R0) of a row, as
// pairs of grid values x = 2 n, 2 n + 1.
struct XTask {
    size_t base;             // first element of the plane (uniform)
    uint32_t lane;           // byte offset of (y, x = 2 j)
    int S0, y, x;            // x of r = 0
    __device__ __forceinline__ XPos at(int r) const { return XPos{base + 2 * (size_t)(r * S0), lane}; }
};

// Runs f(IntC<R>, task, offset of its run in a set, j) over the middle sweep's
// tasks.  Lanes run along the points of a row, so global accesses are contiguous
// runs of M / R0 pairs.
template <RadixSet RSM, class F>
__device__ __forceinline__ void x_middle(const XSArgs &a, const Rows &P, size_t base, F f) {
    const int S0 = (int)a.dS0.d;
    with_radix<RSM>(a.ax.r[0], [&](auto RC) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        const int nt = P.rows * S0;
        for (int i = threadIdx.x; i < nt; i += blockDim.x) {
            const int y = a.dS0.div(i), j = i - y * S0;
            int hi = j;
            if (a.ax.np == 3) {
                const int q1 = a.ax.d2.div(j);           // j = r2 + R2 r1
                hi = q1 + a.ax.r[1] * (j - q1 * a.ax.r[2]);
            }
            const XTask T{base, (uint32_t)(y * 2 * P.M + 2 * j) * 4u, S0, y, 2 * j};
            f(RC, T, P.ypos[y] * P.pitch + hi * (R + a.pad), j);
        }
    });
    __syncthreads();
}
// first inverse x stage (the last to run) from a run, first forward stage to it
template <int R>
__device__ __forceinline__ void run_inverse(const Rows &P, const float2 *e, int j, float2 (&v)[R]) {
#pragma unroll
    for (int d = 0; d < R; ++d) v[d] = e[d];
    twiddle<R, true>(v, P.twx, j);
    Dft<R, true>::template run<1, 0>(v);
}
template <int R>
__device__ __forceinline__ void run_forward(const Rows &P, float2 *e, int j, float2 (&v)[R]) {
    Dft<R, false>::template run<1, 0>(v);
    twiddle<R, false>(v, P.twx, j);
#pragma unroll
    for (int d = 0; d < R; ++d) e[d] = v[d];
}
template <int R>
__device__ __forceinline__ void ld_run(const float *f, const XTask &T, float2 (&v)[R]) {
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = ld2(f, T.at(r));
}
template <int R>
__device__ __forceinline__ void ld_run(const Coef &c, const XTask &T, float2 (&v)[R]) {
    if (c.map) {
        ld_run<R>(c.map, T, v);
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) v[r] = make_float2(c.scalar, c.scalar);
    }
}
template <int R>
__device__ __forceinline__ void st_run(float *f, const XTask &T, const float2 (&v)[R]) {
#pragma unroll
    for (int r = 0; r < R; ++r) st2(f, T.at(r), v[r]);
}

// rows of a global spectrum to LDS, and the x spectrum back (rows in grid order)
__device__ __forceinline__ void x_load(const XSArgs &a, const Rows &P, Lanes L, float2 *sh, const float2 *S) {
    const int nt = P.M * P.rows;
    for (int i = L.first; i < nt; i += L.count) {
        const int y = a.dM.div(i), c = i - y * P.M;
        sh[y * P.pitch + pcol(a, c)] = ld_at(S, (uint32_t)i * 8u);
    }
}
__device__ __forceinline__ void x_store(const XSArgs &a, const Rows &P, Lanes L, const float2 *sh, float2 *S) {
    const int nt = P.M * P.rows;
    for (int i = L.first; i < nt; i += L.count) {
        const int y = a.dM.div(i), c = i - y * P.M;
        st_at(S, (uint32_t)i * 8u, sh[P.ypos[y] * P.pitch + pcol(a, c)]);
    }
}

// position of grid row y between the y transforms (the digits reversed)
__device__ __forceinline__ int row_position(const StageAxis &A, int y) {
    if (A.np == 1) return y;
    if (A.np == 2) return y / A.r[1] + A.r[0] * (y % A.r[1]);
    const int r2 = y % A.r[2], t = y / A.r[2];
    return t / A.r[1] + A.r[0] * (t % A.r[1] + A.r[1] * r2);
}

template <bool PLANES>
__device__ __forceinline__ Rows rows_begin(const XSArgs &a, float2 *lds, const float *pml_y,
                                           const float *pml_z, int row0) {
    const int M = a.x.g.M, ny = a.rows, nyt = PLANES ? ny : 0;
    float2 *const twx = lds, *const twp = lds + M, *const twy = lds + 2 * M;
    int *const ypos = reinterpret_cast<int *>(twy + nyt);
    float *const qy = reinterpret_cast<float *>(ypos + ny), *const qz = qy + ny;
    Rows P{lds + xs_table_slots(M, nyt, ny), twx, twp, twy, ypos, qy, qz, M, ny, a.pitch,
           min(ny, a.x.g.rows - row0)};
    stage_table(twx, a.x.t.tw_x, M);
    stage_table(twp, a.x.t.tw_post, M);
    if (PLANES) stage_table(twy, a.x.t.tw_y, ny);
    for (int y = threadIdx.x; y < P.rows; y += blockDim.x) {
        ypos[y] = PLANES ? row_position(a.ay, y) : y;
        const int row = row0 + y, iz = row / a.x.g.ny;
        qy[y] = pml_y[row - iz * a.x.g.ny];
        qz[y] = pml_z[iz];
    }
    return P;          // (the first barrier is that of to_points)
}

// f(e, ok) over the entries of the CSR list of the block's rows, kPoints to a thread and
// round: entries e[k], those without ok[k] a repeated one that is not to be stored.  The
// entries of neighbouring rows follow each other and name their grid point, so the threads
// share them out whatever the rows hold, and a round's loads are in flight together: a
// plane's points may all be the work of one block, which waits for memory at each step.
// us of the pressure pass, a wavefront a row and one point a lane, and now (beside them
// the engine and its y pass, which spread a plane's points over many blocks): 42 sensors
// in one plane of 64^3 21.5 -> 15.4 (18), at all of its points 25.1 -> 20.4 (20), of 16 x
// 256 57 -> 22 (39); velocity with force sources at half the points of a plane of 16 x 256
// 41 -> 20 (40)
constexpr int kPoints = 4;
template <class F>
__device__ __forceinline__ void for_points(const int *row_ptr, int row0, int ny, F f) {
    const int end = row_ptr[row0 + ny];
    for (int e0 = row_ptr[row0] + threadIdx.x; e0 < end; e0 += kPoints * blockDim.x) {
        int e[kPoints];
        bool ok[kPoints];
#pragma unroll
        for (int k = 0; k < kPoints; ++k) {
            const int i = e0 + k * (int)blockDim.x;
            ok[k] = i < end;
            e[k] = ok[k] ? i : e0;
        }
        f(e, ok);
    }
}
// a source's values at a round's entries, and where
__device__ __forceinline__ void source_values(const SourceDev &src, const int (&e)[kPoints], int (&at)[kPoints],
                                              float (&v)[kPoints]) {
    int el[kPoints];
#pragma unroll
    for (int k = 0; k < kPoints; ++k) {
        at[k] = src.pos[e[k]];
        el[k] = src.elem[e[k]];
        v[k] = src.coef[e[k]];
    }
#pragma unroll
    for (int k = 0; k < kPoints; ++k) v[k] *= src.drive[el[k]];
}
// the values of f at a round's entries of the sensor, and their slots
__device__ __forceinline__ void sensor_values(const SensorDev &s, const float *f, const int (&e)[kPoints],
                                              int (&id)[kPoints], float (&v)[kPoints]) {
    int at[kPoints];
#pragma unroll
    for (int k = 0; k < kPoints; ++k) {
        at[k] = s.pos[e[k]];
        id[k] = s.sid[e[k]];
    }
#pragma unroll
    for (int k = 0; k < kPoints; ++k) v[k] = f[at[k]];
}
// dst[i] = f(dst[i], k) for the entries that count
template <class T, class F>
__device__ __forceinline__ void update_points(T *dst, const int (&id)[kPoints], const bool (&ok)[kPoints], F f) {
    T o[kPoints];
#pragma unroll
    for (int k = 0; k < kPoints; ++k) o[k] = dst[id[k]];
#pragma unroll
    for (int k = 0; k < kPoints; ++k)
        if (ok[k]) dst[id[k]] = f(o[k], k);
}
__device__ __forceinline__ bool rows_have_points(const int *row_ptr, int row0, int ny) {
    return row_ptr && row_ptr[row0 + ny] > row_ptr[row0];
}

// ---- point-wise pieces ------------------------------------------------------------

// sensors at every grid point, non-finite check
struct AllPoints {
    const XSArgs &a;
    int step;
    bool rec;
    template <int R>
    __device__ __forceinline__ void run(const XTask &T, const float2 (&p)[R]) const {
        const SensorDev &s = a.x.sen;
        bool bad = false;
#pragma unroll
        for (int r = 0; r < R; ++r) bad |= !(__builtin_isfinite(p[r].x) && __builtin_isfinite(p[r].y));
        if (bad) atomicMin(a.x.cnt.nonfinite, step);
        if (!rec || !s.all_points) return;
        if (s.p_max) {
            float2 o[R];
#pragma unroll
            for (int r = 0; r < R; ++r) o[r] = ld2(s.p_max, T.at(r));
#pragma unroll
            for (int r = 0; r < R; ++r)
                st2(s.p_max, T.at(r), make_float2(fmaxf(o[r].x, p[r].x), fmaxf(o[r].y, p[r].y)));
        }
        if (s.p_sum2) {
            float2 o[R];
#pragma unroll
            for (int r = 0; r < R; ++r) o[r] = ld2(s.p_sum2, T.at(r));
#pragma unroll
            for (int r = 0; r < R; ++r)
                st2(s.p_sum2, T.at(r), make_float2(o[r].x + p[r].x * p[r].x, o[r].y + p[r].y * p[r].y));
        }
        if (s.p_min) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float2 o = ld2(s.p_min, T.at(r));
                st2(s.p_min, T.at(r), make_float2(fminf(o.x, p[r].x), fminf(o.y, p[r].y)));
            }
        }
        const size_t n = (size_t)a.x.g.nx * a.x.g.rows;
        for (int h = 0; h < s.n_harm && s.harm; ++h) {
            const float c = s.hw[2 * h], sn = s.hw[2 * h + 1];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const XPos e = T.at(r);
                float4 *acc = reinterpret_cast<float4 *>(s.harm + 2 * ((size_t)h * n + e.u + e.l / 4u));
                const float4 o = *acc;
                *acc = make_float4(o.x + p[r].x * c, o.y - p[r].x * sn, o.z + p[r].y * c, o.w - p[r].y * sn);
            }
        }
    }
};

// What a block's rows hold of pressure sources and mask sensors (block-uniform).  Both
// work on a pressure in memory; only a source changes it, so that its forward transform
// waits for a second sweep.  (A second sweep for sensors too, and a wavefront a row in
// for_points: 64^3 water with point sources and sensors 93 us a step, engines 90, now 76)
struct PressurePoints {
    bool source = false, any = false;
    PressurePoints() = default;
    __device__ __forceinline__ PressurePoints(const XArgs &x, int row0, int ny)
        : source(x.src.kind == KW_SOURCE_PRESSURE && rows_have_points(x.src.row_ptr, row0, ny)),
          any(source || (!x.sen.all_points && rows_have_points(x.sen.row_ptr, row0, ny))) {}
};
// the sources and sensors, on a pressure written to p
__device__ __forceinline__ void pressure_points(const XSArgs &a, const Rows &P, const PressurePoints &pts, float *p,
                                                      int row0, int step, bool rec) {
    const XArgs &x = a.x;
    const int ny = P.rows;
    __syncthreads();
    if (pts.source) {
        for_points(x.src.row_ptr, row0, ny, [&](const int (&e)[kPoints], const bool (&ok)[kPoints]) __attribute__((always_inline)) {
            int at[kPoints];
            float v[kPoints];
            source_values(x.src, e, at, v);
            // (a drive of NaN leaves the pressure as it is, as in finish_pressure)
#pragma unroll
            for (int k = 0; k < kPoints; ++k)
                if (ok[k] && v[k] == v[k]) p[at[k]] = v[k];
        });
        __syncthreads();
    }
    const SensorDev &s = x.sen;
    if (rec && !s.all_points && rows_have_points(s.row_ptr, row0, ny)) {
        const int slot = step - s.record_start;
        for_points(s.row_ptr, row0, ny, [&](const int (&e)[kPoints], const bool (&ok)[kPoints]) __attribute__((always_inline)) {
            int id[kPoints];
            float pv[kPoints];
            sensor_values(s, p, e, id, pv);
            if (s.series && slot < s.capacity) {
                float *const row = s.series + (size_t)slot * s.n_points;
#pragma unroll
                for (int k = 0; k < kPoints; ++k)
                    if (ok[k]) row[id[k]] = pv[k];
            }
            if (s.p_max) update_points(s.p_max, id, ok, [&](float o, int k) { return fmaxf(o, pv[k]); });
            if (s.p_min) update_points(s.p_min, id, ok, [&](float o, int k) { return fminf(o, pv[k]); });
            if (s.p_sum2) update_points(s.p_sum2, id, ok, [&](float o, int k) { return o + pv[k] * pv[k]; });
            for (int h = 0; h < s.n_harm; ++h) {
                const float c = s.hw[2 * h], sn = s.hw[2 * h + 1];
                update_points(reinterpret_cast<float2 *>(s.harm) + (size_t)h * s.n_points, id, ok,
                              [&](float2 o, int k) { return make_float2(o.x + pv[k] * c, o.y - pv[k] * sn); });
            }
        });
    }
}

// ---- kernels ---------------------------------------------------------------------

// radices of the x stages but the last (which hold the update's values), and of the
// last one (which holds two butterflies); those of the y stages are in staged.h
constexpr RadixSet kPow2M = radix_bit(1) | radix_bit(2) | radix_bit(4) | radix_bit(8);
constexpr RadixSet kPow2P = radix_bit(2) | radix_bit(4) | radix_bit(8);
constexpr RadixSet kAnyM = kPow2M | radix_bit(3) | radix_bit(5) | radix_bit(6);
constexpr RadixSet kAnyP = kPow2P | radix_bit(3) | radix_bit(5) | radix_bit(6) | radix_bit(9) |
                           radix_bit(10) | radix_bit(12);

#define KW_XS_TEMPLATE template <RadixSet RSY, RadixSet RSM, RadixSet RSP, bool PLANES
// (a density plane block takes up to 168 registers: at 128 it spilled 200 bytes a thread)
#define KW_XS_BOUNDS(PLANE_THREADS, WAVES) __launch_bounds__(PLANES ? PLANE_THREADS : 256, PLANES ? 1 : WAVES)
#define KW_XS_BEGIN(PY, PZ)                                                    \
    extern __shared__ float2 lds_all[];                                        \
    const XArgs &x = a.x;                                                      \
    const int row0 = blockIdx.x * a.rows;                                      \
    const Rows P = rows_begin<PLANES>(a, lds_all, x.t.PY, x.t.PZ, row0);       \
    const size_t soff = (size_t)row0 * x.g.M;   /* of the rows in a spectrum */ \
    const size_t roff = (size_t)row0 * x.g.nx;  /* and in a real field */      \
    (void)soff; (void)roff;

// Spectra of NS fields -> the points before the update, set by set (each step's
// sets between two barriers), and NS sets back to spectra
KW_XS_TEMPLATE, int NS, class Src>
__device__ __forceinline__ void to_points(const XSArgs &a, const Rows &P, Src src) {
    constexpr int ns = NS;
    for_sets<PLANES, NS>(ns, [&](int s, Lanes L) __attribute__((always_inline)) {
        if constexpr (PLANES) y_load_inv<RSY>(a, P, L, P.set(s), src(s));
        else x_load(a, P, L, P.set(s), src(s));
    });
    __syncthreads();
    if constexpr (PLANES) {
#pragma unroll 1
        for (int p = a.ay.np - 2; p >= 0; --p) {
            for_sets<PLANES, NS>(ns, [&](int s, Lanes L) __attribute__((always_inline)) { y_stage<RSY, true>(a, P, L, P.set(s), p); });
            __syncthreads();
        }
    }
    for_sets<PLANES, NS>(ns, [&](int s, Lanes L) __attribute__((always_inline)) { x_pair<RSP, true>(a, P, L, P.set(s)); });
    __syncthreads();
    if (a.ax.np == 3) {
        for_sets<PLANES, NS>(ns, [&](int s, Lanes L) __attribute__((always_inline)) { x_stage1<RSM, true>(a, P, L, P.set(s)); });
        __syncthreads();
    }
}
// SPECTRUM_Y: the y transform too (planes)
KW_XS_TEMPLATE, bool SPECTRUM_Y, int NS, class Dst>
__device__ __forceinline__ void to_spectra(const XSArgs &a, const Rows &P, int ns, Dst dst) {
    if (a.ax.np == 3) {
        for_sets<PLANES, NS>(ns, [&](int s, Lanes L) __attribute__((always_inline)) { x_stage1<RSM, false>(a, P, L, P.set(s)); });
        __syncthreads();
    }
    for_sets<PLANES, NS>(ns, [&](int s, Lanes L) __attribute__((always_inline)) { x_pair<RSP, false>(a, P, L, P.set(s)); });
    __syncthreads();
    if constexpr (PLANES && SPECTRUM_Y) {
#pragma unroll 1
        for (int p = 0; p < a.ay.np - 1; ++p) {
            for_sets<PLANES, NS>(ns, [&](int s, Lanes L) __attribute__((always_inline)) { y_stage<RSY, false>(a, P, L, P.set(s), p); });
            __syncthreads();
        }
        for_sets<PLANES, NS>(ns, [&](int s, Lanes L) __attribute__((always_inline)) { y_store<RSY>(a, P, L, P.set(s), dst(s)); });
        __syncthreads();
        for_sets<PLANES, NS>(ns, [&](int s, Lanes L) __attribute__((always_inline)) { y_store_col0(P, L, P.set(s), dst(s)); });
    } else {
        for_sets<PLANES, NS>(ns, [&](int s, Lanes L) __attribute__((always_inline)) { x_store(a, P, L, P.set(s), dst(s)); });
    }
}

// Eq. (4b), u <- q (q u - dt/rho0 dp); blockIdx.y: the velocity component.
// POINTS: force sources or a velocity series, handled on the stored u between
// the two transforms (the second, from u, only in blocks with force points)
KW_XS_TEMPLATE, bool POINTS>
__global__ void KW_XS_BOUNDS(1024, 4) kw_xvel_s(XSArgs a) {
    KW_XS_BEGIN(pml_sy, pml_sz)
    const int xi = blockIdx.y;
    to_points<RSY, RSM, RSP, PLANES, 1>(a, P, [&](int) __attribute__((always_inline)) { return pick3(x.Sin, xi) + soff; });
    float *const u = pick3(x.fld, xi);
    const Coef dtr = xi == 0 ? x.m.dtr[0] : xi == 1 ? x.m.dtr[1] : x.m.dtr[2];
    const float *const q_rows = xi == 1 ? P.qy : P.qz;
    const bool force = POINTS && x.src.kind == KW_SOURCE_FORCE && xi == x.src.axis &&
                       rows_have_points(x.src.row_ptr, row0, P.rows);        // block-uniform
    x_middle<RSM>(a, P, roff, [&](auto RC, const XTask &T, int off, int j) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        float2 u0[R], d[R], v[R];
        ld_run<R>(u, T, u0);
        ld_run<R>(dtr, T, d);
        run_inverse<R>(P, P.sh + off, j, v);
        const float q1 = q_rows[T.y];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float2 q = xi == 0 ? *reinterpret_cast<const float2 *>(x.t.pml_sx + T.x + 2 * r * T.S0)
                                     : make_float2(q1, q1);
            v[r].x = q.x * (q.x * u0[r].x - d[r].x * v[r].x);
            v[r].y = q.y * (q.y * u0[r].y - d[r].y * v[r].y);
        }
        st_run<R>(u, T, v);
        if (!force) run_forward<R>(P, P.sh + off, j, v);
    });
    if constexpr (POINTS) {
        if (force) {
            for_points(x.src.row_ptr, row0, P.rows, [&](const int (&e)[kPoints], const bool (&ok)[kPoints]) __attribute__((always_inline)) {
                int at[kPoints];
                float v[kPoints];
                source_values(x.src, e, at, v);
                update_points(u, at, ok, [&](float o, int k) { return o + v[k]; });
            });
            __syncthreads();
        }
        // u^(n+1/2) is recorded with p^(n+1): step counter n + 1, already advanced
        const int step = *x.cnt.step, slot = step - x.sen.record_start;
        if (x.sen.u_series && step >= x.sen.record_start && slot < x.sen.capacity)
            for_points(x.sen.row_ptr, row0, P.rows, [&](const int (&e)[kPoints], const bool (&ok)[kPoints]) __attribute__((always_inline)) {
                int id[kPoints];
                float v[kPoints];
                sensor_values(x.sen, u, e, id, v);
                float *const series = x.sen.u_series + ((size_t)slot * 3 + xi) * x.sen.n_points;
#pragma unroll
                for (int k = 0; k < kPoints; ++k)
                    if (ok[k]) series[id[k]] = v[k];
            });
        if (force) {
            x_middle<RSM>(a, P, roff, [&](auto RC, const XTask &T, int off, int j) __attribute__((always_inline)) {
                constexpr int R = decltype(RC)::value;
                float2 v[R];
                ld_run<R>(u, T, v);
                run_forward<R>(P, P.sh + off, j, v);
            });
        }
    }
    to_spectra<RSY, RSM, RSP, PLANES, true, 1>(a, P, 1, [&](int) __attribute__((always_inline)) { return pick3(x.Sout, xi) + soff; });
}

// p = c0^2 rho + nl rho^2 on a task's points (Eq. (6) without absorption)
template <int R>
__device__ __forceinline__ void lossless_eos(const Medium &m, const XTask &T, const float2 (&q)[R], float2 (&p)[R]) {
    ld_run<R>(m.c0sq, T, p);
#pragma unroll
    for (int r = 0; r < R; ++r) p[r] = make_float2(p[r].x * q[r].x, p[r].y * q[r].y);
    if (m.nonlinear) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float2 nl = coef2_at(m.nl, T.at(r));
            p[r].x += nl.x * q[r].x * q[r].x;
            p[r].y += nl.y * q[r].y * q[r].y;
        }
    }
}

// The sums rho of a task's points on: stored and transformed (ABS), or to the pressure,
// which is stored for point sensors and sources and whose transform starts unless a
// source comes first
template <bool ABS, int R>
__device__ __forceinline__ void den_finish(const XSArgs &a, const Rows &P, float2 *out_rho, const XTask &T,
                                           int off, int j, int step, bool rec, const PressurePoints &pts,
                                           float2 (&sr)[R]) {
    if constexpr (ABS) {
        st_run<R>(a.x.rho_total, T, sr);
        run_forward<R>(P, out_rho + off, j, sr);
    } else {
        float2 p[R];
        lossless_eos<R>(a.x.m, T, sr, p);
        if (pts.any) st_run<R>(a.scr, T, p);
        if (!pts.source) {
            AllPoints{a, step, rec}.template run<R>(T, p);
            run_forward<R>(P, P.sh + off, j, p);
        }
    }
}

// Density: Eq. (4d) for the three components of the block's rows, their sums kept in
// registers, then (ABS) the spectra of rho0 sum du (unless the z pass forms it)
// and rho, or the equation of state and the spectrum of p.  Rows with mass source
// points add them to the stored components between the two transforms.
KW_XS_TEMPLATE, bool ABS>
__global__ void KW_XS_BOUNDS(768, 3) kw_xden_s(XSArgs a) {
    KW_XS_BEGIN(pml_y, pml_z)
    to_points<RSY, RSM, RSP, PLANES, 3>(a, P, [&](int g) __attribute__((always_inline)) { return pick3(x.Sin, g) + soff; });
    const bool sumd = ABS && !x.rho0_sum_in_z;
    const bool src = x.src.kind == KW_SOURCE_MASS && rows_have_points(x.src.row_ptr, row0, P.rows);
    const int step = *x.cnt.step;
    const bool rec = step >= x.sen.record_start;
    PressurePoints pts;
    if constexpr (!ABS) pts = PressurePoints(x, row0, P.rows);
    float2 *const out_rho = P.set(sumd ? 1 : 0);
    x_middle<RSM>(a, P, roff, [&](auto RC, const XTask &T, int off, int j) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        float2 r0[R], sr[R], sd[ABS ? R : 1];
        ld_run<R>(x.m.rho0, T, r0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            sr[r] = make_float2(0.0f, 0.0f);
            if constexpr (ABS) sd[r] = make_float2(0.0f, 0.0f);
        }
        const float dt = x.g.dt;
#pragma unroll 1
        for (int g = 0; g < 3; ++g) {
            float *const rho = pick3(x.fld, g);
            const float q1 = (g == 1 ? P.qy : P.qz)[T.y];
            float2 old[R], v[R];
            ld_run<R>(rho, T, old);
            run_inverse<R>(P, P.set(g) + off, j, v);
            if (x.rec_d[0]) st_run<R>(pick3(x.rec_d, g), T, v);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float2 q = g == 0 ? *reinterpret_cast<const float2 *>(x.t.pml_x + T.x + 2 * r * T.S0)
                                        : make_float2(q1, q1);
                const float2 d = v[r];
                float2 nw;
                nw.x = q.x * (q.x * old[r].x - dt * r0[r].x * d.x);
                nw.y = q.y * (q.y * old[r].y - dt * r0[r].y * d.y);
                if (x.m.nonlinear) {
                    // (the hardware reciprocal of 1 + O(dt du), as in kw_xden)
                    nw.x *= __builtin_amdgcn_rcpf(1.0f + 2.0f * dt * d.x);
                    nw.y *= __builtin_amdgcn_rcpf(1.0f + 2.0f * dt * d.y);
                }
                sr[r] = c_add(sr[r], nw);
                if constexpr (ABS) sd[r] = c_add(sd[r], d);
                v[r] = nw;
            }
            st_run<R>(rho, T, v);
            if (x.rec_d[0]) st_run<R>(pick3(x.rec_rho, g), T, v);
        }
        // (the runs of all sets are read: set 0 takes the first output's)
        if constexpr (ABS) {
            if (sumd) {
#pragma unroll
                for (int r = 0; r < R; ++r) sd[r] = make_float2(r0[r].x * sd[r].x, r0[r].y * sd[r].y);
                run_forward<R>(P, P.sh + off, j, sd);
            }
        }
        if (!src) den_finish<ABS, R>(a, P, out_rho, T, off, j, step, rec, pts, sr);
    });
    if (src) {                                               // block-uniform
        // dt M added to each component at the source points, then rho from the
        // components
        for_points(x.src.row_ptr, row0, P.rows, [&](const int (&e)[kPoints], const bool (&ok)[kPoints]) __attribute__((always_inline)) {
            int at[kPoints];
            float v[kPoints];
            source_values(x.src, e, at, v);
#pragma unroll
            for (int g = 0; g < 3; ++g) {
                float *const rec = x.rec_d[0] ? pick3(x.rec_rho, g) : nullptr;
                update_points(pick3(x.fld, g), at, ok, [&](float o, int k) {
                    if (rec) rec[at[k]] = o + v[k];
                    return o + v[k];
                });
            }
        });
        __syncthreads();
        x_middle<RSM>(a, P, roff, [&](auto RC, const XTask &T, int off, int j) __attribute__((always_inline)) {
            constexpr int R = decltype(RC)::value;
            float2 sr[R], w1[R], w2[R];
            ld_run<R>(x.fld[0], T, sr);
            ld_run<R>(x.fld[1], T, w1);
            ld_run<R>(x.fld[2], T, w2);
#pragma unroll
            for (int r = 0; r < R; ++r) sr[r] = c_add(c_add(sr[r], w1[r]), w2[r]);
            den_finish<ABS, R>(a, P, out_rho, T, off, j, step, rec, pts, sr);
        });
    }
    if constexpr (ABS) {
        to_spectra<RSY, RSM, RSP, PLANES, true, 0>(a, P, sumd ? 2 : 1, [&](int s) __attribute__((always_inline)) {
            return (sumd && s == 0 ? x.Sout[0] : x.Sout[1]) + soff;
        });
    } else {
        if (pts.any) pressure_points(a, P, pts, a.scr, row0, step, rec);
        if (pts.source) {
            x_middle<RSM>(a, P, roff, [&](auto RC, const XTask &T, int off, int j) __attribute__((always_inline)) {
                constexpr int R = decltype(RC)::value;
                float2 p[R];
                ld_run<R>(a.scr, T, p);
                AllPoints{a, step, rec}.template run<R>(T, p);
                run_forward<R>(P, P.sh + off, j, p);
            });
        }
        to_spectra<RSY, RSM, RSP, PLANES, false, 1>(a, P, 1, [&](int) __attribute__((always_inline)) { return x.Sout[0] + soff; });
    }
}

// Equation of state of absorbing media (Eq. (6)): p = c0^2 rho + nl rho^2 + ta a +
// tb b (MERGED: one spectrum holds both terms), sensors, x spectrum of p.
// POINTS: mask sensors or a pressure source
KW_XS_TEMPLATE, bool MERGED, bool POINTS>
__global__ void KW_XS_BOUNDS(1024, 4) kw_xeos_s(XSArgs a) {
    KW_XS_BEGIN(pml_y, pml_z)
    to_points<RSY, RSM, RSP, PLANES, MERGED ? 1 : 2>(a, P, [&](int s) __attribute__((always_inline)) { return (s ? x.Sin[1] : x.Sin[0]) + soff; });
    const int step = *x.cnt.step;
    const bool rec = step >= x.sen.record_start;
    PressurePoints pts;
    if constexpr (POINTS) pts = PressurePoints(x, row0, P.rows);
    x_middle<RSM>(a, P, roff, [&](auto RC, const XTask &T, int off, int j) __attribute__((always_inline)) {
        constexpr int R = decltype(RC)::value;
        float2 p[R], v[R], c[MERGED ? 1 : R];
        ld_run<R>(x.rho_total, T, v);
        lossless_eos<R>(x.m, T, v, p);
        if constexpr (!MERGED) ld_run<R>(x.m.ta, T, c);
        run_inverse<R>(P, P.sh + off, j, v);
        if constexpr (MERGED) {
#pragma unroll
            for (int r = 0; r < R; ++r) p[r] = c_add(p[r], v[r]);
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                p[r].x += c[r].x * v[r].x;
                p[r].y += c[r].y * v[r].y;
            }
            ld_run<R>(x.m.tb, T, c);
            run_inverse<R>(P, P.set(1) + off, j, v);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                p[r].x += c[r].x * v[r].x;
                p[r].y += c[r].y * v[r].y;
            }
        }
        if (pts.any) st_run<R>(a.scr, T, p);
        if (!pts.source) {
            AllPoints{a, step, rec}.template run<R>(T, p);
            run_forward<R>(P, P.sh + off, j, p);
        }
    });
    if constexpr (POINTS) {
        if (pts.any) pressure_points(a, P, pts, a.scr, row0, step, rec);
        if (pts.source) {
            x_middle<RSM>(a, P, roff, [&](auto RC, const XTask &T, int off, int j) __attribute__((always_inline)) {
                constexpr int R = decltype(RC)::value;
                float2 p[R];
                ld_run<R>(a.scr, T, p);
                AllPoints{a, step, rec}.template run<R>(T, p);
                run_forward<R>(P, P.sh + off, j, p);
            });
        }
    }
    to_spectra<RSY, RSM, RSP, PLANES, false, 1>(a, P, 1, [&](int) __attribute__((always_inline)) { return x.Sout[0] + soff; });
}

}  // namespace

// the launches of xstaged.h for the radix sets of one file
template <RadixSet RSY, RadixSet RSM, RadixSet RSP>
struct XStagedLaunch {
    struct Shape {
        XSArgs a;
        dim3 grid, block;
        size_t lds;
    };
    static Shape shape(const LaunchCfg &c, const XArgs &x, int pass, int sets, float *scr) {
        const bool planes = c.planes >> pass & 1;
        const GridDev &g = x.g;
        Shape q{};
        XSArgs &a = q.a;
        a.x = x;
        a.ax = c.xs_axis;
        a.ay = c.planes_y;
        a.rows = planes ? g.ny : c.xs_rows[pass];
        a.dM = FastDiv(g.M);
        a.drows = FastDiv(a.rows);
        a.dS0 = FastDiv(g.M / c.xs_axis.r[0]);
        a.pitch = c.xs_pitch;
        a.pad = c.xs_pad;
        a.scr = scr;
        q.grid = dim3((g.rows + a.rows - 1) / a.rows);
        q.block = dim3(planes ? c.planes_threads[pass] : 256);
        q.lds = xs_lds_bytes(g.M, planes ? g.ny : 0, a.rows, sets, c.xs_pitch);
        return q;
    }
#define KW_XS_LAUNCH(KERNEL, ...)                                                                  \
    do {                                                                                           \
        if (planes) hipLaunchKernelGGL((KERNEL<RSY, RSM, RSP, true, __VA_ARGS__>), q.grid, q.block, q.lds, s, q.a); \
        else hipLaunchKernelGGL((KERNEL<RSY, RSM, RSP, false, __VA_ARGS__>), q.grid, q.block, q.lds, s, q.a);       \
    } while (0)
    static hipError_t vel(hipStream_t s, const LaunchCfg &c, const XArgs &x, bool points) {
        Shape q = shape(c, x, XS_VEL, 1, nullptr);
        const bool planes = c.planes >> XS_VEL & 1;
        q.grid.y = 3;
        if (points) KW_XS_LAUNCH(kw_xvel_s, true);
        else KW_XS_LAUNCH(kw_xvel_s, false);
        return hipGetLastError();
    }
    static hipError_t den(hipStream_t s, const LaunchCfg &c, const XArgs &x, float *scr) {
        const Shape q = shape(c, x, XS_DEN, 3, scr);
        const bool planes = c.planes >> XS_DEN & 1;
        if (x.m.absorbing) KW_XS_LAUNCH(kw_xden_s, true);
        else KW_XS_LAUNCH(kw_xden_s, false);
        return hipGetLastError();
    }
    static hipError_t eos(hipStream_t s, const LaunchCfg &c, const XArgs &x, float *scr,
                          bool points, bool merged) {
        const Shape q = shape(c, x, XS_EOS, merged ? 1 : 2, scr);
        const bool planes = c.planes >> XS_EOS & 1;
        if (merged && points) KW_XS_LAUNCH(kw_xeos_s, true, true);
        else if (merged) KW_XS_LAUNCH(kw_xeos_s, true, false);
        else if (points) KW_XS_LAUNCH(kw_xeos_s, false, true);
        else KW_XS_LAUNCH(kw_xeos_s, false, false);
        return hipGetLastError();
    }
#undef KW_XS_LAUNCH
};

}  // namespace kw
