// In-place staged transforms in LDS, of lengths 2^a 3^b 5^c in up to three stages
// (columns: every length up to 1024 but 625; x rows: see stage_axis).
//
// A transform of n = R0 R1 .. points keeps its natural (frequency) order at
// one end.  Stage p combines the elements lo + w d + w R hi (w = R0 .. R_{p-1},
// d < R = R_p, lo < w): the forward transform runs the stages from the first to
// the last and starts from digit-reversed points, the inverse runs them from
// the last to the first and ends there.  The digit-reversed side is only ever
// held between the stages of one kernel: global memory and the update in the
// middle undo it in their index arithmetic.
//
// In place means one barrier a stage (a butterfly writes what it read), and
// any thread may run any butterfly: tasks are dealt out by a flat index, so all
// threads work in every stage whatever its radix.  (The one-butterfly-a-thread
// engine of fft_dev.h leaves threads idle in the passes of larger radices: 125 =
// 5 25 runs its radix-25 pass on 5 threads of 25.)
#pragma once

#include "kernels_impl.h"

namespace kw {

template <bool INV> struct Dft<1, INV> {
    template <int S, int O, int RM>
    __device__ __forceinline__ static void run(float2 (&)[RM]) {}
};

template <int R> struct IntC { static constexpr int value = R; };

// f(IntC<R>) for the run-time radix R of the set RS
template <RadixSet RS, class F>
__device__ __forceinline__ void with_radix(int R, F f) {
    constexpr int q = 63 - __builtin_clzll(RS);
    if constexpr ((RS & (RS - 1)) == 0) {
        f(IntC<q>{});
    } else {
        if (R == q) f(IntC<q>{});
        else with_radix<(RS & ~radix_bit(q))>(R, f);
    }
}

// element at a byte offset of a table in LDS
__device__ __forceinline__ float2 tw_at(const float2 *tw, int off) {
    return *reinterpret_cast<const float2 *>(reinterpret_cast<const char *>(tw) + off);
}
// v[d] *= W^(ts d) (conjugate: INV), d = 1 .. R-1
template <int R, bool INV>
__device__ __forceinline__ void twiddle(float2 (&v)[R], const float2 *tw, int ts) {
    const int step = ts * 8;
    int o = 0;
#pragma unroll
    for (int d = 1; d < R; ++d) {
        o += step;
        const float2 w = tw_at(tw, o);
        v[d] = INV ? c_mulc(v[d], w) : c_mul(v[d], w);
    }
}

// index that the position digits above stage p stand for: hi = r_{p+1} +
// R_{p+1} r_{p+2} + .. is their position, the index counts the last digit lowest
__device__ __forceinline__ int digit_index(const StageAxis &A, int p, int hi) {
    if (p == A.np - 1) return 0;
    if (p == A.np - 2) return hi;
    const int q2 = A.d1.div(hi);             // hi = r1 + R1 r2
    return q2 + A.r[2] * (hi - q2 * A.r[1]);  // r2 + R2 r1
}

// Column 0 before an inverse y transform: C(ky) = A(ky) + i B(ky) from the
// unpacked rows (see col0_type), with A(-ky) = conj A(ky); the rows of A and B
// for row ky, whether they are conjugated, and whether the row is C itself
struct Col0Rows {
    int a, b;
    bool neg, self;
};
__device__ __forceinline__ Col0Rows col0_rows(int ky, int ny) {
    const int h = (ny - 1) / 2;
    const bool self = col0_type(ky, ny) == C0_DOUBLE, neg = ky > h;
    const int j = neg ? ny - ky : ky;
    return Col0Rows{self ? ky : j, self ? ky : ny - 1 - h + j, neg, self};
}
__device__ __forceinline__ float2 col0_join(const Col0Rows &o, float2 A, float2 B) {
    const float s = o.neg ? -1.0f : 1.0f;
    return o.self ? A : make_float2(A.x - s * B.y, s * A.y + B.x);       // A + i B
}

// radices of the kernels built for power-of-two lengths and of the others
constexpr RadixSet kPow2Y = radix_bit(2) | radix_bit(4) | radix_bit(8) | radix_bit(16);
constexpr RadixSet kAnyY = kPow2Y | radix_bit(3) | radix_bit(5) | radix_bit(6) | radix_bit(9) |
                           radix_bit(10) | radix_bit(12) | radix_bit(15);

}  // namespace kw
