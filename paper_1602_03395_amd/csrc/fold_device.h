// Device side of the folded line kernels (any axis length whose pruned length P = M / g has prime
// factors up to 13).
//
// With n = g n1 + n2 and the chirp, the outer g-point transform and the fold collapsed into HT
// (the register form's identity), one term of one line is
//   E_q = IDFT_P( sum_n2 HT_q[n2] . DFT_P( x[g . + n2] TA_q[g .] ) ).
// A workgroup works on rows (one line, one term each). The forward P-point transforms are
// decimation-in-frequency passes in LDS with the radices of FoldPlan, in place: every butterfly
// writes where it read, so a row needs one buffer and a pass one barrier, and the spectrum ends in
// digit-reversed order. Nothing undoes that order: HT is stored in it, and the inverse transform
// is the mirrored decimation in time, which takes it and ends in natural order. The last forward
// stage leaves in each thread the inputs of its own first inverse butterfly, so that stage, the
// product with HT, the sum over the g subsequences and the first inverse stage run in registers.
// P = R0 R1 costs two LDS exchanges per row (M points, then P points), and one of each more per
// further factor.
//
// What bounds it: instruction issue and the latency of a step's barriers, not memory (FP64, 375 points,
// 12 terms, 1500 lines: 56 us, where its 43 MB would take 8 us) except for few terms (FP64, 1080
// points, one term, 9216 lines: 127 us for 318 MB, 62 us at the copy rate). About half of the
// instructions are index arithmetic of the run-time radices; larger radices and full wavefronts in
// every stage (fold_geometry) are what lowers it.
//
// Layout of a row in LDS: subsequence n2 in slot n2 (stride ps); inside a slot, position p at
// p + p / Rl when the last radix Rl is even (the threads of the last stage start Rl elements apart,
// which an even Rl would put on a few banks); all strides of the other stages are multiples of Rl, so
// they stay uniform. Row stride odd.
//
// Table rows (FT): [q][(g + 2) P]: HT_q[n2] in digit-reversed order, then TA_q[g n1], then
// Tf_q[n0(u)]; behind the lam rows the stage twiddles exp(-2 pi i k u / L) as [u - 1][k] per stage.
#pragma once

#include "butterflies.h"

namespace fx {

// One decoded work item of a stage.
struct FoldItem {
    int row;   // row of the tile
    int n2;    // subsequence, or group of subsequences
    int jj;    // butterfly inside the transform
};

// x / d and x mod d for 0 <= x < 2^21, d < 2^13 (host-built reciprocal; the half offset keeps the
// truncation away from the integers by more than the rounding of the product).
__device__ __forceinline__ int fdivu(int x, const FoldDiv& d) {
    return (int)__builtin_fmaf((float)x, d.inv, d.half);
}
__device__ __forceinline__ int fmodu(int x, int q, const FoldDiv& d) { return x - __mul24(q, d.d); }

// Items run over (row / fast, n2, jj, row mod fast), the last fastest: fast = lines of the tile for
// strided lines (the lanes of a wave then walk along the contiguous direction of memory), 1 for
// contiguous ones (the lanes walk along the line).
__device__ __forceinline__ FoldItem fold_item(int idx, int lf, const FoldDiv& dnb, const FoldDiv& dg) {
    FoldItem it;
    const int f = idx & ((1 << lf) - 1);
    const int t = idx >> lf;
    int q = fdivu(t, dnb);
    it.jj = fmodu(t, q, dnb);
    it.n2 = 0;
    if (dg.d > 1) {
        const int rs = fdivu(q, dg);
        it.n2 = fmodu(q, rs, dg);
        q = rs;
    }
    it.row = (q << lf) + f;
    return it;
}

// Offset in a slot of element t = 0 of butterfly jj of stage st, and its k.
__device__ __forceinline__ int fold_at(const FoldStage& st, const FoldPlan& pl, int jj, int& k) {
    const int blk = fdivu(jj, st.m);
    k = fmodu(jj, blk, st.m);
    return __mul24(blk, st.Lp) + k + (pl.pad ? fdivu(k, pl.dRl) : 0);
}

// Calls f.template run<R>() for the runtime radix R of the plan. A kernel holds the radices of one
// class only, since its registers are those of its largest radix: 2..10 in every class, and in the
// stages that hold one set of values also 12, 15, 16 (class 1) or 18, 20, 25 (class 3); class 2 has
// 11, 13 and 14 everywhere.
template <int RC, bool FUSED, typename F> __device__ __forceinline__ void fold_radix(int R, F&& f) {
    switch (R) {
        case 1: if constexpr (FUSED) f.template run<1>(); break;
        case 2: f.template run<2>(); break;
        case 3: f.template run<3>(); break;
        case 4: f.template run<4>(); break;
        case 5: f.template run<5>(); break;
        case 6: f.template run<6>(); break;
        case 7: f.template run<7>(); break;
        case 8: f.template run<8>(); break;
        case 9: f.template run<9>(); break;
        case 10: f.template run<10>(); break;
        default:
            if constexpr (RC == 1 && !FUSED) {
                if (R == 12) f.template run<12>();
                else if (R == 15) f.template run<15>();
                else if (R == 16) f.template run<16>();
            } else if constexpr (RC == 3 && !FUSED) {
                if (R == 18) f.template run<18>();
                else if (R == 20) f.template run<20>();
                else if (R == 25) f.template run<25>();
            } else if constexpr (RC == 2) {
                if (R == 11) f.template run<11>();
                else if (R == 13) f.template run<13>();
                else if (R == 14) f.template run<14>();
            }
            break;
    }
}

// A middle stage of rows x subs transforms, in place.
template <typename T, bool INV> struct FoldMid {
    C<T>* X;
    const C<T>* tw;
    const FoldStage& st;
    const FoldPlan& pl;
    int total, lf;
    const FoldDiv& dsub;
    int rs, ps;
    template <int R> __device__ __forceinline__ void run() {
        const int mp = st.mp, m = st.m.d;
        const C<T>* w = tw + st.tw;
        __syncthreads();
        for (int idx = threadIdx.x; idx < total; idx += blockDim.x) {
            const FoldItem it = fold_item(idx, lf, st.nb, dsub);
            int k;
            C<T>* x = X + it.row * rs + it.n2 * ps + fold_at(st, pl, it.jj, k);
            C<T> v[R];
#pragma unroll
            for (int t = 0; t < R; ++t) v[t] = x[t * mp];
            if constexpr (INV) {
#pragma unroll
                for (int t = 1; t < R; ++t) v[t] = cmulc<T>(v[t], w[(t - 1) * m + k]);
            }
            bfly<T, R, INV>(v);
            if constexpr (!INV) {
#pragma unroll
                for (int t = 1; t < R; ++t) v[t] = cmul<T>(v[t], w[(t - 1) * m + k]);
            }
#pragma unroll
            for (int t = 0; t < R; ++t) x[t * mp] = v[t];
        }
    }
};

}  // namespace fx
