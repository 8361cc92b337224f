// EA with one line per lane (k_EAL): pruned lengths P and g = M / P fixed at compile time, strided lines.
//
// The accumulate commutes with the inverse transform of the samples. With W_q[r] the spectrum that the
// inverse P-point transform of term q takes (r < P; the sum over the g subsequences of HT times their
// P-point transforms), the twiddle of (FFpsi) at the output n0 = P-sample 0 and c' < M is
//   out[c'] = sum_q Tf_q[0] exp(2 pi i q c' / M) sum_r W_q[r] exp(2 pi i r c' (lam / g) / P)
//           = sum_q sum_r Tf_q[0] W_q[r] exp(2 pi i (q + lam r) c' / M),
// so the terms of equal j = q mod g can be added as spectra, H[j][r'] += Tf_q[0] W_q[r], and one
// inverse transform of M points per line (P points over r', g over j) follows at the end instead of
// one P-point transform per term. For r' to be the same slot for every q of a residue, the slot of
// index r must advance with k = (q - j) / g: r = r' + rho0(q), rho0 = -k (lam / g)^-1 mod P, which is a
// modulation of the input by exp(-2 pi i b rho0 / P) and joins the premultiplying phase of (presA).
//
// A workgroup holds 64 lines in LDS, element by element (lane = line: no bank conflicts, no exchange
// between lanes), and has g waves, one per residue j; the terms of a wave run over its residue. Per
// term and subsequence a lane reads its P points, multiplies by the phases (uniform: scalar operands),
// transforms in registers, and adds the product with the term's row of the table (scalar operands
// too) to its P sums. The waves meet once per tile, for the g-point transform over j.
//
// What bounds it: VALU issue. Measured against the forms with a line over several lanes (k_EAW, k_ERG,
// k_EAR), which move every partial sum between lanes and run an inverse transform per term:
// g = 2, P = 32, 50 terms, FP32, 250 x 32768 lines: 36.0 -> 13.1 ms; g = 8, P = 6, 40 terms, FP64, 1600 x 288
// lines: 1057 -> 441 us; g = 8, P = 12, 8 terms, FP64, 8 x 12960 lines: 405 -> 125 us (320 MB, 62 us at the
// copy rate). g = 4, P = 64 (FP32) would need 384 registers for its three sets of P values and ran no
// faster than k_ERG (640 us each), so it is not compiled.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <set>

#include "butterflies.h"
#include "fx_internal.h"

namespace fx {

namespace {

constexpr int kLanes = 64;

// Tables of one axis (build_lane_table): per term the phases of b = 1..P-1 and the rows
// D[n2][r'] = Tf_q[0] HT_q[n2][r' + rho0]; behind the terms the twiddles TW[f][j] of the final transform.
template <typename T, int P, int G>
__global__ __launch_bounds__(kLanes * G) void k_EAL(const C<T>* __restrict__ in, C<T>* __restrict__ out,
                                                    const C<T>* __restrict__ tab, const int* __restrict__ rows,
                                                    int lam, PassGeom g, int accumulate, T* __restrict__ rho) {
    constexpr int M = P * G;
    constexpr int ROW = M + P - 1;
    extern __shared__ __align__(16) unsigned char smem[];
    C<T>* X = (C<T>*)smem;  // [M][64]
    const int lane = threadIdx.x & 63;
    const int j = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // tiles of an XCD are contiguous: neighbouring tiles share memory lines
    const int per = (int)((g.ntiles + 7) >> 3);
    const int tile = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if (tile >= (int)g.ntiles) return;
    const int S = (int)g.S;
    const int nlines = (int)(g.Qin * g.A) * S;
    const int line = min(tile * kLanes + lane, nlines - 1);
    const bool live = tile * kLanes + lane < nlines;
    const int slice = (unsigned)line / (unsigned)S;
    const int64_t base = (int64_t)slice * M * S + (line - slice * S);
    {
        // all loads of a wave issued before the first store
        constexpr int PER = M / G;
        C<T> v[PER];
#pragma unroll
        for (int i = 0; i < PER; ++i) v[i] = in[base + (int64_t)(j + i * G) * S];
#pragma unroll
        for (int i = 0; i < PER; ++i) X[(j + i * G) * kLanes + lane] = v[i];
    }
    __syncthreads();
    C<T> H[P];
#pragma unroll
    for (int r = 0; r < P; ++r) H[r] = mk<T>(0, 0);
    int i0 = (j - g.qb) % G;
    if (i0 < 0) i0 += G;
    for (int i = i0; i < g.qn; i += G) {
        const C<T>* row = tab + (int64_t)(g.qb + i) * ROW;
        C<T> W[P];
#pragma unroll
        for (int r = 0; r < P; ++r) W[r] = mk<T>(0, 0);
#pragma unroll 1
        for (int n2 = 0; n2 < G; ++n2) {
            C<T> v[P];
#pragma unroll
            for (int b = 0; b < P; ++b) v[b] = X[(n2 + G * b) * kLanes + lane];
#pragma unroll
            for (int b = 1; b < P; ++b) v[b] = cmul<T>(v[b], row[b - 1]);
            bfly<T, P, false>(v);
            const C<T>* d = row + P - 1 + n2 * P;
#pragma unroll
            for (int r = 0; r < P; ++r) W[r] = cfma<T>(W[r], d[r], v[r]);
        }
#pragma unroll
        for (int r = 0; r < P; ++r) H[r] = cadd<T>(H[r], W[r]);
    }
    bfly<T, P, true>(H);
    const C<T>* tw = tab + (int64_t)lam * ROW;
#pragma unroll
    for (int f = 0; f < P; ++f) H[f] = cmul<T>(H[f], tw[f * G + j]);
    __syncthreads();
#pragma unroll
    for (int f = 0; f < P; ++f) X[(j * P + f) * kLanes + lane] = H[f];
    __syncthreads();
    for (int f = j; f < P; f += G) {
        C<T> v[G];
#pragma unroll
        for (int i = 0; i < G; ++i) v[i] = X[(i * P + f) * kLanes + lane];
        bfly<T, G, true>(v);
        if (!live) continue;
#pragma unroll
        for (int c = 0; c < G; ++c) {
            const int64_t o = base + (int64_t)rows[f * G + c] * S;
            C<T> z = v[c];
            if (accumulate) z = cadd<T>(z, out[o]);
            out[o] = z;
            if (rho) rho[o] = z.x * z.x + z.y * z.y;
        }
    }
}

template <typename K> hipError_t prep_lds_lane(K kernel, size_t bytes) {
    if (bytes <= 65536) return hipSuccess;
    static std::mutex mu;
    static std::set<const void*> done;
    std::lock_guard<std::mutex> lk(mu);
    if (done.count((const void*)kernel)) return hipSuccess;
    hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       lds_limit_bytes());
    if (e == hipSuccess) done.insert((const void*)kernel);
    return e;
}

template <typename T, int P, int G>
hipError_t launch_eal_pg(const void* in, void* out, const AxisDev& ax, const PassGeom& g, int accumulate, void* rho,
                         hipStream_t st) {
    const size_t lds = (size_t)P * G * kLanes * sizeof(C<T>);
    auto k = k_EAL<T, P, G>;
    hipError_t e = prep_lds_lane(k, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3((unsigned)(((g.ntiles + 7) / 8) * 8)), dim3(kLanes * G), lds, st, (const C<T>*)in,
                       (C<T>*)out, (const C<T>*)ax.LT, ax.LR, ax.lam, g, accumulate, (T*)rho);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_eal_T(const void* in, void* out, const AxisDev& ax, const PassGeom& g, int accumulate, void* rho,
                        hipStream_t st) {
#define FX_EAL(PP, GG) \
    if (ax.P == PP && ax.g == GG) return launch_eal_pg<T, PP, GG>(in, out, ax, g, accumulate, rho, st);
    FX_EAL(2, 8) FX_EAL(3, 8) FX_EAL(4, 8) FX_EAL(6, 8) FX_EAL(8, 8) FX_EAL(12, 8) FX_EAL(16, 8)
    FX_EAL(4, 4) FX_EAL(6, 4) FX_EAL(8, 4) FX_EAL(12, 4) FX_EAL(16, 4)
    FX_EAL(8, 2) FX_EAL(12, 2) FX_EAL(16, 2)
    if constexpr (sizeof(T) == 4) { FX_EAL(32, 2) FX_EAL(32, 4) }
#undef FX_EAL
    return hipErrorInvalidValue;
}

}  // namespace

bool eal_applicable(bool dbl, int M, int g) {
    if (g < 1 || M % g) return false;
    const int P = M / g;
    if ((size_t)M * kLanes * (dbl ? 16 : 8) > (size_t)lds_limit_bytes()) return false;
    auto in = [&](std::initializer_list<int> l) { return std::find(l.begin(), l.end(), P) != l.end(); };
    switch (g) {
        case 8: return in({2, 3, 4, 6, 8, 12, 16});
        case 4: return in({4, 6, 8, 12, 16}) || (!dbl && P == 32);
        case 2: return in({8, 12, 16}) || (!dbl && P == 32);
        default: return false;
    }
}

int eal_tile_lines() { return kLanes; }

hipError_t launch_pass_eal(bool dbl, const void* in, void* out, const AxisDev& ax, const PassGeom& g, int accumulate,
                           void* rho, hipStream_t st) {
    if (!ax.LT || !ax.LR || !eal_applicable(dbl, ax.M, ax.g) || g.TS != kLanes ||
        g.ntiles != (g.Qin * g.A * g.S + kLanes - 1) / kLanes || g.Qin * g.A * g.S >= (int64_t(1) << 31) - kLanes)
        return hipErrorInvalidValue;
    return dbl ? launch_eal_T<double>(in, out, ax, g, accumulate, rho, st)
               : launch_eal_T<float>(in, out, ax, g, accumulate, rho, st);
}

}  // namespace fx
