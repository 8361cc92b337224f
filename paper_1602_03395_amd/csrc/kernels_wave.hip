// E of contiguous lines for the pruned length P = 256: a row (one line, one term) in the registers of 16 lanes.
//
// 16 lanes hold a row, 16 points each. A P-point transform is one 16-point butterfly per lane, the twiddles, one
// exchange through LDS and a second butterfly,
//   V[u + 16 v] = sum_l exp(-2 pi i l v / 16) exp(-2 pi i u l / P) sum_t x[l + 16 t] exp(-2 pi i t u / 16);
// the products with HT add up over the g subsequences in registers, and the inverse transform runs the same
// steps backwards. The lanes of a row are in one wave, so after the line is in LDS nothing waits at a
// barrier, where the folded kernel has three radices and six barriers per step with two waves per SIMD.
//
// What bounds it: latency of the exchange and of the table rows (3 waves per SIMD in FP32, 1 in FP64) for a few
// thousand rows, VALU issue above: 2048 points, g = 8, 40 terms, E + A, FP32, 2560 / 10240 / 40960 rows
// 34 / 104 / 300 -> 32 / 49 / 127 us (the last against the fused folded EA), FP64 54 / 176 / 572 -> 40 / 101 /
// 308 us. Rows straight from global memory (no line in LDS) took 135 us for 20480 rows in FP32: each of the 8 passes
// over a line reads all its memory lines again. The same form for P = 512 in FP32 (one wave per SIMD) gained from
// 10240 rows of g = 8 on only (178 -> 142 us; g = 4, 1280 rows 27 -> 32, 20480 rows 165 -> 194), for P = 128 in FP32 not
// at all (g = 8, 2048 rows 16 -> 20 us).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <set>

#include "butterflies.h"
#include "fx_internal.h"

namespace fx {

namespace {

constexpr int kR = 16, kP = kR * kR;  // lanes and points per lane of a row
constexpr int kLP = kR + 1;           // odd: lanes kLP elements apart share no bank
constexpr int kWaves = 4, kRows = kWaves * (64 / kR);

// Table rows (build_et): the phases TA_q[g b], b = 1..P-1, then HT_q[n2][r]. roots: exp(-2 pi i k / M).
// A workgroup has one line in LDS, subsequence by subsequence, and takes fqpw of its terms, kRows at a time.
template <typename T>
__global__ __launch_bounds__(64 * kWaves) void k_EW(const C<T>* __restrict__ in, C<T>* __restrict__ out,
                                                    const C<T>* __restrict__ tab, const C<T>* __restrict__ roots,
                                                    int gg, PassGeom g) {
    extern __shared__ __align__(16) unsigned char smem[];
    C<T>* tw = (C<T>*)smem;               // exp(-2 pi i u l / P) at u kLP + l
    C<T>* xbuf = tw + kR * kLP;           // exchange buffers of the rows
    C<T>* raw = xbuf + kRows * kR * kLP;  // the line: point g n1 + n2 at n2 (P + 1) + n1
    const int M = kP * gg;
    const int nchunk = (g.qn + g.fqpw - 1) / g.fqpw;
    const int line = (unsigned)blockIdx.x / (unsigned)nchunk;
    const int chunk = (int)blockIdx.x - line * nchunk;
    const C<T>* x = in + (int64_t)line * M;
    for (int e0 = threadIdx.x; e0 < M; e0 += 4 * blockDim.x) {
        C<T> v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = x[min(e0 + k * (int)blockDim.x, M - 1)];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int e = e0 + k * (int)blockDim.x;
            const int n1 = (unsigned)e / (unsigned)gg;
            if (e < M) raw[(e - n1 * gg) * (kP + 1) + n1] = v[k];
        }
    }
    for (int e = threadIdx.x; e < kP; e += blockDim.x) {
        const int u = e / kR, l = e % kR;
        tw[u * kLP + l] = roots[u * l * gg];
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int l = lane % kR, r = w * (64 / kR) + lane / kR;
    C<T>* X = xbuf + r * (kR * kLP);
    const int qi = (unsigned)line / (unsigned)g.A;
    const int i1 = min(g.qn, (chunk + 1) * g.fqpw);
    for (int i0 = chunk * g.fqpw; i0 < i1; i0 += kRows) {
        const int i = min(i0 + r, i1 - 1);
        const C<T>* ta = tab + (int64_t)(g.qb + i) * (M + kP - 1);
        const C<T>* ht = ta + kP - 1 + l;
        C<T> ph[kR], W[kR], v[kR];
#pragma unroll
        for (int t = 0; t < kR; ++t) {
            ph[t] = ta[max(l + kR * t - 1, 0)];
            W[t] = mk<T>(0, 0);
        }
        if (l == 0) ph[0] = mk<T>(1, 0);
#pragma unroll 1
        for (int n2 = 0; n2 < gg; ++n2) {
            C<T> h[kR];
#pragma unroll
            for (int t = 0; t < kR; ++t) h[t] = ht[n2 * kP + kR * t];
#pragma unroll
            for (int t = 0; t < kR; ++t) v[t] = cmul<T>(raw[n2 * (kP + 1) + l + kR * t], ph[t]);
            bfly<T, kR, false>(v);
#pragma unroll
            for (int u = 1; u < kR; ++u) v[u] = cmul<T>(v[u], tw[u * kLP + l]);
            wave_sync();
#pragma unroll
            for (int u = 0; u < kR; ++u) X[u * kLP + l] = v[u];
            wave_sync();
#pragma unroll
            for (int k = 0; k < kR; ++k) v[k] = X[l * kLP + k];
            bfly<T, kR, false>(v);
#pragma unroll
            for (int k = 0; k < kR; ++k) W[k] = cfma<T>(W[k], h[k], v[k]);
        }
        bfly<T, kR, true>(W);
        wave_sync();
#pragma unroll
        for (int c = 0; c < kR; ++c) X[l * kLP + c] = cmulc<T>(W[c], tw[l * kLP + c]);
        wave_sync();
#pragma unroll
        for (int u = 0; u < kR; ++u) v[u] = X[u * kLP + l];
        wave_sync();
        bfly<T, kR, true>(v);
        if (i0 + r >= i1) continue;
        C<T>* o = out + (((int64_t)qi * g.qn + i) * g.A + (line - qi * (int)g.A)) * kP + l;
#pragma unroll
        for (int d = 0; d < kR; ++d) o[kR * d] = v[d];
    }
}

size_t ew_lds(int gg, size_t c) { return ((size_t)kR * kLP * (1 + kRows) + (size_t)(kP + 1) * gg) * c; }

template <typename K> hipError_t prep_lds_ew(K kernel, size_t bytes) {
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

template <typename T>
hipError_t launch_ew_T(const void* in, void* out, const AxisDev& ax, const PassGeom& g, hipStream_t st) {
    const int64_t blocks = g.Qin * g.A * ((g.qn + g.fqpw - 1) / g.fqpw);
    if (blocks >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    const size_t lds = ew_lds(ax.g, sizeof(C<T>));
    auto k = k_EW<T>;
    hipError_t e = prep_lds_ew(k, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(64 * kWaves), lds, st, (const C<T>*)in, (C<T>*)out,
                       (const C<T>*)ax.ET, (const C<T>*)ax.tw, ax.g, g);
    return hipGetLastError();
}

}  // namespace

bool ew_applicable(bool dbl, int M, int g) {
    return g >= 1 && M % g == 0 && M / g == kP && ew_lds(g, dbl ? 16 : 8) <= (size_t)lds_limit_bytes();
}

// Terms per workgroup: one round of its rows, more where there are six workgroups per CU anyway.
int ew_terms(int64_t lines, int qn, int cus) {
    const int64_t rounds = lines * qn / ((int64_t)6 * cus * kRows);
    return (int)std::min<int64_t>((qn + kRows - 1) / kRows, std::max<int64_t>(1, rounds)) * kRows;
}

// Rows of a workgroup that have a term of their own, of the rounds that qn terms take.
double ew_fill(int qn) { return (double)qn / ((qn + kRows - 1) / kRows * kRows); }

hipError_t launch_pass_ew(bool dbl, const void* in, void* out, const AxisDev& ax, const PassGeom& g, hipStream_t st) {
    if (!ax.ET || !ax.tw || !ew_applicable(dbl, ax.M, ax.g) || g.S != 1 || g.fqpw < 1 ||
        g.Qin * g.A * g.qn >= (int64_t(1) << 31))
        return hipErrorInvalidValue;
    return dbl ? launch_ew_T<double>(in, out, ax, g, st) : launch_ew_T<float>(in, out, ax, g, st);
}

}  // namespace fx
