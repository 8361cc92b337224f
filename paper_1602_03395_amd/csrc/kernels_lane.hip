// E, EA and the adjoint of EA with one line per lane: the pruned length P is compiled in (EA: g = M / P
// too), the lines are strided.
//
// The accumulate of EA commutes with the inverse transform of the samples. With W_q[r] the spectrum that
// the inverse P-point transform of term q takes (r < P; the sum over the g subsequences of HT times their
// P-point transforms), the twiddle of (FFpsi) at output c' < M is
//   out[c'] = sum_q Tf_q[0] exp(2 pi i q c' / M) sum_r W_q[r] exp(2 pi i r c' (lam / g) / P)
//           = sum_q sum_r Tf_q[0] W_q[r] exp(2 pi i (q + lam r) c' / M),
// so the terms of equal j = q mod g can be added as spectra, H[j][r'] += Tf_q[0] W_q[r], and one
// inverse transform of M points per line (P points over r', g over j) follows at the end instead of
// one P-point transform per term. For r' to be the same slot for every q of a residue, the slot of
// index r must advance with k = (q - j) / g: r = r' + rho0(q), rho0 = -k (lam / g)^-1 mod P, which is a
// modulation of the input by exp(-2 pi i b rho0 / P) and joins the premultiplying phase of (presA).
//
// A workgroup holds 64 lines in LDS, element by element (lane = line: no bank conflicts, no exchange
// between lanes). EA has a wave per residue j; the terms of a wave run over its residue. Per term and
// subsequence a lane reads its P points, multiplies by the phases (uniform: scalar operands), transforms
// in registers, and adds the product with the term's row of the table (scalar operands too) to its P sums.
// The waves meet once per tile, for the transform over j. Three sets of P values decide the registers:
// from P = 32 (FP64: 16) the even and odd spectral indices go to waves of their own (H = 2: the upper half
// of a subsequence joins the lower on reading, P / 2 points per wave).
//
// What bounds it: VALU issue. Measured against the forms with a line over several lanes (k_EAW, k_ERG,
// k_EAR), which move every partial sum between lanes and run an inverse transform per term:
// g = 2, P = 32, 50 terms, FP32, 250 x 32768 lines: 36.0 -> 11.7 ms (13.2 with H = 1); g = 8, P = 6, 40 terms,
// FP64, 1600 x 288 lines: 1057 -> 441 us; g = 8, P = 12, 8 terms, FP64, 8 x 12960 lines: 405 -> 125 us (320 MB,
// 62 us at the copy rate); g = 4, P = 64, 20 terms, FP32, 1280 x 64 lines: 658 -> 431 us (640 with H = 1),
// its adjoint 983 (k_AHR + k_EHG) -> 393 us. E: g = 8, P = 6, 40 terms, FP64, 92160 lines: 282 (k_ER) -> 110 us
// (425 MB, 83 us at the copy rate); g = 2, P = 32, 50 terms, FP32, 327680 lines: 1460 -> 980 us (4.4 GB: 850 us).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <set>

#include "butterflies.h"
#include "fx_internal.h"

namespace fx {

namespace {

constexpr int kLanes = 64;

// Tile of a workgroup (tiles of one XCD are contiguous: neighbours share memory lines) and its lane's line.
struct LaneTile {
    bool any, live;   // tile exists, lane has a line of its own
    int slice, s;     // line = slice * S + s
};
__device__ __forceinline__ LaneTile lane_tile(const PassGeom& g, int tile) {
    LaneTile t;
    t.any = tile < (int)g.ntiles;
    const int S = (int)g.S, nlines = (int)(g.Qin * g.A) * S;
    const int at = tile * kLanes + (int)(threadIdx.x & 63);
    t.live = at < nlines;
    const int line = min(at, nlines - 1);
    t.slice = (unsigned)line / (unsigned)S;
    t.s = line - t.slice * S;
    return t;
}
__device__ __forceinline__ int lane_block_tile(const PassGeom& g, int nchunk, int& chunk) {
    const int per = (int)((g.ntiles + 7) >> 3);
    const int y = (int)(blockIdx.x >> 3);
    const int tl = (unsigned)y / (unsigned)nchunk;
    chunk = y - tl * nchunk;
    return (int)(blockIdx.x & 7) * per + tl;
}

// Points w, w + NW, ... of the lane's line into LDS, eight loads in flight.
template <typename T, int NW>
__device__ __forceinline__ void lane_load(const C<T>* __restrict__ src, C<T>* __restrict__ X, int M, int64_t S, int w,
                                          int lane) {
    for (int n = w; n < M; n += 8 * NW) {
        C<T> v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            v[i] = mk<T>(0, 0);
            if (n + i * NW < M) v[i] = src[(int64_t)(n + i * NW) * S];
        }
#pragma unroll
        for (int i = 0; i < 8; ++i)
            if (n + i * NW < M) X[(n + i * NW) * kLanes + lane] = v[i];
    }
}

// The P points of subsequence n2 (every `str`-th point from n2), times the phases of the row, transformed.
// With H = 2 the even (or odd) half of a 2 P-point transform: the upper points join the lower ones first.
template <typename T, int P, int H>
__device__ __forceinline__ void lane_forward(const C<T>* __restrict__ X, int n2, int str, int lane,
                                             const C<T>* __restrict__ row, C<T>* v) {
#pragma unroll
    for (int b = 0; b < P; ++b) v[b] = X[(n2 + str * b) * kLanes + lane];
    if constexpr (H == 2) {
#pragma unroll
        for (int b = 0; b < P; ++b) v[b] = cfma<T>(v[b], row[0], X[(n2 + str * (b + P)) * kLanes + lane]);
    }
#pragma unroll
    for (int b = 1; b < P; ++b) v[b] = cmul<T>(v[b], row[H - 2 + b]);
    bfly<T, P, false>(v);
}

// Table rows (build_lt): per term and half the phases (the factor of the upper points when H = 2, then
// b = 1..P-1) and D[n2][r'] = Tf_q[0] HT_q[n2][.]; behind the terms the twiddles TW[f][j] of the final
// transform. P, G: points and waves, G = g H residues; the whole pruned length is P H.
template <typename T, int P, int G, int H>
__global__ __launch_bounds__(kLanes * G) void k_EAL(const C<T>* __restrict__ in, C<T>* __restrict__ out,
                                                    const C<T>* __restrict__ tab, const int* __restrict__ rows,
                                                    int lam, PassGeom g, int accumulate, T* __restrict__ rho) {
    constexpr int M = P * G, g0 = G / H;
    constexpr int ROW = g0 * P + P + H - 2;
    extern __shared__ __align__(16) unsigned char smem[];
    C<T>* X = (C<T>*)smem;  // [M][64]
    const int lane = threadIdx.x & 63;
    const int J = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int chunk;
    const LaneTile t = lane_tile(g, lane_block_tile(g, 1, chunk));
    if (!t.any) return;
    const int64_t S = g.S;
    const int64_t base = (int64_t)t.slice * M * S + t.s;
    lane_load<T, G>(in + base, X, M, S, J, lane);
    __syncthreads();
    C<T> Hs[P];
#pragma unroll
    for (int r = 0; r < P; ++r) Hs[r] = mk<T>(0, 0);
    const int j = J % g0, h = J / g0;
    int i0 = (j - g.qb) % g0;
    if (i0 < 0) i0 += g0;
    for (int i = i0; i < g.qn; i += g0) {
        const C<T>* row = tab + (int64_t)((g.qb + i) * H + h) * ROW;
        C<T> W[P];
#pragma unroll
        for (int r = 0; r < P; ++r) W[r] = mk<T>(0, 0);
#pragma unroll 1
        for (int n2 = 0; n2 < g0; ++n2) {
            C<T> v[P];
            lane_forward<T, P, H>(X, n2, g0, lane, row, v);
            const C<T>* d = row + P + H - 2 + n2 * P;
#pragma unroll
            for (int r = 0; r < P; ++r) W[r] = cfma<T>(W[r], d[r], v[r]);
        }
#pragma unroll
        for (int r = 0; r < P; ++r) Hs[r] = cadd<T>(Hs[r], W[r]);
    }
    bfly<T, P, true>(Hs);
    const C<T>* tw = tab + (int64_t)lam * H * ROW;
#pragma unroll
    for (int f = 0; f < P; ++f) Hs[f] = cmul<T>(Hs[f], tw[f * G + J]);
    __syncthreads();
#pragma unroll
    for (int f = 0; f < P; ++f) X[(J * P + f) * kLanes + lane] = Hs[f];
    __syncthreads();
    for (int f = J; f < P; f += G) {
        C<T> v[G];
#pragma unroll
        for (int i = 0; i < G; ++i) v[i] = X[(i * P + f) * kLanes + lane];
        bfly<T, G, true>(v);
        if (!t.live) continue;
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

// ------------------------------------------------------------------------------------
// EAH: the transpose of k_EAL. The forward M-point transform of the line is taken once; wave (n2, part) then
// adds conj(TA) IDFT_P(conj(D_q[n2]) H[j(q)]) over its terms in registers, P points (2 P with H = 2) of
// the line's subsequence n2; the parts' sums meet in LDS.
// ------------------------------------------------------------------------------------
constexpr int eahl_parts(int g0) { return g0 >= 8 ? 1 : 8 / g0; }

template <typename T, int P, int G, int H>
__global__ __launch_bounds__(kLanes * (G / H) * eahl_parts(G / H)) void k_EAHL(
    const C<T>* __restrict__ in, C<T>* __restrict__ out, const C<T>* __restrict__ tab, const int* __restrict__ rows,
    int lam, PassGeom g, int accumulate) {
    constexpr int M = P * G, g0 = G / H, NP = eahl_parts(g0), NW = g0 * NP;
    constexpr int ROW = g0 * P + P + H - 2;
    extern __shared__ __align__(16) unsigned char smem[];
    C<T>* X = (C<T>*)smem;  // [M][64]
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int chunk;
    const LaneTile t = lane_tile(g, lane_block_tile(g, 1, chunk));
    if (!t.any) return;
    const int64_t S = g.S;
    const int64_t base = (int64_t)t.slice * M * S + t.s;
    const C<T>* tw = tab + (int64_t)lam * H * ROW;
    for (int f = w; f < P; f += NW) {
        C<T> v[G];
#pragma unroll
        for (int c = 0; c < G; ++c) v[c] = in[base + (int64_t)rows[f * G + c] * S];
        bfly<T, G, false>(v);
#pragma unroll
        for (int J = 0; J < G; ++J) X[(J * P + f) * kLanes + lane] = cmulc<T>(v[J], tw[f * G + J]);
    }
    __syncthreads();
    for (int J = w; J < G; J += NW) {
        C<T> v[P];
#pragma unroll
        for (int f = 0; f < P; ++f) v[f] = X[(J * P + f) * kLanes + lane];
        bfly<T, P, false>(v);
#pragma unroll
        for (int f = 0; f < P; ++f) X[(J * P + f) * kLanes + lane] = v[f];
    }
    __syncthreads();
    const int n2 = w % g0, part = w / g0;
    C<T> acc[P * H];
#pragma unroll
    for (int b = 0; b < P * H; ++b) acc[b] = mk<T>(0, 0);
    for (int i = part; i < g.qn; i += NP) {
        const int q = g.qb + i;
        const int j = q % g0;
#pragma unroll 1
        for (int h = 0; h < H; ++h) {
            const C<T>* row = tab + (int64_t)(q * H + h) * ROW;
            const C<T>* d = row + P + H - 2 + n2 * P;
            const C<T>* hs = X + (j + g0 * h) * P * kLanes + lane;
            C<T> v[P];
#pragma unroll
            for (int r = 0; r < P; ++r) v[r] = cmulc<T>(hs[r * kLanes], d[r]);
            bfly<T, P, true>(v);
#pragma unroll
            for (int b = 1; b < P; ++b) v[b] = cmulc<T>(v[b], row[H - 2 + b]);
#pragma unroll
            for (int b = 0; b < P; ++b) acc[b] = cadd<T>(acc[b], v[b]);
            if constexpr (H == 2) {
#pragma unroll
                for (int b = 0; b < P; ++b) acc[b + P] = cfmac<T>(acc[b + P], v[b], row[0]);
            }
        }
    }
    for (int p = 1; p < NP; ++p) {
        __syncthreads();
        if (part == p) {
#pragma unroll
            for (int b = 0; b < P * H; ++b) X[(n2 + g0 * b) * kLanes + lane] = acc[b];
        }
        __syncthreads();
        if (part == 0) {
#pragma unroll
            for (int b = 0; b < P * H; ++b) acc[b] = cadd<T>(acc[b], X[(n2 + g0 * b) * kLanes + lane]);
        }
    }
    if (part != 0 || !t.live) return;
#pragma unroll
    for (int b = 0; b < P * H; ++b) {
        const int64_t o = base + (int64_t)(n2 + g0 * b) * S;
        C<T> z = acc[b];
        if (accumulate) z = cadd<T>(z, out[o]);
        out[o] = z;
    }
}

// ------------------------------------------------------------------------------------
// E with one line per lane (k_EL): P compiled in, any g. As above without the deferred transform: the P
// sums of a term go through its inverse transform in registers and out, 64 lines wide. The waves of a
// workgroup share its tile and take the terms of its chunk in turn.
// Table rows (build_et): the phases b = 1..P-1 of the term, then HT_q[n2][r].
// ------------------------------------------------------------------------------------
constexpr int kElWaves = 8;

template <typename T, int P>
__global__ __launch_bounds__(kLanes * kElWaves) void k_EL(const C<T>* __restrict__ in, C<T>* __restrict__ out,
                                                          const C<T>* __restrict__ tab, int M, int gg, PassGeom g) {
    extern __shared__ __align__(16) unsigned char smem[];
    C<T>* X = (C<T>*)smem;  // [M][64]
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nchunk = (g.qn + g.fqpw - 1) / g.fqpw;
    int chunk;
    const LaneTile t = lane_tile(g, lane_block_tile(g, nchunk, chunk));
    if (!t.any) return;
    const int64_t S = g.S;
    lane_load<T, kElWaves>(in + (int64_t)t.slice * M * S + t.s, X, M, S, w, lane);
    __syncthreads();
    const int qi = (unsigned)t.slice / (unsigned)g.A;
    const int a = t.slice - qi * (int)g.A;
    const int row_len = M + P - 1;
    const int i1 = min(g.qn, (chunk + 1) * g.fqpw);
    for (int i = chunk * g.fqpw + w; i < i1; i += kElWaves) {
        const C<T>* row = tab + (int64_t)(g.qb + i) * row_len;
        C<T> W[P];
#pragma unroll
        for (int r = 0; r < P; ++r) W[r] = mk<T>(0, 0);
#pragma unroll 1
        for (int n2 = 0; n2 < gg; ++n2) {
            C<T> v[P];
            lane_forward<T, P, 1>(X, n2, gg, lane, row, v);
            const C<T>* d = row + P - 1 + n2 * P;
#pragma unroll
            for (int r = 0; r < P; ++r) W[r] = cfma<T>(W[r], d[r], v[r]);
        }
        bfly<T, P, true>(W);
        if (!t.live) continue;
        C<T>* o = out + (((int64_t)qi * g.qn + i) * g.A + a) * P * S + t.s;
#pragma unroll
        for (int u = 0; u < P; ++u) o[u * S] = W[u];
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

template <typename T, int P, int G, int H>
hipError_t launch_eal_pg(Kind kind, const void* in, void* out, const AxisDev& ax, const PassGeom& g, int accumulate,
                         void* rho, hipStream_t st) {
    const size_t lds = (size_t)P * G * kLanes * sizeof(C<T>);
    const dim3 blocks((unsigned)(((g.ntiles + 7) / 8) * 8));
    if (kind == Kind::EA) {
        auto k = k_EAL<T, P, G, H>;
        hipError_t e = prep_lds_lane(k, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k, blocks, dim3(kLanes * G), lds, st, (const C<T>*)in, (C<T>*)out, (const C<T>*)ax.LT,
                           ax.LR, ax.lam, g, accumulate, (T*)rho);
    } else {
        auto k = k_EAHL<T, P, G, H>;
        hipError_t e = prep_lds_lane(k, lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k, blocks, dim3(kLanes * (G / H) * eahl_parts(G / H)), lds, st, (const C<T>*)in, (C<T>*)out,
                           (const C<T>*)ax.LT, ax.LR, ax.lam, g, accumulate);
    }
    return hipGetLastError();
}

template <typename T>
hipError_t launch_eal_T(Kind kind, const void* in, void* out, const AxisDev& ax, const PassGeom& g, int accumulate,
                        void* rho, hipStream_t st) {
#define FX_EAL(PP, GG) \
    if (ax.P == PP && ax.g == GG) return launch_eal_pg<T, PP, GG, 1>(kind, in, out, ax, g, accumulate, rho, st);
    FX_EAL(2, 8) FX_EAL(3, 8) FX_EAL(4, 8) FX_EAL(6, 8) FX_EAL(8, 8) FX_EAL(12, 8)
    FX_EAL(4, 4) FX_EAL(6, 4) FX_EAL(8, 4) FX_EAL(12, 4) FX_EAL(8, 2) FX_EAL(12, 2)
    if constexpr (sizeof(T) == 4) {
        FX_EAL(16, 8) FX_EAL(16, 4) FX_EAL(16, 2)
    } else {
        if (ax.P == 16 && ax.g == 8) return launch_eal_pg<T, 8, 16, 2>(kind, in, out, ax, g, accumulate, rho, st);
        if (ax.P == 16 && ax.g == 4) return launch_eal_pg<T, 8, 8, 2>(kind, in, out, ax, g, accumulate, rho, st);
        if (ax.P == 16 && ax.g == 2) return launch_eal_pg<T, 8, 4, 2>(kind, in, out, ax, g, accumulate, rho, st);
    }
#undef FX_EAL
    if constexpr (sizeof(T) == 4) {
        if (ax.P == 32 && ax.g == 2) return launch_eal_pg<T, 16, 4, 2>(kind, in, out, ax, g, accumulate, rho, st);
        if (ax.P == 32 && ax.g == 4) return launch_eal_pg<T, 16, 8, 2>(kind, in, out, ax, g, accumulate, rho, st);
        if (ax.P == 64 && ax.g == 4) return launch_eal_pg<T, 32, 8, 2>(kind, in, out, ax, g, accumulate, rho, st);
    } else {
        if (ax.P == 32 && ax.g == 2) return launch_eal_pg<T, 16, 4, 2>(kind, in, out, ax, g, accumulate, rho, st);
        if (ax.P == 32 && ax.g == 4) return launch_eal_pg<T, 16, 8, 2>(kind, in, out, ax, g, accumulate, rho, st);
    }
    return hipErrorInvalidValue;
}

template <typename T, int P>
hipError_t launch_el_p(const void* in, void* out, const AxisDev& ax, const PassGeom& g, hipStream_t st) {
    const size_t lds = (size_t)ax.M * kLanes * sizeof(C<T>);
    const int64_t nchunk = (g.qn + g.fqpw - 1) / g.fqpw;
    const int64_t blocks = ((g.ntiles + 7) / 8) * 8 * nchunk;
    if (blocks >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    auto k = k_EL<T, P>;
    hipError_t e = prep_lds_lane(k, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3((unsigned)blocks), dim3(kLanes * kElWaves), lds, st, (const C<T>*)in, (C<T>*)out,
                       (const C<T>*)ax.ET, ax.M, ax.g, g);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_el_T(const void* in, void* out, const AxisDev& ax, const PassGeom& g, hipStream_t st) {
    switch (ax.P) {
        case 2: return launch_el_p<T, 2>(in, out, ax, g, st);
        case 3: return launch_el_p<T, 3>(in, out, ax, g, st);
        case 4: return launch_el_p<T, 4>(in, out, ax, g, st);
        case 5: return launch_el_p<T, 5>(in, out, ax, g, st);
        case 6: return launch_el_p<T, 6>(in, out, ax, g, st);
        case 7: return launch_el_p<T, 7>(in, out, ax, g, st);
        case 8: return launch_el_p<T, 8>(in, out, ax, g, st);
        case 9: return launch_el_p<T, 9>(in, out, ax, g, st);
        case 10: return launch_el_p<T, 10>(in, out, ax, g, st);
        case 12: return launch_el_p<T, 12>(in, out, ax, g, st);
        case 15: return launch_el_p<T, 15>(in, out, ax, g, st);
        case 16: return launch_el_p<T, 16>(in, out, ax, g, st);
        case 32:
            if constexpr (sizeof(T) == 4) return launch_el_p<T, 32>(in, out, ax, g, st);
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
}

// Lines over all slices, as the kernels index them.
bool lane_lines_ok(const PassGeom& g) {
    return g.TS == kLanes && g.ntiles == (g.Qin * g.A * g.S + kLanes - 1) / kLanes &&
           g.Qin * g.A * g.S < (int64_t(1) << 31) - kLanes;
}

}  // namespace

// Half the pruned length per wave where the whole would not fit the registers.
int eal_halves(bool dbl, int M, int g) { return M / g >= (dbl ? 16 : 32) ? 2 : 1; }

bool eal_applicable(bool dbl, int M, int g) {
    if (g < 1 || M % g) return false;
    const int P = M / g;
    if ((size_t)M * kLanes * (dbl ? 16 : 8) > (size_t)lds_limit_bytes()) return false;
    auto in = [&](std::initializer_list<int> l) { return std::find(l.begin(), l.end(), P) != l.end(); };
    switch (g) {
        case 8: return in({2, 3, 4, 6, 8, 12, 16});
        case 4: return in({4, 6, 8, 12, 16, 32}) || (!dbl && P == 64);
        case 2: return in({8, 12, 16, 32});
        default: return false;
    }
}

bool el_applicable(bool dbl, int M, int g) {
    if (g < 1 || M % g || (size_t)M * kLanes * (dbl ? 16 : 8) > (size_t)lds_limit_bytes()) return false;
    switch (M / g) {
        case 2: case 3: case 4: case 5: case 6: case 7: case 8: case 9: case 10: case 12: case 15: case 16: return true;
        case 32: return !dbl;
        default: return false;
    }
}

int lane_tile_lines() { return kLanes; }

hipError_t launch_pass_eal(Kind kind, bool dbl, const void* in, void* out, const AxisDev& ax, const PassGeom& g,
                           int accumulate, void* rho, hipStream_t st) {
    if ((kind != Kind::EA && kind != Kind::EAH) || !ax.LT || !ax.LR || !eal_applicable(dbl, ax.M, ax.g) ||
        !lane_lines_ok(g))
        return hipErrorInvalidValue;
    return dbl ? launch_eal_T<double>(kind, in, out, ax, g, accumulate, rho, st)
               : launch_eal_T<float>(kind, in, out, ax, g, accumulate, rho, st);
}

hipError_t launch_pass_el(bool dbl, const void* in, void* out, const AxisDev& ax, const PassGeom& g, hipStream_t st) {
    if (!ax.ET || !el_applicable(dbl, ax.M, ax.g) || !lane_lines_ok(g) || g.fqpw < 1) return hipErrorInvalidValue;
    return dbl ? launch_el_T<double>(in, out, ax, g, st) : launch_el_T<float>(in, out, ax, g, st);
}

}  // namespace fx
