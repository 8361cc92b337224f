// FP64 phase tables of the prescription (FF), section 5.2, one set per axis.
//
// Every phase is written in cycles (units of 2 pi) as a sum of
//   * an exact rational part (integer numerator reduced modulo its integer
//     denominator in int64),
//   * a small fractional-offset part (|value| <= 1/2 by construction), and
//   * a quadratic part beta * I with beta = pi hbar t / (m lam^2 L^2) and an
//     exact integer I; beta is carried as a double-double (computed in long
//     double) and beta_hi * I is split exactly with an FMA two-product, so the
//     product is reduced modulo 1 without losing the fractional digits that a
//     large chirp argument would otherwise swamp.
// Only the reduced phase (|c| <= 1/2 cycle) goes through sin/cos.
//
// With k = dk * l~ (eq. (kj)), alpha_q = q dk / lam, delta = (abar - a)/dx and
// ell = lam * l~ + q (the fine-lattice wave number of eq. (ulk)):
//   TA[q][n]   : -alpha_q (x_n - a)                      = -(q n) / (lam M)
//   TB[q][m~]  : k (abar - a) - k (k + 2 alpha_q) ht/2m  = l~ delta / M - beta (ell^2 - q^2)
//   Tf[q][nb]  : alpha_q (xbar - a) - alpha_q^2 ht/2m    = q (delta + lam nb) / (lam M) - beta q^2
// For odd M the largest positive coarse wave number is folded to the negative
// side when q >= lam/2 (the umklapp rule stated after (FF)).
//
// Other spectra (section 7.4): with exp(-i t omega_k) in place of the free-particle
// factor, the quadratic parts become -(phi(ell) - phi(q)) in TB and -phi(q) in Tf,
// phi = t omega / (2 pi) in cycles, read from a caller table over the fine wave numbers.
#include <cmath>
#include <cstdint>

#include "fx_internal.h"

namespace fx {
namespace {

constexpr double kTwoPi = 6.283185307179586476925286766559;

inline double reduce_cycles(double c) { return c - std::nearbyint(c); }

// (num mod den) / den in [-1/2, 1/2], exact up to the final division.
inline double rational_cycles(int64_t num, int64_t den) {
    int64_t r = num % den;
    if (r < 0) r += den;
    if (2 * r > den) r -= den;
    return (double)r / (double)den;
}

struct DD { double hi, lo; };

// frac(beta * I) for the double-double beta and an integer I below 2^53.
inline double beta_cycles(DD beta, int64_t I) {
    const double x = (double)I;
    const double p = beta.hi * x;
    const double e = std::fma(beta.hi, x, -p);  // p + e == beta.hi * x exactly
    return reduce_cycles(reduce_cycles(p) + e + beta.lo * x);
}

// exp(-2 pi i k / N), k < N, from one table: the premultiplying phases and the twiddles of HT are all among
// them. Above 2^22 entries they are computed one by one.
class Roots {
public:
    explicit Roots(int64_t N) : N_(N) {
        if (N > (int64_t(1) << 22)) return;
        tab_.resize(2 * (size_t)N);
        for (int64_t k = 0; k < N; ++k) value(k, &tab_[2 * (size_t)k]);
    }
    int64_t size() const { return N_; }
    void get(int64_t k, double* z) const {  // 0 <= k < N
        if (tab_.empty()) return value(k, z);
        z[0] = tab_[2 * (size_t)k];
        z[1] = tab_[2 * (size_t)k + 1];
    }

private:
    void value(int64_t k, double* z) const {
        const double ang = -kTwoPi * rational_cycles(k, N_);
        z[0] = std::cos(ang);
        z[1] = std::sin(ang);
    }
    int64_t N_;
    std::vector<double> tab_;
};

inline void put(std::vector<double>& v, size_t i, double cycles, double amp) {
    const double ang = kTwoPi * reduce_cycles(cycles);
    v[2 * i] = amp * std::cos(ang);
    v[2 * i + 1] = amp * std::sin(ang);
}

int64_t gcd_of(int64_t g, int64_t b) {
    while (b) { const int64_t r = g % b; g = b; b = r; }
    return g;
}

// Chirp-folded table of the register E kernel. With g = gcd(lam, M), P = M / g, input index
// n = g n1 + n2 and spectral index m = r + P c (n1, r < P; n2, c < g), the forward DFT factors as
//   Y[r + P c] = sum_n2 w_g^(n2 c) w_M^(n2 r) V[n2][r],  V[n2][r] = sum_n1 w_P^(n1 r) y[g n1 + n2],
// so the chirp (presB) and the fold over c of the pruned inverse collapse into
//   W[r] = sum_c TB[r + P c] Y[r + P c] = sum_n2 HT[n2][r] V[n2][r],
//   HT[n2][r] = w_M^(n2 r) TA'[n2] sum_c TB[r + P c] w_g^(n2 c) / M,
// where the n2 part of (presA), TA'[n2] = exp(-2 pi i q n2 / (lam M)), and the 1/M of the inverse
// are folded in as well. Layout [q][r][n2] (the g lanes of a line read consecutive values, and the
// P g = M values of one q are contiguous), FP64 complex.
void build_ht(AxisTables& t, int64_t M, int64_t lam, const Roots& roots) {
    const int64_t g = gcd_of(lam, M);
    const int64_t P = M / g;
    const int64_t N = lam * M;
    t.HT.assign(2 * (size_t)(lam * M), 0.0);
    std::vector<double> rg(2 * (size_t)g);  // exp(-2 pi i k / g)
    for (int64_t k = 0; k < g; ++k) put(rg, (size_t)k, -rational_cycles(k, g), 1.0);
    auto at = [&](int64_t q, int64_t r, int64_t n2) { return 2 * (size_t)((q * P + r) * g + n2); };
    for (int64_t q = 0; q < lam; ++q) {
        const double* tb = &t.TB[2 * (size_t)(q * M)];
        for (int64_t n2 = 0; n2 < g; ++n2) {
            for (int64_t r = 0; r < P; ++r) {
                double sr = 0.0, si = 0.0;
                for (int64_t c = 0; c < g; ++c) {
                    const double* z = tb + 2 * (r + P * c);
                    const double* w = &rg[2 * (size_t)((n2 * c) % g)];
                    sr += z[0] * w[0] - z[1] * w[1];
                    si += z[0] * w[1] + z[1] * w[0];
                }
                const size_t i = at(q, r, n2);
                if (n2 == 0) {
                    t.HT[i] = sr * (1.0 / (double)M);
                    t.HT[i + 1] = si * (1.0 / (double)M);
                    continue;
                }
                // exp(-2 pi i (n2 r lam + q n2) / (lam M)) / M
                double z[2];
                roots.get((n2 * (r * lam + q)) % N, z);
                const double er = z[0] / (double)M, ei = z[1] / (double)M;
                t.HT[i] = sr * er - si * ei;
                t.HT[i + 1] = sr * ei + si * er;
            }
        }
    }
}

// The copies of HT that the register kernels read.
void arrange_ht(AxisTables& t, int64_t M, int64_t lam) {
    const int64_t g = gcd_of(lam, M);
    const int64_t P = M / g;
    auto at = [&](int64_t q, int64_t r, int64_t n2) { return 2 * (size_t)((q * P + r) * g + n2); };
    // Second copy for the forward register kernels. Their first cross-lane reduction step pairs
    // lanes n2 and n2 ^ 1; the odd lane keeps the upper half of the P sums. When the odd lane's
    // P values come with their halves exchanged, both lanes keep the lower half and send the upper
    // one, so no per-lane selects are needed:
    //   g >= P (transform, multiply, then reduce): the odd lane's input is modulated by (-1)^n1,
    //     which moves its spectrum by P/2, so its table row is HT[n2][r ^ P/2];
    //   g <  P (transform, multiply, inverse, then reduce): the odd lane's inverse output is moved
    //     by P/2 when its row is modulated by (-1)^r.
    t.HTx = t.HT;
    const bool p2 = (P & (P - 1)) == 0;
    if (p2 && P >= 2 && g >= 2) {
        for (int64_t q = 0; q < lam; ++q) {
            for (int64_t n2 = 1; n2 < g; n2 += 2) {
                for (int64_t r = 0; r < P; ++r) {
                    const size_t d = at(q, r, n2);
                    if (g >= P) {
                        const size_t s = at(q, r ^ (P / 2), n2);
                        t.HTx[d] = t.HT[s];
                        t.HTx[d + 1] = t.HT[s + 1];
                    } else if (r & 1) {
                        t.HTx[d] = -t.HT[d];
                        t.HTx[d + 1] = -t.HT[d + 1];
                    }
                }
            }
        }
    }
    // The table once more in [q][n2][r] order, for kernels whose lanes read their own P values of a
    // row contiguously. For power-of-two P <= min(g, 8) those kernels shift lane n2's spectrum by
    // s = bitrev(n2 mod P) (its input times exp(-2 pi i s n1 / P)), which makes every step of the
    // reduction over the lanes select-free, so the lane's row is turned by s: HTl[q][n2][r] =
    // HT[q][(r + s) mod P][n2] (for P = 2 this is HTx). Otherwise HTl is HTx reordered.
    t.HTl.assign(t.HTx.size(), 0.0);
    int lgp = 0;
    while ((int64_t(1) << lgp) < P) ++lgp;
    const bool rot = p2 && P >= 2 && P <= 8 && g >= P;
    for (int64_t q = 0; q < lam; ++q)
        for (int64_t n2 = 0; n2 < g; ++n2) {
            int64_t sh = 0;
            for (int b = 0; b < lgp; ++b) sh |= ((n2 >> b) & 1) << (lgp - 1 - b);
            for (int64_t r = 0; r < P; ++r) {
                const size_t d = 2 * (size_t)((q * g + n2) * P + r);
                const size_t src = rot ? at(q, (r + sh) % P, n2) : at(q, r, n2);
                const std::vector<double>& from = rot ? t.HT : t.HTx;
                t.HTl[d] = from[src];
                t.HTl[d + 1] = from[src + 1];
            }
        }
}

// Table of the folded line kernels: per term the g rows HT_q[n2] with the spectrum in the digit-reversed
// order in which the plan's forward stages leave it, the premultiplying phases of the subsequences
// TA_q[g n1], and Tf_q[n0(u)] at the output n0(u) < P that reads sample u; then the twiddles
// exp(-2 pi i k u / L) of every stage but the last, [u - 1][k] with u < R, k < m, L = R m.
void build_ft(AxisTables& t, int64_t lam, const FoldPlan& pl) {
    const int64_t M = pl.M, g = pl.g, P = pl.P;
    const int64_t lg = (lam / g) % P;
    t.FT.assign(2 * (size_t)(lam * (g + 2) * P + pl.ntw), 0.0);
    std::vector<int64_t> n0((size_t)P, 0), rev((size_t)P, 0);
    for (int64_t n = 0; n < P; ++n) n0[(size_t)((n * lg) % P)] = n;
    for (int64_t p = 0; p < P; ++p) {
        // position p = sum_s u_s m_s holds frequency r = u_0 + R_0 (u_1 + R_1 (...))
        int64_t rest = p, r = 0, w = 1;
        for (int s = 0; s < pl.n; ++s) {
            r += (rest / pl.st[s].m.d) * w;
            rest %= pl.st[s].m.d;
            w *= pl.st[s].R;
        }
        rev[(size_t)p] = r;
    }
    for (int64_t q = 0; q < lam; ++q) {
        double* row = &t.FT[2 * (size_t)(q * (g + 2) * P)];
        auto set = [&](int64_t at, const std::vector<double>& v, int64_t i) {
            row[2 * at] = v[2 * (size_t)i];
            row[2 * at + 1] = v[2 * (size_t)i + 1];
        };
        for (int64_t n2 = 0; n2 < g; ++n2)
            for (int64_t p = 0; p < P; ++p) set(n2 * P + p, t.HT, (q * P + rev[(size_t)p]) * g + n2);
        for (int64_t n1 = 0; n1 < P; ++n1) {
            set(M + n1, t.TA, q * M + g * n1);
            set(M + P + n1, t.Tf, q * M + n0[(size_t)n1]);
        }
    }
    const size_t tw0 = (size_t)(lam * (g + 2) * P);
    for (int s = 0; s + 1 < pl.n; ++s) {
        const int64_t m = pl.st[s].m.d, R = pl.st[s].R;
        for (int64_t u = 1; u < R; ++u)
            for (int64_t k = 0; k < m; ++k)
                put(t.FT, tw0 + (size_t)(pl.st[s].tw + (u - 1) * m + k), -rational_cycles(k * u, R * m), 1.0);
    }
}

// Table of the lane-per-line EA kernel. With k = (q - q mod g) / g and rho0 = -k (lam / g)^-1 mod P, the
// spectral index in slot r' of term q is r' + rho0 mod P. The slots are taken in `halves` interleaved
// classes h (r' = h + halves r''), P1 = P / halves each. Per term and class: with two classes the factor
// exp(-i pi (q / lam + rho0 + h)) that joins the upper half of a subsequence to the lower; the phases
// exp(-2 pi i b (q + lam (rho0 + h)) / (lam P)), b = 1..P1-1 (the premultiplying phase of (presA) and the
// modulation that moves the class to slot 0); D[n2][r''] = Tf_q[0] HT_q[n2][(rho0 + h + halves r'') mod P].
// Behind the terms, with J = j + g h running over the residues and classes, TW[f][J] = exp(2 pi i
// c1(f) (j + lam h) / M): the P1-point inverse transform over the slots leaves at f the output
// c1(f) = f (lam / g)^-1 mod P1 and those P1 apart, and J is the index of the transform over c2 that
// follows. LR[f][c2] = c1(f) + P1 c2.
void build_lt(AxisTables& t, int64_t M, int64_t lam, int halves) {
    const int64_t g = gcd_of(lam, M), P = M / g, lg = (lam / g) % P, P1 = P / halves, G = g * halves;
    int64_t inv = 0;
    for (int64_t x = 0; x < P; ++x)
        if ((x * lg) % P == 1 % P) { inv = x; break; }
    const int64_t row = g * P1 + P1 + halves - 2;
    t.LT.assign(2 * (size_t)(lam * halves * row + M), 0.0);
    t.LR.assign((size_t)M, 0);
    for (int64_t q = 0; q < lam; ++q) {
        const int64_t k = q / g;
        const int64_t rho0 = (P - (k % P) * inv % P) % P;
        const double fr = t.Tf[2 * (size_t)(q * M)], fi = t.Tf[2 * (size_t)(q * M) + 1];
        for (int64_t h = 0; h < halves; ++h) {
            const int64_t at = (q * halves + h) * row, Q = q + lam * (rho0 + h);
            if (halves == 2) put(t.LT, (size_t)at, -rational_cycles(Q, 2 * lam), 1.0);
            for (int64_t b = 1; b < P1; ++b)
                put(t.LT, (size_t)(at + halves - 2 + b), -rational_cycles(b * Q, lam * P), 1.0);
            for (int64_t n2 = 0; n2 < g; ++n2)
                for (int64_t r = 0; r < P1; ++r) {
                    const double* v = &t.HT[2 * (size_t)((q * P + (rho0 + h + halves * r) % P) * g + n2)];
                    double* d = &t.LT[2 * (size_t)(at + P1 + halves - 2 + n2 * P1 + r)];
                    d[0] = fr * v[0] - fi * v[1];
                    d[1] = fr * v[1] + fi * v[0];
                }
        }
    }
    for (int64_t f = 0; f < P1; ++f) {
        const int64_t c1 = (f * inv) % P1;
        for (int64_t J = 0; J < G; ++J) {
            put(t.LT, (size_t)(lam * halves * row + f * G + J), rational_cycles(c1 * (J % g + lam * (J / g)), M), 1.0);
            t.LR[(size_t)(f * G + J)] = (int)(c1 + P1 * J);
        }
    }
}

// Table of the lane-per-line E and of the rows-in-registers E: per term the phases TA_q[g b], b = 1..P-1, then HT_q[n2][r].
void build_et(AxisTables& t, int64_t M, int64_t lam) {
    const int64_t g = gcd_of(lam, M), P = M / g, row = M + P - 1;
    t.ET.assign(2 * (size_t)(lam * row), 0.0);
    for (int64_t q = 0; q < lam; ++q) {
        double* d = &t.ET[2 * (size_t)(q * row)];
        for (int64_t b = 1; b < P; ++b, d += 2) {
            d[0] = t.TA[2 * (size_t)(q * M + g * b)];
            d[1] = t.TA[2 * (size_t)(q * M + g * b) + 1];
        }
        for (int64_t n2 = 0; n2 < g; ++n2)
            for (int64_t r = 0; r < P; ++r, d += 2) {
                d[0] = t.HT[2 * (size_t)((q * P + r) * g + n2)];
                d[1] = t.HT[2 * (size_t)((q * P + r) * g + n2) + 1];
            }
    }
}

}  // namespace

AxisTables build_axis_tables(const AxisParams& p) {
    const int64_t M = p.M;
    const int64_t lam = p.lam;
    const int64_t N = lam * M;
    AxisTables t;
    t.TA.resize(2 * (size_t)(lam * M));
    t.TB.resize(2 * (size_t)(lam * M));
    t.Tf.resize(2 * (size_t)(lam * M));
    t.tw.resize(2 * (size_t)M);

    // beta = pi * (t / (m/hbar)) / (lam * M * dx)^2 in long double, split into hi + lo.
    const long double pi_l = 3.14159265358979323846264338327950288L;
    const long double Lb = (long double)N * (long double)p.dx;
    const long double beta_l = pi_l * ((long double)p.t / (long double)p.m_over_hbar) / (Lb * Lb);
    DD beta;
    beta.hi = (double)beta_l;
    beta.lo = (double)(beta_l - (long double)beta.hi);

    const double delta = (p.abar - p.a) / p.dx;
    const double di_d = std::nearbyint(delta);
    const int64_t di = (int64_t)di_d;
    const double df = delta - di_d;

    const double inv2pi = 1.0 / kTwoPi;
    const int64_t l0 = N / 2;  // table index of the fine wave number 0
    const Roots roots(N);
    for (int64_t q = 0; q < lam; ++q) {
        const double phq = p.phase ? p.phase[l0 + q] * inv2pi : 0.0;
        for (int64_t n = 0; n < M; ++n) {
            const size_t i = (size_t)(q * M + n);
            // TA: -(q n)/(lam M); q n < lam M
            roots.get(q * n, &t.TA[2 * i]);
            // TB: coarse wave number of eq. (kj) with the odd-M umklapp.
            int64_t lt = (2 * n < M) ? n : n - M;
            if ((M % 2 == 1) && (2 * n == M - 1) && (2 * q >= lam)) lt -= M;
            const int64_t ell = lam * lt + q;
            const int64_t I = ell * ell - q * q;
            const double chirp = p.phase ? reduce_cycles(p.phase[l0 + ell] * inv2pi - phq)
                                         : beta_cycles(beta, I);
            const double tb = rational_cycles(lt * di, M) + (double)lt * df / (double)M - chirp;
            put(t.TB, i, tb, 1.0);
            // Tf: q (delta + lam nb)/(lam M) - beta q^2, amplitude 1/lam.
            const double tf = rational_cycles(q * (di + lam * n), N) + (double)q * df / (double)N
                              - (p.phase ? reduce_cycles(phq) : beta_cycles(beta, q * q));
            put(t.Tf, i, tf, 1.0 / (double)lam);
        }
    }
    for (int64_t k = 0; k < M; ++k) put(t.tw, (size_t)k, -rational_cycles(k, M), 1.0);
    if (p.want_ht || p.lt_halves || p.want_et || p.fold) build_ht(t, M, lam, roots);
    if (p.lt_halves) build_lt(t, M, lam, p.lt_halves);
    if (p.want_et) build_et(t, M, lam);
    if (p.fold) build_ft(t, lam, *p.fold);
    if (p.want_ht) arrange_ht(t, M, lam);
    else t.HT.clear();
    return t;
}

}  // namespace fx
