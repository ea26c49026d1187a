// Eight-point transforms with their input twiddles written as cos (1 + i tan), for the blind rotation that
// keeps one gate in one wavefront.
//
// A 512-point transform at the odd roots, X_k = sum_n z_n psi^(n (1 + 4k)) with psi = exp(i pi / 1024),
// n = j0 + 8 j1 + 64 m and k = k0 + 8 k1 + 64 k2, splits into three eight-point passes whose twiddles
// all sit on the inputs:
//   pass 1 over m    psi^(64 m)             (the same in every lane)          -> k0
//   pass 2 over j1   psi^(8 j1 (1 + 4 k0))                                    -> k1
//   pass 3 over j0   psi^(j0 (1 + 4 k0 + 32 k1))                              -> k2
// and the inverse, z_n = sum_k X_k psi^(-n (1 + 4k)), into
//   pass 3 over k2   no twiddle                                               -> j0
//   pass 2 over k1   psi^(-32 j0 k1)                                          -> j1
//   pass 1 over k0   psi^(-L (1 + 4 k0)), L = j0 + 8 j1                       -> m
//   and psi^(-64 m) on the outputs, whose cosine the caller folds into its rounding.
// The spectra are the ones the four-wave kernels produce (same frequencies, same scale), so both share
// one transformed key.
//
// A twiddle c (1 + i t) costs two fused multiply-adds for the turn by (1 + i t); its cosine is not applied
// to the number but left pending and absorbed, as a ratio of cosines, by the multiply-adds that take
// the place of the transform's additions.  Fourteen instructions twiddle seven inputs instead of
// twenty-eight, and the eight-point transform itself keeps its 52.  Pending factors do not
// cost accuracy however small a cosine is: x (1 + i t) with |t| up to 2^65 and a factor c with c t = 1 is
// as accurate relative to its size as x times the rounded twiddle.
#pragma once
#include <hip/hip_runtime.h>

#include "fft512.h"

namespace fft512 {

// Constants of one transform whose input j carries exp(i phi_j) = c_j (1 + i t_j).
struct Twiddle8 {
    double t[8];         // tan phi_j; t[0] is not used (input 0 carries none, or the caller multiplies it)
    double rho[4];       // c_{j+4} / c_j
    double sig0, sig1;   // c_2 / c_0, c_3 / c_1
    double tau, tauh;    // c_1 / c_0, and the same over sqrt 2
};

FFT_HD double2 cturn(double2 a, double t) { return make_double2(fma(-t, a.y, a.x), fma(t, a.x, a.y)); }
FFT_HD double2 cmadd(double2 a, double s, double2 b) { return make_double2(fma(s, b.x, a.x), fma(s, b.y, a.y)); }      // a + s b
FFT_HD double2 cmaddi(double2 a, double s, double2 b) { return make_double2(fma(-s, b.y, a.x), fma(s, b.x, a.y)); }    // a + i s b

// y[k] = sum_j exp(i phi_j) x[j] w^(j k), w = exp(2 pi i / 8) (INV: exp(-2 pi i / 8)), in place
template <bool INV>
FFT_HD void dft8_twiddled(double2 (&x)[8], const Twiddle8 &w) {
    for (int j = 1; j < 8; ++j) x[j] = cturn(x[j], w.t[j]);
    double2 a[8];
    for (int j = 0; j < 4; ++j) {
        a[j] = cmadd(x[j], w.rho[j], x[j + 4]);
        a[j + 4] = cmadd(x[j], -w.rho[j], x[j + 4]);
    }
    {
        const double2 c0 = cmadd(a[0], w.sig0, a[2]), c1 = cmadd(a[0], -w.sig0, a[2]);
        const double2 c2 = cmadd(a[1], w.sig1, a[3]), d = cmadd(a[1], -w.sig1, a[3]);
        x[0] = cmadd(c0, w.tau, c2);
        x[4] = cmadd(c0, -w.tau, c2);
        const double ti = INV ? -w.tau : w.tau;
        x[2] = cmaddi(c1, ti, d);
        x[6] = cmaddi(c1, -ti, d);
    }
    {
        // sqrt 2 times a5 w and a7 w^3; the 1 / sqrt 2 is in tauh
        const double2 s5 = INV ? make_double2(a[5].x + a[5].y, a[5].y - a[5].x) : make_double2(a[5].x - a[5].y, a[5].x + a[5].y);
        const double2 s7 = INV ? make_double2(a[7].y - a[7].x, -a[7].x - a[7].y) : make_double2(-a[7].x - a[7].y, a[7].x - a[7].y);
        const double s6 = INV ? -w.sig0 : w.sig0;
        const double2 c0 = cmaddi(a[4], s6, a[6]), c1 = cmaddi(a[4], -s6, a[6]);
        const double2 t = cmadd(s5, w.sig1, s7), u = cmadd(s5, -w.sig1, s7);
        x[1] = cmadd(c0, w.tauh, t);
        x[5] = cmadd(c0, -w.tauh, t);
        const double hi = INV ? -w.tauh : w.tauh;
        x[3] = cmaddi(c1, hi, u);
        x[7] = cmaddi(c1, -hi, u);
    }
}

// y[k] = sum_j theta^j x[j] w^(j k): with the twiddles in geometric progression four (cos, tan) pairs --
// theta^4, theta^2, theta, theta w -- serve all twelve butterflies (six instructions each): 72 instead of
// 66, but 16 registers of constants instead of 30.
struct Shift8 {
    double2 h4, h2, h1, h1w;
};
template <bool I>
FFT_HD void bfly(double2 &a, double2 &b, double2 w) {      // a, b <- a +- w b (I: a +- i w b)
    const double2 r = cturn(b, w.y), p = a;
    a = I ? cmaddi(p, w.x, r) : cmadd(p, w.x, r);
    b = I ? cmaddi(p, -w.x, r) : cmadd(p, -w.x, r);
}
FFT_HD void dft8_shifted(double2 (&x)[8], const Shift8 &w) {
    for (int j = 0; j < 4; ++j) bfly<false>(x[j], x[j + 4], w.h4);
    bfly<false>(x[0], x[2], w.h2);
    bfly<false>(x[1], x[3], w.h2);
    bfly<true>(x[4], x[6], w.h2);
    bfly<true>(x[5], x[7], w.h2);
    bfly<false>(x[0], x[1], w.h1);
    bfly<true>(x[2], x[3], w.h1);
    bfly<false>(x[4], x[5], w.h1w);
    bfly<true>(x[6], x[7], w.h1w);
    const double2 y4 = x[1], y2 = x[2], y6 = x[3], y1 = x[4], y3 = x[6], y7 = x[7];
    x[1] = y1; x[2] = y2; x[3] = y3; x[4] = y4; x[6] = y6; x[7] = y7;
}

// ---- the constants in memory, behind the 2,048 powers of psi (offsets in complex words) ----
// Lane-dependent constants are packed two to a complex word, eight words a lane, word-major.
constexpr int kPsiWords = 2048;
constexpr int kFwd2 = kPsiWords;          // [word 8][k0 8]      forward pass 2
constexpr int kInv2 = kFwd2 + 64;         // [word 8][j0 8]      inverse pass 2
constexpr int kInv1 = kInv2 + 64;         // [word 8][L 64]      inverse pass 1
constexpr int kFwd3 = kInv1 + 512;        // [word 4][lane 64]   forward pass 3, lane = 8 k0 + k1: h4, h2, h1, h1w
constexpr int kUniform = kFwd3 + 256;     // 24 doubles of passes 1: tan, rho, sig0, sig1, tau, tauh; then cos
constexpr int kTableWords = kUniform + 12;

FFT_HD Twiddle8 unpack_twiddles(const double2 (&p)[8]) {
    Twiddle8 w;
    w.t[0] = 0.0;
    w.t[1] = p[0].x; w.t[2] = p[0].y; w.t[3] = p[1].x; w.t[4] = p[1].y; w.t[5] = p[2].x; w.t[6] = p[2].y; w.t[7] = p[3].x;
    w.rho[0] = p[3].y; w.rho[1] = p[4].x; w.rho[2] = p[4].y; w.rho[3] = p[5].x;
    w.sig0 = p[5].y; w.sig1 = p[6].x; w.tau = p[6].y; w.tauh = p[6].y * 0.70710678118654752440;
    return w;
}

// All constants, evaluated in extended precision; `tables` holds kTableWords complex words.
inline void fill_tables(double2 *tables) {
    const long double pi = 3.14159265358979323846264338327950288L, unit = pi / 1024;
    for (int j = 0; j < kPsiWords; ++j) tables[j] = make_double2((double)cosl(unit * j), (double)sinl(unit * j));
    auto angle = [&](int e) { return unit * (((e % 2048) + 2048) % 2048); };
    // whole0: input 0 is multiplied by its whole twiddle (word 7) and the ratios count from 1
    auto pack = [&](int base, int width, int lane, const int (&e)[8], bool whole0) {
        long double c[8], t[8];
        for (int j = 0; j < 8; ++j) { c[j] = cosl(angle(e[j])); t[j] = sinl(angle(e[j])) / c[j]; }
        const long double c0 = c[0], s0 = sinl(angle(e[0]));
        if (whole0) c[0] = 1.0L;
        const long double v[16] = {t[1], t[2], t[3], t[4], t[5], t[6], t[7], c[4] / c[0], c[5] / c[1], c[6] / c[2],
                                   c[7] / c[3], c[2] / c[0], c[3] / c[1], c[1] / c[0], c0, s0};
        for (int q = 0; q < 8; ++q) tables[base + q * width + lane] = make_double2((double)v[2 * q], (double)v[2 * q + 1]);
    };
    for (int a = 0; a < 8; ++a) {
        int f[8], g[8];
        for (int j = 0; j < 8; ++j) { f[j] = 8 * j * (1 + 4 * a); g[j] = -32 * a * j; }
        pack(kFwd2, 8, a, f, false);
        pack(kInv2, 8, a, g, false);
    }
    for (int L = 0; L < 64; ++L) {
        int f[8];
        for (int k = 0; k < 8; ++k) f[k] = -L * (1 + 4 * k);
        pack(kInv1, 64, L, f, true);
        const int e = 1 + 4 * (L >> 3) + 32 * (L & 7), h[4] = {4 * e, 2 * e, e, e + 256};
        for (int q = 0; q < 4; ++q)
            tables[kFwd3 + q * 64 + L] = make_double2((double)cosl(angle(h[q])), (double)(sinl(angle(h[q])) / cosl(angle(h[q]))));
    }
    long double c[8], v[24] = {};
    for (int m = 0; m < 8; ++m) { c[m] = cosl(pi * m / 16); v[m] = sinl(pi * m / 16) / c[m]; v[16 + m] = c[m]; }
    for (int m = 0; m < 4; ++m) v[8 + m] = c[m + 4] / c[m];
    v[12] = c[2]; v[13] = c[3] / c[1]; v[14] = c[1]; v[15] = c[1] * sqrtl(0.5L);
    for (int q = 0; q < 12; ++q) tables[kUniform + q] = make_double2((double)v[2 * q], (double)v[2 * q + 1]);
}

}  // namespace fft512
