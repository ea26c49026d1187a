// Eight-point transforms with their input twiddles written as cos (1 + i tan), for the blind rotations.
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
// The spectra are those of fft512.h (same frequencies, same scale), whose steps transform the key.
//
// (The fused-multiply-add form of Linzer and Feig, IEEE Trans. Signal Processing 41, 1993, carried through three passes.)
// A twiddle c (1 + i t) costs two fused multiply-adds for the turn by (1 + i t); its cosine is not applied
// to the number but left pending and absorbed, as a ratio of cosines, by the multiply-adds that take
// the place of the transform's additions.  Fourteen instructions twiddle seven inputs instead of
// twenty-eight, and the eight-point transform itself keeps its 52: 202 to 210 instructions a lane for a whole
// transform instead of 244.  Pending factors do not
// cost accuracy however small a cosine is: x (1 + i t) with |t| up to 2^65 and a factor c with c t = 1 is
// as accurate relative to its size as x times the rounded twiddle.  Largest distance of a product from its integer,
// against the transforms of fft512.h: random operands 7e-7 against 6e-7, extreme magnitudes with random signs
// 1.9e-6 against 2.4e-6, every operand at one end of its range 4.6e-5 against 3.1e-5 (a wrong rounding needs 0.5); on the
// device, over 12,288 gates each, random keys 1.2e-6 either way, keys at one end of the limbs' range 3.6e-5 against 3.1e-5.
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

// The transforms hand out their results one by one, emit(k, y[k]): the four even ones, then -- after
// between() -- the four odd ones, whose half of the additions is still to come.  A caller that stores them to
// LDS so has half of its stores under way while it computes.  The array versions leave them in x.
// w = exp(2 pi i / 8) (INV: exp(-2 pi i / 8)).

// y[k] = sum_j exp(i phi_j) x[j] w^(j k)
template <bool INV, class Emit, class Between>
FFT_HD void dft8_twiddled(double2 (&x)[8], const Twiddle8 &w, Emit &&emit, Between &&between) {
    for (int j = 1; j < 8; ++j) x[j] = cturn(x[j], w.t[j]);
    double2 a[8];
    for (int j = 0; j < 4; ++j) {
        a[j] = cmadd(x[j], w.rho[j], x[j + 4]);
        a[j + 4] = cmadd(x[j], -w.rho[j], x[j + 4]);
    }
    {
        const double2 c0 = cmadd(a[0], w.sig0, a[2]), c1 = cmadd(a[0], -w.sig0, a[2]);
        const double2 c2 = cmadd(a[1], w.sig1, a[3]), d = cmadd(a[1], -w.sig1, a[3]);
        const double ti = INV ? -w.tau : w.tau;
        emit(0, cmadd(c0, w.tau, c2));
        emit(4, cmadd(c0, -w.tau, c2));
        emit(2, cmaddi(c1, ti, d));
        emit(6, cmaddi(c1, -ti, d));
    }
    between();
    {
        // sqrt 2 times a5 w and a7 w^3; the 1 / sqrt 2 is in tauh
        const double2 s5 = INV ? make_double2(a[5].x + a[5].y, a[5].y - a[5].x) : make_double2(a[5].x - a[5].y, a[5].x + a[5].y);
        const double2 s7 = INV ? make_double2(a[7].y - a[7].x, -a[7].x - a[7].y) : make_double2(-a[7].x - a[7].y, a[7].x - a[7].y);
        const double s6 = INV ? -w.sig0 : w.sig0, hi = INV ? -w.tauh : w.tauh;
        const double2 c0 = cmaddi(a[4], s6, a[6]), c1 = cmaddi(a[4], -s6, a[6]);
        const double2 t = cmadd(s5, w.sig1, s7), u = cmadd(s5, -w.sig1, s7);
        emit(1, cmadd(c0, w.tauh, t));
        emit(5, cmadd(c0, -w.tauh, t));
        emit(3, cmaddi(c1, hi, u));
        emit(7, cmaddi(c1, -hi, u));
    }
}

// y[k] = sum_j theta^j x[j] w^(j k): with the twiddles in geometric progression four (cos, tan) pairs --
// theta^4, theta^2, theta, theta w -- serve all twelve butterflies (six instructions each): 72 instead of
// 66, but 16 registers of constants instead of 30.
struct Shift8 {
    double2 h4, h2, h1, h1w;
};
// a +- w b and a +- i w b; b already turned by (1 + i tan)
FFT_HD void bfly(double2 &a, double2 &b, double c) { const double2 p = a, r = b; a = cmadd(p, c, r); b = cmadd(p, -c, r); }
FFT_HD void bfly_i(double2 &a, double2 &b, double c) { const double2 p = a, r = b; a = cmaddi(p, c, r); b = cmaddi(p, -c, r); }

template <bool INV, class Emit, class Between>
FFT_HD void dft8_shifted(double2 (&x)[8], const Shift8 &w, Emit &&emit, Between &&between) {
    const double i2 = INV ? -w.h2.x : w.h2.x, i1 = INV ? -w.h1.x : w.h1.x, i1w = INV ? -w.h1w.x : w.h1w.x;
    for (int j = 0; j < 4; ++j) {
        x[j + 4] = cturn(x[j + 4], w.h4.y);
        bfly(x[j], x[j + 4], w.h4.x);
    }
    x[2] = cturn(x[2], w.h2.y);
    x[3] = cturn(x[3], w.h2.y);
    bfly(x[0], x[2], w.h2.x);
    bfly(x[1], x[3], w.h2.x);
    x[1] = cturn(x[1], w.h1.y);
    x[3] = cturn(x[3], w.h1.y);
    bfly(x[0], x[1], w.h1.x);
    bfly_i(x[2], x[3], i1);
    emit(0, x[0]);
    emit(4, x[1]);
    emit(2, x[2]);
    emit(6, x[3]);
    between();
    x[6] = cturn(x[6], w.h2.y);
    x[7] = cturn(x[7], w.h2.y);
    bfly_i(x[4], x[6], i2);
    bfly_i(x[5], x[7], i2);
    x[5] = cturn(x[5], w.h1w.y);
    x[7] = cturn(x[7], w.h1w.y);
    bfly(x[4], x[5], w.h1w.x);
    bfly_i(x[6], x[7], i1w);
    emit(1, x[4]);
    emit(5, x[5]);
    emit(3, x[6]);
    emit(7, x[7]);
}

template <bool INV>
FFT_HD void dft8_twiddled(double2 (&x)[8], const Twiddle8 &w) {
    double2 y[8];
    dft8_twiddled<INV>(x, w, [&](int k, double2 v) { y[k] = v; }, Nothing());
    for (int k = 0; k < 8; ++k) x[k] = y[k];
}
template <bool INV>
FFT_HD void dft8_shifted(double2 (&x)[8], const Shift8 &w) {
    double2 y[8];
    dft8_shifted<INV>(x, w, [&](int k, double2 v) { y[k] = v; }, Nothing());
    for (int k = 0; k < 8; ++k) x[k] = y[k];
}

// ---- the constants in memory, behind the 2,048 powers of psi (offsets in complex words) ----
// Lane-dependent constants are packed two to a complex word, eight words a lane, word-major.
constexpr int kPsiWords = 2048;
constexpr int kFwd2 = kPsiWords;          // [word 8][k0 8]      forward pass 2
constexpr int kInv2 = kFwd2 + 64;         // [word 8][j0 8]      inverse pass 2
constexpr int kInv1 = kInv2 + 64;         // [word 8][L 64]      inverse pass 1
constexpr int kFwd3 = kInv1 + 512;        // [word 4][lane 64]   forward pass 3, lane = 8 k0 + k1: h4, h2, h1, h1w
constexpr int kFwd2Shift = kFwd3 + 256;   // [word 4][k0 8]      the same form of forward pass 2
constexpr int kInv2Shift = kFwd2Shift + 32;   // [word 4][j0 8]  and of inverse pass 2
constexpr int kUniform = kInv2Shift + 32; // 24 doubles of passes 1: tan, rho, sig0, sig1, tau, tauh; then cos
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
    // theta = psi^e, w = psi^w8
    auto shift = [&](int base, int width, int lane, int e, int w8) {
        const int h[4] = {4 * e, 2 * e, e, e + w8};
        for (int q = 0; q < 4; ++q) {
            const long double c = cosl(angle(h[q]));
            tables[base + q * width + lane] = make_double2((double)c, (double)(sinl(angle(h[q])) / c));
        }
    };
    for (int a = 0; a < 8; ++a) {
        shift(kFwd2Shift, 8, a, 8 * (1 + 4 * a), 256);
        shift(kInv2Shift, 8, a, -32 * a, -256);
        int f[8], g[8];
        for (int j = 0; j < 8; ++j) { f[j] = 8 * j * (1 + 4 * a); g[j] = -32 * a * j; }
        pack(kFwd2, 8, a, f, false);
        pack(kInv2, 8, a, g, false);
    }
    for (int L = 0; L < 64; ++L) {
        int f[8];
        for (int k = 0; k < 8; ++k) f[k] = -L * (1 + 4 * k);
        pack(kInv1, 64, L, f, true);
        shift(kFwd3, 64, L, 1 + 4 * (L >> 3) + 32 * (L & 7), 256);
    }
    long double c[8], v[24] = {};
    for (int m = 0; m < 8; ++m) { c[m] = cosl(pi * m / 16); v[m] = sinl(pi * m / 16) / c[m]; v[16 + m] = c[m]; }
    for (int m = 0; m < 4; ++m) v[8 + m] = c[m + 4] / c[m];
    v[12] = c[2]; v[13] = c[3] / c[1]; v[14] = c[1]; v[15] = c[1] * sqrtl(0.5L);
    for (int q = 0; q < 12; ++q) tables[kUniform + q] = make_double2((double)v[2 * q], (double)v[2 * q + 1]);
}

}  // namespace fft512
