// The rest of a multiplication through the transforms of csrc/fft512.h, for host programs that drive a workgroup's
// lanes one after the other: the inverse steps -- the forward ones backwards, with conjugate twiddles; the
// blind rotations invert with csrc/dft8.h instead -- and the exchanges between the lanes of a wave.
#pragma once
#include "../../paper_1806_03461_amd/csrc/fft512.h"

namespace fft512 {

FFT_HD double2 cmulc(double2 a, double2 b) {   // a * conj(b)
    return make_double2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}

// ---- inverse (unnormalised: 512 times the folded, untwisted points come out) -----------
FFT_HD void inv_pass3_store(double2 (&x)[8], const Lane &ln, double2 *row, int L) {
    radix8<true>(x);
    const int base = (L & 7) * kGrpStride;
    row[base] = x[0];
    for (int j0 = 1; j0 < 8; ++j0) row[base + j0] = cmulc(x[j0], ln.tw2[j0]);
}
FFT_HD void inv_pass2(double2 (&x)[8], const double2 *row, int L) {
    const int j0 = L & 7;
    for (int k = 0; k < 8; ++k) x[k] = row[k * kGrpStride + j0];
    radix8<true>(x);
}
FFT_HD void inv_pass2_store(const double2 (&x)[8], double2 *row, int L) {
    const int j0 = L & 7;
    for (int j1 = 0; j1 < 8; ++j1) row[j0 + 8 * j1] = x[j1];
}
// wave o, from its polynomial's buffer
FFT_HD void inv_pass1(double2 (&x)[8], const Lane &ln, const double2 *poly, int L) {
    for (int k = 0; k < 8; ++k) x[k] = cmulc(poly[k * kRowStride + L], ln.tw1[k]);
    radix8<true>(x);
    for (int m = 1; m < 8; ++m) x[m] = cmulc(x[m], twist_const(m));
}

// gather_rows and scatter_rows written out over the registers of a whole wave (x[lane][register]), for
// host code that drives the lanes one after the other.
inline void gather_rows_wave(double2 (*x)[8]) {
    for (int bit = 5; bit >= 4; --bit) {
        const int d = 1 << bit, rs = bit == 5 ? 4 : 2;      // lane distance, register distance
        for (int L = 0; L < 64; ++L) {
            if (L & d) continue;
            for (int k = 0; k < 8; ++k) {
                if (k & rs) continue;
                const double2 t = x[L][k + rs];
                x[L][k + rs] = x[L + d][k];
                x[L + d][k] = t;
            }
        }
    }
}
inline void scatter_rows_wave(double2 (*x)[8]) {
    for (int bit = 4; bit <= 5; ++bit) {
        const int d = 1 << bit, rs = bit == 5 ? 4 : 2;
        for (int L = 0; L < 64; ++L) {
            if (L & d) continue;
            for (int k = 0; k < 8; ++k) {
                if (k & rs) continue;
                const double2 t = x[L][k + rs];
                x[L][k + rs] = x[L + d][k];
                x[L + d][k] = t;
            }
        }
    }
}

}  // namespace fft512
