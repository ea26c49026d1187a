// Host run of the transforms of csrc/dft8.h, the two forms the blind rotations use: forward pass 2 and inverse
// pass 2 with the twiddles of a table (one gate per wavefront) or as shifted transforms (four waves per gate).
// The key comes, as on the device, from the steps of csrc/fft512.h.  The products
// sum_r digit_r * limb_{r,o} mod X^1024 + 1 are compared with exact 64-bit integers, and their largest distance
// from an integer with that of the same products through the transforms of fft512.h, on random operands and on
// operands at the ends of their ranges.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <vector>

#include "../../paper_1806_03461_amd/csrc/dft8.h"
#include "fft512_inverse.h"

using namespace fft512;

namespace {

constexpr int kN = 1024, kHalf = 512;
enum Form { kFft512, kTable, kShifted, kForms };
const char *const kNames[kForms] = {"fft512", "dft8 table", "dft8 shifted"};
typedef std::vector<int64_t> Poly;

std::vector<double2> g_tables(kTableWords);
Lane g_lane[64];
double2 g_buf[kBufWords], g_tmp[8][64];

Twiddle8 packed(int base, int width, int lane, double2 (&p)[8]) {
    for (int q = 0; q < 8; ++q) p[q] = g_tables[base + q * width + lane];
    return unpack_twiddles(p);
}
Shift8 shift(int base, int width, int lane) {
    Shift8 s;
    s.h4 = g_tables[base + lane]; s.h2 = g_tables[base + width + lane];
    s.h1 = g_tables[base + 2 * width + lane]; s.h1w = g_tables[base + 3 * width + lane];
    return s;
}
const double *uniform() { return reinterpret_cast<const double *>(&g_tables[kUniform]); }

// X[k0 + 8 k1 + 64 k2]
void forward(Form form, const Poly &p, double scale, double2 *X) {
    double2 x[8];
    Twiddle8 w1;
    w1.t[0] = 0.0;
    const double *u = uniform();
    for (int j = 1; j < 8; ++j) w1.t[j] = u[j];
    for (int j = 0; j < 4; ++j) w1.rho[j] = u[8 + j];
    w1.sig0 = u[12]; w1.sig1 = u[13]; w1.tau = u[14]; w1.tauh = u[15];
    for (int L = 0; L < 64; ++L) {
        for (int m = 0; m < 8; ++m) x[m] = make_double2((double)p[L + 64 * m] * scale, (double)p[L + 64 * m + kHalf] * scale);
        if (form == kFft512) { fwd_pass1_store(x, g_lane[L], g_buf, L); continue; }
        dft8_twiddled<false>(x, w1);
        for (int k = 0; k < 8; ++k) g_buf[k * kRowStride + L] = x[k];
    }
    for (int k0 = 0; k0 < 8; ++k0) {
        double2 *row = g_buf + k0 * kRowStride;
        double2 y[8][8], unused[8];
        for (int j0 = 0; j0 < 8; ++j0) {
            if (form == kFft512) { fwd_pass2_load(y[j0], row, j0); continue; }
            for (int j1 = 0; j1 < 8; ++j1) y[j0][j1] = row[j0 + 8 * j1];
            if (form == kTable) dft8_twiddled<false>(y[j0], packed(kFwd2, 8, k0, unused));
            else dft8_shifted<false>(y[j0], shift(kFwd2Shift, 8, k0));
        }
        if (form == kFft512)
            for (int j0 = 0; j0 < 8; ++j0) fwd_pass2_store(y[j0], g_lane[j0], row, j0);
        for (int k1 = 0; k1 < 8; ++k1) {
            if (form == kFft512) {
                fwd_pass3(x, row, k1);
            } else {
                for (int j0 = 0; j0 < 8; ++j0) x[j0] = y[j0][k1];
                dft8_shifted<false>(x, shift(kFwd3, 64, 8 * k0 + k1));
            }
            for (int k2 = 0; k2 < 8; ++k2) X[k0 + 8 * k1 + 64 * k2] = x[k2];
        }
    }
}

void inverse(Form form, const double2 *X, std::vector<double> &out) {
    out.assign(kN, 0.0);
    for (int k0 = 0; k0 < 8; ++k0) {
        double2 *row = g_buf + k0 * kRowStride;
        double2 y[8][8], x[8], unused[8];
        for (int k1 = 0; k1 < 8; ++k1) {
            for (int k2 = 0; k2 < 8; ++k2) y[k1][k2] = X[k0 + 8 * k1 + 64 * k2];
            if (form == kFft512) inv_pass3_store(y[k1], g_lane[k1], row, k1);
            else if (form == kTable) radix8<true>(y[k1]);
            else { for (int k2 = 0; k2 < 8; ++k2) x[k2] = y[k1][k2];
                   radix8<true>(x, [&](int k, double2 v) { y[k1][k] = v; }, Nothing()); }
        }
        for (int j0 = 0; j0 < 8; ++j0) {
            if (form == kFft512) {
                inv_pass2(x, row, j0);
            } else {
                for (int k1 = 0; k1 < 8; ++k1) x[k1] = y[k1][j0];
                if (form == kTable) dft8_twiddled<true>(x, packed(kInv2, 8, j0, unused));
                else dft8_shifted<true>(x, shift(kInv2Shift, 8, j0));
            }
            for (int j1 = 0; j1 < 8; ++j1) g_tmp[k0][j0 + 8 * j1] = x[j1];
        }
    }
    const double *u = uniform();
    for (int L = 0; L < 64; ++L) {
        double2 x[8], p[8];
        if (form == kFft512) {
            for (int k = 0; k < 8; ++k) g_buf[k * kRowStride + L] = g_tmp[k][L];
            inv_pass1(x, g_lane[L], g_buf, L);
        } else {
            const Twiddle8 w = packed(kInv1, 64, L, p);
            for (int k = 0; k < 8; ++k) x[k] = g_tmp[k][L];
            x[0] = cmul(x[0], p[7]);
            dft8_twiddled<true>(x, w);
            for (int m = 1; m < 8; ++m) {
                x[m] = cturn(x[m], -u[m]);
                x[m] = make_double2(u[16 + m] * x[m].x, u[16 + m] * x[m].y);
            }
        }
        for (int m = 0; m < 8; ++m) { out[L + 64 * m] = x[m].x; out[L + 64 * m + kHalf] = x[m].y; }
    }
}

long g_wrong = 0;
double g_worst[kForms] = {};

// digit[r], limb[r] -> sum_r digit[r] * limb[r]
void product(const char *name, const Poly (&digit)[4], const Poly (&limb)[4]) {
    Poly want(kN, 0);
    for (int r = 0; r < 4; ++r)
        for (int i = 0; i < kN; ++i)
            for (int j = 0; j < kN; ++j) {
                const int64_t v = digit[r][i] * limb[r][j];
                if (i + j < kN) want[i + j] += v;
                else want[i + j - kN] -= v;
            }
    static double2 key[4][kHalf], spectrum[4][kHalf], sum[kHalf];
    for (int r = 0; r < 4; ++r) forward(kFft512, limb[r], 1.0 / 512.0, key[r]);
    printf("%-34s", name);
    for (int form = 0; form < kForms; ++form) {
        for (int r = 0; r < 4; ++r) forward((Form)form, digit[r], 1.0, spectrum[r]);
        for (int k = 0; k < kHalf; ++k) {
            sum[k] = make_double2(0.0, 0.0);
            for (int r = 0; r < 4; ++r) {
                const double2 d = spectrum[r][k], b = key[r][k];
                sum[k] = make_double2(fma(-d.y, b.y, fma(d.x, b.x, sum[k].x)), fma(d.y, b.x, fma(d.x, b.y, sum[k].y)));
            }
        }
        std::vector<double> got;
        inverse((Form)form, sum, got);
        double worst = 0.0;
        for (int j = 0; j < kN; ++j) {
            g_wrong += (int64_t)nearbyint(got[j]) != want[j];
            worst = fmax(worst, fabs(got[j] - (double)want[j]));
        }
        printf("  %s %.3g", kNames[form], worst);
        g_worst[form] = fmax(g_worst[form], worst);
    }
    printf("\n");
}

uint64_t g_state = 0x9E3779B97F4A7C15ull;
uint32_t next_u32() {          // xorshift64*
    g_state ^= g_state >> 12; g_state ^= g_state << 25; g_state ^= g_state >> 27;
    return (uint32_t)((g_state * 0x2545F4914F6CDD1Dull) >> 32);
}

}  // namespace

int main() {
    fill_tables(g_tables.data());
    for (int L = 0; L < 64; ++L) lane_init(g_lane[L], g_tables.data(), L);
    Poly digit[4], limb[4];
    auto fill = [&](auto d, auto l) {
        for (int r = 0; r < 4; ++r) {
            digit[r].assign(kN, 0);
            limb[r].assign(kN, 0);
            for (int j = 0; j < kN; ++j) { digit[r][j] = d(r, j); limb[r][j] = l(r, j); }
        }
    };
    auto random_digit = [](int, int) { return (int64_t)(next_u32() % 1024) - 512; };
    auto random_limb = [](int, int) { return (int64_t)(next_u32() % 65536) - 32768; };
    for (int rep = 0; rep < 8; ++rep) { fill(random_digit, random_limb); product("random digits and limbs", digit, limb); }
    for (int rep = 0; rep < 8; ++rep) {
        fill([](int, int) { return next_u32() & 1 ? 511 : -512; }, [](int, int) { return next_u32() & 1 ? 32767 : -32768; });
        product("extreme magnitudes, random signs", digit, limb);
    }
    for (int de : {-512, 511})
        for (int le : {-32768, 32767}) {
            fill([&](int, int) { return de; }, [&](int, int) { return le; });
            product("all digits and limbs at one end", digit, limb);
        }
    for (int at : {0, 1, 63, 511, 512, 1023}) {     // all 4,096 terms of one coefficient have the same sign
        fill([](int, int) { return -512; }, [&](int, int j) { return j <= at ? -32768 : 32767; });
        product("terms of one coefficient aligned", digit, limb);
    }
    fill([](int r, int j) { return (j >> r) & 1 ? 511 : -512; }, [](int r, int j) { return (j ^ r) & 1 ? 32767 : -32768; });
    product("alternating extremes", digit, limb);
    fill([](int r, int j) { return j == 301 * (r + 1) % kN ? 511 : 0; }, random_limb);
    product("monomial digits", digit, limb);
    printf("dft8 exactness: wrong %ld largest distance fft512 %.3g table %.3g shifted %.3g\n", g_wrong, g_worst[kFft512],
           g_worst[kTable], g_worst[kShifted]);
    return g_wrong != 0;
}
