// Host run of the transforms of csrc/dft8.h, the two forms the blind rotations use: forward pass 2 and inverse
// pass 2 with the twiddles of a table (one gate per wavefront) or as shifted transforms (four waves per gate).
// The key comes, as on the device, from the steps of csrc/fft512.h.  The products
// sum_r digit_r * limb_{r,o} mod X^1024 + 1 are compared with exact 64-bit integers, and their largest distance
// from an integer with that of the same products through the transforms of fft512.h, on random operands and on
// operands at the ends of their ranges.  A second part runs whole steps lane by lane as the kernels do, with the exchanges through
// LDS and between lanes: four waves per gate with the key's limbs in slot order, one wave per gate with the factors of
// csrc/sums3.h where the upload stores them for it, up to the two components mod 2^32.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>

#include "../../paper_1806_03461_amd/csrc/dft8.h"
#include "../../paper_1806_03461_amd/csrc/sums3.h"
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

// ---- whole steps, lane by lane ----
typedef double2 Lanes[4][64][8];        // [wave or polynomial][lane][register]
Lanes g_x;
double2 g_key[4][4][kHalf];             // [row][output][slot]
double2 g_sum_key[kSumKeyWords];
struct KeyRows { uint32_t word[4][2][kN]; };        // [row][component]

Twiddle8 pass1() {
    Twiddle8 w;
    const double *u = uniform();
    w.t[0] = 0.0;
    for (int j = 1; j < 8; ++j) w.t[j] = u[j];
    for (int j = 0; j < 4; ++j) w.rho[j] = u[8 + j];
    w.sig0 = u[12]; w.sig1 = u[13]; w.tau = u[14]; w.tauh = u[15];
    return w;
}
template <class P>
void fold(const P *p, int count, double scale) {
    for (int r = 0; r < count; ++r)
        for (int L = 0; L < 64; ++L)
            for (int m = 0; m < 8; ++m)
                g_x[r][L][m] = make_double2((double)p[r][L + 64 * m] * scale, (double)p[r][L + 64 * m + kHalf] * scale);
}
#define LANES for (int L = 0; L < 64; ++L)
#define REGISTERS for (int k = 0; k < 8; ++k)

// the key as the upload stores it: the steps of fft512.h, four polynomials of a row at a time, gathered
void transform_row() {
    for (int w = 0; w < 4; ++w) LANES fwd_pass1_store(g_x[w][L], g_lane[L], g_buf + w * kPolyStride, L);
    for (int w = 0; w < 4; ++w) {
        LANES fwd_pass2_load(g_x[w][L], g_buf + row_of(w, L), L);
        LANES fwd_pass2_store(g_x[w][L], g_lane[L], g_buf + row_of(w, L), L);
        LANES fwd_pass3(g_x[w][L], g_buf + row_of(w, L), L);
        gather_rows_wave(g_x[w]);
    }
}
void store_key(const Poly (&limb)[4][4]) {
    for (int r = 0; r < 4; ++r) {
        fold(limb[r], 4, 1.0 / 512.0);
        transform_row();
        for (int w = 0; w < 4; ++w)
            LANES for (int o = 0; o < 4; ++o)
                for (int q = 0; q < 2; ++q) g_key[r][o][256 * q + 64 * w + L] = g_x[w][L][2 * o + q];
    }
}
void store_sum_key(const KeyRows &key) {
    std::fill(g_sum_key, g_sum_key + kSumKeyWords, make_double2(NAN, NAN));      // a word that is not written shows
    std::vector<double> factor[4];
    for (int r = 0; r < 4; ++r) {
        for (int o = 0; o < 4; ++o) {
            factor[o].assign(kN, 0.0);
            for (int j = 0; j < kN && o < kSums; ++j) factor[o][j] = sum_factor(key.word[r][0][j], key.word[r][1][j], o);
        }
        fold(factor, 4, 1.0 / 512.0);
        transform_row();
        for (int w = 0; w < 4; ++w)
            LANES for (int o = 0; o < kSums; ++o)
                for (int q = 0; q < 2; ++q) g_sum_key[sum_key_word(whole_register(L, q), o, r, whole_lane(w, L))] = g_x[w][L][2 * o + q];
    }
}
// inverse pass 1 and the pending cosines of one lane
void finish(double2 (&x)[8], int L, std::vector<double> &out) {
    double2 p[8];
    const double *u = uniform();
    const Twiddle8 w = packed(kInv1, 64, L, p);
    x[0] = cmul(x[0], p[7]);
    dft8_twiddled<true>(x, w);
    for (int m = 0; m < 8; ++m) {
        if (m) { x[m] = cturn(x[m], -u[m]); x[m] = make_double2(u[16 + m] * x[m].x, u[16 + m] * x[m].y); }
        out[L + 64 * m] = x[m].x;
        out[L + 64 * m + kHalf] = x[m].y;
    }
}
template <class Key>
double2 row_times_key(const double2 (&d)[4], Key &&key) {
    double2 y = make_double2(0.0, 0.0);
    for (int r = 0; r < 4; ++r) {
        const double2 b = key(r);
        y = make_double2(fma(-d[r].y, b.y, fma(d[r].x, b.x, y.x)), fma(d[r].y, b.x, fma(d[r].x, b.y, y.y)));
    }
    return y;
}

// four waves per gate: wave r transforms polynomial r in pass 1 and holds rows 2 w, 2 w + 1 of all afterwards
void step_four_waves(const Poly (&digit)[4], std::vector<double> (&out)[4]) {
    fold(digit, 4, 1.0);
    const Twiddle8 w1 = pass1();
    for (int w = 0; w < 4; ++w) LANES {
        dft8_twiddled<false>(g_x[w][L], w1);
        REGISTERS g_buf[w * kPolyStride + k * kRowStride + L] = g_x[w][L][k];
    }
    for (int w = 0; w < 4; ++w) {
        auto mine = [&](int L) { return g_buf + row_of(w, L); };
        auto k0 = [&](int L) { return 2 * w + (L >> 3 & 1); };
        double2 (&x)[64][8] = g_x[w];
        LANES REGISTERS x[L][k] = mine(L)[(L & 7) + 8 * k];
        LANES dft8_shifted<false>(x[L], shift(kFwd2Shift, 8, k0(L)));
        LANES REGISTERS mine(L)[k * kGrpStride + (L & 7)] = x[L][k];
        LANES REGISTERS x[L][k] = mine(L)[(L & 7) * kGrpStride + k];
        LANES dft8_shifted<false>(x[L], shift(kFwd3, 64, 8 * k0(L) + (L & 7)));
        gather_rows_wave(x);
        LANES {
            double2 y[8];
            for (int o = 0; o < 4; ++o)
                for (int q = 0; q < 2; ++q) {
                    const double2 d[4] = {x[L][q], x[L][2 + q], x[L][4 + q], x[L][6 + q]};
                    y[2 * o + q] = row_times_key(d, [&](int r) { return g_key[r][o][256 * q + 64 * w + L]; });
                }
            REGISTERS x[L][k] = y[k];
        }
        scatter_rows_wave(x);
        LANES radix8<true>(x[L]);
        LANES REGISTERS mine(L)[(L & 7) * kGrpStride + k] = x[L][k];
        LANES REGISTERS x[L][k] = mine(L)[k * kGrpStride + (L & 7)];
        LANES dft8_shifted<true>(x[L], shift(kInv2Shift, 8, L & 7));
        LANES REGISTERS mine(L)[(L & 7) + 8 * k] = x[L][k];
    }
    for (int o = 0; o < 4; ++o) LANES {
        REGISTERS g_x[o][L][k] = g_buf[o * kPolyStride + k * kRowStride + L];
        finish(g_x[o][L], L, out[o]);
    }
}

// one wave per gate: each polynomial through the wave's one buffer, lane = 8 k0 + (j0 or k1)
void step_one_wave(const Poly (&digit)[4], std::vector<double> (&out)[kSums]) {
    fold(digit, 4, 1.0);
    const Twiddle8 w1 = pass1();
    double2 p[8];
    auto mine = [&](int L) { return g_buf + (L >> 3) * kRowStride; };
    for (int r = 0; r < 4; ++r) {
        double2 (&x)[64][8] = g_x[r];
        LANES { dft8_twiddled<false>(x[L], w1); REGISTERS g_buf[k * kRowStride + L] = x[L][k]; }
        LANES REGISTERS x[L][k] = mine(L)[(L & 7) + 8 * k];
        LANES dft8_twiddled<false>(x[L], packed(kFwd2, 8, L >> 3, p));
        LANES REGISTERS mine(L)[k * kGrpStride + (L & 7)] = x[L][k];
        LANES REGISTERS x[L][k] = mine(L)[(L & 7) * kGrpStride + k];
        LANES dft8_shifted<false>(x[L], shift(kFwd3, 64, L));
    }
    LANES REGISTERS {
        const double2 d[4] = {g_x[0][L][k], g_x[1][L][k], g_x[2][L][k], g_x[3][L][k]};
        for (int o = 0; o < kSums; ++o) g_x[o][L][k] = row_times_key(d, [&](int r) { return g_sum_key[sum_key_word(k, o, r, L)]; });
    }
    for (int o = 0; o < kSums; ++o) {
        double2 (&x)[64][8] = g_x[o];
        LANES radix8<true>(x[L]);
        LANES REGISTERS mine(L)[(L & 7) * kGrpStride + k] = x[L][k];
        LANES REGISTERS x[L][k] = mine(L)[k * kGrpStride + (L & 7)];
        LANES dft8_twiddled<true>(x[L], packed(kInv2, 8, L & 7, p));
        LANES REGISTERS mine(L)[(L & 7) + 8 * k] = x[L][k];
        LANES { REGISTERS x[L][k] = g_buf[k * kRowStride + L]; finish(x[L], L, out[o]); }
    }
}

// the four-wave kernels' step against exact integers; returns the number of wrong coefficients
long steps(const Poly (&digit)[4], const Poly (&limb)[4][4], double &worst) {
    store_key(limb);
    std::vector<double> out[4];
    for (auto &o : out) o.assign(kN, 0.0);
    step_four_waves(digit, out);
    long wrong = 0;
    for (int o = 0; o < 4; ++o) {
        Poly want(kN, 0);
        for (int r = 0; r < 4; ++r)
            for (int i = 0; i < kN; ++i)
                for (int j = 0; j < kN; ++j) {
                    const int64_t v = digit[r][i] * limb[r][o][j];
                    if (i + j < kN) want[i + j] += v;
                    else want[i + j - kN] -= v;
                }
        for (int j = 0; j < kN; ++j) {
            wrong += (int64_t)nearbyint(out[o][j]) != want[j];
            worst = fmax(worst, fabs(out[o][j] - (double)want[j]));
        }
    }
    return wrong;
}
// the wave kernel's step, both components mod 2^32; returns the number of wrong coefficients
long sum_steps(const Poly (&digit)[4], const KeyRows &key) {
    store_sum_key(key);
    std::vector<double> out[kSums];
    for (auto &o : out) o.assign(kN, 0.0);
    step_one_wave(digit, out);
    auto low_word = [](double v) { uint64_t b; std::memcpy(&b, &v, 8); return (uint32_t)b; };
    long wrong = 0;
    for (int j = 0; j < kN; ++j) {
        uint32_t q = low_word(kIntegerShift + out[0][j]);
        for (int c = 0; c < 2; ++c) {
            uint32_t want = 0;
            for (int r = 0; r < 4; ++r)
                for (int i = 0; i < kN; ++i) {
                    const uint32_t v = (uint32_t)digit[r][i] * key.word[r][c][(j - i) & (kN - 1)];
                    want += i <= j ? v : 0u - v;
                }
            wrong += minus_product(q, low_word(kHalfShift - out[1 + c][j])) != 0u - want;
        }
    }
    return wrong;
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
    {
        Poly rows[4][4];
        double worst = 0.0;
        long wrong = 0;
        for (int rep = 0; rep < 4; ++rep) {
            fill(random_digit, random_limb);
            for (int r = 0; r < 4; ++r)
                for (int o = 0; o < 4; ++o) {
                    rows[r][o].assign(kN, 0);
                    for (int j = 0; j < kN; ++j) rows[r][o][j] = rep == 3 ? (next_u32() & 1 ? 32767 : -32768) : random_limb(r, j);
                }
            if (rep == 2) fill([](int r, int j) { return j == 301 * (r + 1) % kN ? 511 : 0; }, random_limb);
            wrong += steps(digit, rows, worst);
            static KeyRows key;
            for (auto &row : key.word) for (auto &component : row) for (uint32_t &word : component) word = rep == 3 ? 0x80000000u - (next_u32() & 1) : next_u32();
            wrong += sum_steps(digit, key);
        }
        printf("whole steps: wrong %ld largest distance %.3g\n", wrong, worst);
        g_wrong += wrong;
    }
    printf("dft8 exactness: wrong %ld largest distance fft512 %.3g table %.3g shifted %.3g\n", g_wrong, g_worst[kFft512],
           g_worst[kTable], g_worst[kShifted]);
    return g_wrong != 0;
}
