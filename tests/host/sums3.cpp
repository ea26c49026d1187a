// Host run of the three sums of csrc/sums3.h, with the transforms the wave blind rotation applies: both components of
// sum_r digit_r * key_r mod (X^1024 + 1, 2^32) against 64-bit integers, on random operands and on operands at the ends
// of their ranges.  Prints the wrong coefficients and the largest distance of a value from where it is rounded to.
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>

#include "../../paper_1806_03461_amd/csrc/dft8.h"
#include "../../paper_1806_03461_amd/csrc/sums3.h"

using namespace fft512;

namespace {

constexpr int kN = 1024, kHalf = 512;
std::vector<double2> g_tables(kTableWords);
Lane g_lane[64];
const double *uniform() { return reinterpret_cast<const double *>(&g_tables[kUniform]); }

Twiddle8 packed(int base, int width, int lane, double2 (&p)[8]) {
    for (int q = 0; q < 8; ++q) p[q] = g_tables[base + q * width + lane];
    return unpack_twiddles(p);
}

// X[k0 + 8 k1 + 64 k2], by the steps of fft512.h (the key's) or those of dft8.h (the digits')
void forward(const double *v, bool key, double2 *X) {
    static double2 buf[8 * kRowStride];
    double2 x[8], p[8];
    Twiddle8 w1;
    const double *u = uniform();
    w1.t[0] = 0.0;
    for (int j = 1; j < 8; ++j) w1.t[j] = u[j];
    for (int j = 0; j < 4; ++j) w1.rho[j] = u[8 + j];
    w1.sig0 = u[12]; w1.sig1 = u[13]; w1.tau = u[14]; w1.tauh = u[15];
    for (int L = 0; L < 64; ++L) {
        for (int m = 0; m < 8; ++m) x[m] = make_double2(v[L + 64 * m], v[L + 64 * m + kHalf]);
        if (key) { fwd_pass1_store(x, g_lane[L], buf, L); continue; }
        dft8_twiddled<false>(x, w1);
        for (int k = 0; k < 8; ++k) buf[k * kRowStride + L] = x[k];
    }
    for (int k0 = 0; k0 < 8; ++k0) {
        double2 y[8][8];
        for (int j0 = 0; j0 < 8; ++j0) {
            for (int j1 = 0; j1 < 8; ++j1) y[j0][j1] = buf[k0 * kRowStride + j0 + 8 * j1];
            if (!key) { dft8_twiddled<false>(y[j0], packed(kFwd2, 8, k0, p)); continue; }
            radix8<false>(y[j0]);
            for (int k = 1; k < 8; ++k) y[j0][k] = cmul(y[j0][k], g_lane[j0].tw2[k]);
        }
        for (int k1 = 0; k1 < 8; ++k1) {
            for (int j0 = 0; j0 < 8; ++j0) x[j0] = y[j0][k1];
            if (key) {
                radix8<false>(x);
            } else {
                Shift8 s;
                double2 *const h[4] = {&s.h4, &s.h2, &s.h1, &s.h1w};
                for (int q = 0; q < 4; ++q) *h[q] = g_tables[kFwd3 + 64 * q + 8 * k0 + k1];
                dft8_shifted<false>(x, s);
            }
            for (int k2 = 0; k2 < 8; ++k2) X[k0 + 8 * k1 + 64 * k2] = x[k2];
        }
    }
}

void inverse(const double2 *X, double *out) {
    double2 tmp[8][64], x[8], p[8];
    for (int k0 = 0; k0 < 8; ++k0) {
        double2 y[8][8];
        for (int k1 = 0; k1 < 8; ++k1) {
            for (int k2 = 0; k2 < 8; ++k2) y[k1][k2] = X[k0 + 8 * k1 + 64 * k2];
            radix8<true>(y[k1]);
        }
        for (int j0 = 0; j0 < 8; ++j0) {
            for (int k1 = 0; k1 < 8; ++k1) x[k1] = y[k1][j0];
            dft8_twiddled<true>(x, packed(kInv2, 8, j0, p));
            for (int j1 = 0; j1 < 8; ++j1) tmp[k0][j0 + 8 * j1] = x[j1];
        }
    }
    const double *u = uniform();
    for (int L = 0; L < 64; ++L) {
        const Twiddle8 w = packed(kInv1, 64, L, p);
        for (int k = 0; k < 8; ++k) x[k] = tmp[k][L];
        x[0] = cmul(x[0], p[7]);
        dft8_twiddled<true>(x, w);
        for (int m = 0; m < 8; ++m) {
            if (m) { x[m] = cturn(x[m], -u[m]); x[m] = make_double2(u[16 + m] * x[m].x, u[16 + m] * x[m].y); }
            out[L + 64 * m] = x[m].x;
            out[L + 64 * m + kHalf] = x[m].y;
        }
    }
}

uint32_t low_word(double v) { uint64_t b; std::memcpy(&b, &v, 8); return (uint32_t)b; }

long g_wrong = 0;

template <class Digit, class Key>
void run(const char *name, Digit &&digit_at, Key &&key_at) {
    static int32_t digit[4][kN];
    static uint32_t key[4][2][kN];
    for (int r = 0; r < 4; ++r)
        for (int j = 0; j < kN; ++j) {
            digit[r][j] = digit_at(r, j);
            for (int c = 0; c < 2; ++c) key[r][c][j] = key_at(r, c, j);
        }
    static double2 D[kHalf], K[kHalf], sum[kSums][kHalf];
    std::memset(sum, 0, sizeof sum);
    for (int r = 0; r < 4; ++r) {
        double v[kN];
        for (int j = 0; j < kN; ++j) v[j] = digit[r][j];
        forward(v, false, D);
        for (int o = 0; o < kSums; ++o) {
            for (int j = 0; j < kN; ++j) v[j] = sum_factor(key[r][0][j], key[r][1][j], o) * (1.0 / 512.0);
            forward(v, true, K);
            for (int k = 0; k < kHalf; ++k)
                sum[o][k] = make_double2(fma(-D[k].y, K[k].y, fma(D[k].x, K[k].x, sum[o][k].x)), fma(D[k].y, K[k].x, fma(D[k].x, K[k].y, sum[o][k].y)));
        }
    }
    static double value[kSums][kN];
    for (int o = 0; o < kSums; ++o) inverse(sum[o], value[o]);
    double worst[kSums] = {};
    long wrong = 0;
    for (int j = 0; j < kN; ++j) {
        uint32_t want[2] = {0, 0};
        for (int r = 0; r < 4; ++r)
            for (int i = 0; i < kN; ++i) {
                const int k = (j - i) & (kN - 1);
                const uint32_t d = (uint32_t)(i <= j ? digit[r][i] : -digit[r][i]);
                want[0] += d * key[r][0][k];
                want[1] += d * key[r][1][k];
            }
        uint32_t q = low_word(kIntegerShift + value[0][j]);
        worst[0] = fmax(worst[0], fabs(value[0][j] - nearbyint(value[0][j])));
        for (int c = 0; c < 2; ++c) {
            const uint32_t got = 0u - minus_product(q, low_word(kHalfShift - value[1 + c][j]));
            wrong += got != want[c];
            const double rest = value[1 + c][j] - (double)(want[c] & kSumMask) / (1 << kSumBits);
            worst[1 + c] = fmax(worst[1 + c], fabs(rest - nearbyint(rest)));
        }
    }
    g_wrong += wrong;
    printf("%-28s wrong %ld distance low %.3g top %.3g %.3g\n", name, wrong, worst[0], worst[1], worst[2]);
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
    auto random_digit = [](int, int) { return (int32_t)(next_u32() % 1024) - 512; };
    auto random_key = [](int, int, int) { return next_u32(); };
    for (int rep = 0; rep < 4; ++rep) run("random", random_digit, random_key);
    for (int rep = 0; rep < 2; ++rep)
        run("extremes, random signs", [](int, int) { return next_u32() & 1 ? 511 : -512; },
            [](int, int, int) { return next_u32() & 1 ? 0x7FFFFFFFu : 0x80000000u; });
    // the largest factors of the top sums (2^31) and of the low one (2^21, reached at 0x200000 + 2^11 * 0)
    for (int32_t d : {-512, 511})
        for (uint32_t k : {0x80000000u, 0x7FFFFFFFu, 0x80008000u, 0x00200000u, 0x001FFFFFu, 0xFFFFFFFFu})
            run("all at one end", [&](int, int) { return d; }, [&](int, int c, int) { return c && (k == 0x00200000u || k == 0x001FFFFFu) ? 0u : k; });
    for (int at : {0, 511, 1023})                   // all 4,096 terms of one coefficient have the same sign, in either direction
        for (int flip : {0, 1}) {
            run("terms aligned, top", [&](int, int) { return -512; }, [&](int, int, int j) { return (j <= at) != flip ? 0x80000000u : 0x7FFFFFFFu; });
            run("terms aligned, low", [&](int, int) { return -512; }, [&](int, int c, int j) { return c ? 0u : (j <= at) != flip ? 0x00200000u : 0x001FFFFFu; });
        }
    run("monomial digits", [](int r, int j) { return j == 301 * (r + 1) % kN ? 511 : 0; }, random_key);
    printf("sums3: wrong %ld\n", g_wrong);
    return g_wrong != 0;
}
