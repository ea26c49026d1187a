// gfx950 kernels: transform-domain bootstrapping key, blind rotation, key switch, output gather.
//
// The bootstrapped gate is the CGGI gate the TAPAS paper builds its circuits from
// (Sec. 3.1.2, Sec. 4.1); the paper gives no construction, the steps are the public ones.
//
// Exactness.  Each blind-rotation step needs, for both TRLWE components c,
//     sum_{r<4} digit_r(X) * BK_i[r][c](X)   mod (X^1024 + 1, 2^32),
// digit_r with coefficients in [-512, 512).  The products are integer ones, computed with double-precision FFTs whose
// rounding error stays far below 1/2, so rounding the inverse transforms gives them exactly.  The key's 32 bits a
// coefficient are too many for one such product.  The four-wave kernels split every coefficient into two signed 16-bit
// limbs, key = lo + 2^16 hi (mod 2^32): four products for the two components, coefficients below 2^36, and the result is
// lo-sum + 2^16 * hi-sum (mod 2^32).  The wave kernel gets both components from three products (sums3.h).  MI355X
// issues FP64 FMAs at full vector rate, which makes this cheaper than any 32-bit-integer number-theoretic transform on
// its VALU.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstddef>
#include <cstdlib>

#include "common.h"
#include "dft8.h"
#include "fft512.h"
#include "kernels.h"
#include "sums3.h"

namespace tfhe {

using namespace fft512;

namespace {

constexpr int kN = 1024;
constexpr int kHalf = 512;
constexpr int kThreadsPerGate = 256;
constexpr uint32_t kEighth = 1u << 29;

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ------------------------------------------------------------------------------------------
// Bootstrapping key -> transform domain, in both forms: with the key's limbs for the four-wave kernels, with the factors of
// sums3.h for the wave kernel.  Two workgroups per sample row (i, r), one for each form: the four waves of the first
// transform the four polynomials o = 2*component + limb with the very steps the blind rotation applies to its four digit
// polynomials, so the spectra land in the slot order the products use; of the second's waves, three the three factors.
// bk_raw [n][4][2][1024] uint32  ->  bk_fft [n][4 rows][o][512] complex, and behind all of it [n][k2 8][3 sums][4 rows][64 lanes].
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void bk_to_spectrum_kernel(const uint32_t *__restrict__ bk_raw,
                                                             double2 *__restrict__ bk_fft,
                                                             const double2 *__restrict__ tables) {
    __shared__ double2 buf[kBufWords];
    const int L = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const size_t row = blockIdx.x >> 1;            // i * 4 + r
    const bool sums = blockIdx.x & 1;
    const int c = wv >> 1, limb = wv & 1;          // pass 1: wave o = 2 c + limb, or o of sums3.h
    const uint32_t *src = bk_raw + row * 2 * kN;
    Lane ln;
    lane_init(ln, tables, L);
    double2 x[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        const int j = L + 64 * m;
        double v[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (sums) {
                v[h] = wv < kSums ? sum_factor(src[j + h * kHalf], src[kN + j + h * kHalf], wv) : 0.0;
            } else {
                const uint32_t w = src[c * kN + j + h * kHalf];
                const int32_t lo = (int16_t)(w & 0xFFFFu);
                const int32_t hi = (int16_t)(((w - (uint32_t)lo) >> 16) & 0xFFFFu);
                v[h] = (double)(limb ? hi : lo);
            }
        }
        // the 1/512 of the inverse transform is folded into the key (exact: a power of two)
        x[m] = make_double2(v[0] * (1.0 / 512.0), v[1] * (1.0 / 512.0));
    }
    fwd_pass1_store(x, ln, buf + wv * kPolyStride, L);
    __syncthreads();
    double2 *mine = buf + row_of(wv, L);
    fwd_pass2_load(x, mine, L);
    wave_sync();
    fwd_pass2_store(x, ln, mine, L);
    wave_sync();
    fwd_pass3(x, mine, L);
    gather_rows(x);
    if (sums) {
        double2 *out = bk_fft + (size_t)(gridDim.x >> 1) * 4 * kHalf + (row >> 2) * (size_t)kSumKeyWords;
#pragma unroll
        for (int o = 0; o < kSums; ++o)
#pragma unroll
            for (int q = 0; q < 2; ++q) out[sum_key_word(whole_register(L, q), o, (int)(row & 3), whole_lane(wv, L))] = x[2 * o + q];
        return;
    }
    double2 *out = bk_fft + row * (size_t)(4 * kHalf);
#pragma unroll
    for (int o = 0; o < 4; ++o)
#pragma unroll
        for (int q = 0; q < 2; ++q) out[(size_t)o * kHalf + 256 * q + threadIdx.x] = x[2 * o + q];
}

// ------------------------------------------------------------------------------------------
// Blind rotation, one gate per workgroup of 256 threads (4 waves).
//   prologue  c = (0, kappa) + m (s0 c0 + s1 c1); abar_j = round(c_j * 2N / 2^32); ACC = (0, X^-bbar v)
//   n steps   D = X^abar_i ACC - ACC; wave r = (component, digit) decomposes its digit polynomial
//             and runs pass 1 of its forward FFT; after a barrier wave w carries the frequencies
//             k0 = 2w, 2w+1 of all four polynomials through passes 2 and 3, gathers the four
//             spectra of each of its frequencies into one lane, multiplies them with the key row
//             in registers, scatters the four output spectra o = (component, limb) back and runs
//             the inverse passes 3 and 2; after a second barrier wave o runs inverse pass 1,
//             rounds and adds into ACC; a third barrier closes the step
//   epilogue  sample extraction of coefficient 0 -> ext[gate][1025]
// A workgroup takes gates blockIdx.x, blockIdx.x + gridDim.x, ...; launches normally have one
// workgroup per gate (see resident_groups()).
// ------------------------------------------------------------------------------------------
constexpr int kMirror = 64;       // coefficients 0..63 of each accumulator component are kept a second time
struct GateLds {
    // accumulator (mask, body), stored bitwise complemented: c = ~ACC = -ACC - 1.  Behind each component
    // sits a mirror of its first 64 coefficients, stored as -c - 2: a rotated read of 64 consecutive
    // coefficients that runs past X^N continues into the mirror, and the value found there already
    // carries the sign change of X^N = -1 (see the rotation in blind_rotate_body)
    uint32_t acc[2][kN + kMirror];
    // the four polynomials' transform buffers, without the gap behind the last: the LDS of a workgroup is
    // given out in units of 1,280 bytes, and with it three of them would not fit a CU
    double2 buf[kBufWords - 16];
    double2 inv1[5 * 64];         // words 0..4 of the constants of inverse pass 1 (dft8.h)
    uint16_t bar[1032];           // abar_0 .. abar_{n-1}, bbar
};
static_assert(3 * ((sizeof(GateLds) + 1279) / 1280 * 1280) <= 160 * 1024, "three workgroups share a CU's LDS");

__device__ __forceinline__ void gate_constants(int op, uint32_t &kappa, uint32_t &mult) {
    switch (op) {
    case TFHE_NAND: kappa = kEighth;          mult = 0xFFFFFFFFu; break;
    case TFHE_AND:  kappa = 0u - kEighth;     mult = 1u;          break;
    case TFHE_OR:   kappa = kEighth;          mult = 1u;          break;
    case TFHE_NOR:  kappa = 0u - kEighth;     mult = 0xFFFFFFFFu; break;
    case TFHE_XOR:  kappa = 2u * kEighth;     mult = 2u;          break;
    default:        kappa = 0u - 2u * kEighth; mult = 0xFFFFFFFEu; break;   // XNOR
    }
}

// 16-byte load from a buffer: descriptor and soffset are scalar, voffset is the lane's byte offset
__device__ __forceinline__ double2 load_key(__amdgpu_buffer_rsrc_t rsrc, uint32_t voffset, uint32_t soffset) {
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)voffset, (int)soffset, 0);
    double2 out;
    out.x = __hiloint2double((int)v.y, (int)v.x);
    out.y = __hiloint2double((int)v.w, (int)v.z);
    return out;
}

// The constants that are the same in every lane come through the scalar cache, in most kernels once a step (the pointer is
// made opaque, or the compiler keeps all of them in scalar registers over the loop and spills).
typedef __attribute__((address_space(4))) const double const_double;
__device__ __forceinline__ const_double *uniform_constants(const double2 *tables) {
    const_double *p = (const_double *)(uintptr_t)(tables + kUniform);
    asm volatile("" : "+s"(p));
    return p;
}
__device__ __forceinline__ Twiddle8 pass1_twiddles(const_double *u) {
    Twiddle8 w;
    w.t[0] = 0.0;
#pragma unroll
    for (int j = 1; j < 8; ++j) w.t[j] = u[j];
#pragma unroll
    for (int j = 0; j < 4; ++j) w.rho[j] = u[8 + j];
    w.sig0 = u[12]; w.sig1 = u[13]; w.tau = u[14]; w.tauh = u[15];
    return w;
}

// A step's key values of one thread come in four parts of 8 (32 registers): part p = 2 q + h holds
// rows r = 0..3 x outputs o = 2h, 2h+1 at the thread's slot 256 q + tid.
// AHEAD: the variants for one or two workgroups per CU request the key row in eight portions of four loads, ahead of the products that
// use it.  With two workgroups all eight are of the row of step i + 1 and stand between the phases that follow the products of step i.
// LONE: one workgroup per CU.  A portion keeps the CU's one address unit busy for 4 x 16 clocks per wave, and a wave alone
// on its SIMD cannot issue anything else meanwhile, so all 32 loads in one place stall all four waves.  Six portions are of step i + 1: two
// after the products, two and one in the waits for the inverse exchanges, one behind the step's last barrier; the other two (3 and 7)
// are of step i itself, behind its first barrier, still an exchange and two passes ahead of their use.  All stand where the wave waits
// anyway; which of these places, and which of them the scheduler may not move instructions across, was found by timing about 250
// arrangements: one portion after each of eight phases 1.530 ms for 8 gates and 1.588 for 256, this one 1.482 and 1.524, most
// others 1.50 to 1.64.  What tells them apart is how four waves in step meet at the address unit and at LDS, which no rule here predicts:
// another compiler's order of instructions may want another one.  The way from L2 is longer than with single portions (counted 104
// clocks then, 178 to 189 now that portions stand in pairs) and is covered.
// Two workgroups per CU hide that behind each other; there the last two portions go with earlier ones, a step's length
// ahead of their use, which also saves the registers of the loads in flight across forward passes 2 and 3 (301 gates 1.96 -> 1.94 ms, and no scratch).
// At three workgroups per CU the others cover the loads and holding registers for them does not pay:
// with two parts kept in flight (registers freed by moving the pass-2 twiddles to LDS) a launch of
// 65,536 gates took 390-410 ms instead of 266-278.  The wait for a key row that no workgroup of the
// XCD has touched yet is what keeps the workgroups of an XCD within the few rows its L2 holds.
template <bool MARGIN, int AHEAD, bool LONE>
__device__ __forceinline__ void blind_rotate_body(const BlindRotateArgs &a) {
    extern __shared__ __align__(4096) unsigned char lds_raw[];
    GateLds &my = *reinterpret_cast<GateLds *>(lds_raw);
    static_assert(AHEAD == 0 || AHEAD == 4, "no key values or a whole step's ahead");

    // The accumulator's components: with their mirrors in the throughput kernel, 4 KB each from a multiple of
    // 4 KB on, without mirrors, in the latency kernel (see the rotation).
    auto acc = [&](int c) -> uint32_t * { return LONE ? reinterpret_cast<uint32_t *>(lds_raw) + c * kN : my.acc[c]; };

    const int tid = threadIdx.x;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);     // wave, in a scalar register
    const int L = tid & 63;

    // Constants of the passes (dft8.h).  Those of inverse pass 1 are the largest set: five of its eight words
    // wait in LDS, read while the barrier before the pass is waited for.
    const int k0 = 2 * wv + (L >> 3 & 1);
    Shift8 f2, f3, i2;
    f2.h4 = a.tables[kFwd2Shift + k0]; f2.h2 = a.tables[kFwd2Shift + 8 + k0];
    f2.h1 = a.tables[kFwd2Shift + 16 + k0]; f2.h1w = a.tables[kFwd2Shift + 24 + k0];
    f3.h4 = a.tables[kFwd3 + 8 * k0 + (L & 7)]; f3.h2 = a.tables[kFwd3 + 64 + 8 * k0 + (L & 7)];
    f3.h1 = a.tables[kFwd3 + 128 + 8 * k0 + (L & 7)]; f3.h1w = a.tables[kFwd3 + 192 + 8 * k0 + (L & 7)];
    i2.h4 = a.tables[kInv2Shift + (L & 7)]; i2.h2 = a.tables[kInv2Shift + 8 + (L & 7)];
    i2.h1 = a.tables[kInv2Shift + 16 + (L & 7)]; i2.h1w = a.tables[kInv2Shift + 24 + (L & 7)];
    // With the key row ahead and the rounding distance recorded, two workgroups per CU have no registers for the other three.
    constexpr bool kSpare = MARGIN && AHEAD && !LONE;
    double2 i1[3];
    for (int q = 0; q < 3; ++q) i1[q] = a.tables[kInv1 + (5 + q) * 64 + L];
    for (int e = tid; e < 5 * 64; e += kThreadsPerGate) my.inv1[e] = a.tables[kInv1 + e];
    auto pause = [] { __builtin_amdgcn_sched_barrier(0); };
    auto pause_if_shared = [] { if (!LONE) __builtin_amdgcn_sched_barrier(0); };
    auto lone_pause = [] { if (LONE) __builtin_amdgcn_sched_barrier(0); };
    // The constants that are the same in every lane.  With one or two workgroups per CU nobody covers the waits for them, which
    // also wait for every LDS read in flight: forward pass 1 keeps its own over the loop, and a lone workgroup, whose rotation
    // needs no scalar registers, the cosines of the rounding too (8 gates 1.555 -> 1.53 ms a call; 301 gates 2.02 -> 1.975, 512 gates
    // 2.32 -> 2.21; there with the cosines 2.02 and 2.26).
    const_double *const kept = uniform_constants(a.tables);
    const Twiddle8 kept_w1 = pass1_twiddles(kept);
    double kept_cos[8];
    for (int m = 1; m < 8; ++m) kept_cos[m] = kept[16 + m];
    const __amdgpu_buffer_rsrc_t key_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<double2 *>(a.bk_fft), 0, (int)((size_t)a.n * 16 * kHalf * sizeof(double2)), 0x00020000);
    const uint32_t voff = (uint32_t)tid * (uint32_t)sizeof(double2);
    // value of row r, output 2 (part & 1) + o2 at slot 256 (part >> 1) + tid; the two slots of a thread share the scalar
    // offset, so that the compiler forms it once for both (against one each: 64 gates 1.59 -> 1.54 ms, 301 gates and more equal)
    auto key = [&](int row, int part, int r, int o2) {
        return load_key(key_rsrc, voff + (part >> 1 ? 4096u : 0u),
                        (uint32_t)row * 16u * kHalf * (uint32_t)sizeof(double2) +
                            (uint32_t)((r * 4 + 2 * (part & 1) + o2) * kHalf * sizeof(double2)));
    };

    const int comp = wv >> 1;                   // pass 1 forward: component of D; inverse: component of ACC
    const int sel = wv & 1;                     // pass 1 forward: digit index; inverse: limb
    // Signed digit `sel` of x: add the rounding constant and the half-bases of the lower digits
    // (not its own: its two's-complement field then already is the centred digit), move the
    // field to the top of the word, shift back down arithmetically.
    const uint32_t dround = 1u << (31 - 2 * a.bgbit);
    const uint32_t doffset = sel ? dround : dround + (1u << (31 - a.bgbit));
    const uint32_t dfield = (uint32_t)(32 - a.bgbit * (1 + sel));   // lowest bit of the digit's field
    double2 *const poly = my.buf + wv * kPolyStride;      // pass 1: this wave's polynomial
    double2 *const mine = my.buf + row_of(wv, L);         // passes 2, 3: this lane's row
    double worst = 0.0;
    // Wave priority, throughput kernel only (two or three workgroups share a CU): the phases that lead up to a
    // barrier or follow one directly -- rotation and forward pass 1, inverse pass 1 and the accumulation -- issue
    // first, forward passes 2 and 3 next, and the other workgroups' gather, products and scatter, which wait
    // on swaps and key loads anyway, last.  Measured against one high level for all of the former: 301 gates
    // 2.23 -> 2.21 ms, 512 gates 2.29 -> 2.27, 768 gates 3.42 -> 3.34; raising the gather instead costs up to 30 %.
    auto priority = [](int level) {
        if (LONE) return;                // a lone workgroup per CU has nobody to overtake
        if (level == 2) __builtin_amdgcn_s_setprio(2);
        else if (level == 1) __builtin_amdgcn_s_setprio(1);
        else __builtin_amdgcn_s_setprio(0);
    };

    for (size_t gi = a.first + blockIdx.x; gi < a.count; gi += gridDim.x) {
    // ---- prologue ----
    {
        int op = a.uniform_op;
        size_t i0 = gi, i1 = gi;
        uint32_t s0 = 1u, s1 = 1u;
        const uint32_t *src1 = a.in1;
        if (a.recs) {
            const tfhe_gate_rec r = a.recs[gi];
            op = r.op; i0 = (size_t)r.in0; i1 = (size_t)r.in1;
            s0 = r.neg0 ? 0xFFFFFFFFu : 1u; s1 = r.neg1 ? 0xFFFFFFFFu : 1u;
        } else if (op == TFHE_MUX) {
            i0 = i1 = gi >> 1;
            if (gi & 1) { op = TFHE_MUX_ELSE; src1 = a.in1_alt; }
        }
        // a multiplexer half is an AND whose result stays under the ring key:
        // AND(s, a), then AND(NOT s, b)
        if (op == TFHE_MUX_ELSE) s0 = 0u - s0;
        if (op >= TFHE_MUX) op = TFHE_AND;
        uint32_t kappa, mult;
        gate_constants(op, kappa, mult);
        const size_t w = (size_t)a.n + 1;
        for (int j = tid; j <= a.n; j += kThreadsPerGate) {
            uint32_t c = mult * (s0 * a.in0[i0 * w + j] + s1 * src1[i1 * w + j]);
            if (j == a.n) c += kappa;
            my.bar[j] = (uint16_t)(((c + (1u << 20)) >> 21) & 2047u);
        }
    }
    __syncthreads();
    {
        const int bbar = my.bar[a.n];
        const int bb = bbar & (kN - 1);
        const uint32_t first = bbar < kN ? kEighth : 0u - kEighth;   // X^-bbar v, closed form
        for (int j = tid; j < kN; j += kThreadsPerGate) {
            const uint32_t c = ~(j < kN - bb ? first : 0u - first);
            acc(0)[j] = ~0u;
            acc(1)[j] = c;
            if (!LONE && j < kMirror) { my.acc[0][kN + j] = 0u - ~0u - 2u; my.acc[1][kN + j] = 0u - c - 2u; }
        }
    }
    __syncthreads();

    double2 ahead[AHEAD ? AHEAD : 1][4][2];     // [part][row][output of the pair]
    // portion e of 8: rows 2 (e & 1), 2 (e & 1) + 1 of part e >> 1
    auto load_ahead = [&](int row, int e) {
        if (!AHEAD) return;
#pragma unroll
        for (int r = 2 * (e & 1); r < 2 * (e & 1) + 2; ++r)
#pragma unroll
            for (int o2 = 0; o2 < 2; ++o2)
                ahead[e >> 1][r][o2] = key(row, e >> 1, r, o2);
    };
#pragma unroll
    for (int e = 0; e < 8; ++e)
        if (!LONE || (e & 3) != 3) load_ahead(0, e);      // a lone workgroup requests portions 3 and 7 in the step itself

    int abar_next = my.bar[0];
    for (int i = 0; i < a.n; ++i) {
        double2 x[8];
        priority(2);
        {
        // ---- rotate, subtract, decompose, fold and twist ----
        // read one step ahead (off the critical path); the same in every lane, so it goes to a scalar
        // register and everything below that does not depend on the lane is scalar arithmetic
        const int abar = __builtin_amdgcn_readfirstlane(abar_next);
        typedef __attribute__((address_space(3))) const uint32_t lds_word;
        const uint32_t acc_at = (uint32_t)(uintptr_t)(lds_word *)acc(comp);
        const uint32_t lane4 = (uint32_t)L << 2;
        const uint32_t back4 = (uint32_t)(0 - abar) << 2;       // X^abar reads abar coefficients back, mod 8192 bytes
        // Coefficient j = L + 64 m + 512 h of X^abar ACC is +-ACC[(j - abar) mod N].  The 64 lanes read 64
        // consecutive source coefficients starting at lane 0's, whose byte offset and sign are scalar.  The
        // run wraps past X^N in exactly one of the sixteen (m, h), from some lane on; those lanes read
        // on into the mirror behind the component, which holds mu = -c - 2 for the first 64 coefficients.
        // With ACC stored as c = ~ACC, the step's  +-ACC[src] - ACC[j] + doffset  is
        //   source not past X^N (flip = ~0):  -c[src] + c[j] + doffset = (c[src] ^ ~0) + c[j] + doffset + 1
        //   source past X^N (flip = 0):        c[src] + c[j] + doffset + 2
        // i.e. (c[src] ^ flip) + c[j] + (doffset + 2 + flip); a lane in the mirror needs the other flip,
        // and (mu ^ flip) + flip = (c ^ ~flip) + ~flip for either flip: two vector instructions per
        // coefficient, whatever the lane.
        // A wave alone on its SIMD pays for scalar instructions like for vector ones; the latency kernel
        // therefore keeps address and sign per lane (five vector instructions per coefficient instead of three
        // and five scalar ones) and needs no mirror: bit 12 of a lane's own sum is its sign, the bits below are its
        // offset, and (c ^ flip) + flip is +-ACC - 1 for either flip.
        uint32_t from[8][2], flip[8][2], bias[8][2];
        if (LONE) {
            uint32_t low12 = 4095u;
            asm("" : "+v"(low12));                   // in a vector register: one v_and_or_b32 takes no second constant
#pragma unroll
            for (int m = 0; m < 8; ++m)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t s = (lane4 + back4 + 4096u) + (uint32_t)(64 * m + h * kHalf) * 4u;
                    from[m][h] = (s & low12) | acc_at;
                    flip[m][h] = (uint32_t)__builtin_amdgcn_sbfe((int32_t)s, 12, 1);
                    bias[m][h] = doffset + 2u;
                }
        } else
#pragma unroll
        for (int m = 0; m < 8; ++m)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                // + 4096: bit 12 of the sum then says "lane 0's source not past X^N"
                const uint32_t s = back4 + (uint32_t)(64 * m + h * kHalf) * 4u + 4096u;
                from[m][h] = acc_at + (s & 4095u);
                flip[m][h] = (uint32_t)((int32_t)(s << 19) >> 31);
                bias[m][h] = doffset + 2u + flip[m][h];
                asm("" : "+s"(from[m][h]), "+s"(flip[m][h]), "+s"(bias[m][h]));
            }
        // all sixteen rotated reads are issued before any of them is consumed
        uint32_t rot[8][2];
#pragma unroll
        for (int m = 0; m < 8; ++m)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                rot[m][h] = *(lds_word *)(uintptr_t)(LONE ? from[m][h] : lane4 + from[m][h]);
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            int32_t dig[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int j = L + 64 * m + h * kHalf;
                uint32_t d = (rot[m][h] ^ flip[m][h]) + acc(comp)[j];
                if (LONE) asm("" : "+v"(d));             // v_xad_u32, and one v_add3_u32 for the other two
                d += LONE ? flip[m][h] + bias[m][h] : bias[m][h];
                dig[h] = __builtin_amdgcn_sbfe((int32_t)d, dfield, (uint32_t)a.bgbit);    // signed field
            }
            x[m] = make_double2((double)dig[0], (double)dig[1]);
        }
        }
        lone_pause();
        {
            const Twiddle8 w1 = AHEAD ? kept_w1 : pass1_twiddles(uniform_constants(a.tables));
            dft8_twiddled<false>(x, w1, [&](int k, double2 v) { poly[k * kRowStride + L] = v; }, pause);
        }
        __syncthreads();
        if (LONE) { load_ahead(i, 3); load_ahead(i, 7); }
        lone_pause();

        // ---- this wave's frequencies of all four polynomials ----
        priority(1);
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = mine[(L & 7) + 8 * j];
        wave_sync();
        dft8_shifted<false>(x, f2, [&](int k, double2 v) { mine[k * kGrpStride + (L & 7)] = v; }, pause_if_shared);
        wave_sync();
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = mine[(L & 7) * kGrpStride + j];
        dft8_shifted<false>(x, f3);
        priority(0);
        gather_rows(x);                      // x[2 r + q]: digit polynomial r at slot 256 q + tid

        // ---- products with the key row, in registers: y[2 o + q] = sum_r x[2 r + q] key[r][o] ----
        double2 y[8];
#pragma unroll
        for (int part = 0; part < 4; ++part) {
            const int q = part >> 1;
            double2 k[4][2];
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int o2 = 0; o2 < 2; ++o2)
                    k[r][o2] = part < AHEAD ? ahead[part < AHEAD ? part : 0][r][o2]
                                            : key(i, part, r, o2);
#pragma unroll
            for (int o2 = 0; o2 < 2; ++o2) {
                // one chain of fused multiply-adds per real output (four independent chains per part)
                const double2 d0 = x[q];
                double yr = d0.x * k[0][o2].x, yi = d0.x * k[0][o2].y;
                yr = fma(-d0.y, k[0][o2].y, yr);
                yi = fma(d0.y, k[0][o2].x, yi);
#pragma unroll
                for (int r = 1; r < 4; ++r) {
                    const double2 d = x[2 * r + q];
                    yr = fma(d.x, k[r][o2].x, yr);
                    yi = fma(d.x, k[r][o2].y, yi);
                    yr = fma(-d.y, k[r][o2].y, yr);
                    yi = fma(d.y, k[r][o2].x, yi);
                }
                y[2 * (2 * (part & 1) + o2) + q] = make_double2(yr, yi);
            }
        }
        const int next = i + 1 < a.n ? i + 1 : i;     // the last step requests its own row again
        load_ahead(next, 0);
        if (LONE) load_ahead(next, 2);

        // ---- back: scatter the four output spectra to their lanes, inverse passes 3 and 2 ----
        scatter_rows(y);
        radix8<true>(y, [&](int k, double2 v) { mine[(L & 7) * kGrpStride + k] = v; }, pause);
        wave_sync();
        load_ahead(next, 1);
        if (LONE) load_ahead(next, 6);
#pragma unroll
        for (int k = 0; k < 8; ++k) y[k] = mine[k * kGrpStride + (L & 7)];
        wave_sync();
        if (!LONE) load_ahead(next, 2);
        dft8_shifted<true>(y, i2, [&](int k, double2 v) { mine[(L & 7) + 8 * k] = v; }, pause);
        if (LONE) load_ahead(next, 4);
        double2 p[8];
#pragma unroll
        for (int q = 0; q < 8; ++q)
            p[q] = q < 5 ? my.inv1[q * 64 + L] : kSpare ? a.tables[kInv1 + q * 64 + L] : i1[q < 5 ? 0 : q - 5];
        __syncthreads();
        abar_next = my.bar[i + 1];           // bar[n] exists (it holds bbar)
        lone_pause();
        if (!LONE) { load_ahead(next, 3); load_ahead(next, 6); }

        // ---- inverse pass 1 of output polynomial o = wave, exact rounding, accumulate ----
        priority(2);
#pragma unroll
        for (int k = 0; k < 8; ++k) x[k] = poly[k * kRowStride + L];
        x[0] = cmul(x[0], p[7]);
        dft8_twiddled<true>(x, unpack_twiddles(p));
        const_double *u = AHEAD ? kept : uniform_constants(a.tables);
        double tan_m[8], cos_m[8];
#pragma unroll
        for (int m = 1; m < 8; ++m) { tan_m[m] = AHEAD ? kept_w1.t[m] : u[m]; cos_m[m] = LONE ? kept_cos[m] : u[16 + m]; }
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            if (m) x[m] = cturn(x[m], -tan_m[m]);
            const double part[2] = {x[m].x, x[m].y};
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                // 1.5 * 2^52 - value leaves round-to-nearest(-value) = -round(value) mod 2^32 in the low word (ties
                // go to even either way); the complemented accumulator takes it: ~(ACC + r) = ~ACC - r.
                // The value's pending cosine rides in the multiply-add, so it is rounded once.
                const double shifted = m ? fma(-cos_m[m], part[h], 6755399441055744.0) : 6755399441055744.0 - part[h];
                uint32_t r = (uint32_t)__double2loint(shifted);
                if (MARGIN) worst = fmax(worst, fabs((m ? cos_m[m] * part[h] : part[h]) + (shifted - 6755399441055744.0)));
                if (sel) r <<= 16;
                if (!LONE && m == 3 && h == 1) load_ahead(next, 4);
                atomicAdd(&acc(comp)[L + 64 * m + h * kHalf], r);
                if (!LONE && m == 0 && h == 0) atomicSub(&my.acc[comp][kN + L], r);      // the mirror holds -c - 2
            }
        }
        __syncthreads();
        lone_pause();
        load_ahead(next, 5);
        if (!LONE) load_ahead(next, 7);
    }

    // ---- epilogue: the constant coefficient as an LWE sample under the ring key ----
    {
        uint32_t *ext = a.ext + gi * (size_t)(kN + 1);
        // ACC = ~c, -ACC = c + 1
        for (int j = tid; j < kN; j += kThreadsPerGate) ext[j] = j == 0 ? ~acc(0)[0] : acc(0)[kN - j] + 1u;
        if (tid == 0) ext[kN] = ~acc(1)[0];
    }
    __syncthreads();          // the next gate's prologue overwrites the accumulator
    }
    if (MARGIN) {
        // non-negative doubles order like their bit patterns
        atomicMax(reinterpret_cast<unsigned long long *>(a.margin),
                  (unsigned long long)__double_as_longlong(worst));
    }
}

template <bool MARGIN>
__global__ __launch_bounds__(kThreadsPerGate) __attribute__((amdgpu_waves_per_eu(3, 3))) void blind_rotate_kernel(BlindRotateArgs a) {
    blind_rotate_body<MARGIN, 0, false>(a);
}

// The same step for two gates per CU, where 256 registers a wave hold the key row of step i + 1 while step i runs.  With the
// row loaded where it is used, the way from L2 costs a fifth of such a launch (512 gates 2.25 ms; 1.83 if every load hit L1, 2.25
// if every one hit L2), and a third workgroup that would cover it is not there: 301 gates 2.20 -> 1.94 ms, 400 gates 2.30 -> 1.96, 512 gates
// 2.25 -> 2.10 to 2.18.  Half of the row ahead: 2.29, 2.29, 2.33.  The priorities matter more here: without them 301 gates 2.42.
template <bool MARGIN>
__global__ __launch_bounds__(kThreadsPerGate) __attribute__((amdgpu_waves_per_eu(2, 2))) void blind_rotate_pair_kernel(BlindRotateArgs a) {
    blind_rotate_body<MARGIN, 4, false>(a);
}

// The same step for batches of at most one gate per CU, where a gate's latency is all that
// counts: six of the eight portions of a key row are requested a step ahead, the other two in the step.
template <bool MARGIN>
__global__ __launch_bounds__(kThreadsPerGate) __attribute__((amdgpu_waves_per_eu(1, 1))) void blind_rotate_latency_kernel(BlindRotateArgs a) {
    blind_rotate_body<MARGIN, 4, true>(a);
}

// ------------------------------------------------------------------------------------------
// Blind rotation of large batches: one gate per wavefront, four gates per workgroup of 256 threads, two
// workgroups per CU (256 VGPRs a wave).
//
// A lane holds all four digit spectra of its eight frequencies (x[4][8], 128 registers), so the products
// need no exchange between lanes and no barrier stands between a wave and its data: against the four-wave
// kernel the 256 lane swaps of a gate's step and three barriers are gone, and both digits of a component come
// from one rotated read and one subtraction.  The two components of the result come from three sums (sums3.h): seven transforms a
// step and 96 KB of key instead of eight and 128 KB.  A polynomial passes through one 9 KB buffer that belongs to the wave; LDS
// operations of a wave execute in order, so the stores of one polynomial may follow the loads of the one
// before it at once.
//
// What bounds it: vector issue, LDS and the key stream through L1 side by side, at a clock that power lowers (2.18 GHz in whole rounds,
// 2.39 with a workgroup per CU).  An exchange of a polynomial (8 KB) costs its wave eight stores of 28 clocks of issue and eight
// loads of about 14, and the CU's LDS 13 and 5 clocks each (a 16-byte store as two of 8 bytes costs the same): fourteen exchanges are about
// 2,000 clocks of LDS a gate-step beside 2,240 of vector issue.  So at most one exchange stands in a region between two scheduling barriers,
// its stores nine vector instructions apart, and, but for the step's first, one more piece of arithmetic comes before its result is
// used; the step's first reads go before the rounding of the step before.  Calls, against two exchanges in a region, closer and used
// at once: 1,024 gates 4.26 -> 3.80 ms, 16,384 gates 52.2 -> 49.8, 65,536 gates 205.5 -> 199.8 (four sums 236, the four-wave kernel 284).
// Without the barrier before the products + 1 %; without any exchange - 15 %, without key loads - 8 % (half of which is clock), without both
// - 27 % (with the exchanges as they stood before).  Key rows brought to LDS and read from there by all four waves instead of four L1
// reads: equal.  Products spread over the forward half, a digit polynomial or a component at a time: registers spill.
//
// Barrier before the products: the four waves of a workgroup then read the key row together and three
// quarters of their reads hit L1; without it the waves of
// an XCD spread over more rows than its L2 holds.
// Priorities: the inverse transforms and the beginning of the forward ones, up to the second exchange, issue ahead of the rest and the
// products, so that the two waves of a SIMD fall into opposite halves: one computes while the other waits for LDS and keys.
// 16,384 gates, lowered behind the first second pass 51.6 ms, up to eight pieces later 51.9 to 53.3; raised a piece later 53.
// Two waves per SIMD in the lone form too, with the same priorities: alone it has one, but launches for two keys on two streams then
// share the CUs.  800, 900 and 1,024 gates for each of two keys: 6.36, 6.61 and 6.74 ms; 6.78, 7.06 and 7.21 without priorities; 7.74,
// 7.55 and 7.59 compiled for one wave, one launch after the other.  One of them alone 3.75, 3.75 and 3.82 in either form.
// ------------------------------------------------------------------------------------------
constexpr int kWaveGates = 4;      // waves (= gates) of a workgroup

struct WaveLds {
    double2 buf[kWaveGates][8 * kRowStride];
    uint32_t acc[kWaveGates][2][kN + kMirror];     // as in GateLds
    // lane-dependent constants of dft8.h, a piece of the table in memory: forward pass 2, inverse passes 2 and 1
    double2 constants[kFwd3 - kFwd2];
};
static_assert(kFwd2 < kInv2 && kInv2 < kInv1 && kInv1 < kFwd3, "the table's order");
static_assert(2 * sizeof(WaveLds) <= 160 * 1024, "two workgroups share a CU's LDS");

// Scheduling patterns of the instructions between two region ends.  EXCHANGE: eight stores to LDS, then eight loads, each followed by nine
// vector instructions of other work as long as there is any.  A store of 16 bytes a lane holds its wave's issue for 28 clocks, and for 52
// where four waves store in step, unless six or more multiply-adds stand behind each (nine against five and three:
// 1,024 gates 3.80, 3.98 and 4.47 ms, 16,384 gates 49.8, 51.3 and 52.0).  KEYS: a key load, then four multiply-adds,
// instead of four loads in a row (16,384 gates 50.1 -> 49.8 ms).
#define REGION_END() __builtin_amdgcn_sched_barrier(0)
#define ONE_OF(KIND, V) __builtin_amdgcn_sched_group_barrier(KIND, 1, 0); __builtin_amdgcn_sched_group_barrier(0x002, V, 0);
#define FOUR_OF(KIND, V) ONE_OF(KIND, V) ONE_OF(KIND, V) ONE_OF(KIND, V) ONE_OF(KIND, V)
#define EXCHANGE_BESIDE() FOUR_OF(0x200, 9) FOUR_OF(0x200, 9) FOUR_OF(0x100, 9) FOUR_OF(0x100, 9)
#define KEYS_BESIDE() FOUR_OF(0x020, 4)

template <bool MARGIN, bool SHARE>
__global__ __launch_bounds__(64 * kWaveGates) __attribute__((amdgpu_waves_per_eu(2, 2))) void blind_rotate_wave_kernel(BlindRotateArgs a) {
    // Key batches (one sum at one frequency: four 16-byte loads) in registers.  A lone wave covers the way from L2 with one more
    // (1,024 gates 3.92 -> 3.80 ms); with two on a SIMD five or six are no faster than four.
    constexpr int kKeyRing = SHARE ? 4 : 5;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    WaveLds &my = *reinterpret_cast<WaveLds *>(lds_raw);
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int L = threadIdx.x & 63;
    // the items are spread evenly over the workgroups, at most one a wave
    const size_t items = a.count - a.first, begin = a.first + items * blockIdx.x / gridDim.x;
    const size_t end = a.first + items * (blockIdx.x + 1) / gridDim.x;
    const size_t gi = begin + wv;
    uint32_t (&acc)[2][kN + kMirror] = my.acc[wv];
    double2 *const buf = my.buf[wv];
    double2 *const mine = buf + (L >> 3) * kRowStride;          // passes 2, 3: lane = 8 k0 + (j0 or k1)
    for (int e = threadIdx.x; e < kFwd3 - kFwd2; e += 64 * kWaveGates) my.constants[e] = a.tables[kFwd2 + e];
    Shift8 f3;
    f3.h4 = a.tables[kFwd3 + L];
    f3.h2 = a.tables[kFwd3 + 64 + L];
    f3.h1 = a.tables[kFwd3 + 128 + L];
    f3.h1w = a.tables[kFwd3 + 192 + L];
    const __amdgpu_buffer_rsrc_t key_rsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<double2 *>(a.bk_fft + (size_t)a.n * 16 * kHalf), 0, (int)((size_t)a.n * kSumKeyWords * sizeof(double2)), 0x00020000);
    const uint32_t voff = (uint32_t)sum_key_word(0, 0, 0, L) * (uint32_t)sizeof(double2);
    double worst = 0.0;
    __syncthreads();
    if (gi >= end) return;            // a wave without a gate: the barriers below wait for the others only

    int op = a.uniform_op;
    size_t i0 = gi, i1 = gi;
    uint32_t s0 = 1u, s1 = 1u;
    const uint32_t *src1 = a.in1;
    if (a.recs) {
        const tfhe_gate_rec r = a.recs[gi];
        op = r.op; i0 = (size_t)r.in0; i1 = (size_t)r.in1;
        s0 = r.neg0 ? 0xFFFFFFFFu : 1u; s1 = r.neg1 ? 0xFFFFFFFFu : 1u;
    } else if (op == TFHE_MUX) {
        i0 = i1 = gi >> 1;
        if (gi & 1) { op = TFHE_MUX_ELSE; src1 = a.in1_alt; }
    }
    if (op == TFHE_MUX_ELSE) s0 = 0u - s0;
    if (op >= TFHE_MUX) op = TFHE_AND;
    uint32_t kappa, mult;
    gate_constants(op, kappa, mult);
    const uint32_t *c0 = a.in0 + i0 * ((size_t)a.n + 1), *c1 = src1 + i1 * ((size_t)a.n + 1);
    auto rotation = [&](int j) -> int {
        uint32_t c = mult * (s0 * c0[j] + s1 * c1[j]);
        if (j == a.n) c += kappa;
        return (int)(((c + (1u << 20)) >> 21) & 2047u);
    };
    {
        const int bbar = __builtin_amdgcn_readfirstlane(rotation(a.n));
        const int bb = bbar & (kN - 1);
        const uint32_t first = bbar < kN ? kEighth : 0u - kEighth;
        for (int j = L; j < kN; j += 64) {
            const uint32_t c = ~(j < kN - bb ? first : 0u - first);
            acc[0][j] = ~0u;
            acc[1][j] = c;
            if (j < kMirror) { acc[0][kN + j] = 0u - ~0u - 2u; acc[1][kN + j] = 0u - c - 2u; }
        }
    }
    wave_sync();

    const uint32_t dround = 1u << (31 - 2 * a.bgbit), dhalf = 1u << (31 - a.bgbit);
    const uint32_t field0 = (uint32_t)(32 - a.bgbit), field1 = (uint32_t)(32 - 2 * a.bgbit);
    int bars = 0;                               // the rotation amounts of 64 steps, one per lane
    uint32_t back4 = 0;                         // bytes that the step's rotation reads back
    // The lane's number, counted again where it is needed once in 64 steps or at the end: kept, it and the addresses formed from it take
    // registers that the lone form does not have.
    auto lane_again = [] {
        uint32_t all = ~0u;
        asm volatile("" : "+s"(all));
        return (int)__builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0u));
    };
    auto set_step = [&](int i) {
        if ((i & 63) == 0) {
            const int j = i + lane_again();
            bars = rotation(j < a.n ? j : a.n);
        }
        back4 = (uint32_t)(0 - __builtin_amdgcn_readfirstlane(__builtin_amdgcn_readlane(bars, i & 63))) << 2;
    };
    // Rotated and plain reads of a component (see blind_rotate_body for the mirror and the sign).  A lone wave pays for every scalar
    // instruction: it keeps the sixteen addresses of component 0 for component 1 (1,024 gates 3.86 -> 3.80 ms).  With two waves on a
    // SIMD that is slower (16,384 gates 49.8 -> 50.5 ms).
    typedef __attribute__((address_space(3))) const uint32_t lds_word;
    const uint32_t lane_at = (uint32_t)(uintptr_t)(lds_word *)acc[0] + ((uint32_t)L << 2);
    uint32_t rot[8][2], own[8][2], at[8][2];
    auto read_component = [&](int comp) {
        const uint32_t acc_at = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_word *)acc[comp]);
#pragma unroll
        for (int m = 0; m < 8; ++m)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t back = (back4 + (uint32_t)(64 * m + h * kHalf) * 4u) & 4095u;
                if (SHARE) {
                    rot[m][h] = *(lds_word *)(uintptr_t)(((uint32_t)L << 2) + __builtin_amdgcn_readfirstlane(acc_at + back));
                } else {
                    if (comp == 0) at[m][h] = lane_at + __builtin_amdgcn_readfirstlane(back);
                    rot[m][h] = ((lds_word *)(uintptr_t)at[m][h])[comp * (kN + kMirror)];
                }
                own[m][h] = acc[comp][L + 64 * m + h * kHalf];
            }
        wave_sync();
    };
    set_step(0);
    read_component(0);
    for (int i = 0; i < a.n; ++i) {
        double2 x[4][8];

        // ---- the pieces of a step ----
        // both digits of the difference, folded: x[2 comp] and x[2 comp + 1]
        auto digits = [&](int comp) {
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                int32_t hi[2], lo[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t s = back4 + (uint32_t)(64 * m + h * kHalf) * 4u + 4096u;
                    const uint32_t flip = __builtin_amdgcn_readfirstlane((uint32_t)((int32_t)(s << 19) >> 31));
                    const uint32_t bias = __builtin_amdgcn_readfirstlane(dround + 2u + flip);
                    const uint32_t d = (rot[m][h] ^ flip) + own[m][h] + bias;
                    lo[h] = __builtin_amdgcn_sbfe((int32_t)d, field1, (uint32_t)a.bgbit);
                    hi[h] = (int32_t)(d + dhalf) >> field0;
                }
                x[2 * comp][m] = make_double2((double)hi[0], (double)hi[1]);
                x[2 * comp + 1][m] = make_double2((double)lo[0], (double)lo[1]);
            }
        };
        // lane-dependent constants are read again where they are needed: kept in registers they would
        // leave none for the key loads in flight
        typedef __attribute__((address_space(3))) const double2 lds_words;
        auto load_twiddles = [&](const double2 *table, int width, int lane, double2 (&p)[8]) {
#pragma unroll
            for (int q = 0; q < 8; ++q) p[q] = *(const double2 *)((lds_words *)(table + lane) + q * width);
        };
        auto store_columns = [&](const double2 (&v)[8]) {            // element k of lane L at row k, column L
#pragma unroll
            for (int k = 0; k < 8; ++k) buf[k * kRowStride + L] = v[k];
            wave_sync();
        };
        auto load_columns = [&](double2 (&v)[8]) {
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = buf[k * kRowStride + L];
            wave_sync();
        };
        auto store_row = [&](const double2 (&v)[8]) {                // row L / 8: element k at L % 8 + 8 k
#pragma unroll
            for (int k = 0; k < 8; ++k) mine[(L & 7) + 8 * k] = v[k];
            wave_sync();
        };
        auto load_row = [&](double2 (&v)[8]) {
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = mine[(L & 7) + 8 * k];
            wave_sync();
        };
        auto store_across = [&](const double2 (&v)[8]) {             // the inner transpose, groups of 8 lanes
#pragma unroll
            for (int k = 0; k < 8; ++k) mine[k * kGrpStride + (L & 7)] = v[k];
            wave_sync();
        };
        auto load_across = [&](double2 (&v)[8]) {
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = mine[k * kGrpStride + (L & 7)];
            wave_sync();
        };
        auto store_along = [&](const double2 (&v)[8]) {
#pragma unroll
            for (int k = 0; k < 8; ++k) mine[(L & 7) * kGrpStride + k] = v[k];
            wave_sync();
        };
        auto load_along = [&](double2 (&v)[8]) {
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = mine[(L & 7) * kGrpStride + k];
            wave_sync();
        };
        constexpr uint32_t kWord = sizeof(double2);
        const uint32_t row = (uint32_t)i * kSumKeyWords * kWord;
        double2 ring[kKeyRing][4];
        // Sum b % 3 at frequency k2 = b / 3: four rows of 1 KB behind each other, which one scalar offset and the immediate offsets of
        // the loads reach.
        auto load_batch = [&](int b) {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                ring[b % kKeyRing][r] = load_key(key_rsrc, voff + kWord * sum_key_word(0, 0, r, 0), row + kWord * sum_key_word(b / kSums, b % kSums, 0, 0));
        };

        // ---- forward: four polynomials.  An exchange stands beside the arithmetic of another polynomial, and one more piece of arithmetic
        // comes between it and its own polynomial's next pass, so that its latency is covered too: at most one exchange a region.  The
        // step's beginning has no other arithmetic yet: polynomial 1's first exchange stands beside the reads of component 1 alone, and
        // is what comes between polynomial 0's first exchange and its next pass ----
        {
            double2 p[8];
            load_twiddles(my.constants, 8, L >> 3, p);
            const Twiddle8 w2 = unpack_twiddles(p);
            const Twiddle8 w1 = pass1_twiddles(uniform_constants(a.tables));

            digits(0);
            dft8_twiddled<false>(x[0], w1);
            REGION_END();
            store_columns(x[0]); load_row(x[0]);
            dft8_twiddled<false>(x[1], w1);
            EXCHANGE_BESIDE()
            REGION_END();
            read_component(1);
            store_columns(x[1]); load_row(x[1]);
            REGION_END();
            dft8_twiddled<false>(x[0], w2);
            REGION_END();
            __builtin_amdgcn_s_setprio(0);
            store_across(x[0]); load_along(x[0]);
            digits(1);
            dft8_twiddled<false>(x[2], w1);
            EXCHANGE_BESIDE()
            REGION_END();
            store_columns(x[2]); load_row(x[2]);
            dft8_twiddled<false>(x[1], w2);
            EXCHANGE_BESIDE()
            REGION_END();
            store_across(x[1]); load_along(x[1]);
            dft8_twiddled<false>(x[3], w1);
            EXCHANGE_BESIDE()
            REGION_END();
            store_columns(x[3]); load_row(x[3]);
            dft8_twiddled<false>(x[2], w2);
            EXCHANGE_BESIDE()
            REGION_END();
            store_across(x[2]); load_along(x[2]);
            dft8_shifted<false>(x[0], f3);
            EXCHANGE_BESIDE()
            REGION_END();
            dft8_twiddled<false>(x[3], w2);
            REGION_END();
            load_batch(0);
            store_across(x[3]); load_along(x[3]);
            dft8_shifted<false>(x[1], f3);
            EXCHANGE_BESIDE()
            REGION_END();
            load_batch(1);
            dft8_shifted<false>(x[2], f3);
            REGION_END();
            load_batch(2);
            dft8_shifted<false>(x[3], f3);
            REGION_END();
            if (!SHARE) load_batch(3);
        }

        // ---- products with the key row: at every frequency the four digit spectra give way to the three sums ----
        if (SHARE) __builtin_amdgcn_s_barrier();     // no data passes: the four waves read the key row together
#pragma unroll
        for (int k2 = 0; k2 < 8; ++k2) {
            double2 y[kSums];
#pragma unroll
            for (int o = 0; o < kSums; ++o) {
                const int b = kSums * k2 + o;
                if (b + kKeyRing - 1 < 8 * kSums) load_batch(b + kKeyRing - 1);
                if (!SHARE) REGION_END();
                const double2 (&k)[4] = ring[b % kKeyRing];
                const double2 d0 = x[0][k2];
                double yr = d0.x * k[0].x, yi = d0.x * k[0].y;
                yr = fma(-d0.y, k[0].y, yr);
                yi = fma(d0.y, k[0].x, yi);
#pragma unroll
                for (int r = 1; r < 4; ++r) {
                    const double2 d = x[r][k2];
                    yr = fma(d.x, k[r].x, yr);
                    yi = fma(d.x, k[r].y, yi);
                    yr = fma(-d.y, k[r].y, yr);
                    yi = fma(d.y, k[r].x, yi);
                }
                y[o] = make_double2(yr, yi);
                if (SHARE) { KEYS_BESIDE() }
                REGION_END();
            }
#pragma unroll
            for (int o = 0; o < kSums; ++o) x[o][k2] = y[o];
        }

        // ---- back: inverse transforms, exact rounding, accumulate ----
        __builtin_amdgcn_s_setprio(2);
        {
            double2 p[8];
            load_twiddles(my.constants + (kInv2 - kFwd2), 8, L & 7, p);
            const Twiddle8 w2 = unpack_twiddles(p);
            load_twiddles(my.constants + (kInv1 - kFwd2), 64, L, p);
            const Twiddle8 w1 = unpack_twiddles(p);
            const double2 w10 = p[7];
            double tan_m[8], cos_m[8];
            const_double *u = uniform_constants(a.tables);
#pragma unroll
            for (int m = 1; m < 8; ++m) { tan_m[m] = u[m]; cos_m[m] = u[16 + m]; }
            uint32_t low[8][2];            // the low sum, then what it leaves for component 1 (sums3.h)
            // pass 1 and rounding of sum o, and the accumulation of component o - 1
            auto finish = [&](int o) {
                double2 (&v)[8] = x[o];
                v[0] = cmul(v[0], w10);
                dft8_twiddled<true>(v, w1);
#pragma unroll
                for (int m = 0; m < 8; ++m) {
                    if (m) v[m] = cturn(v[m], -tan_m[m]);
                    const double part[2] = {v[m].x, v[m].y};
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        // the value's pending cosine rides in the multiply-add, so it is rounded once
                        if (o == 0) {
                            const double shifted = m ? fma(cos_m[m], part[h], kIntegerShift) : kIntegerShift + part[h];
                            low[m][h] = (uint32_t)__double2loint(shifted);
                            if (MARGIN) worst = fmax(worst, fabs((m ? cos_m[m] * part[h] : part[h]) - (shifted - kIntegerShift)));
                        } else {
                            const double shifted = m ? fma(-cos_m[m], part[h], kHalfShift) : kHalfShift - part[h];
                            // the complemented accumulator takes -P: ~(ACC + P) = ~ACC - P
                            const uint32_t t = minus_product(low[m][h], (uint32_t)__double2loint(shifted));
                            if (MARGIN) {
                                const double rest = (m ? cos_m[m] * part[h] : part[h]) - (double)((0u - t) & kSumMask) * (1.0 / (1 << kSumBits));
                                worst = fmax(worst, fabs(rest - rint(rest)));
                            }
                            atomicAdd(&acc[o - 1][L + 64 * m + h * kHalf], t);
                            if (m == 0 && h == 0) atomicSub(&acc[o - 1][kN + L], t);      // the mirror holds -c - 2
                        }
                    }
                }
            };
            radix8<true>(x[0]);
            REGION_END();
            store_along(x[0]); load_across(x[0]);
            radix8<true>(x[1]);
            EXCHANGE_BESIDE()
            REGION_END();
            store_along(x[1]); load_across(x[1]);
            radix8<true>(x[2]);
            EXCHANGE_BESIDE()
            REGION_END();
            store_along(x[2]); load_across(x[2]);
            dft8_twiddled<true>(x[0], w2);
            EXCHANGE_BESIDE()
            REGION_END();
            store_row(x[0]); load_columns(x[0]);
            dft8_twiddled<true>(x[1], w2);
            EXCHANGE_BESIDE()
            REGION_END();
            store_row(x[1]); load_columns(x[1]);
            dft8_twiddled<true>(x[2], w2);
            EXCHANGE_BESIDE()
            REGION_END();
            store_row(x[2]); load_columns(x[2]);
            finish(0);
            EXCHANGE_BESIDE()
            REGION_END();
            finish(1);
            wave_sync();
            REGION_END();
            // component 0 is complete: the next step's reads of it go before the rounding of component 1 (after the last step they
            // are not used)
            set_step(i + 1 < a.n ? i + 1 : i);
            read_component(0);
            finish(2);
            wave_sync();
            REGION_END();
        }
    }

    uint32_t *ext = a.ext + gi * (size_t)(kN + 1);
    const int lane = lane_again();
    for (int j = lane; j < kN; j += 64) ext[j] = j == 0 ? ~acc[0][0] : acc[0][kN - j] + 1u;
    if (lane == 0) ext[kN] = ~acc[1][0];
    if (MARGIN)
        atomicMax(reinterpret_cast<unsigned long long *>(a.margin), (unsigned long long)__double_as_longlong(worst));
}

// ------------------------------------------------------------------------------------------
// Key switch, one workgroup per gate:  out = (0, b') - sum_{i,j} KSK[i][j][digit_ij]
// over the t base-2^basebit digits of the rounded mask words; digit 0 reads the zero row
// appended to the key so that all loads of one mask word can be in flight together.
// ------------------------------------------------------------------------------------------
template <int T>
__global__ __launch_bounds__(256) void key_switch_kernel(KeySwitchArgs a) {
    __shared__ uint32_t ext[kN + 1];
    const int tid = threadIdx.x;
    // with a.splits > 1 the mask words of one gate are shared out over that many workgroups,
    // each adding its partial result into the (zeroed) output with integer atomics
    const size_t gi = blockIdx.x / a.splits;
    const int part = (int)(blockIdx.x % a.splits);
    // the second half of a multiplexer has been added into the first: nothing to switch
    if (a.recs ? a.recs[gi].op == TFHE_MUX_ELSE : (a.uniform_mux && (gi & 1))) return;
    const uint32_t *src = a.ext + gi * (size_t)(kN + 1);
    for (int j = tid; j <= kN; j += 256) ext[j] = src[j];
    __syncthreads();

    const int words = a.n + 1;
    constexpr int kMaxPerThread = 5;              // ceil(1025 / 256)
    uint32_t acc[kMaxPerThread];
#pragma unroll
    for (int q = 0; q < kMaxPerThread; ++q) {
        const int w = tid + 256 * q;
        acc[q] = (w == a.n && part == 0) ? ext[kN] : 0u;
    }
    const int values = (1 << a.basebit) - 1;
    const uint32_t round = 1u << (31 - T * a.basebit);
    const size_t zero_row = (size_t)kN * T * values;   // appended row of zeros
    const int per_thread = (words + 255) >> 8;
    const int i_begin = part * (kN / a.splits), i_end = i_begin + kN / a.splits;
    for (int i = i_begin; i < i_end; ++i) {
        const uint32_t ai = ext[i] + round;
        const uint32_t *rows[T];
#pragma unroll
        for (int j = 0; j < T; ++j) {
            const uint32_t v = (ai >> (32 - a.basebit * (j + 1))) & (uint32_t)values;
            const size_t row = v ? ((size_t)i * T + j) * values + (v - 1) : zero_row;
            rows[j] = a.ksk + row * (size_t)a.stride;
        }
        for (int q = 0; q < per_thread; ++q) {
            const int w = tid + 256 * q;
            if (w < words) {
                uint32_t part_sum[T];
#pragma unroll
                for (int j = 0; j < T; ++j) part_sum[j] = rows[j][w];
                uint32_t sum = 0;
#pragma unroll
                for (int j = 0; j < T; ++j) sum += part_sum[j];
                acc[q] -= sum;
            }
        }
    }
    const size_t out_index = a.recs ? (size_t)a.recs[gi].out : (a.uniform_mux ? gi >> 1 : gi);
    uint32_t *out = a.out + out_index * (size_t)words;
#pragma unroll
    for (int q = 0; q < kMaxPerThread; ++q) {
        const int w = tid + 256 * q;
        if (w < words) {
            if (a.splits > 1) atomicAdd(out + w, acc[q]);
            else out[w] = acc[q];
        }
    }
}

// zero the output samples that the split key switch accumulates into
__global__ void zero_outputs_kernel(KeySwitchArgs a) {
    const size_t gi = blockIdx.x;
    if (a.recs ? a.recs[gi].op == TFHE_MUX_ELSE : (a.uniform_mux && (gi & 1))) return;
    const size_t out_index = a.recs ? (size_t)a.recs[gi].out : (a.uniform_mux ? gi >> 1 : gi);
    uint32_t *out = a.out + out_index * (size_t)(a.n + 1);
    for (int w = threadIdx.x; w <= a.n; w += blockDim.x) out[w] = 0u;
}

// ------------------------------------------------------------------------------------------
// Key switch as a dense contraction on the matrix cores (t = 8 digits in base 4, N = 1024, n + 1 <= 512).
// With one-hot digits the sum is a matrix product
//     S[g][c] = sum_{i, j, v} [digit_ij(g) == v] * KSK[i][j][v][c]      (v = 0: a zero row)
// with K = 1024 * 8 * 4 = 32,768.  The 32-bit key words are split into four balanced signed
// bytes, x = s0 + 2^8 s1 + 2^16 s2 + 2^24 s3 (mod 2^32), |s| <= 128, so every plane is an exact
// int8 x int8 -> int32 product (|sum| <= 2^20) and S is recombined with shifts.
//
// v_mfma_i32_32x32x32_i8: lane l supplies row (A) / column (B) l % 32 and the 16 bytes of
// k-group l / 32; both operands use the same byte <-> k map, which is all the contraction needs.
// One k-step of 32 is one mask word i: its 8 digits x 4 values.  A lane's A operand is built
// in registers: 4 digits -> 4 words 1 << (8 * digit).  The key is pre-tiled so that a B operand
// (32 columns x 32 k) is 1 KB contiguous in lane order: tiles[block of 32 words][i][plane][lane].
//
// A workgroup takes 32 TILES gates, 32 output words and a share of the mask words, of which each of its four
// waves takes a quarter.  The waves' sums meet in LDS and go into the zeroed outputs with one integer atomic
// per word and workgroup (order-independent: still exact).  Few gates are bound by the one pass over the 64 MB
// of key tiles and by the latency of getting them started, many by the tiles' way from L2 (64 MB per 32 TILES
// gates), which two workgroups on a CU keep busier than one with more gates.  Measured against 256 gates x 64 words a
// workgroup, one wave per SIMD, with up to 32 partial sums of every word added by atomics:
// the kernel alone, 8 gates 26.5 -> 13.3 us, 64 gates 36 -> 17, 256 gates 56 -> 33, 512 gates 82 -> 65, 1,536 gates 237 -> 121,
// 4,096 gates 403 -> 291, 16,384 gates 1,457 -> 1,353.
// ------------------------------------------------------------------------------------------
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

// tiles[((cb * 1024 + i) * 4 + plane) * 64 + lane] = 16 bytes: byte q is plane `plane` of
// KSK[i][4 * (lane / 32) + q / 4][q % 4][32 * cb + lane % 32]  (value 0 and words past n: 0)
__global__ __launch_bounds__(256) void ksk_to_tiles_kernel(const uint32_t *__restrict__ ksk, int stride, int words,
                                                           v4i *__restrict__ tiles) {
    const int i = blockIdx.x, cb = blockIdx.y;
    const int plane = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int c = 32 * cb + (lane & 31);
    uint32_t packed[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int j = 4 * (lane >> 5) + (q >> 2), v = q & 3;
        uint32_t x = (v && c < words) ? ksk[((size_t)(i * 8 + j) * 3 + (v - 1)) * stride + c] : 0u;
        int32_t digit = 0;
#pragma unroll
        for (int b = 0; b <= 3; ++b) {
            digit = (int8_t)(x & 0xFFu);
            x = (x - (uint32_t)digit) >> 8;            // exact: the low byte is zero after the subtraction
            if (b == plane) break;
        }
        packed[q >> 2] |= ((uint32_t)digit & 0xFFu) << (8 * (q & 3));
    }
    v4i t;
    t.x = (int)packed[0]; t.y = (int)packed[1]; t.z = (int)packed[2]; t.w = (int)packed[3];
    tiles[(((size_t)cb * kN + i) * 4 + plane) * 64 + lane] = t;
}

constexpr int kKsShare = 128;     // mask words of a workgroup at most

template <int TILES>
struct KsLds {
    union {
        uint32_t mask_words[kKsShare][32 * TILES + 1];
        uint32_t partial[4][16 * TILES][64];
    };
    int32_t out_row[32 * TILES];
};

template <int TILES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(TILES == 4 ? 1 : 2, TILES == 4 ? 1 : 2)))
void key_switch_mfma_kernel(KeySwitchArgs a) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    KsLds<TILES> &lds = *reinterpret_cast<KsLds<TILES> *>(lds_raw);
    constexpr int kRows = 32 * TILES;
    constexpr int kAhead = TILES == 1 ? 8 : 4;                  // mask words whose key tiles are in flight
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int cb = blockIdx.y;
    const size_t g0 = (size_t)blockIdx.x * kRows;
    const int words = a.n + 1;
    if (tid < kRows) {
        const size_t gi = g0 + tid;
        int32_t row = -1;
        if (gi < a.count) {
            if (a.recs) { if (a.recs[gi].op != TFHE_MUX_ELSE) row = a.recs[gi].out; }
            else if (!a.uniform_mux) row = (int32_t)gi;
            else if (!(gi & 1)) row = (int32_t)(gi >> 1);
        }
        lds.out_row[tid] = row;
    }
    const int share = kN / a.splits, share_shift = 31 - __builtin_clz(share);      // a power of two, 64 or 128
    const int i_begin = (int)blockIdx.z * share;
    const int mine = share >> 2, first = wave * mine;           // this wave's mask words, from i_begin + first on
    const v4i *tiles = reinterpret_cast<const v4i *>(a.ksk_tiles) + ((size_t)cb * kN + i_begin + first) * 4 * 64 + lane;
    v4i ring[kAhead][4];
#pragma unroll
    for (int s = 0; s < kAhead; ++s)
#pragma unroll
        for (int b = 0; b < 4; ++b) ring[s][b] = tiles[(s * 4 + b) * 64];
    v16i acc[TILES][4];
#pragma unroll
    for (int rt = 0; rt < TILES; ++rt)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[rt][b][r] = 0;
    const uint32_t round = 1u << (31 - 16);
    // consecutive lanes read consecutive mask words of one gate; a row without an output is summed up and dropped
#pragma unroll 8
    for (int idx = tid; idx < share * kRows; idx += 256) {
        const int g = idx >> share_shift, ii = idx & (share - 1);
        const size_t gi = g0 + g < a.count ? g0 + g : a.count - 1;
        lds.mask_words[ii][g] = a.ext[gi * (size_t)(kN + 1) + i_begin + ii] + round;
    }
    __syncthreads();
    const int byte_shift = 24 - 8 * (lane >> 5);
    for (int i1 = 0; i1 < mine; i1 += kAhead) {
#pragma unroll
        for (int s = 0; s < kAhead; ++s) {
#pragma unroll
            for (int rt = 0; rt < TILES; ++rt) {
                const uint32_t w = (lds.mask_words[first + i1 + s][(lane & 31) + 32 * rt] >> byte_shift) & 0xFFu;
                v4i at;
                at.x = (int)(1u << (((w >> 6) & 3u) << 3));
                at.y = (int)(1u << (((w >> 4) & 3u) << 3));
                at.z = (int)(1u << (((w >> 2) & 3u) << 3));
                at.w = (int)(1u << ((w & 3u) << 3));
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    acc[rt][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(at, ring[s][b], acc[rt][b], 0, 0, 0);
            }
            if (i1 + kAhead < mine) {
#pragma unroll
                for (int b = 0; b < 4; ++b) ring[s][b] = tiles[((size_t)(i1 + s + kAhead) * 4 + b) * 64];
            }
        }
    }
    __syncthreads();                                            // the mask words give way to the partial sums
#pragma unroll
    for (int rt = 0; rt < TILES; ++rt) {
        // With four tiles the accumulators are all 256 accumulation registers; left alone the compiler copies every one of
        // them to vector registers first and spills three.  The last tile stays where it is until the others are stored (212
        // vector registers; by events around the zeroing and this kernel, with the spills and now: 128 gates 30.5 and 30.4 us,
        // 256 gates 40.5 and 40.4, 512 gates 72.0 and 71.6).
        if constexpr (TILES == 4)
            if (rt == TILES - 1) asm volatile("" : "+a"(acc[rt][0]), "+a"(acc[rt][1]), "+a"(acc[rt][2]), "+a"(acc[rt][3]));
#pragma unroll
        for (int r = 0; r < 16; ++r)
            lds.partial[wave][16 * rt + r][lane] = (uint32_t)acc[rt][0][r] + ((uint32_t)acc[rt][1][r] << 8) +
                                                   ((uint32_t)acc[rt][2][r] << 16) + ((uint32_t)acc[rt][3][r] << 24);
        if constexpr (TILES == 4) __builtin_amdgcn_sched_barrier(0);
    }
    __syncthreads();
    // accumulator register r of lane l: row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32
    const int c = 32 * cb + (lane & 31);
    if (c >= words) return;
#pragma unroll
    for (int e = 0; e < 4 * TILES; ++e) {
        const int at = wave * 4 * TILES + e, rt = at >> 4, r = at & 15;
        const int g = 32 * rt + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        const int32_t row = lds.out_row[g];
        if (row < 0) continue;
        const uint32_t sum = lds.partial[0][at][lane] + lds.partial[1][at][lane] + lds.partial[2][at][lane] + lds.partial[3][at][lane];
        const uint32_t body = (c == a.n && blockIdx.z == 0) ? a.ext[(g0 + g) * (size_t)(kN + 1) + kN] : 0u;
        atomicAdd(a.out + (size_t)row * words + c, body - sum);
    }
}

// Multiplexer: the two half results (ring-key samples of AND(s,a) and AND(NOT s,b)) are summed,
// 1/8 is added to the body, and the sum is what the key switch of the first half consumes.
__global__ void mux_combine_kernel(uint32_t *ext, const tfhe_gate_rec *recs, size_t count) {
    const size_t e = blockIdx.x;
    const bool first = recs ? recs[e].op == TFHE_MUX : (e & 1) == 0;
    if (!first || e + 1 >= count) return;
    uint32_t *dst = ext + e * (size_t)(kN + 1);
    const uint32_t *add = dst + (kN + 1);
    for (int j = threadIdx.x; j <= kN; j += blockDim.x) dst[j] += add[j] + (j == kN ? kEighth : 0u);
}

// out[k] = +-wires[ref.wire]  or the noiseless sample of the constant bit
__global__ void gather_outputs_kernel(const uint32_t *wires, const tfhe_out_ref *refs, uint32_t *out,
                                      size_t count, int words) {
    const size_t k = blockIdx.x;
    if (k >= count) return;
    const tfhe_out_ref r = refs[k];
    for (int w = threadIdx.x; w < words; w += blockDim.x) {
        uint32_t v;
        if (r.wire >= 0) {
            v = wires[(size_t)r.wire * words + w];
            if (r.value) v = 0u - v;
        } else {
            v = w == words - 1 ? (r.value ? kEighth : 0u - kEighth) : 0u;
        }
        out[k * (size_t)words + w] = v;
    }
}

__global__ void fill_trivial_kernel(uint32_t *ct, int words, uint32_t body) {
    for (int w = threadIdx.x; w < words; w += blockDim.x) ct[w] = w == words - 1 ? body : 0u;
}

// Register-resident double-precision FMA loop: what the vector ALU of this device sustains when
// nothing but arithmetic is in the way (16 independent chains per lane, no memory traffic).  The
// blind rotation's achieved rate is quoted against this measured figure beside the published peak.
constexpr int kPeakChains = 16, kPeakUnroll = 8;
__global__ __launch_bounds__(256) void fp64_fma_peak_kernel(double *sink, int iters, double a, double b) {
    double v[kPeakChains];
#pragma unroll
    for (int c = 0; c < kPeakChains; ++c) v[c] = (double)(threadIdx.x + c) * 1e-9;
    for (int i = 0; i < iters; ++i)
#pragma unroll
        for (int u = 0; u < kPeakUnroll; ++u)
#pragma unroll
            for (int c = 0; c < kPeakChains; ++c) v[c] = fma(v[c], a, b);
    double total = 0.0;
#pragma unroll
    for (int c = 0; c < kPeakChains; ++c) total += v[c];
    if (total == 12345.678) sink[0] = total;       // never true: keeps the chains alive
}

}  // namespace

// Compute units of the current device (cached).
static int device_cus() {
    static const int cus = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess)
            return n;
        return 0;
    }();
    return cus;
}

// Largest batch that goes to the latency variant: one gate per compute unit of the device.
static int latency_batch_limit() {
    static const int limit = [] {
        if (const char *e = getenv("TFHE_LATENCY_BATCH")) return atoi(e);
        return device_cus();
    }();
    return limit;
}

// Largest batch that goes to the variant for two gates per compute unit.
static int pair_batch_limit() {
    static const int limit = [] {
        if (const char *e = getenv("TFHE_PAIR_BATCH")) return atoi(e);
        return 2 * latency_batch_limit();
    }();
    return limit;
}

// Upper bound on the workgroups of a launch of blind_rotate_kernel, 0 = none (one workgroup per gate, the
// default).  With a bound -- three per CU is what stays resident -- each workgroup takes every
// grid-th gate and all of them walk the key rows together from the first gate to the last.
// Measured on 12,288 gates, when this kernel took them: workgroups that start together stay in the same phase of the step,
// so their transform, product and key-load phases coincide instead of overlapping, and the
// launch takes 68 ms against 56 ms with one workgroup per gate, whose start times spread out.
static int resident_groups() {
    static const int groups = [] {
        if (const char *e = getenv("TFHE_RESIDENT_GROUPS")) { const int v = atoi(e); if (v > 0) return v; }
        return 0;
    }();
    return groups;
}

// TFHE_WAVE_GATES_FROM overrides the rule of launch_blind_rotate: batches from this size on run whole on the
// one-gate-per-wave kernel, smaller ones on the four-wave kernels.
static long wave_gates_from() {
    static const long from = [] {
        const char *e = getenv("TFHE_WAVE_GATES_FROM");
        return e ? atol(e) : -1L;
    }();
    return from;
}

// Kernels that use more than 64 KB of dynamic LDS have to be told so once per device;
// `done` is that kernel's own bit mask of devices.
static int allow_dynamic_lds(const void *kernel, size_t bytes, std::atomic<uint64_t> &done) {
    int dev = 0;
    TFHE_HIP(hipGetDevice(&dev));
    const uint64_t bit = 1ull << (dev & 63);
    if (done.load(std::memory_order_acquire) & bit) return TFHE_OK;
    TFHE_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
    done.fetch_or(bit, std::memory_order_release);
    return TFHE_OK;
}

size_t blind_rotate_lds_bytes() { return sizeof(GateLds); }

// ------------------------------------------------------------------------------------------
// Scratch of the entry point that allocates nothing: the extracted samples between the blind
// rotation and the key switch of at most kStaticGates gates.  Every device the library runs on
// holds its own copy of the array at its own address, looked up once per device at key upload;
// host code only ever uses that looked-up pointer, never the array's name.
// ------------------------------------------------------------------------------------------
constexpr size_t kStaticGates = TFHE_NOALLOC_MAX_GATES;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) uint32_t scratch[kStaticGates * (kN + 1)];
static std::atomic<uint32_t *> scratch_of_device[kMaxDevices];

size_t static_scratch_gates() { return kStaticGates; }

int static_scratch_init() {
    int dev = 0;
    TFHE_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return set_error(TFHE_E_HIP, "device index %d out of range", dev);
    if (scratch_of_device[dev].load(std::memory_order_acquire)) return TFHE_OK;
    uint32_t *ptr = nullptr;
    TFHE_HIP(hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch)));
    if (!ptr) return set_error(TFHE_E_HIP, "no device address for the static scratch array");
    scratch_of_device[dev].store(ptr, std::memory_order_release);
    return TFHE_OK;
}

uint32_t *static_scratch_ptr() {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    return scratch_of_device[dev].load(std::memory_order_acquire);
}

int launch_bk_to_spectrum(const uint32_t *bk_raw, double2 *bk_fft, const double2 *tables, int n,
                          hipStream_t stream) {
    hipLaunchKernelGGL(bk_to_spectrum_kernel, dim3((unsigned)n * 8), dim3(256), 0, stream, bk_raw, bk_fft, tables);
    TFHE_HIP(hipGetLastError());
    return TFHE_OK;
}

// The blind rotations, each plain and with the rounding distance recorded (the launcher chooses without regard to that, so
// that what is recorded is of the kernel that serves the same call otherwise), and the widest matrix-core key
// switch, with their dynamic LDS sizes and per-device "attribute set" masks
namespace {
enum Rotation { kFourWaves, kLatency, kPair, kWaveMeet, kWaveLone, kRotations };
struct BigLdsKernel { const void *fn; size_t lds; std::atomic<uint64_t> done; };
BigLdsKernel rotation_kernels[kRotations][2] = {
    {{reinterpret_cast<const void *>(&blind_rotate_kernel<false>), sizeof(GateLds), {0}},
     {reinterpret_cast<const void *>(&blind_rotate_kernel<true>), sizeof(GateLds), {0}}},
    {{reinterpret_cast<const void *>(&blind_rotate_latency_kernel<false>), sizeof(GateLds), {0}},
     {reinterpret_cast<const void *>(&blind_rotate_latency_kernel<true>), sizeof(GateLds), {0}}},
    {{reinterpret_cast<const void *>(&blind_rotate_pair_kernel<false>), sizeof(GateLds), {0}},
     {reinterpret_cast<const void *>(&blind_rotate_pair_kernel<true>), sizeof(GateLds), {0}}},
    {{reinterpret_cast<const void *>(&blind_rotate_wave_kernel<false, true>), sizeof(WaveLds), {0}},
     {reinterpret_cast<const void *>(&blind_rotate_wave_kernel<true, true>), sizeof(WaveLds), {0}}},
    {{reinterpret_cast<const void *>(&blind_rotate_wave_kernel<false, false>), sizeof(WaveLds), {0}},
     {reinterpret_cast<const void *>(&blind_rotate_wave_kernel<true, false>), sizeof(WaveLds), {0}}},
};
BigLdsKernel widest_key_switch = {reinterpret_cast<const void *>(&key_switch_mfma_kernel<4>), sizeof(KsLds<4>), {0}};
int allow(BigLdsKernel &k) { return allow_dynamic_lds(k.fn, k.lds, k.done); }

static_assert(kThreadsPerGate == 64 * kWaveGates, "workgroups of one size");
int launch_rotation(Rotation which, size_t groups, const BlindRotateArgs &a, hipStream_t stream) {
    BigLdsKernel &k = rotation_kernels[which][a.margin ? 1 : 0];
    if (int rc = allow(k)) return rc;
    BlindRotateArgs args = a;
    void *params[] = {&args};
    (void)hipLaunchKernel(k.fn, dim3((unsigned)groups), dim3(kThreadsPerGate), params, k.lds, stream);
    TFHE_HIP(hipGetLastError());
    return TFHE_OK;
}
}  // namespace

// Everything a launch would otherwise set up on first use (dynamic-LDS permissions, the cached
// device properties, the address of the static scratch), done once per device at key upload so
// that later calls only launch.
int prepare_kernels() {
    (void)pair_batch_limit();
    (void)resident_groups();
    (void)wave_gates_from();
    for (auto &forms : rotation_kernels)
        for (BigLdsKernel &k : forms)
            if (int rc = allow(k)) return rc;
    if (int rc = allow(widest_key_switch)) return rc;
    return static_scratch_init();
}

// Items first .. count - 1 of a batch with the four-wave kernels.
static int launch_four_waves(const BlindRotateArgs &a, hipStream_t stream) {
    const size_t items = a.count - a.first, bound = (size_t)resident_groups();
    if (items <= (size_t)latency_batch_limit()) return launch_rotation(kLatency, items, a, stream);
    if (items <= (size_t)pair_batch_limit()) return launch_rotation(kPair, items, a, stream);
    return launch_rotation(kFourWaves, bound ? std::min(items, bound) : items, a, stream);
}

static_assert(kRoundPerCu == 2 * kWaveGates, "two workgroups of the wave kernel per CU");

// Items first .. count - 1 with the wave kernel.  With more than one workgroup per CU the waves of a workgroup meet before the
// products, so that their key reads hit L1 (8,192 gates 26.0 -> 25.2 ms); a lone workgroup leaves L1 and L2 idle enough
// and loses by waiting (a call of 1,024 gates 3.77 ms on the form without, 4.50 on the form with).
// Five or six gates per CU are spread over two workgroups on every CU instead of filling half of the CUs with two whole ones:
// calls of 1,280 gates 5.52 -> 5.16 ms, 1,536 gates 5.64 -> 5.16, 3,584 gates 12.5 -> 11.85.  Seven are not: the CUs that end early
// leave the others their power (1,554 gates 5.66 ms as they are, 5.90 spread; 1,792 gates 5.84 and 6.01).  Four at a time and the others in
// a launch of their own is slower: 1,280 gates 5.37 against 5.20 ms, 1,536 gates 5.91 against 5.23.
// Two lone launches for two keys, on two streams, do share the CUs (see the kernel).
static int launch_wave(const BlindRotateArgs &a, size_t cus, hipStream_t stream) {
    const size_t items = a.count - a.first, least = (items + kWaveGates - 1) / kWaveGates;
    if (items <= kWaveGates * cus) return launch_rotation(kWaveLone, least, a, stream);
    return launch_rotation(kWaveMeet, items <= 6 * cus ? 2 * cus : least, a, stream);
}

// Whole rounds go to the wave kernel, and what remains follows on the kernel that serves it fastest (times in kernels.h): seven
// gates per CU in the same launch, four to six in one of their own (behind the rounds of the same launch their workgroups would
// go to whichever CU ended first), fewer on the four-wave kernels.
int launch_blind_rotate(const BlindRotateArgs &args, hipStream_t stream) {
    if (args.count == 0) return TFHE_OK;
    BlindRotateArgs a = args;
    a.first = 0;
    const size_t cus = device_cus() > 0 ? (size_t)device_cus() : 256;
    size_t rest = a.count % (kRoundPerCu * cus);
    RestKernel kernel = rest_kernel((rest + cus - 1) / cus, rest < a.count);
    if (wave_gates_from() >= 0) {
        kernel = a.count >= (size_t)wave_gates_from() ? RestKernel::kWithRounds : RestKernel::kFourWaves;
        rest = a.count;
    }
    if (kernel == RestKernel::kWithRounds) rest = 0;
    if (rest < args.count) {
        a.count = args.count - rest;
        if (int rc = launch_wave(a, cus, stream)) return rc;
    }
    if (!rest) return TFHE_OK;
    a.first = args.count - rest;
    a.count = args.count;
    return kernel == RestKernel::kWave ? launch_wave(a, cus, stream) : launch_four_waves(a, stream);
}

int launch_ksk_to_tiles(const uint32_t *ksk, int stride, int words, void *tiles, hipStream_t stream) {
    hipLaunchKernelGGL(ksk_to_tiles_kernel, dim3(kN, 16), dim3(256), 0, stream, ksk, stride, words,
                       reinterpret_cast<v4i *>(tiles));
    TFHE_HIP(hipGetLastError());
    return TFHE_OK;
}

size_t ksk_tiles_bytes() { return (size_t)16 * kN * 4 * 64 * sizeof(v4i); }

int launch_key_switch(const KeySwitchArgs &a, hipStream_t stream) {
    if (a.count == 0) return TFHE_OK;
    if (a.ksk_tiles && a.matrix && a.t == 8 && a.basebit == 2 && a.n + 1 <= 512) {
        // Gates of a workgroup: as many as there are, up to 128 while one workgroup per CU serves them all; beyond,
        // 64, of which two workgroups share a CU (64 against 128: 512 gates 87 against 65 us, 1,024 gates 94
        // against 125).  A sixteenth of the mask words each fills the chip for up to 128 gates (against an
        // eighth: 128 gates 23 against 29 us, 256 gates 43 against 33).
        KeySwitchArgs m = a;
        const unsigned tiles = a.count <= 32 ? 1 : a.count <= 64 || a.count > 512 ? 2 : 4;
        m.splits = a.count <= 128 ? 16 : 8;
        hipLaunchKernelGGL(zero_outputs_kernel, dim3((unsigned)a.count), dim3(256), 0, stream, m);
        TFHE_HIP(hipGetLastError());
        const dim3 grid((unsigned)((a.count + 32 * tiles - 1) / (32 * tiles)), 16, (unsigned)m.splits);
        if (tiles == 1) {
            hipLaunchKernelGGL(key_switch_mfma_kernel<1>, grid, dim3(256), sizeof(KsLds<1>), stream, m);
        } else if (tiles == 2) {
            hipLaunchKernelGGL(key_switch_mfma_kernel<2>, grid, dim3(256), sizeof(KsLds<2>), stream, m);
        } else {
            if (int rc = allow(widest_key_switch)) return rc;
            hipLaunchKernelGGL(key_switch_mfma_kernel<4>, grid, dim3(256), sizeof(KsLds<4>), stream, m);
        }
        TFHE_HIP(hipGetLastError());
        return TFHE_OK;
    }
    if (a.splits < 1 || (a.splits & (a.splits - 1)) || a.splits > 64)
        return set_error(TFHE_E_PARAM, "key-switch splits must be a power of two <= 64");
    if (a.splits > 1) {
        hipLaunchKernelGGL(zero_outputs_kernel, dim3((unsigned)a.count), dim3(256), 0, stream, a);
        TFHE_HIP(hipGetLastError());
    }
    const dim3 grid((unsigned)(a.count * a.splits)), block(256);
    switch (a.t) {
#define KS_CASE(T) case T: hipLaunchKernelGGL(key_switch_kernel<T>, grid, block, 0, stream, a); break;
        KS_CASE(1) KS_CASE(2) KS_CASE(3) KS_CASE(4) KS_CASE(5) KS_CASE(6) KS_CASE(7) KS_CASE(8)
        KS_CASE(9) KS_CASE(10) KS_CASE(11) KS_CASE(12)
#undef KS_CASE
    default: return set_error(TFHE_E_PARAM, "unsupported key-switch digit count %d", a.t);
    }
    TFHE_HIP(hipGetLastError());
    return TFHE_OK;
}

int launch_mux_combine(uint32_t *ext, const tfhe_gate_rec *recs, size_t count, hipStream_t stream) {
    if (count == 0) return TFHE_OK;
    hipLaunchKernelGGL(mux_combine_kernel, dim3((unsigned)count), dim3(256), 0, stream, ext, recs, count);
    TFHE_HIP(hipGetLastError());
    return TFHE_OK;
}

int launch_gather_outputs(const uint32_t *wires, const tfhe_out_ref *refs, uint32_t *out, size_t count,
                          int words, hipStream_t stream) {
    if (count == 0) return TFHE_OK;
    hipLaunchKernelGGL(gather_outputs_kernel, dim3((unsigned)count), dim3(256), 0, stream, wires, refs, out,
                       count, words);
    TFHE_HIP(hipGetLastError());
    return TFHE_OK;
}

// Time the FMA loop with HIP events on `stream`; *tflops = achieved double-precision rate.
int measure_fp64_fma_peak(hipStream_t stream, double *sink, double *tflops) {
    const int cus = device_cus() > 0 ? device_cus() : 256;
    const int blocks = cus * 8, iters = 4096;               // 8 workgroups of 4 waves per CU: 8 waves per SIMD
    hipEvent_t t0, t1;
    TFHE_HIP(hipEventCreate(&t0));
    TFHE_HIP(hipEventCreate(&t1));
    float best = 0.0f;
    int rc = TFHE_OK;
    for (int rep = 0; rep < 3 && rc == TFHE_OK; ++rep) {      // the first launch warms the clocks up
        hipError_t e = hipEventRecord(t0, stream);
        hipLaunchKernelGGL(fp64_fma_peak_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, sink, iters, 0.999999, 1e-7);
        if (e == hipSuccess) e = hipGetLastError();
        if (e == hipSuccess) e = hipEventRecord(t1, stream);
        if (e == hipSuccess) e = hipEventSynchronize(t1);
        float ms = 0.0f;
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, t0, t1);
        if (e != hipSuccess) { rc = set_error(TFHE_E_HIP, "FMA peak measurement failed: %s", hipGetErrorString(e)); break; }
        if (rep == 0 || ms < best) best = ms;
    }
    (void)hipEventDestroy(t0);
    (void)hipEventDestroy(t1);
    if (rc) return rc;
    const double flops = 2.0 * kPeakChains * kPeakUnroll * (double)iters * 256.0 * (double)blocks;
    *tflops = flops / ((double)best * 1e-3) / 1e12;
    return TFHE_OK;
}

int launch_fill_trivial(uint32_t *ct, int words, int bit, hipStream_t stream) {
    hipLaunchKernelGGL(fill_trivial_kernel, dim3(1), dim3(256), 0, stream, ct, words,
                       bit ? kEighth : 0u - kEighth);
    TFHE_HIP(hipGetLastError());
    return TFHE_OK;
}

}  // namespace tfhe
