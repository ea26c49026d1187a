// Launchers of the gfx950 kernels (kernels.hip), called by the host executor.
#pragma once
#include "common.h"

namespace tfhe {

struct BlindRotateArgs {
    const tfhe_gate_rec *recs;   // device; NULL: gate i reads in0[i], in1[i] with uniform_op
    int uniform_op;
    const uint32_t *in0, *in1;   // device wire arrays the records index into
    const uint32_t *in1_alt;     // uniform TFHE_MUX only: launch item 2g is AND(in0[g], in1[g]),
                                 // item 2g+1 is AND(NOT in0[g], in1_alt[g])
    uint32_t *ext;               // device [count][1025]: extracted samples
    size_t count;
    size_t first;                // set by the launcher: a launch takes items first .. count - 1
    const double2 *bk_fft;       // device [n][4][4][512], and behind it [n][8][3][4][64] (sums3.h)
    const double2 *tables;       // device: exp(i pi j / 1024), j < 2048, and the constants of dft8.h
    int n, bgbit;
    double *margin;              // device, optional: largest rounding distance seen
};

struct KeySwitchArgs {
    const uint32_t *ext;         // device [count][1025]
    const tfhe_gate_rec *recs;   // device; NULL: gate i writes out[i]
    uint32_t *out;               // device wire array
    size_t count;
    const uint32_t *ksk;         // device [1024][t][2^basebit - 1][stride] plus one zero row
    int n, t, basebit;
    int uniform_mux;             // recs == NULL: items come in pairs, item 2g carries the sum and writes out[g]
    int splits;                  // gather kernel: workgroups sharing one gate's mask words (power of two)
    int stride;                  // words per key row on the device: n+1 rounded up to even, pad = 0
    const void *ksk_tiles;       // device, optional: the key as signed-byte tiles for the matrix-core kernel
    int matrix;                  // use the matrix-core kernel (needs ksk_tiles, t = 8, basebit = 2, n + 1 <= 512)
};

// What the scheduler of narrow circuits weighs launches by: the milliseconds that a blind rotation of `items` gates took on a device
// with `cus` compute units (256 of them, n = 500) before the wave kernel's step was cut as it is.  It takes now, by events around the rotation:
//   wave kernel       eight gates per CU at a time: 6.0 ms a round, 3.68 with at most four per CU in it, 5.0 to 5.25 with five or six,
//                     spread evenly over the CUs, 5.58 with seven
//   four-wave kernels 1.46 to 1.48 ms, 1.90 to 2.08 and 2.99 to 3.26 for one, two and three gates per CU, 5.3 for five
// The table is not these: filled by them, 213 dense layers of up to 110,000 gates whose schedule changes would by these times take 0.4 % less on
// average (4 % less to 1.8 % more), ten scores of 256 inputs, measured, 52.9 ms instead of 53.5 and five other circuits the same within
// 0.2 %, while of the 22,593 gates of 24 sorting networks of 64 inputs none would move.  The launcher's rule does not use it.
inline double rest_ms(size_t per_cu) {      // a launch of less than a round
    const double ms[9] = {0.0, 1.55, 2.1, 3.32, 4.15, 5.4, 5.85, 6.0, 6.42};
    return ms[per_cu];
}
// The kernel that serves a batch's last, partial round fastest: the wave kernel together with the whole rounds or in a launch of its
// own, or the four-wave kernels.  Calls on the wave kernel and on the four-wave ones: four gates per CU, 1,024 gates 3.77 and 5.48 ms,
// 3,072 (behind a round) 10.6 and 11.95; five, 1,025 gates 5.33 and 5.93, 1,280 gates 5.16 and 5.97, behind a round 3,073 gates
// 12.62 and 12.51, 3,328 gates 11.97 and 11.96.
enum class RestKernel { kFourWaves, kWave, kWithRounds };
inline RestKernel rest_kernel(size_t per_cu, bool behind_rounds) {
    if (per_cu >= 7) return RestKernel::kWithRounds;
    return per_cu == 4 || per_cu == 6 || (per_cu == 5 && !behind_rounds) ? RestKernel::kWave : RestKernel::kFourWaves;
}
constexpr size_t kRoundPerCu = 8;
inline double rotation_ms(size_t items, size_t cus) {
    const size_t round = kRoundPerCu * cus, rest = items % round;
    return 6.42 * (double)(items / round) + rest_ms((rest + cus - 1) / cus);
}

// complex words of the key's spectra, both forms
inline size_t bk_spectrum_words(size_t n) { return n * 4 * (4 + 3) * 512; }

size_t blind_rotate_lds_bytes();
int launch_bk_to_spectrum(const uint32_t *bk_raw, double2 *bk_fft, const double2 *tables, int n,
                          hipStream_t stream);
int launch_blind_rotate(const BlindRotateArgs &a, hipStream_t stream);
int launch_key_switch(const KeySwitchArgs &a, hipStream_t stream);
// the key-switching key (device, padded rows) as int8 operand tiles; `tiles` holds ksk_tiles_bytes()
size_t ksk_tiles_bytes();
int launch_ksk_to_tiles(const uint32_t *ksk, int stride, int words, void *tiles, hipStream_t stream);
// ext[e] += ext[e+1]; ext[e].body += 1/8 for every first half e of a multiplexer
int launch_mux_combine(uint32_t *ext, const tfhe_gate_rec *recs, size_t count, hipStream_t stream);
int launch_gather_outputs(const uint32_t *wires, const tfhe_out_ref *refs, uint32_t *out, size_t count,
                          int words, hipStream_t stream);
// per-device set-up at key upload: kernel attributes, address of the static scratch array
int prepare_kernels();
// the static scratch of the current device (NULL before prepare_kernels ran on it) and the
// number of extracted samples ([1025] words each) it holds
uint32_t *static_scratch_ptr();
size_t static_scratch_gates();
// achieved TFLOP/s of a register-resident FP64 FMA loop on the current device (synchronises `stream`)
int measure_fp64_fma_peak(hipStream_t stream, double *sink, double *tflops);
int launch_fill_trivial(uint32_t *ct, int words, int bit, hipStream_t stream);

}  // namespace tfhe
