// Stand-ins for the launchers of kernels.hip in host builds of the library: none may be reached.
#pragma once
#include <cstdio>
#include <cstdlib>

#include "../../paper_1806_03461_amd/csrc/kernels.h"

namespace tfhe {
static int unreachable(const char *what) { std::fprintf(stderr, "device launcher %s reached\n", what); std::abort(); }
size_t blind_rotate_lds_bytes(int) { return 0; }
int launch_bk_to_spectrum(const uint32_t *, double2 *, const double2 *, int, hipStream_t) { return unreachable("bk"); }
int launch_blind_rotate(const BlindRotateArgs &, hipStream_t) { return unreachable("blind_rotate"); }
int launch_key_switch(const KeySwitchArgs &, hipStream_t) { return unreachable("key_switch"); }
size_t ksk_tiles_bytes() { return 0; }
int launch_ksk_to_tiles(const uint32_t *, int, int, void *, hipStream_t) { return unreachable("tiles"); }
int launch_mux_combine(uint32_t *, const tfhe_gate_rec *, size_t, hipStream_t) { return unreachable("mux"); }
int launch_gather_outputs(const uint32_t *, const tfhe_out_ref *, uint32_t *, size_t, int, hipStream_t) { return unreachable("gather"); }
int launch_fill_trivial(uint32_t *, int, int, hipStream_t) { return unreachable("fill"); }
int prepare_kernels() { return unreachable("prepare"); }
int measure_fp64_fma_peak(hipStream_t, double *, double *) { return unreachable("peak"); }
uint32_t *static_scratch_ptr() { return nullptr; }
size_t static_scratch_gates() { return 4096; }
}  // namespace tfhe
