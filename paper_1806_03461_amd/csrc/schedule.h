// The schedule of a circuit (executor.cpp): levels, launch-sized levels and the wire pool.  Host code without device
// work, declared here so that host programs can run it by itself.
#pragma once
#include "common.h"

namespace tfhe {

struct Levels {
    std::vector<int32_t> level;     // per record
    std::vector<size_t> start;      // records of level l occupy sorted positions [start[l], start[l+1])
    int32_t max_level = 0;
    bool any_mux = false;
};

// Validation and earliest-possible levels of a topologically ordered gate list.
int levelize(const tfhe_gate_rec *gates, size_t ngates, size_t nwires, Levels &lv);

// Gates with slack moved to later levels where that fills launches on a device with `cus` compute units; `lv`
// comes from levelize and keeps its number of levels.  Circuits whose levels average more than kRounds full
// rounds of the blind rotation, and circuits without a level of more than one gate per CU, stay as they are.
constexpr size_t kRounds = 16;
void fill_levels(const tfhe_gate_rec *gates, size_t ngates, size_t nwires, size_t cus, Levels &lv);

// Records sorted by level, in slots of a wire pool.
int plan_wire_pool(const tfhe_gate_rec *gates, size_t ngates, size_t nwires, size_t n_fixed, const Levels &lv,
                   tfhe_gate_rec *sorted, tfhe_out_ref *outs, size_t nouts, size_t *pool_wires);

}  // namespace tfhe
