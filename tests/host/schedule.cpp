// Host run of the schedule that layer calls and gate streams use (csrc/schedule.h): earliest levels, levels filled by
// launch size, wire pool.  Random circuits with multiplexers and lowered layers, on devices of 1 to 256 compute units.
// A filled schedule has to keep the number of levels, run no gate before what it reads, keep the two records
// of a multiplexer side by side, and on a wire pool hand every gate and every output the wire it names, where
// all of a level's reads come before its writes.  Prints the gates that filling moved, per group of circuits.
#include <algorithm>
#include <chrono>
#include <cstring>

#include "../../paper_1806_03461_amd/csrc/schedule.h"
#include "device_stubs.h"

using namespace tfhe;

#define CHECK(cond) do { if (!(cond)) { std::fprintf(stderr, "%s:%d: %s\n", __FILE__, __LINE__, #cond); std::exit(1); } } while (0)

namespace {

uint64_t g_state = 0xD1B54A32D192ED03ull;
uint32_t next_u32() {          // xorshift64*
    g_state ^= g_state >> 12; g_state ^= g_state << 25; g_state ^= g_state >> 27;
    return (uint32_t)((g_state * 0x2545F4914F6CDD1Dull) >> 32);
}
uint32_t below(uint32_t n) { return next_u32() % n; }

struct Circuit {
    std::vector<tfhe_gate_rec> gates;
    std::vector<tfhe_out_ref> outs;
    size_t nwires = 0, n_fixed = 0;
    void gate(int op, int32_t a, int32_t b, int32_t out) { gates.push_back({(uint8_t)op, (uint8_t)below(2), (uint8_t)below(2), 0, a, b, out}); }
};

// Inputs come from the last `reach` wires, rarely from anywhere: a small reach makes a deep and narrow circuit.
Circuit random_circuit(size_t fixed, size_t ngates, size_t reach, uint32_t mux_percent) {
    Circuit c;
    c.n_fixed = c.nwires = fixed;
    auto pick = [&] {
        const size_t from = c.nwires > reach && below(16) ? c.nwires - reach : 0;
        return (int32_t)(from + below((uint32_t)(c.nwires - from)));
    };
    while (c.gates.size() < ngates) {
        const int32_t out = (int32_t)c.nwires, a = pick(), b = pick();
        if (below(100) < mux_percent) {
            c.gate(TFHE_MUX, a, b, out);
            const uint8_t selector = c.gates.back().neg0;
            c.gate(TFHE_MUX_ELSE, a, pick(), out);
            c.gates.back().neg0 = selector;
        } else {
            c.gate((int)below(6), a, b, out);
        }
        ++c.nwires;
    }
    for (int k = 0; k < 20; ++k) c.outs.push_back({(int32_t)below((uint32_t)c.nwires), (int32_t)below(2)});
    return c;
}

Circuit lowered(int d, int p, uint32_t flags) {
    std::vector<int8_t> W((size_t)d * p);
    std::vector<int32_t> T(p);
    for (int8_t &w : W) w = below(20) ? (below(2) ? 1 : -1) : 0;
    for (int32_t &t : T) t = (int32_t)(d / 3 + below((uint32_t)(d / 3)));
    tfhe_gate_rec *g = nullptr; tfhe_out_ref *o = nullptr; size_t ng = 0, no = 0;
    Circuit c;
    CHECK(bnn_dense_lower_opts(d, W.data(), T.data(), p, 0, flags, &g, &ng, &o, &no, &c.nwires) == TFHE_OK);
    c.gates.assign(g, g + ng);
    c.outs.assign(o, o + no);
    c.n_fixed = (size_t)d + 2;
    tfhe_free_buffer(g); tfhe_free_buffer(o);
    return c;
}

// One wide level and a chain at whose every step one more gate becomes ready that nothing reads: its latest level is
// the circuit's last.
Circuit deep_circuit(size_t depth, size_t wide) {
    Circuit c;
    c.n_fixed = c.nwires = 2;
    for (size_t k = 0; k < wide; ++k) c.gate(TFHE_AND, 0, 1, (int32_t)c.nwires++);
    for (int32_t chain = 0, k = 0; k < (int32_t)depth; ++k, c.nwires += 2) {
        c.gate(TFHE_AND, chain, 1, (int32_t)c.nwires);
        c.gate(TFHE_OR, chain, 1, (int32_t)c.nwires + 1);
        chain = (int32_t)c.nwires;
    }
    return c;
}

// Levels and plan of `c` on `cus` compute units; returns how many records filling moved.
size_t check(const Circuit &c, size_t cus) {
    const std::vector<tfhe_gate_rec> &g = c.gates;
    Levels early, lv;
    CHECK(levelize(g.data(), g.size(), c.nwires, early) == TFHE_OK);
    lv = early;
    fill_levels(g.data(), g.size(), c.nwires, cus, lv);
    CHECK(lv.max_level == early.max_level && lv.any_mux == early.any_mux);
    CHECK(lv.level.size() == g.size() && lv.start.size() == (size_t)lv.max_level + 2);

    std::vector<int32_t> ready(c.nwires, 0);          // level that writes a wire
    std::vector<size_t> width(lv.start.size(), 0);
    size_t moved = 0;
    for (size_t k = 0; k < g.size(); ++k) {
        const int32_t l = lv.level[k];
        CHECK(l >= 1 && l <= lv.max_level && ready[g[k].in0] < l && ready[g[k].in1] < l);
        if (g[k].op == TFHE_MUX) CHECK(lv.level[k + 1] == l && ready[g[k + 1].in1] < l);
        else ready[g[k].out] = l;
        ++width[(size_t)l];
        CHECK(l >= early.level[k]);
        moved += l != early.level[k];
    }
    size_t at = 0;
    for (int32_t l = 0; l <= lv.max_level + 1; ++l) {
        CHECK(lv.start[(size_t)l] == at);
        if (l >= 1 && l <= lv.max_level) CHECK(width[(size_t)l] > 0);
        at += l <= lv.max_level ? width[(size_t)l] : 0;
    }
    CHECK(at == g.size());

    std::vector<tfhe_gate_rec> sorted(g.size());
    std::vector<tfhe_out_ref> outs = c.outs;
    size_t pool = 0;
    CHECK(plan_wire_pool(g.data(), g.size(), c.nwires, c.n_fixed, lv, sorted.data(), outs.data(), outs.size(), &pool) == TFHE_OK);
    CHECK(pool >= c.n_fixed && pool <= c.nwires);
    std::vector<size_t> from(g.size()), next(lv.start.begin(), lv.start.end());      // the record at each sorted position
    for (size_t k = 0; k < g.size(); ++k) from[next[(size_t)lv.level[k]]++] = k;
    std::vector<int32_t> holds(pool, -1);              // the wire whose value a slot holds
    for (size_t w = 0; w < c.n_fixed; ++w) holds[w] = (int32_t)w;
    for (int32_t l = 1; l <= lv.max_level; ++l) {
        const size_t lo = lv.start[(size_t)l], hi = lv.start[(size_t)l + 1];
        for (size_t k = lo; k < hi; ++k) {
            const tfhe_gate_rec &s = sorted[k], &r = g[from[k]];
            CHECK(s.op == r.op && s.neg0 == r.neg0 && s.neg1 == r.neg1);
            CHECK(s.in0 >= 0 && (size_t)s.in0 < pool && s.in1 >= 0 && (size_t)s.in1 < pool);
            CHECK(s.out >= (int32_t)c.n_fixed && (size_t)s.out < pool);
            CHECK(holds[s.in0] == r.in0 && holds[s.in1] == r.in1);
            if (s.op == TFHE_MUX) CHECK(k + 1 < hi && sorted[k + 1].op == TFHE_MUX_ELSE && sorted[k + 1].out == s.out);
        }
        for (size_t k = lo; k < hi; ++k) holds[sorted[k].out] = -2 - (int32_t)k;      // written by two gates of a level?
        for (size_t k = lo; k < hi; ++k) {
            if (sorted[k].op != TFHE_MUX) CHECK(holds[sorted[k].out] == -2 - (int32_t)k);
        }
        for (size_t k = lo; k < hi; ++k) holds[sorted[k].out] = g[from[k]].out;
    }
    for (size_t k = 0; k < outs.size(); ++k) {
        CHECK(outs[k].value == c.outs[k].value);
        if (c.outs[k].wire >= 0) CHECK(holds[outs[k].wire] == c.outs[k].wire);
        else CHECK(outs[k].wire == c.outs[k].wire);
    }
    return moved;
}

// today's times of a blind rotation on 256 CUs; the table that levels are filled by holds those of earlier kernels
double measured_ms(size_t items, size_t cus) {
    const double rest[8] = {0.0, 1.48, 2.08, 3.26, 3.68, 5.15, 5.15, 5.58};
    const size_t round = kRoundPerCu * cus, left = items % round;
    return 6.0 * (double)(items / round) + rest[(left + cus - 1) / cus];
}

// time of the blind rotations, as the scheduler's table has it, or by the times above
double estimate(const Circuit &c, size_t cus, bool filled, double (*time)(size_t, size_t) = rotation_ms) {
    Levels lv;
    CHECK(levelize(c.gates.data(), c.gates.size(), c.nwires, lv) == TFHE_OK);
    if (filled) fill_levels(c.gates.data(), c.gates.size(), c.nwires, cus, lv);
    double ms = 0.0;
    for (int32_t l = 1; l <= lv.max_level; ++l) ms += time(lv.start[(size_t)l + 1] - lv.start[(size_t)l], cus);
    return ms;
}

}  // namespace

int main() {
    size_t moved = 0, circuits = 0;
    for (size_t cus : {1, 2, 5, 16, 256})
        for (uint32_t mux : {0u, 30u, 100u})
            for (size_t reach : {3, 40, 700, 5000})
                for (int rep = 0; rep < 3; ++rep, ++circuits)
                    moved += check(random_circuit(1 + below(40), 1 + below(6000), reach, mux), cus);
    std::printf("random circuits %zu moved %zu\n", circuits, moved);
    CHECK(moved > 0);

    // layers, wider than a gate per CU; every way to lower them that gives other gates
    const uint32_t flags[] = {0, TFHE_LOWER_MUX_COMPARATOR, TFHE_LOWER_PLUS_ONE, TFHE_LOWER_SHARE_GATES, TFHE_LOWER_SORTING_NETWORK};
    for (uint32_t f : flags) {
        const Circuit c = lowered(64, 24, f);
        const size_t m = check(c, 256), few = check(c, 3);
        const double early = estimate(c, 256, false, measured_ms), filled = estimate(c, 256, true, measured_ms);
        std::printf("layer 64 -> 24, flags %u: moved %zu of %zu (3 CUs: %zu), estimate %.1f -> %.1f ms, by today's times %.1f -> %.1f\n", f, m,
                    c.gates.size(), few, estimate(c, 256, false), estimate(c, 256, true), early, filled);
        CHECK(m > 0 && estimate(c, 256, true) <= estimate(c, 256, false));
        CHECK(filled <= early);
    }
    // circuits that keep their earliest levels: no level of more than a gate per CU, and levels of more than kRounds rounds
    CHECK(check(lowered(33, 4, 0), 256) == 0);
    const Circuit big = lowered(64, 24, 0);
    Levels lv;
    CHECK(levelize(big.gates.data(), big.gates.size(), big.nwires, lv) == TFHE_OK);
    CHECK(big.gates.size() > kRounds * kRoundPerCu * (size_t)lv.max_level && check(big, 1) == 0);
    // Filling takes time in proportion to the circuit, not to its depth squared: 0.02 s on one core, where looking
    // through every level between a gate's and the last took 8 s.
    {
        const Circuit c = deep_circuit(100000, 600);
        CHECK(levelize(c.gates.data(), c.gates.size(), c.nwires, lv) == TFHE_OK);
        const auto start = std::chrono::steady_clock::now();
        fill_levels(c.gates.data(), c.gates.size(), c.nwires, 256, lv);
        const double s = std::chrono::duration<double>(std::chrono::steady_clock::now() - start).count();
        std::printf("100,000 levels: %.3f s\n", s);
        CHECK(s < 2.0);
    }
    std::puts("schedule: ok");
    return 0;
}
