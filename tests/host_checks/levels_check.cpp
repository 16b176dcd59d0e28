// The level scheduler (she_circuits.cpp: levelize, even_levels) on the host: whatever the circuit and the device, evened levels
// hold every entry once, each after its operands, in as many levels as the circuit is deep, none empty, MUXes behind gates, and
// their estimated time is at most that of the earliest levels; level_time grows with the level up to its steps and beyond.
#include <chrono>
#include <cstdio>
#include <random>

#include "she_internal.h"

static int failures = 0;
#define CHECK(c, ...) do { if (!(c)) { failures++; std::printf(__VA_ARGS__); } } while (0)
using namespace she;

static Netlist circuit(std::mt19937 &rng, uint32_t cap, size_t entries, uint32_t reach, bool muxes)
{
    Netlist nl(cap, false, true);
    std::vector<uint32_t> wires;
    for (size_t k = 0; k < entries; k++) {
        auto pick = [&]() -> uint32_t {
            const uint32_t r = rng() % (reach + 4);
            if (r >= reach || wires.empty()) return rng() % (cap + 2);               // an input or a constant
            return wires[wires.size() - 1 - rng() % std::min<size_t>(reach, wires.size())];
        };
        const uint32_t kind = rng() % 4;
        wires.push_back(kind == 0 && muxes ? nl.mux(pick(), pick(), pick()) : kind == 1 ? nl.gate3(SHE_MAJ3, pick(), pick(), pick())
                                                                                     : nl.gate(SHE_AND, pick(), pick()));
    }
    return nl;
}

static double estimate(const Netlist &nl, const std::vector<size_t> &bounds, uint32_t cus)
{
    double us = 0;
    for (size_t lv = 0; lv + 1 < bounds.size(); lv++) {
        uint64_t r = 0;
        for (size_t g = bounds[lv]; g < bounds[lv + 1]; g++) r += is_mux_type(nl.type[g]) ? 2 : 1;
        us += level_time(r, cus);
    }
    return us;
}

static void check(const Netlist &nl, uint32_t cus, const char *what)
{
    Netlist early = nl, even = nl;
    std::vector<size_t> m0, m1;
    const std::vector<size_t> b0 = early.levelize(&m0), b1 = even.levelize(&m1, cus);
    CHECK(b0.size() == b1.size(), "%s: %zu levels, %zu evened\n", what, b0.size() - 1, b1.size() - 1);
    CHECK(even.type.size() == nl.type.size() && b1.back() == nl.type.size(), "%s: %zu entries\n", what, even.type.size());
    CHECK(estimate(even, b1, cus) <= estimate(early, b0, cus) * (1 + 1e-12), "%s: %.0f us at the earliest, %.0f evened\n", what,
          estimate(early, b0, cus), estimate(even, b1, cus));
    const uint32_t first = nl.cap + 2;
    std::vector<int> level(nl.next_temp - first, -1);
    std::vector<size_t> was(nl.next_temp - first);
    for (size_t g = 0; g < nl.type.size(); g++) was[nl.out[g] - first] = g;
    for (size_t lv = 0; lv + 1 < b1.size(); lv++) {
        CHECK(b1[lv] < b1[lv + 1] && b1[lv] <= m1[lv] && m1[lv] <= b1[lv + 1], "%s: level %zu\n", what, lv);
        for (size_t g = b1[lv]; g < b1[lv + 1]; g++) {
            CHECK(is_mux_type(even.type[g]) == (g >= m1[lv]), "%s: kinds of level %zu\n", what, lv);
            const size_t w = was[even.out[g] - first];
            CHECK(even.type[g] == nl.type[w] && even.in0[g] == nl.in0[w] && even.in1[g] == nl.in1[w] && even.in2[g] == nl.in2[w],
                  "%s: an entry changed\n", what);
            for (uint32_t op : {even.in0[g], even.in1[g], has_third_operand(even.type[g]) ? even.in2[g] : 0u})
                CHECK(op < first || (level[op - first] >= 0 && level[op - first] < (int)lv), "%s: an operand is not there yet\n", what);
        }
        for (size_t g = b1[lv]; g < b1[lv + 1]; g++) {
            CHECK(level[even.out[g] - first] < 0, "%s: an entry twice\n", what);
            level[even.out[g] - first] = (int)lv;
        }
    }
    CHECK(even.compact_temporaries(b1) > 0, "%s: a temporary lost its slot\n", what);
}

int main()
{
    std::mt19937 rng(7);
    check(Netlist(4), 256, "empty");
    for (uint32_t cus : {1u, 4u, 64u, 256u})
        for (size_t entries : {1, 2, 17, 300, 3000})
            for (uint32_t reach : {0u, 1u, 5u, 60u, 700u})
                for (bool muxes : {false, true}) {
                    char what[96];
                    std::snprintf(what, sizeof what, "%zu entries, reach %u, %u compute units%s", entries, reach, cus, muxes ? ", MUXes" : "");
                    check(circuit(rng, 8, entries, reach, muxes), cus, what);
                }
    for (uint32_t cus : {1u, 64u, 256u, 304u})
        for (uint64_t r = 1; r < 40 * (uint64_t)cus; r++)
            CHECK(level_time(r, cus) > 0 && (level_time(r + 4 * (uint64_t)cus, cus) > level_time(r, cus)), "%llu rotations on %u\n",
                  (unsigned long long)r, cus);
    std::printf("failures %d\n", failures);
    Netlist big = circuit(rng, 8, 26000, 4000, true);
    const auto t0 = std::chrono::steady_clock::now();
    Netlist copy = big; copy.levelize(nullptr);
    const auto t1 = std::chrono::steady_clock::now();
    copy = big; const size_t levels = copy.levelize(nullptr, 256).size() - 1;
    const auto t2 = std::chrono::steady_clock::now();
    std::printf("26000 entries, %zu levels: %.2f ms, evened %.2f ms\n", levels, std::chrono::duration<double>(t1 - t0).count() * 1e3,
                std::chrono::duration<double>(t2 - t1).count() * 1e3);
    return failures != 0;
}
