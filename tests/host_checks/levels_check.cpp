// The level scheduler (she_circuits.cpp: levelize, even_levels) on the host: whatever the circuit and the device, evened levels
// hold every entry once, each after its operands, in as many levels as the circuit is deep, none empty, MUXes behind gates, and
// their estimated time is at most that of the earliest levels; circuits with room to gain gain it, and ones without stay as they
// are; level_time grows with the level and steps where the launch gets another kernel or another division among its forms.
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
        uint64_t gates = 0, muxes = 0;
        for (size_t g = bounds[lv]; g < bounds[lv + 1]; g++) (is_mux_type(nl.type[g]) ? muxes : gates)++;
        us += level_time(gates, 2 * muxes, cus);
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

// `wide` entries that nobody reads beside a chain of `depth`: with more of them than the first level has room for
static Netlist slack(uint32_t wide, uint32_t depth, bool muxes)
{
    Netlist nl(8, false, true);
    uint32_t w = nl.gate(SHE_AND, 0, 1);
    for (uint32_t k = 1; k < depth; k++) w = nl.gate(SHE_OR, w, k % 8);
    for (uint32_t k = 0; k < wide; k++)
        if (muxes) nl.mux(k % 8, (k + 1) % 8, (k + 2) % 8);
        else nl.gate(SHE_AND, k % 8, (k + 3) % 8);
    return nl;
}

// evened levels must take less than `share` of the earliest ones' time, and hand out the netlist as it was
static void gains(const Netlist &nl, uint32_t cus, double share, const char *what)
{
    Netlist early = nl, even = nl, unsorted(0);
    const std::vector<size_t> b0 = early.levelize(), b1 = even.levelize(nullptr, cus, &unsorted);
    const double t0 = estimate(early, b0, cus), t1 = estimate(even, b1, cus);
    CHECK(b1 != b0 && t1 < share * t0, "%s: %.0f us at the earliest, %.0f evened\n", what, t0, t1);
    CHECK(unsorted.type == nl.type && unsorted.in0 == nl.in0 && unsorted.in1 == nl.in1 && unsorted.in2 == nl.in2 &&
          unsorted.out == nl.out && unsorted.next_temp == nl.next_temp, "%s: not the netlist as it was\n", what);
}

static void gains_nothing(const Netlist &nl, uint32_t cus, const char *what)
{
    Netlist early = nl, even = nl, unsorted(0);
    const std::vector<size_t> b0 = early.levelize(), b1 = even.levelize(nullptr, cus, &unsorted);
    CHECK(b1 == b0 && even.out == early.out && unsorted.type.empty(), "%s: moved entries\n", what);
}

// what a launch runs: kernel, full rounds, and the forms beside them
struct Form {
    RotationKernel kernel; uint32_t waves; bool pairs, quads; uint64_t rounds;
    bool operator!=(const Form &o) const
    {
        return kernel != o.kernel || waves != o.waves || pairs != o.pairs || quads != o.quads || rounds != o.rounds;
    }
};
static Form form(uint64_t r, uint32_t cus)
{
    const MixedBlocks b = mixed_blocks(r, cus, 6 * (size_t)cus);
    const RotationKernel kernel = rotation_kernel(r, cus, 6 * (size_t)cus);
    return {kernel, b.waves, b.pairs > 0, b.quads > 0, kernel == RotationKernel::WAVES ? (r - 1) / (4 * (uint64_t)cus) : 0};
}

int main()
{
    std::mt19937 rng(7);
    gains(slack(300, 6, false), 256, 0.9, "300 gates beside a chain");                   // 3.4 ms and five of 1.8 -> six of 1.8
    gains(slack(780, 12, false), 256, 0.9, "780 gates beside a chain");
    gains(slack(150, 6, true), 256, 0.9, "150 MUXes beside a chain");
    gains(slack(75, 6, false), 64, 0.9, "75 gates beside a chain on 64 compute units");
    gains_nothing(slack(255, 6, false), 256, "a level of one gate per compute unit");
    gains_nothing(slack(300, 1, false), 256, "one level");
    gains_nothing(slack(40000, 2, false), 256, "levels of many rounds");
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
    for (uint32_t cus : {64u, 256u, 304u})
        for (uint64_t r = 1; r < 40 * (uint64_t)cus; r++) {
            const double up = level_time(r + 1, cus) - level_time(r, cus);
            const bool changes = form(r, cus) != form(r + 1, cus);
            CHECK(up >= 0, "%llu rotations on %u: less for one more\n", (unsigned long long)r, cus);
            CHECK(up < 100 || changes, "%llu rotations on %u: a step of %.0f us within one form\n", (unsigned long long)r, cus, up);
            CHECK(up > 200 || !changes || r > 6 * (uint64_t)cus, "%llu rotations on %u: no step to another form\n", (unsigned long long)r, cus);
        }
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
