// The library's host files on a fake device (fake_device.h):
//   1. a call that runs out of memory says so and leaves no error for the next launch (or the next call of another library in
//      the process) to find;
//   2. a context whose scratch has grown gives everything back;
//   3. a circuit that runs in some amount of memory runs in any larger amount, and one whose levels are evened out in no more
//      than it needs at its earliest levels.
#include <cstdint>
#include <vector>

#include "fake_device.h"

static int failures = 0;
#define CHECK(c, ...) do { if (!(c)) { failures++; std::printf(__VA_ARGS__); } } while (0)

static she_ctx *context(uint32_t N, uint32_t capacity, uint32_t n = 4)
{
    she_params P{};
    P.n = n; P.N = N; P.k = 1; P.bg_bit = 7; P.l = 3; P.ks_t = 1; P.ks_basebit = 1;
    she_ctx *c = nullptr;
    if (she_keygen(&P, 3, capacity, &c)) { std::printf("keygen: %s\n", she_last_error(nullptr)); std::exit(1); }
    return c;
}

// without memory the call fails and nothing stays behind; with memory it works
template <class F> static void short_of_memory(const char *what, F &&call)
{
    fake::limit = fake::held;
    int rc = call();
    CHECK(rc == SHE_ENOMEM, "%s without memory returns %d\n", what, rc);
    CHECK(hipGetLastError() == hipSuccess, "%s leaves an error behind\n", what);
    fake::limit = ~(size_t)0;
    rc = call();
    CHECK(rc == SHE_OK, "%s with memory returns %d\n", what, rc);
}

// A circuit on the pool's first 64 slots; the results that no entry reads are its outputs.
struct Circuit {
    std::vector<uint8_t> type;
    std::vector<uint32_t> in0, in1, in2, refs, out;
    uint32_t add(uint8_t t, uint32_t a, uint32_t b, uint32_t c = 0)
    {
        type.push_back(t); in0.push_back(a); in1.push_back(b); in2.push_back(c);
        return SHE_WIRE_GATE | (uint32_t)(type.size() - 1);
    }
    void finish()
    {
        std::vector<uint8_t> read(type.size(), 0);
        for (const auto *in : {&in0, &in1, &in2})
            for (uint32_t w : *in)
                if (w & SHE_WIRE_GATE) read[w & ~SHE_WIRE_GATE] = 1;
        for (uint32_t g = 0; g < type.size(); g++)
            if (!read[g]) { refs.push_back(SHE_WIRE_GATE | g); out.push_back(64 + (uint32_t)out.size()); }
    }
    int run(she_ctx *c) const
    {
        return she_eval_circuit(c, type.data(), in0.data(), in1.data(), in2.data(), type.size(), refs.data(), out.data(), out.size(), nullptr);
    }
};

// Runs the circuit in fresh contexts with more and more memory.  Returns the least it ran in, and how it ran.
struct Walk { size_t least = 0, schedules = 0; bool chunks = false; };
static Walk walk(const char *what, uint32_t N, uint32_t n, const Circuit &circuit, bool split, size_t from, size_t to, size_t step)
{
    Walk w;
    std::vector<uint64_t> schedule;
    for (size_t free = from; free <= to; free += step) {
        she_ctx *c = context(N, 1 << 12, n);
        she_set_option(c, SHE_OPT_NATIVE_MUX, 1);
        if (!split) she_set_option(c, SHE_OPT_SPLIT_BELOW, 0);
        fake::limit = fake::held + free;
        fake::rotations.clear();
        const int rc = circuit.run(c);
        CHECK(rc == SHE_OK || rc == SHE_ENOMEM, "%s with %zu bytes: %s\n", what, free, she_last_error(c));
        CHECK(hipGetLastError() == hipSuccess, "%s with %zu bytes leaves an error behind\n", what, free);
        CHECK(rc == SHE_OK || !w.least, "%s runs in %zu bytes and not in %zu\n", what, w.least, free);
        if (rc == SHE_OK) {
            if (!w.least) w.least = free;
            size_t levels = 0;
            she_last_level_sizes(c, nullptr, nullptr, 0, &levels);
            std::vector<uint64_t> gates(levels), muxes(levels);
            she_last_level_sizes(c, gates.data(), muxes.data(), levels, nullptr);
            if (fake::rotations.size() > levels) w.chunks = true;
            if (gates != schedule) { schedule = gates; w.schedules++; }
        }
        fake::limit = ~(size_t)0;
        CHECK(circuit.run(c) == SHE_OK, "%s after a try with %zu bytes: %s\n", what, free, she_last_error(c));
        she_free(c);
        CHECK(fake::held == 0, "%s: %zu bytes are still held after she_free\n", what, fake::held);
    }
    CHECK(w.least > from && w.least < to, "%s: does not start to run between %zu and %zu bytes\n", what, from, to);
    return w;
}

static void circuits_short_of_memory()
{
    // one level of 300 gates and 150 MUXes
    Circuit level;
    for (uint32_t k = 0; k < 450; k++) level.add(k < 300 ? SHE_AND : SHE_CIRCUIT_MUX, k % 64, (k + 1) % 64, (k + 2) % 64);
    level.finish();
    CHECK(walk("a level of gates and MUXes", 256, 630, level, true, 700000, 1800000, 25000).chunks, "a level never ran in parts\n");

    // 306 gates in the second level, of which 50 can wait for a level with room: the fourth, 460 gates, as the third holds
    // 1024; the 100 first gates that they read stay alive while the third level's results come on top
    Circuit c;
    std::vector<uint32_t> first, second, third, fourth;
    for (uint32_t k = 0; k < 612; k++) first.push_back(c.add(SHE_AND, k % 64, (k + 7) % 64));
    for (uint32_t k = 0; k < 306; k++) second.push_back(c.add(SHE_AND, first[2 * k], first[2 * k + 1]));
    for (uint32_t k = 0; k < 1024; k++) third.push_back(c.add(SHE_MAJ3, second[k % 256], second[(k + 1) % 256], first[512 + k % 100]));
    for (uint32_t k = 0; k < 460; k++) fourth.push_back(c.add(SHE_MAJ3, third[2 * k], third[2 * k + 1], third[1023 - k % 104]));
    for (uint32_t k = 0; k < 154; k++) c.add(SHE_XOR3, fourth[k], fourth[154 + k], fourth[306 + k]);
    for (uint32_t k = 0; k < 50; k++) c.add(SHE_XOR, second[256 + k], fourth[k]);
    c.finish();
    const Walk evened = walk("a circuit with evened levels", 1024, 64, c, true, 2000000, 3400000, 7000);
    const Walk earliest = walk("a circuit at its earliest levels", 1024, 64, c, false, 2000000, 3400000, 7000);
    CHECK(evened.schedules == 2 && earliest.schedules == 1, "%zu schedules, %zu at the earliest levels\n", evened.schedules, earliest.schedules);
    CHECK(evened.least <= earliest.least, "evened levels need %zu bytes, the earliest %zu\n", evened.least, earliest.least);
}

int main()
{
    circuits_short_of_memory();
    std::vector<uint32_t> a(64), b(64), s(64), out(64);
    std::vector<uint8_t> bits(64, 1), types(64, 0);
    for (uint32_t k = 0; k < 64; k++) { a[k] = k; b[k] = 63 - k; s[k] = k; out[k] = 64 + k; }
    she_ctx *c = context(256, 128);
    short_of_memory("she_encrypt_bits", [&] { return she_encrypt_bits(c, bits.data(), 64, 5, a.data()); });
    short_of_memory("she_eval_gates", [&] { return she_eval_gates(c, types.data(), a.data(), b.data(), out.data(), 8); });
    short_of_memory("she_eval_mux", [&] { return she_eval_mux(c, s.data(), a.data(), b.data(), out.data(), 16); });
    short_of_memory("she_leveled_init", [&] { return she_leveled_init(c, 2, 64); });
    for (uint32_t k = 0; k < 64; k++) { s[k] = 0; a[k] = k % 8; b[k] = 8 + k % 8; out[k] = 16 + k % 48; }
    short_of_memory("she_eval_cmux", [&] { return she_eval_cmux(c, s.data(), a.data(), b.data(), out.data(), 48); });
    she_free(c);
    CHECK(fake::held == 0, "%zu bytes are still held after she_free\n", fake::held);

    // gate levels grow the scratch that MUX levels share
    c = context(256, 128);
    for (uint32_t k = 0; k < 64; k++) { s[k] = k; a[k] = k; b[k] = 63 - k; out[k] = 64 + k; }
    for (size_t count : {4, 16, 64}) {
        CHECK(she_eval_mux(c, s.data(), a.data(), b.data(), out.data(), count / 4) == SHE_OK, "%zu MUX gates\n", count / 4);
        CHECK(she_eval_gates(c, types.data(), a.data(), b.data(), out.data(), count) == SHE_OK, "%zu gates\n", count);
    }
    she_free(c);
    CHECK(fake::held == 0, "%zu bytes are still held after she_free of a context whose scratch grew\n", fake::held);
    std::printf("failures %d\n", failures);
    return failures != 0;
}
