// The launches that a level of gates and native MUXes gets, on a fake device (fake_device.h): every rotation once, the gates
// first and with their outputs, those of the MUXes as samples; one launch or two, whichever was measured to be shorter.
#include <cstdint>
#include <vector>

#include "fake_device.h"

static int failures = 0;
#define CHECK(c, ...) do { if (!(c)) { failures++; std::printf(__VA_ARGS__); } } while (0)

// ms at n = 630 on 256 compute units; sizes where the two differ by more than 2 %
struct Level { uint32_t N, l; size_t gates, muxes; double one, two; };
static const Level measured[] = {
    {1024, 3, 1157, 579, 13.79, 12.50}, {1024, 3, 1220, 599, 13.75, 12.85}, {1024, 3, 1536, 100, 9.62, 9.14}, {1024, 3, 1335, 760, 16.04, 14.96},
    {1024, 3, 250, 128, 3.35, 3.40}, {1024, 3, 600, 400, 7.26, 9.3}, {1024, 3, 1024, 256, 7.53, 9.1}, {1024, 3, 96, 416, 5.6, 7.0},
    {1024, 3, 3000, 40, 15.55, 17.4}, {1024, 3, 1200, 170, 9.47, 9.95},
    {1024, 2, 2048, 64, 12.37, 10.96}, {1024, 2, 1565, 273, 12.62, 11.26}, {1024, 2, 1542, 392, 12.62, 11.76}, {1024, 2, 250, 128, 3.1, 5.14},
    {1024, 2, 1024, 256, 7.3, 7.77}, {1024, 2, 1536, 100, 7.34, 10.1}, {1024, 4, 2048, 64, 20.1, 17.64}, {1024, 4, 450, 545, 11.9, 16.0},
    {1024, 1, 528, 800, 8.59, 7.79}, {512, 3, 2048, 64, 8.84, 8.10}, {512, 3, 3000, 40, 12.22, 11.04}, {512, 3, 528, 1412, 12.74, 11.66},
    {512, 3, 1030, 255, 5.9, 6.95}, {512, 3, 96, 416, 3.22, 5.15}, {512, 2, 2048, 64, 6.7, 6.32}, {512, 2, 3000, 40, 9.28, 8.51},
    {512, 2, 1130, 205, 4.5, 5.37}, {512, 4, 1667, 834, 16.14, 14.92}, {256, 3, 800, 370, 4.85, 4.55}, {256, 3, 2048, 64, 6.91, 6.12},
    {256, 3, 1038, 579, 6.94, 6.17}, {256, 3, 1280, 128, 3.56, 4.42}, {256, 3, 250, 128, 1.55, 2.57}, {256, 2, 1038, 562, 5.24, 5.12},
};

static void check(she_ctx *c, const she_params &P, size_t gates, size_t muxes, int wanted)
{
    const size_t n = gates + muxes;
    std::vector<uint8_t> type(n, 1);
    std::vector<uint32_t> in(n), out(n), refs(n);
    for (size_t g = 0; g < n; g++) {
        if (g >= gates) type[g] = SHE_CIRCUIT_MUX;
        in[g] = g % 8; out[g] = (uint32_t)(8 + g); refs[g] = SHE_WIRE_GATE | (uint32_t)g;
    }
    fake::rotations.clear();
    const int rc = she_eval_circuit(c, type.data(), in.data(), in.data(), in.data(), n, refs.data(), out.data(), n, nullptr);
    CHECK(rc == SHE_OK, "N %u, l %u, %zu gates and %zu MUXes: %s\n", P.N, P.l, gates, muxes, she_last_error(c));
    const auto &launches = fake::rotations;
    CHECK(!wanted || launches.size() == (size_t)wanted, "N %u, l %u, %zu gates and %zu MUXes: %zu launches, %d wanted\n", P.N, P.l,
          gates, muxes, launches.size(), wanted);
    size_t done = 0;
    for (const fake::Rotations &r : launches) {
        CHECK(r.bar == launches[0].bar + done * ((P.n + 2) / 2 * 2), "N %u, l %u, %zu and %zu: a launch from %zu elsewhere\n", P.N, P.l,
              gates, muxes, done);
        const size_t direct = r.mux ? r.direct : r.count;
        CHECK(direct == std::min(r.count, gates - std::min(done, gates)), "N %u, l %u, %zu and %zu: %zu direct from %zu on\n", P.N, P.l,
              gates, muxes, direct, done);
        CHECK(r.out == (direct > 0), "N %u, l %u, %zu and %zu: outputs\n", P.N, P.l, gates, muxes);
        done += r.count;
    }
    CHECK(done == gates + 2 * muxes, "N %u, l %u, %zu and %zu: %zu rotations\n", P.N, P.l, gates, muxes, done);
}

int main()
{
    for (const uint32_t N : {256u, 512u, 1024u})
        for (const uint32_t l : {1u, 2u, 3u, 4u}) {
            she_params P{};
            P.n = 4; P.N = N; P.k = 1; P.bg_bit = 6; P.l = l; P.ks_t = 1; P.ks_basebit = 1;
            she_ctx *c = nullptr;
            if (she_keygen(&P, 3, 8 + 5000, &c)) { std::printf("keygen: %s\n", she_last_error(nullptr)); return 1; }
            she_set_option(c, SHE_OPT_NATIVE_MUX, 1);
            for (const Level &m : measured)
                if (m.N == N && m.l == l) check(c, P, m.gates, m.muxes, m.one < m.two ? 1 : 2);
            for (size_t gates : {0, 1, 31, 256, 257, 1000, 1536, 2049, 3100})
                for (size_t muxes : {0, 1, 127, 300, 769, 1024, 1800})
                    if (gates + muxes) check(c, P, gates, muxes, gates && muxes ? 0 : 1);
            she_set_option(c, SHE_OPT_SPLIT_BELOW, 0);                     // full rounds only: small levels share one
            for (const Level &m : measured)
                if (m.N == N && m.l == l && m.one < m.two) check(c, P, m.gates, m.muxes, 1);
            she_free(c);
        }
    std::printf("failures %d\n", failures);
    return failures != 0;
}
