// she_trlwe_read and she_trlwe_phase on a fake device (fake_device.h) with no memory left beside the pools: they return what
// they return with memory to spare, and leave no error for the next launch to find.
#include <cstdint>
#include <vector>

#include "fake_device.h"

static int failures = 0;
#define CHECK(c, ...) do { if (!(c)) { failures++; std::printf(__VA_ARGS__); } } while (0)

int main()
{
    for (uint32_t N : {256u, 512u, 1024u, 2048u}) {
        she_params P{};
        P.n = 4; P.N = N; P.k = 1; P.bg_bit = 7; P.l = 3; P.ks_t = 1; P.ks_basebit = 1; P.lwe_std = 0; P.bk_std = 0;
        she_ctx *c = nullptr;
        if (she_keygen(&P, 3, 4, &c)) { std::printf("keygen: %s\n", she_last_error(nullptr)); return 1; }
        constexpr uint32_t COUNT = 1025, SLOTS = 9;                           // more than a chunk
        const size_t words = (size_t)2 * N;
        std::vector<uint32_t> raw(SLOTS * words), ids(COUNT), to(SLOTS), got(COUNT * words), phases(COUNT * N), want;
        for (size_t w = 0; w < raw.size(); w++) raw[w] = (uint32_t)(w * 2654435761u);
        for (uint32_t k = 0; k < SLOTS; k++) to[k] = k;
        for (uint32_t k = 0; k < COUNT; k++) ids[k] = k * 5 % SLOTS;
        CHECK(!she_leveled_init(c, 1, SLOTS) && !she_trlwe_write(c, raw.data(), SLOTS, to.data()), "N %u: setup\n", N);
        for (const bool full : {true, false, true}) {
            fake::limit = full ? fake::held : ~(size_t)0;
            const int rc = she_trlwe_read(c, ids.data(), COUNT, got.data());
            CHECK(rc == SHE_OK, "N %u, memory full %d: read returns %d\n", N, full, rc);
            for (uint32_t k = 0; k < COUNT && rc == SHE_OK; k++)
                CHECK(!std::memcmp(&got[k * words], &raw[ids[k] * words], words * 4), "N %u, memory full %d: sample %u\n", N, full, k);
            CHECK(she_trlwe_phase(c, ids.data(), COUNT, phases.data()) == SHE_OK, "N %u, memory full %d: phase\n", N, full);
            if (want.empty()) want = phases;
            CHECK(phases == want, "N %u, memory full %d: phases\n", N, full);
            CHECK(hipGetLastError() == hipSuccess, "N %u, memory full %d: an error is left behind\n", N, full);
        }
        fake::limit = ~(size_t)0;
        she_free(c);
    }
    std::printf("failures %d\n", failures);
    return failures != 0;
}
