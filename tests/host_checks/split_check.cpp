// How the key switch splits its coefficient range (she_internal.h: key_switch_split), on the host: every split is one that
// the kernel takes, and at sizes whose times were measured for all splits the one chosen is within 8 % of the best (the
// medians repeat to 3 %, and a split stands for a whole range of sizes and for keys in and out of the caches).
#include <algorithm>
#include <cstdio>

#include "she_internal.h"

static int failures = 0;
#define CHECK(c, ...) do { if (!(c)) { failures++; std::printf(__VA_ARGS__); } } while (0)

constexpr uint32_t CUS = 256, GATES_PER_BLOCK = 256;
static uint32_t chosen(uint32_t N, uint32_t n, size_t gates, uint32_t cus)
{
    return she::key_switch_split(N, gates, (uint32_t)((gates + GATES_PER_BLOCK - 1) / GATES_PER_BLOCK), (n + 1 + 31) / 32, cus);
}

// us of k_key_switch_mfma with 1, 2, .. 32 splits on 256 compute units, the mean of a key in the caches and a key from
// memory (0: not measured, and far from the best)
struct Measured { uint32_t N, n; size_t gates; int us[6]; };
static const Measured MEASURED[] = {
    {1024, 630, 1, {0, 0, 123, 68, 42, 31}},
    {1024, 630, 256, {0, 0, 134, 79, 54, 46}},
    {1024, 630, 512, {0, 236, 133, 84, 64, 80}},
    {1024, 630, 700, {446, 236, 134, 86, 104, 109}},
    {1024, 630, 1100, {444, 238, 140, 158, 150, 163}},
    {1024, 630, 2048, {448, 253, 181, 175, 200, 241}},
    {1024, 630, 2304, {449, 262, 181, 192, 217, 272}},
    {1024, 630, 2305, {449, 266, 275, 236, 240, 292}},
    {1024, 630, 4096, {471, 319, 298, 316, 346, 458}},
    {1024, 500, 256, {0, 0, 121, 74, 48, 41}},
    {1024, 500, 513, {0, 217, 122, 82, 62, 78}},
    {1024, 500, 4096, {398, 245, 256, 241, 276, 352}},
    {1024, 800, 83, {0, 238, 133, 80, 54, 58}},
    {1024, 800, 2048, {456, 261, 282, 244, 252, 311}},
    {1024, 1024, 1, {0, 227, 125, 76, 51, 49}},
    {1024, 1024, 513, {440, 238, 148, 149, 132, 149}},
    {1024, 1024, 2048, {481, 319, 295, 278, 307, 391}},
    {512, 500, 256, {0, 0, 69, 45, 33, 30}},
    {512, 500, 700, {0, 118, 70, 50, 44, 57}},
    {512, 500, 3000, {205, 131, 98, 111, 139, 201}},
    {1024, 2048, 1, {512, 268, 148, 89, 90, 76}},
    {1024, 2048, 513, {517, 288, 290, 235, 233, 281}},
    {1024, 2048, 1536, {539, 555, 455, 436, 478, 615}},
    {1024, 4096, 257, {536, 337, 312, 285, 306, 398}},
    {1024, 4096, 513, {543, 552, 438, 400, 429, 520}},
    {1024, 4096, 1536, {1077, 864, 775, 788, 913, 0}},
    {1024, 4096, 3000, {1607, 1429, 1379, 1461, 0, 0}},
};

int main()
{
    for (const Measured &m : MEASURED) {
        int best = 1 << 30, at = 0;
        for (int us : m.us) if (us) best = std::min(best, us);
        const uint32_t split = chosen(m.N, m.n, m.gates, CUS);
        while (1u << at < split) at++;
        CHECK(at < 6 && m.us[at] && m.us[at] * 100 <= best * 108, "N %u n %u, %zu gates: split %u takes %d us, the best %d\n", m.N,
              m.n, m.gates, split, at < 6 ? m.us[at] : 0, best);
    }
    // a power of two that leaves every workgroup eight coefficients or more (the kernel takes two at a time)
    for (uint32_t N : {256u, 512u, 1024u})
        for (uint32_t n : {1u, 31u, 32u, 630u, 4096u})
            for (uint32_t cus : {1u, 64u, 256u, 304u})
                for (size_t gates : {1, 255, 256, 257, 4095, 32767, 32768}) {
                    const uint32_t s = chosen(N, n, gates, cus);
                    CHECK(s >= 1 && s <= 32 && !(s & (s - 1)) && N / s >= 8, "N %u n %u, %zu gates on %u: split %u\n", N, n, gates, cus, s);
                }
    std::printf("failures %d\n", failures);
    return failures != 0;
}
