// How a launch is divided among the forms of k_blind_rotate_mixed (she_internal.h: mixed_blocks), on the host: the forms hold
// every gate exactly once whatever the level's size, the device and SHE_OPT_SPLIT_BELOW, and a launch that the option rules
// out is none of them.
#include <cstdio>

#include "she_internal.h"

static int failures = 0;
#define CHECK(c, ...) do { if (!(c)) { failures++; std::printf(__VA_ARGS__); } } while (0)

int main()
{
    for (uint32_t cus : {1u, 2u, 64u, 256u, 304u})
        for (size_t split_below : {(size_t)0, (size_t)1, (size_t)cus, 2 * (size_t)cus + 1, 6 * (size_t)cus, ~(size_t)0})
            for (size_t gates = 1; gates <= 20 * (size_t)cus + 5; gates++) {
                const she::MixedBlocks b = she::mixed_blocks(gates, cus, split_below);
                const size_t rest = gates % (4 * (size_t)cus), in_waves = 4 * (size_t)b.waves;
                if (!(b.pairs + b.quads)) {
                    CHECK(!b.waves, "%zu gates on %u: wavefronts alone\n", gates, cus);
                    continue;
                }
                CHECK(rest <= split_below, "%zu gates on %u: a rest of %zu above %zu\n", gates, cus, rest, split_below);
                CHECK(in_waves == gates - rest, "%zu gates on %u: %zu in rounds\n", gates, cus, in_waves);
                // first_quad = gates - quads in the kernel: pairs hold what lies between, the last one possibly one gate
                const size_t in_pairs = gates - b.quads - in_waves;
                CHECK(in_waves + b.quads <= gates && b.pairs == (in_pairs + 1) / 2, "%zu gates on %u: %u pairs for %zu\n", gates,
                      cus, b.pairs, in_pairs);
                CHECK(b.pairs + b.quads <= 2 * (size_t)cus, "%zu gates on %u: %u + %u workgroups\n", gates, cus, b.pairs, b.quads);
            }
    std::printf("failures %d\n", failures);
    return failures != 0;
}
