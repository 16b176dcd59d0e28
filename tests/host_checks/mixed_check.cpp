// How a launch is divided among the forms of k_blind_rotate_mixed (she_internal.h: mixed_blocks), on the host: the forms hold
// every gate exactly once whatever the level's size, the device and SHE_OPT_SPLIT_BELOW; quads, pairs, or both are there for
// the rests that they are meant for, and for no others; and the launches without them get the kernels of their sizes.
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
                const size_t rest = gates % (4 * (size_t)cus), in_waves = 4 * (size_t)b.waves, rounds = gates / (4 * (size_t)cus);
                const bool allowed = rest && rest <= split_below, third = rest > 2 * (size_t)cus && rest <= 3 * (size_t)cus;
                const bool quads = allowed && ((rounds && rest <= cus) || (rounds != 1 && third));
                const bool pairs = allowed && ((rounds && rest > cus && rest <= 2 * (size_t)cus) || (rounds != 1 && third));
                CHECK((b.quads > 0) == quads && (b.pairs > 0) == pairs, "%zu gates on %u, %zu: %u pairs and %u quads\n", gates, cus,
                      split_below, b.pairs, b.quads);
                using K = she::RotationKernel;
                const K kernel = she::rotation_kernel(gates, cus, split_below);
                const K wanted = quads || pairs ? K::MIXED : gates > split_below ? K::WAVES : gates <= cus ? K::WIDE :
                                 gates <= 2 * (size_t)cus ? K::QUAD : K::SPLIT;
                CHECK(kernel == wanted, "%zu gates on %u, %zu: kernel %d, not %d\n", gates, cus, split_below, (int)kernel, (int)wanted);
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
                CHECK(b.pairs <= cus && b.quads <= cus, "%zu gates on %u: %u pairs, %u quads\n", gates, cus, b.pairs, b.quads);
            }
    std::printf("failures %d\n", failures);
    return failures != 0;
}
