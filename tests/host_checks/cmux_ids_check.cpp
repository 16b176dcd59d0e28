// The block of ids that small CMux levels put into the kernel's arguments (she_internal.h: fill_cmux_ids): the lists in
// their places, and nothing of what was in the memory before.
#include <cstdio>
#include <cstring>
#include <vector>

#include "she_internal.h"

static int failures = 0;
#define CHECK(c, ...) do { if (!(c)) { failures++; std::printf(__VA_ARGS__); } } while (0)

int main()
{
    for (size_t count : {(size_t)1, (size_t)2, she::CMUX_ARG_IDS - 1, she::CMUX_ARG_IDS}) {
        std::vector<uint32_t> lists(4 * count);
        for (size_t k = 0; k < lists.size(); k++) lists[k] = (uint32_t)(1000 + k);
        she::CmuxIds ids;
        std::memset(&ids, 0xA5, sizeof ids);
        she::fill_cmux_ids(ids, &lists[0], &lists[count], &lists[2 * count], &lists[3 * count], count);
        for (size_t q = 0; q < 4; q++)
            for (size_t k = 0; k < she::CMUX_ARG_IDS; k++)
                CHECK(ids.id[q][k] == (k < count ? lists[q * count + k] : 0), "%zu entries, list %zu: place %zu holds %x\n", count,
                      q, k, ids.id[q][k]);
    }
    std::printf("failures %d\n", failures);
    return failures != 0;
}
