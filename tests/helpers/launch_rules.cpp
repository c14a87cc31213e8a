// The index and choice rules that kernels and their host code share, checked on the host
// for tests/test_launch_rules_cpu.py.  Prints "rules ok".
#include <cstdio>
#include <cstdlib>

#include "bits.h"

using namespace pbit;

#define CHECK(c)                                                                 \
    do {                                                                         \
        if (!(c)) {                                                              \
            std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c); \
            std::exit(2);                                                        \
        }                                                                        \
    } while (0)

// The group cursor of bit_tile.h's sweep over any number of groups: every pass works on
// the groups in order, and no index passes the last one.
static void group_cursor()
{
    for (int G : {1, 2, 3, 4, 5, 255}) {
        int at = bit_group_at(0, G), next = bit_group_at(G > 1 ? 1 : 0, G);
        for (int s = 0; s < 5; ++s)
            for (int c = 0; c < G; ++c) {
                const int g = at;
                at = next;
                next = bit_group_at(c + 2, G);
                CHECK(g == c && next >= 0 && next < G);
            }
    }
}

int main()
{
    group_cursor();
    std::printf("rules ok\n");
    return 0;
}
