// The index and choice rules that kernels and their host code share, checked on the host
// for tests/test_launch_rules_cpu.py.  Prints "rules ok".
#include <cstdio>
#include <cstdlib>

#include "bits.h"
#include "bq.h"

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

// Reads of the FP4 tiles' coupling codes: a lane reads 8 bytes at 8 lane + a K step from the
// uniform start of a wave's ring, the first block's or the next one's, in sides of every padding.
static void coupling_codes()
{
    for (int na_p = 64; na_p <= 1152; na_p += 64)
        for (int nb_p = 64; nb_p <= 1152; nb_p += 64)
            for (int waves : {8, 16}) {
                const int64_t bytes = bq_code_bytes(na_p, nb_p);
                auto reads = [&](int64_t from, int steps) {
                    CHECK(from >= 0 && from + (int64_t)kCodeUnit * (steps - 1) + 8 * 63 + 8 <= bytes);
                };
                for (int side = 0; side < 2; ++side) {
                    const int blocks = (side == 0 ? na_p : nb_p) / 32, steps = (side == 0 ? nb_p : na_p) / 64;
                    for (int wave = 0; wave < waves; ++wave) {
                        reads(bq_code_start(na_p, nb_p, side, wave), kCodeRing);
                        for (int blk = wave; blk < blocks; blk += waves) {
                            const int64_t at = (side == 0 ? 0 : na_p * nb_p / 4) + (int64_t)kCodeUnit * steps * blk;
                            reads(at, steps > kCodeRing ? steps : kCodeRing);
                        }
                    }
                }
            }
}

// Reads of the cluster kernel's exchange words: octet by octet up to the widest side its operands
// hold, within the octets the side has.
static void exchange_octets()
{
    for (int steps : {4, 8, 16, 32})
        for (int blocks = 1; blocks <= 2 * steps; ++blocks) {
            const int octets = (blocks + 7) / 8;
            for (int k = 0; k < (steps + 3) / 4; ++k) {
                const int at = bq_octet(k, octets);
                CHECK(at >= 0 && 1024 * at + 512 + 16 * 31 + 16 <= 1024 * octets && (k >= octets || at == k));
            }
        }
}

int main()
{
    group_cursor();
    coupling_codes();
    exchange_octets();
    std::printf("rules ok\n");
    return 0;
}
