// Fields computed from the bit-held sweep's site records (bits_host.cpp), for
// tests/test_bit_records_cpu.py: reads a problem and one spin configuration from stdin,
// builds the records, decodes every pair and prints form, positions, wide pairs and the
// fields by site.
#include <cstdio>
#include <vector>

#include "bits.h"

using namespace pbit;

int main()
{
    int n, groups, lx, ends;
    if (scanf("%d %d %d %d", &n, &groups, &lx, &ends) != 4) return 1;
    std::vector<int32_t> start(n + 1), nbr(ends);
    std::vector<int8_t> J(ends), h(n), m(n);
    std::vector<uint8_t> group(n);
    auto get = [](auto &v) {
        for (auto &x : v) {
            int t;
            if (scanf("%d", &t) != 1) return false;
            x = (typename std::remove_reference<decltype(x)>::type)t;
        }
        return true;
    };
    if (!get(start) || !get(nbr) || !get(J) || !get(h) || !get(group) || !get(m)) return 1;
    BitHost b;
    if (!bit_build(n, start.data(), nbr.data(), J.data(), h.data(), group.data(), groups, lx, b)) {
        printf("refused\n");
        return 0;
    }
    // elements by index from LDS address 0: the tables' space, the positions, the constant
    std::vector<int> el(kBitElBase / 2 + b.n_pos + 2, 0);  // 1: spin -1
    for (int p = 0; p < b.n_pos; ++p)
        if (b.pos_site[p] != kBitNoSite) el[kBitElBase / 2 + p] = m[b.pos_site[p]] < 0;
    std::vector<int> field(n, 1 << 20);
    auto word = [&](const std::vector<uint32_t> &r, int pairs, int p, int w) {
        return r[((size_t)(w / 4) * pairs + p) * 4 + w % 4];
    };
    for (int c = 0; c < groups; ++c) {
        const int32_t *g = &b.groups[4 * c];
        for (int p = 0; p < g[1] + g[3]; ++p)
            for (int hh = 0; hh < 2; ++hh) {
                const int at = 2 * (g[0] + g[2] + p) + hh;
                const bool wide = p < g[1];
                const std::vector<uint32_t> &r = wide ? b.wide : b.rec;
                const int pairs = wide ? b.n_wide : b.n_pairs, q = wide ? g[0] + p : g[2] + p - g[1];
                auto half = [&](int w) { return (word(r, pairs, q, w) >> (16 * hh)) & 0xFFFFu; };
                const int K = wide ? kBitSlotsWide : b.form == kBitGeneral ? kBitSlots : 6;
                const bool four = !wide && b.form == kBitCube4;
                int neg = 0;
                for (int u = 0; u < K; ++u) {
                    uint32_t idx, mask = half(four ? 4 + u : K + u);
                    if (!four)
                        idx = half(u);
                    else if (u < 5)
                        idx = ((word(r, pairs, q, u / 2) >> (16 * (u % 2))) & 0xFFFFu) + hh;
                    else
                        idx = hh ? word(r, pairs, q, 3) & 0xFFFFu : word(r, pairs, q, 2) >> 16;
                    if (idx >= el.size() || (mask != 0u && mask != 0xFFFFu)) return 2;
                    neg += el[idx] ^ (mask ? 1 : 0);
                }
                const uint32_t odd = K == 6 ? 0u : half(2 * K), site = half(four ? 10 : K == 6 ? 12 : 2 * K + 1);
                const uint32_t real = b.pos_site[at];
                if (real == kBitNoSite) continue;
                if (site != real || field[real] != 1 << 20) return 3;
                field[real] = K - 2 * neg - (odd ? 1 : 0);
            }
    }
    printf("%d %d %d\n", b.form, b.n_pos, b.n_wide);
    for (int i = 0; i < n; ++i) printf("%d ", field[i]);
    printf("\n");
    return 0;
}
