// bits_host.cpp — site records of the bit-held sparse sweep (bits.h).
#include <algorithm>
#include <utility>

#include "bits.h"

namespace pbit {

namespace {

// One site's terms: element index and sign (1: the term is -m) per slot, and whether an
// unpaired +1 was needed to fill them.
struct Slots {
    uint32_t idx[kBitSlotsWide];
    bool neg[kBitSlotsWide];
    bool odd;
};

}  // namespace

bool bit_build(int n, const int32_t *start, const int32_t *nbr, const int8_t *J, const int8_t *h,
               const uint8_t *group, int n_groups, int cube_lx, BitHost &out)
{
    std::vector<int> terms((size_t)n, 0);  // bonds with J != 0, and the field
    bool six = true;                       // every site: six bonds, no field
    for (int i = 0; i < n; ++i) {
        for (int32_t e = start[i]; e < start[i + 1]; ++e) terms[i] += J[e] != 0;
        six = six && terms[i] == 6 && !(h && h[i]);
        terms[i] += h && h[i] ? 1 : 0;
        if (terms[i] > kBitSlotsWide) return false;
    }
    // positions: group by group, sites with more than kBitSlots terms first; a cube's colour
    // follows the lattice rows (ascending site)
    std::vector<std::vector<uint32_t>> members((size_t)n_groups);
    for (int i = 0; i < n; ++i) members[group[i]].push_back((uint32_t)i);
    out = BitHost();
    out.n = n;
    out.n_groups = n_groups;
    std::vector<uint32_t> pos((size_t)n);
    for (int c = 0; c < n_groups; ++c) {
        auto &m = members[c];
        auto wide_end = std::stable_partition(m.begin(), m.end(), [&](uint32_t i) { return terms[i] > kBitSlots; });
        int n_wide = (int)(wide_end - m.begin());
        if (n_wide & 1) {  // the last wide pair takes an ordinary site
            if (wide_end != m.end()) ++n_wide;
        }
        const int wp = (n_wide + 1) / 2, op = ((int)m.size() - n_wide + 1) / 2;
        out.groups.insert(out.groups.end(), {out.n_wide, wp, out.n_pairs, op});
        size_t q = 0;
        for (int p = 0; p < 2 * (wp + op); ++p) {
            // padding closes the wide pairs and the ordinary pairs of the group
            const bool real = p < 2 * wp ? (int)q < n_wide : q < m.size();
            if (real) {
                pos[m[q]] = (uint32_t)out.pos_site.size();
                out.pos_site.push_back((uint16_t)m[q++]);
            } else {
                out.pos_site.push_back(kBitNoSite);
            }
        }
        out.n_wide += wp;
        out.n_pairs += op;
        out.max_pairs = std::max(out.max_pairs, wp + op);
    }
    out.n_pos = (int)out.pos_site.size();
    if (out.n_pos > kBitMaxPositions) return false;
    for (uint32_t &p : pos) p += kBitElBase / 2;
    const uint32_t constant = (uint32_t)out.n_pos + kBitElBase / 2;  // the constant +1 spin
    out.form = six && out.n_pos == n ? (cube_lx > 0 && cube_lx % 4 == 0 ? kBitCube4 : kBitCube) : kBitGeneral;

    auto slots = [&](uint32_t site, int k, Slots &s) {
        int u = 0;
        if (site != kBitNoSite) {
            for (int32_t e = start[site]; e < start[site + 1]; ++e)
                if (J[e] != 0) {
                    s.idx[u] = pos[nbr[e]];
                    s.neg[u++] = J[e] < 0;
                }
            if (h && h[site]) {
                s.idx[u] = constant;
                s.neg[u++] = h[site] < 0;
            }
        }
        // padding terms: pairs of -1 and +1, and a +1 left over if their number is odd
        const int pad = k - u;
        for (int q = 0; q < pad; ++q) {
            s.idx[u + q] = constant;
            s.neg[u + q] = q < pad / 2;
        }
        s.odd = pad & 1;
    };
    auto mask = [](int lo, int hi) { return (lo ? 0x0000FFFFu : 0u) | (hi ? 0xFFFF0000u : 0u); };
    auto put = [](std::vector<uint32_t> &rec, int pairs, int pair, const uint32_t *words, int n_words) {
        for (int w = 0; w < n_words; ++w) rec[((size_t)(w / 4) * pairs + pair) * 4 + w % 4] = words[w];
    };
    const int words = out.form == kBitCube4 ? 12 : 16;
    out.rec.assign((size_t)words * out.n_pairs, 0u);
    out.wide.assign((size_t)32 * out.n_wide, 0u);
    for (int c = 0; c < n_groups; ++c) {
        const int32_t *g = &out.groups[(size_t)4 * c];
        for (int p = 0; p < g[1] + g[3]; ++p) {
            const bool wide = p < g[1];
            const uint32_t at = 2u * (uint32_t)(g[0] + g[2] + p);
            const uint32_t s0 = out.pos_site[at], s1 = out.pos_site[at + 1];
            const int k = wide ? kBitSlotsWide : (out.form == kBitGeneral ? kBitSlots : 6);
            Slots a, b;
            slots(s0, k, a);
            slots(s1, k, b);
            uint32_t w[2 * kBitSlotsWide + 2];
            int nw = 0;
            if (out.form == kBitCube4) {
                // the five slots whose neighbours are one aligned pair of elements, (2 q, 2 q + 1)
                // of the first and the second site, go to the front
                int front = 0;
                for (int u = 0; u < 6 && front < 5; ++u) {
                    if (a.idx[u] & 1) continue;
                    int v = front;
                    while (v < 6 && b.idx[v] != a.idx[u] + 1) ++v;
                    if (v == 6) continue;
                    std::swap(a.idx[front], a.idx[u]);
                    std::swap(a.neg[front], a.neg[u]);
                    std::swap(b.idx[front], b.idx[v]);
                    std::swap(b.neg[front], b.neg[v]);
                    ++front;
                }
                if (front < 5) return false;  // not a cube in row order
                w[nw++] = a.idx[0] | a.idx[1] << 16;
                w[nw++] = a.idx[2] | a.idx[3] << 16;
                w[nw++] = a.idx[4] | a.idx[5] << 16;
                w[nw++] = b.idx[5];
            } else {
                for (int u = 0; u < k; ++u) w[nw++] = a.idx[u] | b.idx[u] << 16;
            }
            for (int u = 0; u < k; ++u) w[nw++] = mask(a.neg[u], b.neg[u]);
            if (k != 6) w[nw++] = mask(a.odd, b.odd);
            w[nw++] = s0 | s1 << 16;
            if (wide)
                put(out.wide, out.n_wide, g[0] + p, w, nw);
            else
                put(out.rec, out.n_pairs, g[2] + p - g[1], w, nw);
        }
    }
    return true;
}

}  // namespace pbit
