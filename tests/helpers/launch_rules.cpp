// The index and choice rules that kernels and their host code share, checked on the host
// for tests/test_launch_rules_cpu.py.  Prints "rules ok".
#include <cstdio>
#include <cstdlib>
#include <mutex>
#include <random>
#include <thread>
#include <utility>
#include <vector>

#include "bits.h"
#include "bq.h"
#include "bq_tune.h"
#include "sweep_cost.h"
#include "meet.h"

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

// Meeting words as memory that performs an unordered add as late as it may: after the thread's
// next ordered operation, or, where arrivals order nothing (ordered = false), a while after it.
struct MeetMemory {
    std::mutex mu;
    uint32_t word[10] = {};
};
struct MeetThread {
    MeetMemory &m;
    std::mt19937 rng;
    bool ordered;
    int patience;
    std::vector<int> pending;
    int until = 0;
    void perform()
    {
        for (int w : pending) ++m.word[w];
        pending.clear();
    }
    void operation()
    {
        if (--until <= 0) perform();
    }
    uint32_t add(int w, uint32_t)
    {
        std::lock_guard<std::mutex> lk(m.mu);
        pending.push_back(w);
        until = 20;
        return m.word[w];  // (a slot is not used before the meeting ends)
    }
    uint32_t arrive()
    {
        std::lock_guard<std::mutex> lk(m.mu);
        if (ordered) perform();
        return m.word[0]++;
    }
    uint32_t read(int w)
    {
        std::lock_guard<std::mutex> lk(m.mu);
        operation();
        return m.word[w];
    }
    bool swap(uint32_t &seen, uint32_t v)
    {
        std::lock_guard<std::mutex> lk(m.mu);
        operation();
        if (m.word[0] != seen) {
            seen = m.word[0];
            return false;
        }
        m.word[0] = v;
        return true;
    }
    bool late() { return patience >= 0 && patience-- == 0; }
    void pause()
    {
        if (rng() % 4 == 0) std::this_thread::yield();
    }
};

// Sixteen workgroups, two on each XCD: all of them go, or none does.  Returns how many went.
static int meeting(unsigned seed, bool ordered, bool impatient, int short_xcd)
{
    MeetMemory memory;
    constexpr int kGroups = 16;
    std::vector<char> went(kGroups, 2);
    std::vector<std::thread> pool;
    for (int k = 0; k < kGroups; ++k)
        pool.emplace_back([&, k] {
            std::mt19937 rng(seed * 100 + k);
            const int patience = impatient && rng() % 3 == 0 ? (int)(rng() % 60) : -1;
            MeetThread t{memory, rng, ordered, patience, {}, 0};
            uint32_t slot;
            const int xcc = k % 8 == short_xcd ? 0 : k % 8;
            went[k] = meet(t, kGroups, 2u, (uint32_t)xcc, slot);
        });
    for (auto &t : pool) t.join();
    int n = 0;
    for (char w : went) {
        CHECK(w == 0 || w == 1);
        n += w;
    }
    return n;
}

static void meetings()
{
    int went = 0, unordered = 0;
    for (unsigned s = 0; s < 200; ++s) {
        CHECK(meeting(s, true, false, -1) == 16);
        CHECK(meeting(s, true, false, 3) == 0);  // an XCD with too few
        const int n = meeting(s, true, true, -1);
        CHECK(n == 0 || n == 16);
        went += n == 16;
        unordered += meeting(s, false, false, -1) != 16;
    }
    std::printf("impatient meetings held: %d of 200\n", went);
    CHECK(unordered > 0);  // the model does tell arrivals that order nothing
}

// Timings of a kernel whose launches may not run: each has to have run.
static void run_times()
{
    for (int lost = 0; lost < 4; ++lost) {  // the launch that does not run (3: none)
        int launch = 0;
        double one = 0.0, more = 0.0;
        const bool ok = time_runs([&](int n) { return launch++ == lost ? 2.0 : 0.1 + 0.01 * n; },
                                  [&] { return launch - 1 != lost; }, 32, &one, &more);
        CHECK(ok == (lost > 1));
        CHECK(!ok || (one < 0.2 && more < 0.5 && launch == 2));
    }
}

// The cheapest of the timed kernels: the cluster kernel's place in the cache does not hide the
// others from anneals that cannot take it (static scratch, graphs, short runs).
static void timed_kernels()
{
    const std::vector<BqCost> costs = {{BqVariant::Small, 0, 0.0, 0.030}, {BqVariant::Bits, 256, 0.0, 0.021},
                                       {BqVariant::Bits, 64, 0.0, 0.013}, {BqVariant::Cluster, 0, 0.040, 0.004}};
    auto chunk = [](BqVariant v) { return v == BqVariant::Cluster ? 20000 : 1; };
    const BqCost *c = cheapest(costs, true, 100, 100, chunk);
    CHECK(c && c->variant == BqVariant::Cluster);
    c = cheapest(costs, false, 100, 100, chunk);
    CHECK(c && c->variant == BqVariant::Bits && c->rt == 64);
    c = cheapest(costs, true, 2, 2, chunk);
    CHECK(c && c->variant == BqVariant::Bits);
    // a launch for every energy check: 100 sweeps in runs of 3
    c = cheapest(costs, true, 100, 3, chunk);
    CHECK(c && c->variant == BqVariant::Bits);
    c = cheapest(costs, true, 100, 10, chunk);
    CHECK(c && c->variant == BqVariant::Cluster);
    CHECK(!cheapest(std::vector<BqCost>(), true, 100, 100, chunk));
}

// Graphs as bits or as bytes: the faster form of shapes measured on the device (us per sweep in
// bytes and in the best width of bits; random, regular, bipartite and dimerized graphs, and
// graphs of some wide sites), and both estimates within a quarter of the measured times.
static void graph_forms()
{
    struct Case {
        GraphShape g;
        int max_pairs, R;
        double bytes, bits;
    };
    const Case cases[] = {
        {{4, 0, 252, 0, 250, 744, 4, 4, 0}, 48, 16, 2.4, 2.9},  // reg3
        {{5, 0, 502, 0, 500, 1992, 5, 5, 0}, 86, 1024, 3.2, 3.7},  // reg4
        {{6, 0, 502, 0, 500, 2990, 6, 12, 0}, 69, 512, 4.6, 4.4},  // reg6
        {{8, 8, 0, 506, 500, 4952, 8, 24, 0}, 54, 128, 8.1, 9.3},  // reg10
        {{8, 8, 0, 1006, 1000, 9950, 8, 24, 0}, 105, 1024, 8.7, 9.9},  // reg10
        {{8, 8, 0, 2006, 2000, 19964, 8, 24, 0}, 210, 4096, 16.3, 21.5},  // reg10
        {{6, 6, 26, 476, 500, 3966, 6, 12, 443}, 63, 1024, 5.5, 7.5},  // reg8
        {{7, 7, 40, 3962, 4000, 31954, 11, 22, 3909}, 485, 128, 18.6, 12.4},  // reg8
        {{9, 9, 0, 4004, 4000, 51914, 14, 56, 0}, 357, 512, 21.4, 14.5},  // reg13
        {{6, 5, 366, 136, 500, 2978, 6, 17, 3}, 75, 512, 5.8, 6.7},  // rnd6
        {{7, 7, 2792, 1212, 4000, 23980, 13, 40, 45}, 602, 1024, 13.9, 11.4},  // rnd6
        {{5, 5, 486, 16, 500, 1990, 5, 10, 0}, 95, 16, 4.2, 6.1},  // rnd4
        {{5, 5, 3844, 158, 4000, 15984, 10, 25, 1}, 729, 4096, 17.4, 12.4},  // rnd4
        {{4, 2, 250, 4, 250, 1004, 4, 8, 0}, 42, 128, 3.5, 4.0},  // hub0.01
        {{6, 6, 3600, 402, 4000, 18786, 11, 43, 0}, 684, 1024, 13.5, 9.1},  // hub0.1
        {{6, 6, 86, 36, 120, 694, 6, 21, 0}, 20, 4096, 8.4, 7.1},  // hub0.3
        {{2, 2, 0, 500, 500, 6346, 2, 8, 0}, 125, 128, 3.3, 2.4},  // bip13
        {{2, 2, 62, 1938, 2000, 15936, 4, 8, 1872}, 500, 1024, 8.1, 4.3},  // bip8
        {{2, 0, 8000, 0, 8000, 23992, 16, 16, 0}, 2000, 4096, 21.0, 13.7},  // bip3
        {{5, 2, 250, 4, 250, 1000, 5, 10, 0}, 49, 512, 4.0, 4.6},  // dimer
        {{5, 5, 5478, 14, 5488, 21952, 14, 28, 0}, 1101, 4096, 21.3, 14.6},  // dimer
        {{4, 0, 8002, 0, 8000, 23994, 17, 17, 0}, 1496, 16, 10.9, 7.2},  // reg3
    };
    for (const Case &c : cases) {
        BitView v{};
        v.form = kBitGeneral;
        v.n = (int)c.g.n;
        v.n_pos = (int)(c.g.sites + c.g.wide_sites);
        v.n_groups = c.g.groups;
        v.max_pairs = c.max_pairs;
        bool close = false;
        CHECK(graph_bits_cheaper(c.g, v, c.R, 256, &close) == (c.bits < c.bytes));
        const int Rp = (c.R + 15) / 16 * 16, rs = byte_pick_rs(v.n, Rp, 256, 0);
        double bits = 1e9;
        for (int w : {4, 8, 16}) bits = std::min(bits, graph_bits_us(c.g, v, w, Rp, 256));
        const double bytes = graph_bytes_us(c.g, rs, Rp, 256);
        CHECK(bits < 1.25 * c.bits && c.bits < 1.25 * bits && bytes < 1.25 * c.bytes && c.bytes < 1.25 * bytes);
    }
    CHECK(byte_pick_rs(39936, 4096, 256, 0) == 4 && byte_pick_rs(39937, 4096, 256, 0) == 0);
    CHECK(byte_pick_rs(5488, 4096, 256, 0) == 8 && byte_pick_rs(500, 16384, 256, 0) == 16 && byte_pick_rs(500, 64, 256, 16) == 16);
}

// Cubes of more than 8192 sites, in tiles or by a launch per half-sweep (us per sweep of the faster of
// the two launch kernels, and of the best tiles, measured): what the estimate decides is the faster
// form, or within 5 % of it, and the rest is timed.
static void cube_forms()
{
    struct Case {
        int n;
        bool fields;
        int R;
        double launches, tiles;
    };
    const Case cases[] = {
        {8712, false, 16, 9.3, 5.7},  // 22x22x18
        {8712, true, 128, 12.8, 6.2},  // 22x22x18
        {10240, true, 64, 8.8, 6.7},  // 64x16x10
        {11520, true, 16, 9.2, 8.3},  // 32x20x18
        {13824, false, 16, 10.0, 7.8},  // 24x24x24
        {13824, true, 128, 16.2, 9.4},  // 24x24x24
        {17576, false, 64, 9.2, 11.2},  // 26x26x26
        {17576, false, 256, 19.0, 11.2},  // 26x26x26
        {17576, true, 512, 17.3, 12.0},  // 26x26x26
        {18432, false, 256, 12.3, 10.2},  // 32x24x24
        {21952, true, 16, 10.1, 14.7},  // 28x28x28
        {21952, true, 512, 17.2, 14.7},  // 28x28x28
        {27000, false, 64, 9.5, 16.6},  // 30x30x30
        {27000, false, 256, 22.5, 16.7},  // 30x30x30
        {32768, false, 512, 16.2, 18.6},  // 32x32x32
        {32768, false, 1024, 26.3, 18.5},  // 32x32x32
        {32768, false, 4096, 69.6, 49.5},  // 32x32x32
        {46080, false, 16, 9.2, 25.8},  // 48x32x30
        {46080, true, 128, 21.4, 30.5},  // 48x32x30
        {46080, true, 1024, 34.7, 30.6},  // 48x32x30
        {46080, false, 4096, 95.7, 70.0},  // 48x32x30
        {38880, false, 64, 11.5, 21.6},  // 36x36x30
        {38880, false, 512, 29.6, 21.8},  // 36x36x30
    };
    int timed = 0;
    for (const Case &c : cases) {
        BitView v{};
        v.form = c.fields ? kBitGeneral : kBitCube4;
        v.n = v.n_pos = c.n;
        v.n_groups = 2;
        v.max_pairs = c.n / 4;
        double tiles = 1e9;
        for (int rs : {4, 8, 16}) tiles = std::min(tiles, cube_bits_us(v, rs, (c.R + 15) / 16 * 16, 256));
        const CubeForm f = cube_form(tiles, c.n, c.R, 1000, true);
        CHECK(f != CubeForm::Tiles || c.tiles < 1.05 * c.launches);
        CHECK(f != CubeForm::Launches || c.launches < 1.05 * c.tiles);
        timed += f == CubeForm::Time;
        CHECK(cube_form(tiles, c.n, c.R, 2, false) != CubeForm::Time);
    }
    CHECK(timed >= 10);
    // without matrix-core tiles and too short to time: the stencil takes 17.4 and 9.2 us a sweep of 26^3
    CHECK(cube_form(11.2, 17576, 128, 100, false) == CubeForm::Tiles);
    CHECK(cube_form(11.2, 17576, 64, 100, false) == CubeForm::Launches);
}

int main()
{
    group_cursor();
    coupling_codes();
    exchange_octets();
    meetings();
    run_times();
    timed_kernels();
    graph_forms();
    cube_forms();
    std::printf("rules ok\n");
    return 0;
}
