// sweep_cost.h — what a sweep costs in the forms a cube or general graph can take, in
// microseconds on MI355X (host only).
//
// Graphs, in tiles that hold their spins as bits (bit_tile.h) or as bytes (graph_tile_item): both
// were timed over 835 shapes: 60 to 8000 spins, 3 to 15 terms a site (regular, random,
// bipartite, dimerized, and with 1 to 30 % of sites of 8 to 15 terms among sites of four), 2 to 9
// update groups, 16 to 4096 replicas, bits in each tile width.  The formulas below, fitted to
// that, are within 6 % (one standard deviation) of either form.  A sweep is a serial chain per
// group (latency) beside the work of its sites (throughput); neither hides the other fully.
#pragma once

#include <algorithm>
#include <cmath>

#include "batch.h"
#include "bits.h"

namespace pbit {

// Counted when a graph is loaded.
struct GraphShape {
    int groups = 0;         // update groups
    int wide_groups = 0;    // groups with a pair of sites of more than seven terms
    double sites = 0;       // positions of ordinary pairs
    double wide_sites = 0;  // positions of wide pairs
    // byte tiles: sites, bond ends, chunks of 512 sites of a group, the longest adjacency of each
    // chunk in steps of four bonds, and sites of eight bonds that follow one of eight (their
    // adjacencies, 32 bytes apart, take 1.7 ns a site more)
    double n = 0, ends = 0, chunks = 0, steps = 0, eights = 0;
};

// Anneals shorter than this keep an estimate where longer ones time the forms (0.3 ms, once a
// shape and context).
constexpr double kTimedAnnealUs = 3000.0;

inline double chain_and_work(double chain, double work, double norm)
{
    return std::pow(std::pow(chain, norm) + std::pow(work, norm), 1.0 / norm);
}

// Microseconds of a sweep of one tile of rs replicas with `beside` of them on its compute unit.
inline double graph_bit_tile_us(const GraphShape &g, int rs, int beside)
{
    const int i = rs == 4 ? 0 : rs == 8 ? 1 : 2;
    static const double many[3] = {0.72, 0.845, 0.95}, two[3] = {0.46, 0.50, 0.54}, wide[3] = {0.48, 0.26, 0.24};
    static const double site[3] = {0.61e-3, 1.0e-3, 1.64e-3}, wide_site[3] = {1.33e-3, 2.95e-3, 6.2e-3};
    const double chain = g.groups * (g.groups == 2 ? two : many)[i] + g.wide_groups * wide[i];
    const double work = g.sites * site[i] + g.wide_sites * wide_site[i];
    return chain_and_work(chain, work * (1 + 0.96 * (beside - 1)), 1.09);
}

inline double graph_byte_tile_us(const GraphShape &g, int rs, int beside)
{
    const double chain = 0.41 * g.groups + (rs == 4 ? 0.0 : 0.166) * g.chunks + (rs == 4 ? 0.196 : 0.24) * g.steps;
    const double work = (0.59e-3 * g.n + 0.112e-3 * g.ends + 1.72e-3 * g.eights) * (rs / 4);
    return chain_and_work(chain, work * (1 + 0.064 * (beside - 1)), 1.21);
}

// Byte tiles a compute unit holds, of eight waves each: `most` by registers, and their rows' LDS.
constexpr int kByteSlabsPerCu = 4, kByteTilesPerCu = 3;  // per-instance kernels (up to 49), batched kernel (71)
inline int byte_tiles_per_cu(double n, int rs, int most)
{
    return std::max(1, std::min(most, (int)(160 * 1024 / (n * rs + 2304))));
}

// Microseconds of a sweep of Rp replicas in tiles of rs on `cus` compute units.
inline double graph_bits_us(const GraphShape &g, const BitView &v, int rs, int Rp, int cus)
{
    const int tiles = (Rp + rs - 1) / rs, per_cu = bit_tiles_per_cu(v, rs);
    const int rounds = (tiles + cus * per_cu - 1) / (cus * per_cu), beside = std::min(per_cu, (tiles + cus - 1) / cus);
    return rounds * graph_bit_tile_us(g, rs, beside);
}

// Replicas per byte tile: the narrowest of 4, 8 and 16 that fits LDS and leaves at most two
// workgroups per compute unit, else the widest that fits (0: none, or the forced one does not).  A
// workgroup's sweep costs about the same at any tile width up to two per CU, so narrow tiles
// spread small replica counts over more CUs, and past two per CU the wider tile wins.
inline int byte_pick_rs(int64_t n, int Rp, int cus, int forced)
{
    int best = 0;
    for (int rs : {4, 8, 16}) {
        if (Rp % rs != 0 || n * rs > kGraphSlabLds || (forced && rs != forced)) continue;
        best = rs;
        if (Rp / rs <= 2 * cus) break;
    }
    return best;
}

inline double graph_bytes_us(const GraphShape &g, int rs, int Rp, int cus)
{
    const int tiles = Rp / rs, per_cu = byte_tiles_per_cu(g.n, rs, kByteSlabsPerCu);
    const int rounds = (tiles + cus * per_cu - 1) / (cus * per_cu), beside = std::min(per_cu, (tiles + cus - 1) / cus);
    return rounds * graph_byte_tile_us(g, rs, beside);
}

// Whether a graph's sweeps are faster with its spins as bits than as bytes.  Over the shapes the
// costs were fitted to, the choice loses less than 5 % in 95 of 100 and 18 % at most; *close says
// that they are within 15 %, where all of those lie.  Measured in us per sweep, bytes and bits, at
// 1024 replicas: 500 sites of 10 terms 7.8 and 9.1, of 6 terms 4.7 and 4.4; 2000 sites of 8 terms
// 11.1 and 9.9; 250 dimerized ones 4.0 and 4.6.
inline bool graph_bits_cheaper(const GraphShape &g, const BitView &v, int R, int cus, bool *close)
{
    const int Rp = (R + 15) / 16 * 16, rs = byte_pick_rs(v.n, Rp, cus, 0);
    double bits = graph_bits_us(g, v, 4, Rp, cus);
    for (int w : {8, 16}) bits = std::min(bits, graph_bits_us(g, v, w, Rp, cus));
    const double bytes = rs ? graph_bytes_us(g, rs, Rp, cus) : 2.0 * bits;
    if (close) *close = bits < 1.15 * bytes && bytes < 1.15 * bits;
    return bits < bytes;
}

// A cube's sweep in tiles of rs replicas: measured 0.58 ns per site and tile of 4 replicas (0.70
// with fields or zero couplings), 1.6 and 2.7 times that with 8 and 16, at 12^3 to 36^3, and what an
// update group costs at least (4^3 to 8^3).
inline double cube_bits_us(const BitView &v, int rs, int Rp, int cus)
{
    const int tiles = (Rp + rs - 1) / rs, slots = cus * bit_tiles_per_cu(v, rs);
    const double c = rs == 4 ? 1.0 : rs == 8 ? 1.62 : 2.7;
    return ((tiles + slots - 1) / slots) *
           (0.28 * v.n_groups + c * (v.form == kBitGeneral ? 0.70e-3 : 0.58e-3) * (double)v.n);
}

// How a cube of more sites than always stay in LDS runs, given the cost of its best tiles: in
// tiles, by the launch-per-half-sweep kernels, or as a timing of all of them says.  Those were
// measured at 0.93 to 2.4 times 8 us + 0.5 ps per spin and sweep (8.4 to 132 us from 8320 to 61 952
// sites and 16 to 4096 replicas: the stencil's launches of 128 replicas and more, and shapes without
// matrix-core tiles, are far above the line), so the estimate decides only where the tiles need
// less than 0.8 of that or more than 2.5 times it.  Without matrix-core tiles, where no anneal
// was timed before, it also decides for short anneals.
enum class CubeForm { Tiles, Launches, Time };
inline double cube_launch_us(int64_t n, int R, bool matrix_tiles)
{
    const double least = 8.0 + 0.5e-6 * (double)n * R;
    return matrix_tiles || R < 128 ? least : std::max(least, 10.0 + 0.4e-3 * (double)n);
}
inline CubeForm cube_form(double tiles_us, int64_t n, int R, int sweeps, bool matrix_tiles)
{
    const double launches = cube_launch_us(n, R, matrix_tiles);
    if (tiles_us < 0.8 * launches) return CubeForm::Tiles;
    if (tiles_us > 2.5 * launches) return CubeForm::Launches;
    if (!matrix_tiles && sweeps * std::min(tiles_us, launches) < kTimedAnnealUs)
        return tiles_us < launches ? CubeForm::Tiles : CubeForm::Launches;
    return CubeForm::Time;
}

}  // namespace pbit
