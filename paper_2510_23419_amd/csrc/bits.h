// bits.h — sparse problems (cubes and general graphs) with their spins held as
// bits in LDS: host-built site records and the launchers of bit_kernels.hip.
//
// Sites are numbered by position: update group by update group, each group padded
// to an even count, so that positions 2 p and 2 p + 1 form pair p.  Every site's
// field is a sum of K terms +-m, one per slot: its bonds, its external field (a
// slot on a constant +1 spin), and padding (slots on that spin, as many -1 as +1).
// With n of the K terms negative, I = K - 2 n - odd, where odd = 1 for a site whose
// terms needed an unpaired +1 to reach K.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

namespace pbit {

constexpr int kBitSlots = 7;      // slots per site, ordinary pairs
constexpr int kBitSlotsWide = 15; // slots per site, pairs with a site of more than kBitSlots terms
// A tile's LDS: tables, then 16-bit elements by position and one constant +1 spin behind
// them.  Records hold element indices from LDS address 0, so half the tables' bytes are
// added to a position.
constexpr uint32_t kBitElBase = 7168;
constexpr uint32_t kBitNoSite = 0xFFFFu;  // a padding position
constexpr int kBitMaxPositions = 65536 - (int)kBitElBase / 2 - 2;

// Record forms of the ordinary pairs.
enum BitForm : int {
    kBitCube4 = 0,   // six bonds, five neighbour pairs aligned (dense cubes without fields, Lx a multiple of 4)
    kBitCube = 1,    // six bonds (other dense cubes without fields)
    kBitGeneral = 2  // seven slots and the odd mask, with wide pairs
};

struct BitView {
    int form;               // BitForm
    int n, n_pos, n_groups; // sites, positions, update groups
    int n_pairs;            // ordinary pairs over all groups
    int n_wide;             // wide pairs over all groups
    int max_pairs;          // most pairs of one group
    // per group {first wide pair, wide pairs, first ordinary pair, ordinary pairs}: the group's
    // positions start at twice the sum of both firsts, wide pairs first
    const int4 *groups;
    // records, [16-byte word][pair]: kBitCube4 three words (eight 16-bit element indices: the
    // low element of slots 0..4, both elements of slot 5; six masks; sites), kBitCube and
    // kBitGeneral four words (slot indices, masks, odd mask, sites), wide pairs eight
    const uint4 *rec, *wide;
    const uint16_t *pos_site;  // [n_pos] site of a position, kBitNoSite for padding
    const int8_t *h;           // device [n] by site, or null (energies)
};

struct BitHost {
    int form = 0, n = 0, n_pos = 0, n_groups = 0, n_pairs = 0, n_wide = 0, max_pairs = 0;
    std::vector<int32_t> groups;     // [n_groups][4]
    std::vector<uint32_t> rec, wide; // [word][pair][4]
    std::vector<uint16_t> pos_site;
};

// Builds the records of a problem given as per-site neighbour lists in CSR form
// (start[n + 1], neighbour and coupling in {-1, 0, +1} per entry; an entry per bond
// end), fields h (or null) and update groups.  `cube_lx` is the cube's first side
// for a cube whose groups are its two colours (0 otherwise): its positions then
// follow the lattice rows.  False where a site has more than kBitSlotsWide terms
// or the positions exceed kBitMaxPositions.
bool bit_build(int n, const int32_t *start, const int32_t *nbr, const int8_t *J, const int8_t *h,
               const uint8_t *group, int n_groups, int cube_lx, BitHost &out);

// Update group that a sweep's cursor c (up to two past the last of its `groups` groups) stands on:
// the groups of the next sweep follow.
constexpr __host__ __device__ int bit_group_at(int c, int groups) { return groups == 1 ? 0 : c < groups ? c : c - groups; }

// One anneal's tiles: tile t holds replicas [rs t, rs t + rs).
struct BitJobDev {
    BitView v;
    const uint32_t *table;  // [S][width] thresholds, row s = local sweep s
    int8_t *state;          // spins by site: [n][row_stride] matrix (row_stride > 0, tile t = columns
                            // [rs t, + rs)), or [tiles][n][rs] (row_stride = 0)
    int32_t *energy;        // [tiles * rs] energies after a tile's item, or null
    int width, rs, row_stride;
    uint32_t sweep0, rq0, k0, k1;
};

// LDS a tile needs, whatever its replica count.
inline size_t bit_lds(int n_pos) { return kBitElBase + 4 * ((size_t)(n_pos + 3) / 2); }
constexpr size_t kBitMaxLds = 160 * 1024 - 4096;

// Threads of a per-instance tile of rs replicas: enough for the largest group in its
// finest units, between the decision tables' entries and 1024; and how many such tiles a
// compute unit holds (four waves per SIMD, LDS).
inline int bit_threads(const BitView &v, int rs)
{
    const int units = (2 * v.max_pairs * (rs / 4) + 63) / 64 * 64, least = v.form == kBitGeneral ? 256 : 64;
    return units > 1024 ? 1024 : units < least ? least : units;
}
inline int bit_tiles_per_cu(const BitView &v, int rs)
{
    const int by_waves = 1024 / bit_threads(v, rs), by_lds = (int)(kBitMaxLds / bit_lds(v.n_pos));
    return by_waves < by_lds ? by_waves : by_lds < 1 ? 1 : by_lds;
}

// Sweeps [s_begin, s_end) of tiles [0, tiles), one workgroup per tile.
hipError_t bit_slab(const BitJobDev &jb, int tiles, int s_begin, int s_end, hipStream_t st);

}  // namespace pbit
