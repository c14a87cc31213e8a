// bq.h — biclique problem view and launchers (declarations shared by the
// host runtime and the biclique kernels).
#pragma once

#include "internal.h"

namespace pbit {

struct BqView {
    int na, nb;      // real side sizes
    int na_p, nb_p;  // padded to kBqPad (extra couplings and spins are zero)
    const int8_t *J;   // [na_p][nb_p]
    const int8_t *JT;  // [nb_p][na_p]
    const int8_t *hA;  // [na_p]
    const int8_t *hB;  // [nb_p]
    // for the kernels on spin bits: the couplings as E2M1 numbers in the order the widened
    // bits take (spin_bits_fp4), scaled so that every product is 2 J b, rows of
    // bq_row_bytes(nb_p) and bq_row_bytes(na_p), and each site's field plus its coupling sum
    const uint8_t *J4;
    const uint8_t *JT4;
    const int32_t *hA2;  // [na_p]
    const int32_t *hB2;  // [nb_p]
    // for the batched FP4 tiles: couplings as two-bit codes, 16 per word, in MFMA fragment
    // order (see load_biclique), side A's sites (na_p * nb_p / 16 words), then side B's, then
    // the words that the tiles' rings read past them (bq_code_bytes)
    const uint32_t *J2;
};

// Bytes of a row of four-bit couplings: whole stages of 256 sites for the per-launch bit kernel
// (zeros past ko_p) where it can take the side.
constexpr int bq_row_bytes(int ko_p) { return ko_p % 128 == 0 ? (ko_p + 255) / 256 * 128 : ko_p / 2; }
// Coupling codes of the batched FP4 tiles: bytes of one K step (64 sites of the other side) of a
// block of 32 sites, K steps a wave reads ahead, where a block of a side starts (the block of a
// wave past the side's last one is the last), and the bytes of both sides with what a ring that
// starts on the last block reads past it.
constexpr int kCodeUnit = 512, kCodeRing = 4;
constexpr __host__ __device__ int bq_code_start(int na_p, int nb_p, int side, int wave)
{
    const int blocks = (side == 0 ? na_p : nb_p) / 32, per_block = kCodeUnit * ((side == 0 ? nb_p : na_p) / 64);
    return (side == 0 ? 0 : na_p * nb_p / 4) + per_block * (wave < blocks ? wave : blocks - 1);
}
constexpr __host__ __device__ int64_t bq_code_bytes(int na_p, int nb_p)
{
    return (int64_t)na_p * nb_p / 2 + (kCodeRing - 1) * kCodeUnit;
}
// Exchange words of the cluster kernel come in octets of blocks; the octet that K steps 4 k to
// 4 k + 3 of a side of `octets` octets read (the last one's past it, whose products are left out).
constexpr __host__ __device__ int bq_octet(int k, int octets) { return k < octets ? k : octets - 1; }
constexpr int kBqPad = 64;       // site padding of small biclique sides (MFMA K and N tiles)
constexpr int kBqPadLarge = 128; // site padding of sides with at least kBqLargeSide sites
constexpr int kBqLargeSide = 512;
constexpr int kBqRPad = 128;     // replica padding of biclique spin matrices (MFMA M tile)
constexpr int kMaxTableWidth = 4096;  // threshold-row entries a biclique kernel stages in LDS (16 KiB)

// ---- biclique launchers; spins are device MA [Rp][na_p], MB [Rp][nb_p] -----
// Kernel variants of a biclique half-sweep.  Small: 64 x 64 tiles straight from
// global memory (any padding); Dma: 128 x 128 tiles with K stages of 128 bytes
// moved by the global-to-LDS DMA into a ring of 4 stages (sides padded to 128,
// Rp a multiple of 128); Bits: tiles of 64 sites x 256, 128 or 64 replicas on spins
// held as bits, widened for the FP4 MFMA (bqb_*; sides padded to 128, Rp a multiple
// of 256); Slab: sides of
// at most 512 sites, couplings and 16- or 8-replica slices held in LDS for runs of
// sweeps in one launch (bq_slab).
// Cluster: couplings in registers across an XCD for runs of sweeps (bq_cluster).
enum class BqVariant : int { Auto = 0, Small = 1, Dma = 2, Bits = 3, Slab = 4, Cluster = 5 };
// The LDS-resident form for small sides: sweeps [s_begin, s_end) (table rows), absolute
// index sweep0 + s, of all Rp replicas (Rp / rs workgroups of rs-replica slices) on MA / MB
// in place.  rs is 16 or 8; 0 picks 16 when that gives a workgroup to every compute unit,
// else 8.  bq_slab_rs returns the slice that a launch with rs uses (0: none fits Rp).
int bq_slab_rs(int Rp, int rs);
bool bq_slab_supported(const BqView &p, int Rp, int width, int rs = 0);
hipError_t bq_slab(const BqView &p, int8_t *MA, int8_t *MB, int Rp, const uint32_t *table, int width, int s_begin,
                   int s_end, uint32_t sweep0, uint32_t rq0, Key key, hipStream_t st, int rs = 0);
// The form whose couplings stay in registers across an XCD (bq_cluster.hip), for sides of at
// most 2048 sites and threshold rows of at most 256 entries: sweeps [s_begin, s_end) of
// replicas [0, R) on MA / MB in place, with `work` (bq_cluster_bytes) as exchange memory and a
// workgroup on each of `cus` compute units, which wait up to `meet_us` for each other
// (kMeetUs: an idle device takes some 10 us).  work[1] is 0 afterwards if the sweeps ran, 1
// if the workgroups could not be resident together (MA / MB untouched), 2 after a lost flag.
bool bq_cluster_supported(const BqView &p, int width);
size_t bq_cluster_bytes(const BqView &p, int R);
constexpr int kMeetUs = 2000;
hipError_t bq_cluster(const BqView &p, int8_t *MA, int8_t *MB, int R, int Rp, const uint32_t *table, int width,
                      int s_begin, int s_end, uint32_t sweep0, uint32_t rq0, Key key, void *work, int cus,
                      int meet_us, hipStream_t st);
hipError_t bq_init(const BqView &p, int8_t *MA, int8_t *MB, int R, uint32_t rq0, Key key, hipStream_t st);
hipError_t bq_from_rows(const BqView &p, const int8_t *src_rn, int R, int8_t *MA, int8_t *MB, hipStream_t st);
hipError_t bq_to_rows(const BqView &p, const int8_t *MA, const int8_t *MB, int8_t *dst_rn, int R, hipStream_t st);
hipError_t bq_halfsweep(const BqView &p, int side, int8_t *MA, int8_t *MB, int R, int Rp, const uint32_t *trow,
                        int width, uint32_t sweep, uint32_t rq0, Key key, hipStream_t st, BqVariant variant);
hipError_t bq_energy(const BqView &p, const int8_t *MA, const int8_t *MB, int R, int Rp, int32_t *E, hipStream_t st);

// ---- the same with spins held as bits (set = -1), 32 sites per word, by blocks of 128 sites:
// word w of replica r at ((w / 4) Rp + r) 4 + (w % 2) 2 + (w / 2) % 2 of MAb (na_p / 32 words per
// replica) or MBb
bool bqb_supported(const BqView &p, int Rp);
hipError_t bqb_pack(const BqView &p, const int8_t *MA, const int8_t *MB, uint32_t *MAb, uint32_t *MBb, int Rp,
                    hipStream_t st);
hipError_t bqb_unpack(const BqView &p, const uint32_t *MAb, const uint32_t *MBb, int8_t *MA, int8_t *MB, int Rp,
                      hipStream_t st);
// rt: replicas per tile, 64, 128 or 256; 0 (or a value that does not divide Rp): 256
// where that gives at least 256 workgroups, else 128
hipError_t bqb_halfsweep(const BqView &p, int side, uint32_t *MAb, uint32_t *MBb, int Rp, const uint32_t *trow,
                         int width, uint32_t sweep, uint32_t rq0, Key key, hipStream_t st, int rt = 0);

}  // namespace pbit
