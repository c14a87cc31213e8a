// batch_kernels.hip — persistent batched sweep for many independent jobs.
//
// Each workgroup repeatedly takes a work item (job, replica tile, sweep range)
// from a device queue and runs it with the tile's spins held in LDS, so the
// half-sweeps of a tile need only workgroup barriers, never a grid-wide one:
// replicas are independent runs (paper Sec. 1.3.3), and inside a tile the two
// update groups alternate (Sec. 1.2.2).  Jobs of uneven sizes therefore share
// one launch.  The arithmetic, the Philox counters and the decision rule are
// the same as in the per-instance kernels, so a job's result does not depend on
// which items it was batched with.
#include <type_traits>

#include "batch.h"
#include "device.h"
#include "bq.h"

namespace pbit {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));


__device__ __forceinline__ int take_item(int32_t *counter, int *slot)
{
    if (threadIdx.x == 0) *slot = atomicAdd(counter, 1);
    __syncthreads();
    const int it = __builtin_amdgcn_readfirstlane(*slot);
    __syncthreads();
    return it;
}

__device__ __forceinline__ uint32_t neg2(uint32_t m, uint32_t keep, uint32_t flip) { return (m & keep) ^ flip; }

// ---------------------------------------------------------------- graph tiles

// General graphs with k update groups (Sec. 1.2.2) whose sites have more terms than the bit
// records hold (bits.h): the spins of 4W replicas of the whole graph live in LDS as W dwords
// per site (byte p of dword k = replica 4k + p, +1 = 0x01, -1 = 0xFF).  The classes
// are swept in ascending colour order with a workgroup barrier between them; a
// thread takes one site of the class at a time, reads its record and adjacency
// words from global memory (class-major, as for the per-instance sweep) and its
// neighbours' rows from LDS, and counts negative products bytewise exactly as
// the per-instance kernel does (0x02 per negative product, degree <= 127), so
// that the field, the Philox counters and the carry decision are the same.
constexpr int kGraphOff = kGraphMaxDegree + 1;  // |I| <= degree + |h|
constexpr int kGraphSlots = 2 * kGraphOff + 1;

template <int W>
__device__ __forceinline__ void graph_tile_item(const WorkItem &w, const GraphJobDev &jb, uint4 *tile_rows,
                                                uint64_t *gtab, int32_t *eacc, uint32_t one)
{
    typedef uint32_t V __attribute__((ext_vector_type(W)));
    constexpr int RS = 4 * W;
    V *rows = reinterpret_cast<V *>(tile_rows);  // [n]
    const int tid = threadIdx.x;
    const int n = jb.n;
    const uint32_t rgw = jb.rq0 + (uint32_t)W * (uint32_t)w.tile;  // Philox counter word 2 of the tile's first group
    // the tile's rows: contiguous (batch state) or strided columns of the per-instance spins
    const size_t rstride = jb.row_stride ? (size_t)jb.row_stride : (size_t)RS;
    int8_t *gst = jb.state + (size_t)w.tile * (jb.row_stride ? (size_t)RS : (size_t)n * RS);

    if (w.init) {
        for (int i = tid; i < n; i += kGraphTileThreads) {
            V d;
#pragma unroll
            for (int k = 0; k < W; ++k) {
                const Block4 b = philox((uint32_t)i, 0u, rgw + (uint32_t)k, kDomainInit, jb.k0, jb.k1);
                uint32_t packed = 0;
#pragma unroll
                for (int p = 0; p < 4; ++p) packed |= (uint32_t)(uint8_t)init_spin(b.w[p]) << (8 * p);
                d[k] = packed;
            }
            rows[i] = d;
        }
    } else {
        for (int i = tid; i < n; i += kGraphTileThreads) rows[i] = load_global<V>(gst + rstride * i);
    }

    for (int s = w.s_begin; s < w.s_end; ++s) {
        __syncthreads();
        // decision words by descending field value: entry k is S(I) for I = kGraphOff - k
        const uint32_t *trow = jb.table + (size_t)s * jb.width;
        for (int k = tid; k < kGraphSlots; k += kGraphTileThreads) {
            const int I = kGraphOff - k;
            const uint32_t T = load_global<uint32_t>(trow + min(I >= 0 ? I : -I, jb.width - 1));
            gtab[k] = I >= 0 ? (uint64_t)T : ((uint64_t)1 << 32) - T;
        }
        __syncthreads();
        const uint32_t t = jb.sweep0 + (uint32_t)s;
        for (int c = 0; c < jb.n_colours; ++c) {
            const int p0 = load_global<int32_t>(jb.class_start + c), p1 = load_global<int32_t>(jb.class_start + c + 1);
            for (int j = p0 + tid; j < p1; j += kGraphTileThreads) {
                const v4i mv = load_global<v4i>(jb.meta + j);  // site, first entry, end entry, nnz + h
                const int4 m = make_int4(mv[0], mv[1], mv[2], mv[3]);
                const int i = m.x;
                uint32_t cnt[W];
#pragma unroll
                for (int k = 0; k < W; ++k) cnt[k] = 0u;
                // four adjacency entries, then their four rows, in flight together; an entry
                // past the end reads as 0 (row 0, no coupling), so it adds nothing
                for (int e = m.y; e < m.z; e += 4) {
                    uint32_t a[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) a[u] = e + u < m.z ? load_global<uint32_t>(jb.adj + e + u) : 0u;
                    V v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = rows[a[u] >> 2];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        // 0x02 in every byte where J != 0 (keep) and where J = -1 (flip)
                        const uint32_t keep = (uint32_t)((int32_t)(a[u] << 31) >> 31) & 0x02020202u;
                        const uint32_t flip = (uint32_t)((int32_t)(a[u] << 30) >> 31) & 0x02020202u;
#pragma unroll
                        for (int k = 0; k < W; ++k) cnt[k] += neg2(v[u][k], keep, flip);
                    }
                }
                // a byte c of cnt (two per negative product) gives I = base - c: entry kGraphOff - base + c
                const char *tb = reinterpret_cast<const char *>(gtab) + 8 * (kGraphOff - m.w);
                V out;
#pragma unroll
                for (int k = 0; k < W; ++k) {
                    const Block4 b = philox((uint32_t)i, t, rgw + (uint32_t)k, kDomainSweep, jb.k0, jb.k1);
                    uint32_t sgn[4];  // 1: the replica's new spin is -1
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const uint32_t cb = (cnt[k] >> (8 * p)) & 0xFFu;
                        const uint64_t S = *static_cast<const uint64_t *>(__builtin_assume_aligned(tb + 8 * cb, 8));
                        sgn[p] = (uint32_t)(((uint64_t)b.w[p] * one + S) >> 32);
                    }
                    const uint32_t lo = __builtin_amdgcn_perm(sgn[1], sgn[0], 0x0C0C0400u);
                    const uint32_t hi = __builtin_amdgcn_perm(sgn[3], sgn[2], 0x0C0C0400u);
                    out[k] = __builtin_amdgcn_perm(0u, 0xFF01u, __builtin_amdgcn_perm(hi, lo, 0x05040100u));
                }
                rows[i] = out;
            }
            __syncthreads();
        }
    }

    // energies from scratch: E = -sum_bonds J m_i m_j - sum_i h_i m_i; a product is -1
    // where the two bytes differ (bit 1 of their xor)
    if (tid < RS) eacc[tid] = 0;
    __syncthreads();
    int32_t er[RS];
#pragma unroll
    for (int r = 0; r < RS; ++r) er[r] = 0;
    for (int b = tid; b < jb.n_bonds; b += kGraphTileThreads) {
        const int J = load_global<int8_t>(jb.bJ + b);
        if (J == 0) continue;
        const V mi = rows[load_global<int32_t>(jb.bi + b)], mj = rows[load_global<int32_t>(jb.bj + b)];
#pragma unroll
        for (int k = 0; k < W; ++k) {
            const uint32_t d = ((mi[k] ^ mj[k]) >> 1) & 0x01010101u;
#pragma unroll
            for (int p = 0; p < 4; ++p) er[4 * k + p] -= J * (1 - 2 * (int)((d >> (8 * p)) & 1u));
        }
    }
    if (jb.h)
        for (int i = tid; i < n; i += kGraphTileThreads) {
            const int hv = load_global<int8_t>(jb.h + i);
            if (hv == 0) continue;
            const V mi = rows[i];
#pragma unroll
            for (int k = 0; k < W; ++k)
#pragma unroll
                for (int p = 0; p < 4; ++p) er[4 * k + p] -= hv * (int)(int8_t)(mi[k] >> (8 * p));
        }
#pragma unroll
    for (int r = 0; r < RS; ++r) {
        int v = er[r];
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
        if ((tid & 63) == 0) atomicAdd(&eacc[r], v);
    }
    __syncthreads();
    if (tid < RS) jb.energy[RS * w.tile + tid] = eacc[tid];
    for (int i = tid; i < n; i += kGraphTileThreads) *reinterpret_cast<V *>(gst + rstride * i) = rows[i];
}

// Persistent graph-tile kernel: items of any tile width share the launch.
__global__ __launch_bounds__(kGraphTileThreads) void k_graph_tiles(const GraphJobDev *__restrict__ jobs,
                                                                   const WorkItem *__restrict__ items,
                                                                   const int32_t *__restrict__ n_items_p,
                                                                   int32_t *__restrict__ counter, uint32_t one)
{
    extern __shared__ uint4 tile_rows[];
    __shared__ uint64_t gtab[kGraphSlots];
    __shared__ int32_t eacc[16];
    __shared__ int slot;
    const int n_items = *n_items_p;
    for (;;) {
        const int it = take_item(counter, &slot);
        if (it >= n_items) break;
        const WorkItem w = items[it];
        const GraphJobDev jb = jobs[w.job];
        if (jb.rs == 16)
            graph_tile_item<4>(w, jb, tile_rows, gtab, eacc, one);
        else if (jb.rs == 8)
            graph_tile_item<2>(w, jb, tile_rows, gtab, eacc, one);
        else
            graph_tile_item<1>(w, jb, tile_rows, gtab, eacc, one);
        __syncthreads();  // the next item's first LDS writes wait for this item's last reads
    }
}

// The per-instance graph sweep held in LDS: workgroup t runs tile t (replicas
// [4 W t, + 4 W)) of the job for sweeps [s_begin, s_end), reading and writing its
// columns of the per-instance spins.
template <int W>
__global__ __launch_bounds__(kGraphTileThreads) void k_graph_slab(GraphJobDev jb, int s_begin, int s_end,
                                                                  uint32_t one)
{
    extern __shared__ uint4 tile_rows[];
    __shared__ uint64_t gtab[kGraphSlots];
    __shared__ int32_t eacc[16];
    const WorkItem w{0, (int)blockIdx.x, s_begin, s_end, 0, {0, 0, 0}};
    graph_tile_item<W>(w, jb, tile_rows, gtab, eacc, one);
}

// ---------------------------------------------------------------- biclique tiles

// A tile holds RB x 32 replicas of both sides in LDS, one row per replica, padding zero.
// Each half-sweep is an MFMA product of the LDS spin rows with the couplings
// streamed from global memory (L2-resident, shared by all tiles of the job),
// followed by the decision epilogue writing the new side into LDS.
constexpr int kRing = 4;      // K-units of J fragments in flight per site block (bit tiles)

// The FP4 operand (32 K values of a lane) of two words of coupling codes: nibble i of dword
// 2 d + e is bits 3 - e (sign) and 1 - e (set: +-1, else 0) of nibble i of word d.
__device__ __forceinline__ v4i widen_codes(v2i_t x, uint32_t mask)
{
    const int m = (int)mask;
    return v4i{x[0] & m, (x[0] << 1) & m, x[1] & m, (x[1] << 1) & m};
}

// Biclique tiles with the spins held as bits in LDS: row r holds one bit per site (set = -1), 32 sites per word, side A
// in words [0, na_p / 32), side B after it, with an odd row pitch so that the 32
// rows a fragment read touches sit on distinct banks.  A K step of 64 sites is two words per
// replica, one in each lane half, widened in registers to four-bit numbers and multiplied on
// the FP4 MFMA by the couplings stored in the same order (J4, JT4): the sum is
// 2 sum_k J_sk b_k and the field is I = (h + sum_k J) - the sum, exact.
// A bit row is an eighth of an int8 row, so 128 replicas fit LDS at any side
// length and each coupling fragment feeds RB MFMAs: couplings reach the CU at
// 1 / (64 RB) bytes per multiply-add.  The 64
// decisions of a wave for one (replica group, p) form a ballot mask, and the
// words of the 32 replicas of a block are written by one lane each.
template <int RB>
__global__ __launch_bounds__(kBqTileThreads) void k_bq_tiles_bits(const BqJobDev *__restrict__ jobs,
                                                                  const WorkItem *__restrict__ items,
                                                                  const int32_t *__restrict__ n_items_p,
                                                                  int32_t *__restrict__ counter, uint32_t one)
{
    constexpr int RS = 32 * RB;
    extern __shared__ uint4 dyn[];
    __shared__ int32_t eacc[RS];
    __shared__ int slot;
    const int tid = threadIdx.x;
    const int lane = tid & 63, ln = lane & 31, kg = lane >> 5;
    const int wave = tid >> 6;
    const int n_items = *n_items_p;

    for (;;) {
        const int it = take_item(counter, &slot);
        if (it >= n_items) break;
        const WorkItem w = items[it];
        const BqJobDev jb = jobs[w.job];
        const int na = jb.na, nb = jb.nb, na_p = jb.na_p, nb_p = jb.nb_p;
        const int wa = na_p / 32, wb = nb_p / 32;  // spin words of each side in a row
        const int PW = wa + wb, pitch = PW + 1;    // words per row in global memory / in LDS
        uint32_t *sw = reinterpret_cast<uint32_t *>(dyn);
        // decision words after the rows, 8-byte aligned
        uint64_t *Sw = reinterpret_cast<uint64_t *>(sw + ((RS * pitch + 1) & ~1));
        const char *Sb = reinterpret_cast<const char *>(Sw);
        uint32_t *gst = reinterpret_cast<uint32_t *>(jb.state) + (size_t)w.tile * RS * PW;
        const uint32_t rg0 = jb.rq0 + (uint32_t)(w.tile * (RS / 4));

        if (w.init) {
            for (int k = tid; k < RS * pitch; k += kBqTileThreads) sw[k] = 0u;
            __syncthreads();
            // thread (site, replica group): the four replicas' spins of one site
            for (int k = tid; k < (na + nb) * (RS / 4); k += kBqTileThreads) {
                const int g = k % (RS / 4), i = k / (RS / 4);  // site id: A first, then B
                const int col = i < na ? i : na_p + (i - na);
                const Block4 b = philox((uint32_t)i, 0u, rg0 + (uint32_t)g, kDomainInit, jb.k0, jb.k1);
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    if (init_spin(b.w[p]) < 0) atomicOr(&sw[(4 * g + p) * pitch + col / 32], 1u << (col % 32));
            }
        } else {
            for (int k = tid; k < RS * PW; k += kBqTileThreads) {
                const int r = k / PW, c = k % PW;
                sw[r * pitch + c] = gst[(size_t)r * PW + c];
            }
        }
        if (tid < RS) eacc[tid] = 0;

        for (int s = w.s_begin; s < w.s_end; ++s) {
            __syncthreads();
            const uint32_t *trow = jb.table + (size_t)s * jb.width;
            const int top = jb.width - 1;
            for (int e = tid; e <= 2 * top; e += kBqTileThreads) {
                const int I = e - top;
                const uint32_t Tm = load_global<uint32_t>(trow + (I >= 0 ? I : -I));
                Sw[e] = I >= 0 ? (uint64_t)Tm : ((uint64_t)1 << 32) - Tm;
            }
            __syncthreads();
            const uint32_t t = jb.sweep0 + (uint32_t)s;
            const bool last = s + 1 == w.s_end;
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const int ns_p = side == 0 ? na_p : nb_p;
                const int ns = side == 0 ? na : nb;
                const int ko = side == 0 ? nb_p : na_p;  // coupling bytes per row (the other side)
                const int in_w = side == 0 ? wa : 0;     // word column of the other side
                const int out_w = side == 0 ? 0 : wa;    // word column of this side
                const uint8_t *Jx = side == 0 ? jb.J4 : jb.JT4;
                const int32_t *hs2 = side == 0 ? jb.hA2 : jb.hB2;
                const uint32_t site_base = side == 0 ? 0u : (uint32_t)na;
                // one 32-site block per wave at a time; its coupling fragments stream
                // from global memory through a ring kRing K-units (32 bytes) ahead,
                // which past the end of a block fills with the wave's next block
                const int nku = ko / 64, row = bq_row_bytes(ko);
                constexpr int kStep = kBqTileThreads / 64;
                const int nblk = ns_p / 32;
                v4i ring[kRing];
                if (wave < nblk) {
                    const uint8_t *br0 = Jx + (size_t)(wave * 32 + ln) * row + 16 * kg;
#pragma unroll
                    for (int u = 0; u < kRing; ++u) ring[u] = load_global<v4i>(br0 + 32 * min(u, nku - 1));
                }
                for (int blk = wave; blk < nblk; blk += kStep) {
                    const int site = blk * 32 + ln;
                    const uint8_t *br = Jx + (size_t)site * row + 16 * kg;
                    const uint8_t *bn = blk + kStep < nblk ? br + (size_t)kStep * 32 * row : br;
                    v16f_t acc[RB];
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                        for (int j = 0; j < 16; ++j) acc[rb][j] = __uint_as_float(kFieldBase);
                    const uint32_t *abase = sw + ln * pitch + in_w + kg;
                    for (int kb = 0; kb < nku; kb += kRing) {
#pragma unroll
                        for (int u = 0; u < kRing; ++u) {
                            const int ku = kb + u;
                            if (ku < nku) {
                                const v4i b = ring[u];
                                const int kn = ku + kRing;
                                ring[u] = load_global<v4i>(kn < nku ? br + 32 * kn : bn + 32 * min(u, nku - 1));
#pragma unroll
                                for (int rb = 0; rb < RB; ++rb) {
                                    const v4i a = spin_bits_fp4(abase[rb * 32 * pitch + 2 * ku]);
                                    acc[rb] = mfma_fp4(a, b, acc[rb]);
                                }
                            }
                        }
                    }
                    // decisions; padding sites take bits that nothing reads (their
                    // couplings and fields are zero and they are never returned)
                    const int h2 = hs2[site];  // field plus coupling sum; site < ns_p
                    const bool site_ok = site < ns;
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        uint32_t outw = 0u;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int r4 = rb * 32 + 8 * q + 4 * kg;  // first replica of the group in the tile
                            const Block4 b = philox(site_base + (uint32_t)site, t, rg0 + (uint32_t)(r4 >> 2),
                                                    kDomainSweep, jb.k0, jb.k1);
#pragma unroll
                            for (int p = 0; p < 4; ++p) {
                                // the accumulator's bits are kFieldBase + 8 sum J b
                                const int I = h2 - ((int)(__float_as_uint(acc[rb][4 * q + p]) - kFieldBase) >> 2);
                                const int Ic = min(max(I, -top), top);
                                const uint64_t S = *static_cast<const uint64_t *>(
                                    __builtin_assume_aligned(Sb + 8 * (Ic + top), 8));
                                const bool neg = (((uint64_t)b.w[p] * one + S) >> 32) != 0;  // new spin -1
                                // energy after the last side-B update: E = -sum_b m_b I_b - sum_a h_a m_a
                                if (side == 1 && last && site_ok) atomicAdd(&eacc[r4 + p], neg ? I : -I);
                                const uint64_t m = __ballot(neg);
                                const int L = 8 * q + p;
                                outw = (uint32_t)lane_write((int)(uint32_t)m, L, (int)outw);
                                outw = (uint32_t)lane_write((int)(uint32_t)(m >> 32), L + 4, (int)outw);
                            }
                        }
                        if (lane < 32) sw[(rb * 32 + lane) * pitch + out_w + blk] = outw;
                    }
                }
                __syncthreads();
            }
        }

        // field part of side A, then the energies and the spins go back to global memory
        for (int k = tid; k < RS * na; k += kBqTileThreads) {
            const int r = k / na, a = k % na;
            const int m = (sw[r * pitch + a / 32] >> (a % 32)) & 1u ? -1 : 1;
            const int v = (int)jb.hA[a] * m;
            if (v != 0) atomicAdd(&eacc[r], -v);
        }
        __syncthreads();
        if (tid < RS) jb.energy[w.tile * RS + tid] = eacc[tid];
        for (int k = tid; k < RS * PW; k += kBqTileThreads) {
            const int r = k / PW, c = k % PW;
            gst[(size_t)r * PW + c] = sw[r * pitch + c];
        }
    }
}

// A tile holds RB x 32 replicas of both sides in LDS, one row per replica, side A first:
// four bits a site, +1, -1 or (padding) 0 as E2M1 numbers, 32 sites in 16 bytes with site
// 4 i + j at nibble i of dword j.  A half-sweep multiplies the rows by the couplings on the
// FP4 MFMA, 64 sites a step: products are -1, 0 or 1 and the float sums stay below 2^20 from
// a start of 1.5 x 2^21, where the accumulator's bits are kFieldBase + 4 sum exactly, so |4 I| is
// one v_sad away and indexes the sweep's threshold row.  Couplings stream from the L2 (shared
// by all tiles of the job) as two-bit codes, two instructions from the MFMA's operand, and
// each fragment feeds RB MFMAs.
//
// What bounds it: instruction issue.  A block of 32 sites x 32 replicas takes about 140 vector
// instructions for its random words and as many for its decisions, and each K step an MFMA of
// 32 cycles and 6 instructions for the codes, which do not overlap (56 cycles a step); the
// sum of these is the measured 13.5 us a sweep of a tile at 1022 sites per side.  A tile of 32
// replicas alone on a compute unit took 33 us there with int8 operands (27 against 11 at 876,
// where 16 waves against 8 gave 15 to 19): half the MFMA time, an eighth of the LDS reads.
// Deeper rings than four steps changed nothing at 16 waves.
template <int RB, int THREADS>
__global__ __launch_bounds__(THREADS) void k_bq_tiles(const BqJobDev *__restrict__ jobs,
                                                             const WorkItem *__restrict__ items,
                                                             const int32_t *__restrict__ n_items_p,
                                                             int32_t *__restrict__ counter)
{
    constexpr int RS = 32 * RB;
    extern __shared__ uint4 dyn[];
    __shared__ int32_t eacc[RS];
    __shared__ int slot;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), ln = lane & 31, kg = lane >> 5;
    const int n_items = *n_items_p;
    v16f_t bias;
#pragma unroll
    for (int j = 0; j < 16; ++j) bias[j] = __uint_as_float(kFieldBase);

    for (;;) {
        const int it = take_item(counter, &slot);
        if (it >= n_items) break;
        const WorkItem w = items[it];
        const BqJobDev jb = jobs[w.job];
        const int na = jb.na, nb = jb.nb, na_p = jb.na_p, nb_p = jb.nb_p;
        const int PR = na_p + nb_p, pitch = PR / 2 + 16;  // sites of a row, bytes between rows (an odd number of 16)
        uint8_t *sp = reinterpret_cast<uint8_t *>(dyn);
        uint32_t *rows = reinterpret_cast<uint32_t *>(sp + (size_t)RS * pitch);  // threshold rows of some sweeps
        const int n_rows = bq_tile_rows(jb.width);
        int8_t *fields = reinterpret_cast<int8_t *>(rows + n_rows * jb.width);  // of both sides
        uint8_t *gst = jb.state + (size_t)w.tile * RS * PR;
        const uint32_t rg0 = jb.rq0 + (uint32_t)(w.tile * (RS / 4));
        // the dword and bit of a site (side B's from na_p on) in its row
        auto dword = [&](int r, int i) { return reinterpret_cast<uint32_t *>(sp + r * pitch) + 4 * (i >> 5) + (i & 3); };
        auto shift = [](int i) { return (i & 28); };

        if (w.init) {
            for (int k = tid; k < RS * pitch / 16; k += THREADS) dyn[k] = make_uint4(0, 0, 0, 0);
            __syncthreads();
            // thread (site, replica group): one nibble in each of four rows
            for (int k = tid; k < (na + nb) * (RS / 4); k += THREADS) {
                const int g = k % (RS / 4), i = k / (RS / 4);
                const int at = i < na ? i : na_p + (i - na);
                const Block4 b = philox((uint32_t)i, 0u, rg0 + (uint32_t)g, kDomainInit, jb.k0, jb.k1);
#pragma unroll
                for (int p = 0; p < 4; ++p)
                    atomicOr(dword(4 * g + p, at), (init_spin(b.w[p]) < 0 ? 0xAu : 0x2u) << shift(at));
            }
        } else {
            // 16 int8 spins of a row to a halfword in each of four dwords
            for (int k = tid; k < RS * (PR / 16); k += THREADS) {
                const int r = k / (PR / 16), c16 = k % (PR / 16);
                const uint4 x = *reinterpret_cast<const uint4 *>(gst + (size_t)r * PR + 16 * c16);
                const uint32_t y[4] = {x.x, x.y, x.z, x.w};
                uint32_t h[4] = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t t = ((y[i] >> 4) & 0x08080808u) | ((y[i] & 0x01010101u) << 1);
#pragma unroll
                    for (int j = 0; j < 4; ++j) h[j] |= ((t >> (8 * j)) & 15u) << (4 * i);
                }
                uint16_t *d = reinterpret_cast<uint16_t *>(dword(r, 16 * c16)) + (c16 & 1);
#pragma unroll
                for (int j = 0; j < 4; ++j) d[2 * j] = (uint16_t)h[j];
            }
        }
        if (tid < RS) eacc[tid] = 0;
        for (int k = tid; k < PR; k += THREADS) fields[k] = k < na_p ? jb.hA[k] : jb.hB[k - na_p];

        // coupling codes of both sides, read by a uniform offset and the lane's own (the uniform
        // offset is outside the buffer's range check: every start is a block of the side)
        const int side_b = na_p * nb_p / 4;
        const __amdgpu_buffer_rsrc_t codes = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint32_t *>(jb.J2), 0, (uint32_t)bq_code_bytes(na_p, nb_p), 0x00027000);
        constexpr int kUnit = kCodeUnit;
        constexpr int kStep = THREADS / 64;
        auto fetch = [&](int from, int u) {
            return __builtin_bit_cast(v2i_t, __builtin_amdgcn_raw_buffer_load_b64(codes, 8 * lane + kUnit * u, from, 0));
        };
        v2i_t ring[kCodeRing];
#pragma unroll
        for (int u = 0; u < kCodeRing; ++u) ring[u] = fetch(bq_code_start(na_p, nb_p, 0, wave), u);

        for (int s = w.s_begin; s < w.s_end; ++s) {
            const int kr = (s - w.s_begin) % n_rows;
            if (kr == 0) {
                __syncthreads();
                const uint32_t *trow = jb.table + (size_t)s * jb.width;
                const int count = min(n_rows, w.s_end - s) * jb.width;
                for (int e = tid; e < count; e += THREADS) rows[e] = load_global<uint32_t>(trow + e);
                __syncthreads();
            }
            const uint32_t row = lds_address(rows) + 4u * (uint32_t)(kr * jb.width);
            const uint32_t row_end = row + 4u * (uint32_t)(jb.width - 1);
            const uint32_t t = jb.sweep0 + (uint32_t)s;
            const bool last = s + 1 == w.s_end;
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const int ns = side == 0 ? na : nb;
                const int no = side == 0 ? nb : na, no_p = side == 0 ? nb_p : na_p;  // the other side
                const uint8_t *in = sp + (side == 0 ? na_p / 2 : 0) + ln * pitch + 16 * kg;
                uint8_t *out = sp + (side == 0 ? 0 : na_p / 2);
                const uint32_t site_base = side == 0 ? 0u : (uint32_t)na;
                // one 32-site block per wave at a time; its coupling codes stream from global
                // memory through a ring kCodeRing K steps ahead.  Past the end of a block the
                // ring fills with the first steps of the wave's next block, of the other side
                // after the last one, so that they arrive during the decisions and the barrier.
                const int nku = (no + 63) / 64, nblk = (ns + 31) / 32;
                const int per_block = kUnit * (no_p / 64);
                const int start = side == 0 ? 0 : side_b;
                const int other_start = bq_code_start(na_p, nb_p, 1 - side, wave);
                if (wave >= nblk)
#pragma unroll
                    for (int u = 0; u < kCodeRing; ++u) ring[u] = fetch(other_start, u);
                for (int blk = wave; blk < nblk; blk += kStep) {
                    const int site = blk * 32 + ln;
                    const int br = start + per_block * blk;
                    const int bn = blk + kStep < nblk ? br + per_block * kStep : other_start;
                    const int hval = fields[(side == 0 ? 0 : na_p) + site];  // padded fields are zero
                    v16f_t acc[RB];
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) acc[rb] = bias;
                    for (int kb = 0; kb < nku; kb += kCodeRing) {
                        const int ahead = br + kUnit * (kb + kCodeRing);
                        v4i a[kCodeRing][RB];
#pragma unroll
                        for (int u = 0; u < kCodeRing; ++u)
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb)
                                a[u][rb] = *reinterpret_cast<const v4i *>(in + rb * 32 * pitch + 32 * (kb + u));
#pragma unroll
                        for (int u = 0; u < kCodeRing; ++u) {
                            const v4i b = widen_codes(ring[u], kb + u < nku ? 0xAAAAAAAAu : 0u);
                            // slot u takes the step a ring ahead in this block, or, after this
                            // block's last step of its residue class, step u of the next block
                            ring[u] = fetch(kb + kCodeRing + u < nku ? ahead : bn, u);
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb) acc[rb] = mfma_fp4(a[u][rb], b, acc[rb]);
                        }
                    }
                    const uint32_t mid = kFieldBase - 4u * (uint32_t)hval;  // the accumulator at I = 0
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        uint32_t x[16], T[16];
#pragma unroll
                        for (int j = 0; j < 16; ++j) {
                            x[j] = __float_as_uint(acc[rb][j]);
                            T[j] = lds_word(min(sad(x[j], mid, row), row_end));  // at most its last entry
                        }
                        __builtin_amdgcn_sched_barrier(0);  // the reads go out together, before the random words
                        uint32_t outw = 0u;
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const int r4 = rb * 32 + 8 * q + 4 * kg;  // first replica of the group in the tile
                            const Block4 b = philox(site_base + (uint32_t)site, t, rg0 + (uint32_t)(r4 >> 2),
                                                    kDomainSweep, jb.k0, jb.k1);
#pragma unroll
                            for (int p = 0; p < 4; ++p) {
                                const uint64_t m = heat_bath(b.w[p], T[4 * q + p], x[4 * q + p], mid);
                                // energy after the last side-B update: E = -sum_b m_b I_b - sum_a h_a m_a
                                if (side == 1 && last && site < ns) {
                                    const int I = (int)(x[4 * q + p] - mid) >> 2;
                                    atomicAdd(&eacc[r4 + p], (m >> lane) & 1u ? I : -I);
                                }
                                const int L = 8 * q + p;
                                outw = (uint32_t)lane_write((int)(uint32_t)m, L, (int)outw);
                                outw = (uint32_t)lane_write((int)(uint32_t)(m >> 32), L + 4, (int)outw);
                            }
                        }
                        // lane r: the 32 new spins of replica r (padding sites take any value:
                        // their couplings and fields are zero and they are never returned)
                        if (lane < 32)
                            *reinterpret_cast<v4i *>(out + (rb * 32 + lane) * pitch + 16 * blk) = spin_nibbles(outw);
                    }
                }
                __syncthreads();
            }
        }

        // field part of side A, then the energies and the spins go back to global memory
        __syncthreads();
        for (int k = tid; k < RS * na; k += THREADS) {
            const int r = k / na, a = k % na;
            const int v = (int)jb.hA[a];
            if (v != 0) atomicAdd(&eacc[r], (*dword(r, a) >> shift(a)) & 8u ? v : -v);
        }
        __syncthreads();
        if (tid < RS) jb.energy[w.tile * RS + tid] = eacc[tid];
        for (int k = tid; k < RS * (PR / 16); k += THREADS) {
            const int r = k / (PR / 16), c16 = k % (PR / 16);
            const uint16_t *d = reinterpret_cast<const uint16_t *>(dword(r, 16 * c16)) + (c16 & 1);
            uint32_t y[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t n = (uint32_t)d[2 * j] >> (4 * i);
                    y[i] |= (n & 2u ? (n & 8u ? 0xFFu : 1u) : 0u) << (8 * j);
                }
            *reinterpret_cast<uint4 *>(gst + (size_t)r * PR + 16 * c16) = make_uint4(y[0], y[1], y[2], y[3]);
        }
        __syncthreads();
    }
}

}  // namespace

size_t graph_tile_lds(int64_t N, int rs) { return (size_t)N * rs; }

size_t bq_tile_lds(int rs, int na_p, int nb_p, int width, int mode)
{
    // spin rows, then one 64-bit decision word per field value in [-(width - 1), width - 1]
    size_t rows;
    if (mode != kTileBits)  // four bits a site, threshold rows of some sweeps, fields
        return (size_t)rs * ((size_t)(na_p + nb_p) / 2 + 16) + sizeof(uint32_t) * (size_t)(bq_tile_rows(width) * width) +
               (size_t)(na_p + nb_p);
    rows = sizeof(uint32_t) * (size_t)((rs * ((na_p + nb_p) / 32 + 1) + 1) & ~1);
    return rows + sizeof(uint64_t) * (size_t)(2 * width - 1);
}

template <int W>
static hipError_t graph_slab_launch(const GraphJobDev &jb, int tiles, int s_begin, int s_end, hipStream_t st)
{
    static const hipError_t lds_attr = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_graph_slab<W>),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                                           160 * 1024 - 4096);
    if (lds_attr != hipSuccess) return lds_attr;
    hipLaunchKernelGGL(k_graph_slab<W>, dim3((unsigned)tiles), dim3(kGraphTileThreads), graph_tile_lds(jb.n, 4 * W),
                       st, jb, s_begin, s_end, 1u);
    return hipGetLastError();
}

hipError_t graph_slab(const GraphJobDev &jb, int tiles, int s_begin, int s_end, hipStream_t st)
{
    if (tiles < 1 || jb.row_stride % 16 != 0 || jb.row_stride < tiles * jb.rs || s_end < s_begin ||
        graph_tile_lds(jb.n, jb.rs) > (size_t)(160 * 1024 - 4096))
        return hipErrorInvalidValue;
    if (jb.rs == 16) return graph_slab_launch<4>(jb, tiles, s_begin, s_end, st);
    if (jb.rs == 8) return graph_slab_launch<2>(jb, tiles, s_begin, s_end, st);
    if (jb.rs == 4) return graph_slab_launch<1>(jb, tiles, s_begin, s_end, st);
    return hipErrorInvalidValue;
}

hipError_t tiles_set_lds_limit()
{
    const int max_lds = 160 * 1024 - 4096;  // leave room for the static shared variables
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_graph_tiles),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, max_lds);
    if (e == hipSuccess) e = bit_tiles_set_lds_limit();
    const void *bq_kernels[] = {reinterpret_cast<const void *>(&k_bq_tiles_bits<1>),
                                reinterpret_cast<const void *>(&k_bq_tiles_bits<2>),
                                reinterpret_cast<const void *>(&k_bq_tiles_bits<4>),
                                reinterpret_cast<const void *>(&k_bq_tiles<1, 1024>),
                                reinterpret_cast<const void *>(&k_bq_tiles<2, 512>)};
    for (const void *k : bq_kernels)
        if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, max_lds);
    return e;
}

hipError_t graph_tiles(const GraphJobDev *jobs, const WorkItem *items, const int32_t *n_items, int32_t *counter,
                       int grid, size_t lds_bytes, hipStream_t st)
{
    hipLaunchKernelGGL(k_graph_tiles, dim3((unsigned)grid), dim3(kGraphTileThreads), lds_bytes, st, jobs, items,
                       n_items, counter, 1u);
    return hipGetLastError();
}

hipError_t bq_tiles(const BqJobDev *jobs, const WorkItem *items, const int32_t *n_items, int32_t *counter, int rs,
                    int mode, int grid, size_t lds_bytes, hipStream_t st)
{
#define PBIT_BQ_TILES(K, THREADS, ...)                                                                             \
    hipLaunchKernelGGL(K, dim3((unsigned)grid), dim3(THREADS), lds_bytes, st, jobs, items, n_items, counter, ##__VA_ARGS__)
    const int rb = rs == 128 ? 4 : rs == 64 ? 2 : rs == 32 ? 1 : 0;
    if (rb == 0 || (mode != kTileFp4 && mode != kTileBits)) return hipErrorInvalidValue;
    if (mode == kTileBits) {
        if (rb == 4) PBIT_BQ_TILES((k_bq_tiles_bits<4>), kBqTileThreads, 1u);
        else if (rb == 2) PBIT_BQ_TILES((k_bq_tiles_bits<2>), kBqTileThreads, 1u);
        else PBIT_BQ_TILES((k_bq_tiles_bits<1>), kBqTileThreads, 1u);
    } else {
        // FP4 rows come in 32- and 64-replica tiles (128 replicas would spill registers); 16 waves
        // hide more than 8 (12 against 15.5 us a sweep at 689 sites), but two replica blocks
        // do not fit their registers
        if (rb == 4) return hipErrorInvalidValue;
        if (rb == 2) PBIT_BQ_TILES((k_bq_tiles<2, 512>), 512);
        else PBIT_BQ_TILES((k_bq_tiles<1, 1024>), 1024);
    }
#undef PBIT_BQ_TILES
    return hipGetLastError();
}

}  // namespace pbit
