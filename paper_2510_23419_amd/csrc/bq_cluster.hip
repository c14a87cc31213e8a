// bq_cluster.hip — bicliques whose couplings stay in the registers of one XCD's compute
// units for a whole run of sweeps.
//
// A half-sweep of a mid-sized biclique is a few hundred nanoseconds of matrix work, far
// below what a launch costs, and its couplings do not fit one compute unit.  Here the 32
// compute units of an XCD form a cluster that anneals row tiles of 32 replicas: workgroup
// c of a cluster owns sites 32 c .. 32 c + 31 of both sides (two such blocks where a side has
// more than 1024) and keeps their coupling rows as MFMA operands in registers (one wave per
// SIMD, so 512 of them; 256 hold a block's couplings at 2048 sites per side, four bits each).
// Each of its four waves takes row tiles of its own, and the waves with
// the same row tile in the other workgroups are all it ever talks to: after an update a
// wave stores its 32 x 32 new spins as 32 words and raises its flag, and before one it
// waits for the flags of the other side's blocks and reads their words, all within the
// XCD's own L2.  No other synchronisation takes place inside a run.
//
// What bounds it: a serial chain per half-sweep, with one wave per SIMD.  At 1024 sites per
// side, 16 MFMAs with the widening of their spin bits (55 cycles each, not overlapped), 16
// decisions and the random words (some 1.5 k cycles), the store, flag, poll and load
// through the L2 (1.5 k), behind which half of the random words are drawn.
//
// Measured, us per sweep, the kernel it was taken for (a launch per half-sweep, or the
// LDS-resident form at 512) and this one:
//   2048 x 2048, 1024 replicas   17.9 ->  8.2 (9.2 with the two row tiles of a wave in turn)
//   1024 x 1024, 1024 replicas   13.3 ->  3.8 (4.4 with int8 operands)
//   1024 x 1024, 16 replicas     21.5 ->  3.7
//    512 x 512, 1024 replicas     4.5 ->  3.3; below 256 sites the LDS-resident form wins
// Words and flags are stored at workgroup scope and read, by other workgroups of the XCD, at agent
// scope.  That is this machine's guarantee, not the language's: a gfx950 compute unit writes stores
// of that scope through to the L2 that the whole XCD shares (vmcnt counts them there), and the
// loads bypass the reader's own cache.  Stores with agent scope made 1024 x 1024 9.2 us; threshold rows loaded every sweep instead of 16 at a time, and a table of carry
// words rebuilt every sweep instead of the rows themselves, cost 0.5 and 0.3 us.
//
// The workgroups have to be resident together, and spread evenly over the XCDs: they
// meet before touching anything (meet.h), and if they do not all arrive in time or an XCD has
// too few of them, all leave and the caller runs the sweeps another way.
//
// Arithmetic, counters and decisions are the bit kernel's (bq_kernels.hip): spin bits
// widened for the FP4 MFMA, exact sums, thresholds by |I|.
#include <algorithm>
#include <type_traits>

#include "bq.h"
#include "device.h"
#include "meet.h"

namespace pbit {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kMaxWidth = 256;            // threshold row entries
constexpr int kRows = 16;                 // threshold rows held per wave
constexpr int kMaxBlocks = 64;            // a wave's lanes watch one flag each
constexpr int kPollLimit = 1 << 21;       // a second or so: never reached by resident workgroups

struct Args {
    const uint8_t *J[2];    // J4, JT4: coupling rows of side A's and side B's sites
    const int32_t *h2[2];   // field plus coupling sum
    int8_t *M[2];           // int8 spins [Rp][n_p]
    uint32_t *X[2];         // spin words [row tile][block / 8][block % 2][32 replicas][block / 2 % 4]
    uint32_t *flags;        // [2][row tiles][kMaxBlocks]: updates a block has published
    uint32_t *ctl;          // arrivals, status, 8 per-XCD counts
    const uint32_t *table;
    int n[2], n_p[2], blocks[2];
    int width, tiles, s_begin, s_end, members;
    uint32_t sweep0, rq0, k0, k1;
    uint64_t meet_ticks;  // longest wait for the other workgroups, of the 100 MHz clock
};

__device__ __forceinline__ uint32_t agent_load(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t agent_add(uint32_t *p, uint32_t v)
{
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The meeting words (meet.h) in device memory.
struct MeetDevice {
    uint32_t *ctl;
    uint64_t limit, t0;
    __device__ uint32_t add(int word, uint32_t v) { return agent_add(ctl + word, v); }
    __device__ uint32_t read(int word) { return agent_add(ctl + word, 0u); }
    __device__ uint32_t arrive()
    {
        return __hip_atomic_fetch_add(ctl, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ bool swap(uint32_t &seen, uint32_t v)
    {
        return __hip_atomic_compare_exchange_strong(ctl, &seen, v, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ bool late() { return __builtin_amdgcn_s_memrealtime() - t0 > limit; }
    __device__ void pause() { __builtin_amdgcn_s_sleep(2); }
};

// Exchange words of one side and row tile as a buffer of whole octets of blocks (its range check
// leaves the uniform offset out: see bq_octet).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc(uint32_t *p, int octets)
{
    return __builtin_amdgcn_make_buffer_rsrc(p, 0, 1024 * octets, 0x00027000);
}

// KS: K steps of 64 sites a side may have (the couplings take 8 KS registers).  BPW: blocks of
// a workgroup, one a wave: all four waves on one block, each with a row tile of its own, or
// two waves on each of two.  TILES: row tiles a wave advances together, one's half-sweep in
// the shadow of the other's exchange.
template <int KS, int BPW, int TILES>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void k_bq_cluster(Args g)
{
    extern __shared__ uint32_t lds[];  // per wave kRows threshold rows; starts at LDS address 0
    uint32_t *joined = lds;            // before the rows are loaded
    if (threadIdx.x == 0) {
        const uint32_t xcc = __builtin_amdgcn_s_getreg(20 | (0 << 6) | (31 << 11)) & 15u;  // HW_REG_XCC_ID
        uint32_t slot = 0u;
        MeetDevice mem{g.ctl, g.meet_ticks, __builtin_amdgcn_s_memrealtime()};
        const bool ok = meet(mem, gridDim.x, (uint32_t)g.members, xcc, slot);
        joined[0] = ok;
        joined[1] = xcc;
        joined[2] = slot;
        if (!ok) __hip_atomic_store(g.ctl + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    const int ok = __builtin_amdgcn_readfirstlane((int)joined[0]);
    const int cluster = __builtin_amdgcn_readfirstlane((int)joined[1]);
    const int slot = __builtin_amdgcn_readfirstlane((int)joined[2]);
    __syncthreads();
    if (!ok || (uint32_t)slot >= (uint32_t)g.members) return;

    const int lane = threadIdx.x & 63, ln = lane & 31, kg = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int c = BPW * slot + wave % BPW;  // this wave's block
    const bool has[2] = {c < g.blocks[0], c < g.blocks[1]};
    if (!has[0] && !has[1]) return;
    // coupling operands: row 32 c + ln, 16 bytes of K step u at 32 u + 16 kg; zero past the row
    v4i_t jr[2][KS];
    int h2[2];
#pragma unroll
    for (int side = 0; side < 2; ++side) {
        const int ko = g.n_p[1 - side];
        const uint8_t *row = g.J[side] + (size_t)(32 * c + ln) * bq_row_bytes(ko) + 16 * kg;
#pragma unroll
        for (int u = 0; u < KS; ++u)
            jr[side][u] = has[side] && 64 * u < ko ? *reinterpret_cast<const v4i_t *>(row + 32 * u) : v4i_t{0, 0, 0, 0};
        h2[side] = has[side] ? g.h2[side][32 * c + ln] : 0;
    }
    const int top = g.width - 1;
    // An accumulator's bits are kFieldBase + 4 (2 sum_k J b) = mid - 4 I with mid =
    // kFieldBase + 4 h2, and |4 I| is the byte offset of Tm(|I|).
    v16f_t bias;
#pragma unroll
    for (int j = 0; j < 16; ++j) bias[j] = __uint_as_float(kFieldBase);
    const uint32_t mid[2] = {kFieldBase + 4u * (uint32_t)h2[0], kFieldBase + 4u * (uint32_t)h2[1]};
    const uint32_t rows = (uint32_t)wave * kRows * 4u * (uint32_t)g.width;  // LDS address of this wave's threshold rows

    auto each_tile = [](auto f) {
        f(std::integral_constant<int, 0>{});
        if constexpr (TILES > 1) f(std::integral_constant<int, 1>{});
    };
    constexpr int kStep = kXcds * (kWaves / BPW);
    for (int t0 = cluster + kXcds * (wave / BPW); t0 < g.tiles; t0 += kStep * TILES) {
        auto present = [&](int i) { return i == 0 || t0 + kStep * i < g.tiles; };
        uint32_t *flag[TILES][2];
        const int octets[2] = {(g.blocks[0] + 7) / 8, (g.blocks[1] + 7) / 8};  // blocks / 8 of a side
        uint32_t *xt[TILES][2];
        __amdgpu_buffer_rsrc_t xr[TILES][2];
#pragma unroll
        for (int i = 0; i < TILES; ++i)
#pragma unroll
            for (int side = 0; side < 2; ++side) {
                const size_t t = (size_t)(present(i) ? t0 + kStep * i : t0);
                flag[i][side] = g.flags + kMaxBlocks * (side * (size_t)g.tiles + t);
                xt[i][side] = g.X[side] + t * octets[side] * 256;
                xr[i][side] = rsrc(xt[i][side], octets[side]);
            }
        int out[TILES][2] = {};  // lane r: this block's word of replica r
        // random words of one update: two of the four blocks at a time
        uint32_t w[TILES][16];
        auto draw = [&](auto ic, int side, uint32_t sweep, int q0) {
            constexpr int i = decltype(ic)::value;
            const int t = t0 + kStep * i;
            const uint32_t site = (uint32_t)(side ? g.n[0] : 0) + 32u * (uint32_t)c + (uint32_t)ln;
#pragma unroll
            for (int q = q0; q < q0 + 2; ++q) {
                const Block4 b = philox(site, sweep, g.rq0 + (uint32_t)(8 * t + 2 * q + kg), kDomainSweep, g.k0, g.k1);
#pragma unroll
                for (int p = 0; p < 4; ++p) w[i][4 * q + p] = b.w[p];
            }
#pragma unroll
            for (int j = 4 * q0; j < 4 * q0 + 8; ++j) asm volatile("" : "+v"(w[i][j]));  // drawn here, not where they are used
        };
        // publish the own block (sequence number seq of its side), drawing the next update's
        // words (side ns, sweep next) while the stores travel and the first look at the flags
        // that update waits for is under way
        uint32_t peek[TILES] = {};
        auto publish = [&](auto ic, int side, uint32_t seq, int ns, uint32_t next) {
            constexpr int i = decltype(ic)::value;
            if (lane < 32)
                __hip_atomic_store(xt[i][side] + (((c >> 3) * 2 + (c & 1)) * 128 + 4 * lane + ((c >> 1) & 3)), (uint32_t)out[i][side],
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __builtin_amdgcn_sched_barrier(0);
            draw(ic, ns, next, 0);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the words are in L2
            asm volatile("" ::: "memory");
            if (lane == 0)
                __hip_atomic_store(flag[i][side] + c, seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            peek[i] = agent_load(flag[i][1 - ns] + lane);
            __builtin_amdgcn_sched_barrier(0);
            draw(ic, ns, next, 2);
            __builtin_amdgcn_sched_barrier(0);
        };
        const int first = has[0] ? 0 : 1;  // the side this block updates first in a sweep
        // initial spins of the own block of both sides
        auto start = [&](auto ic) {
            constexpr int i = decltype(ic)::value;
            if (!present(i)) return;
#pragma unroll
            for (int side = 0; side < 2; ++side)
                if (has[side]) {
                    const int8_t *m = g.M[side] + (size_t)(32 * (t0 + kStep * i) + 16 * kg) * g.n_p[side] + 32 * c + ln;
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const uint64_t b = __ballot(m[(size_t)r * g.n_p[side]] < 0);
                        out[i][side] = lane_write((int)(uint32_t)b, r, out[i][side]);
                        out[i][side] = lane_write((int)(uint32_t)(b >> 32), r + 16, out[i][side]);
                    }
                }
            if (has[1]) {
                publish(ic, 1, 1u, first, g.sweep0 + (uint32_t)g.s_begin);
            } else {
                draw(ic, first, g.sweep0 + (uint32_t)g.s_begin, 0);
                draw(ic, first, g.sweep0 + (uint32_t)g.s_begin, 2);
                peek[i] = agent_load(flag[i][1 - first] + lane);
            }
        };
        each_tile(start);

        bool lost = false;
        auto half = [&](auto ic, auto side_c, uint32_t row, uint32_t need, uint32_t seq, int ns, uint32_t next) {
            constexpr int i = decltype(ic)::value, side = decltype(side_c)::value;
            if (!present(i)) return;
            const uint32_t *f = flag[i][1 - side] + lane;
            const bool watch = lane < g.blocks[1 - side];
            int polls = 0;
            while (!__all(!watch || peek[i] >= need)) {
                if (++polls > kPollLimit) {
                    lost = true;
                    return;
                }
                peek[i] = agent_load(f);
            }
            asm volatile("" ::: "memory");
            // words of replica ln, of four even blocks a load in lanes 0-31 and of four odd ones
            // in lanes 32-63: the halves of four K steps
            constexpr int KO = (KS + 3) / 4;
            v4i_t v[KO];
#pragma unroll
            for (int k = 0; k < KO; ++k)
                v[k] = __builtin_bit_cast(v4i_t, __builtin_amdgcn_raw_buffer_load_b128(xr[i][1 - side], 512 * kg + 16 * ln,
                                                                                      1024 * bq_octet(k, octets[1 - side]),
                                                                                      16 /* sc1 */));
            v16f_t acc = bias;
#pragma unroll
            for (int k = 0; k < KO; ++k)
                if (k < octets[1 - side]) {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        acc = mfma_fp4(spin_bits_fp4((uint32_t)v[k][u]), jr[side][4 * k + u], acc);
                }
            uint32_t x[16], T[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                x[j] = __float_as_uint(acc[j]);
                T[j] = lds_word(min(sad(x[j], mid[side], row), row + 4u * (uint32_t)top));  // at most the last entry
            }
            uint64_t minus[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) minus[j] = heat_bath(w[i][j], T[j], mid[side], x[j]);  // I >= 0 up to mid
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int r = 8 * (j >> 2) + (j & 3);
                out[i][side] = lane_write((int)(uint32_t)minus[j], r, out[i][side]);
                out[i][side] = lane_write((int)(uint32_t)(minus[j] >> 32), r + 4, out[i][side]);
            }
            publish(ic, side, seq, ns, next);
        };

        // kRows sweeps' threshold rows at a time in LDS (a row loaded every sweep would put a
        // memory latency into every wait below), then each sweep's decision words
        for (int s = g.s_begin; s < g.s_end; ++s) {
            const int k = (s - g.s_begin) % kRows;
            if (k == 0) {
                const int count = min(kRows, g.s_end - s) * g.width;
                const uint32_t *src = g.table + (size_t)s * g.width;
                for (int e = 0; e < count; e += 64)
                    if (e + lane < count)
                        __builtin_amdgcn_global_load_lds(src + e + lane, lds + wave * kRows * g.width + e, 4, 0, 0);
                __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
                asm volatile("" ::: "memory");
            }
            const uint32_t row = rows + 4u * (uint32_t)(k * g.width);
            const uint32_t done = (uint32_t)(s - g.s_begin);
            const uint32_t sweep = g.sweep0 + (uint32_t)s;
            if (has[0])
                each_tile([&](auto ic) {
                    half(ic, std::integral_constant<int, 0>{}, row, done + 1u, done + 1u, has[1] ? 1 : 0,
                         has[1] ? sweep : sweep + 1u);
                });
            if (lost) break;
            if (has[1])
                each_tile([&](auto ic) {
                    half(ic, std::integral_constant<int, 1>{}, row, done + 1u, done + 2u, first, sweep + 1u);
                });
            if (lost) break;
        }
        if (lost) {
            if (lane == 0) __hip_atomic_store(g.ctl + 1, 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        // spins out, zero at padding sites
        each_tile([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            if (!present(i)) return;
#pragma unroll
            for (int side = 0; side < 2; ++side)
                if (has[side]) {
                    int8_t *m = g.M[side] + (size_t)(32 * (t0 + kStep * i) + 16 * kg) * g.n_p[side] + 32 * c + ln;
                    const bool real = 32 * c + ln < g.n[side];
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane(out[i][side], r);
                        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane(out[i][side], r + 16);
                        const uint32_t b = ((kg ? hi : lo) >> ln) & 1u;
                        m[(size_t)r * g.n_p[side]] = real ? (b ? (int8_t)-1 : (int8_t)1) : (int8_t)0;
                    }
                }
        });
    }
}

constexpr size_t kCtlWords = 16;

int blocks_of(int n) { return (n + 31) / 32; }

template <int KS, int BPW, int TILES>
hipError_t launch_tiles(const Args &g, int cus, size_t lds, hipStream_t st)
{
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_bq_cluster<KS, BPW, TILES>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL((k_bq_cluster<KS, BPW, TILES>), dim3((unsigned)cus), dim3(kThreads), lds, st, g);
    return hipGetLastError();
}

template <int KS, int BPW>
hipError_t launch(const Args &g, int cus, size_t lds, hipStream_t st)
{
    // two row tiles a wave wherever some wave has two
    if (g.tiles > kXcds * (kWaves / BPW)) return launch_tiles<KS, BPW, 2>(g, cus, lds, st);
    return launch_tiles<KS, BPW, 1>(g, cus, lds, st);
}

}  // namespace

bool bq_cluster_supported(const BqView &p, int width)
{
    return p.J4 && blocks_of(p.na) <= kMaxBlocks && blocks_of(p.nb) <= kMaxBlocks && width >= 1 && width <= kMaxWidth;
}

size_t bq_cluster_bytes(const BqView &p, int R)
{
    const size_t tiles = (size_t)(R + 31) / 32;
    const size_t octets = (size_t)(blocks_of(p.na) + 7) / 8 + (size_t)(blocks_of(p.nb) + 7) / 8;
    return 4 * (kCtlWords + 2 * tiles * kMaxBlocks + tiles * octets * 256);
}

hipError_t bq_cluster(const BqView &p, int8_t *MA, int8_t *MB, int R, int Rp, const uint32_t *table, int width,
                      int s_begin, int s_end, uint32_t sweep0, uint32_t rq0, Key key, void *work, int cus,
                      int meet_us, hipStream_t st)
{
    const int tiles = (R + 31) / 32;
    if (!bq_cluster_supported(p, width) || s_end < s_begin || 32 * tiles > Rp || cus < kXcds) return hipErrorInvalidValue;
    if (s_end == s_begin) return hipSuccess;
    uint32_t *w = static_cast<uint32_t *>(work);
    hipError_t e = fill_i32((int32_t *)w, (int64_t)(bq_cluster_bytes(p, R) / 4), 0, st);
    if (e != hipSuccess) return e;
    Args g{};
    g.J[0] = p.J4;
    g.J[1] = p.JT4;
    g.h2[0] = p.hA2;
    g.h2[1] = p.hB2;
    g.M[0] = MA;
    g.M[1] = MB;
    g.ctl = w;
    g.flags = w + kCtlWords;
    g.X[0] = g.flags + 2 * tiles * kMaxBlocks;
    g.X[1] = g.X[0] + (size_t)tiles * ((blocks_of(p.na) + 7) / 8) * 256;
    g.table = table;
    g.n[0] = p.na;
    g.n[1] = p.nb;
    g.n_p[0] = p.na_p;
    g.n_p[1] = p.nb_p;
    g.blocks[0] = blocks_of(p.na);
    g.blocks[1] = blocks_of(p.nb);
    const int blocks = std::max(g.blocks[0], g.blocks[1]);
    g.members = blocks <= 32 ? blocks : (blocks + 1) / 2;
    g.width = width;
    g.tiles = tiles;
    g.s_begin = s_begin;
    g.s_end = s_end;
    g.sweep0 = sweep0;
    g.rq0 = rq0;
    g.k0 = key.k0;
    g.k1 = key.k1;
    g.meet_ticks = 100u * (uint64_t)meet_us;
    const size_t lds = sizeof(uint32_t) * (size_t)std::max(kRows * width * kWaves, 4);
    if (blocks <= 8) return launch<4, 1>(g, cus, lds, st);
    if (blocks <= 16) return launch<8, 1>(g, cus, lds, st);
    return blocks <= 32 ? launch<16, 1>(g, cus, lds, st) : launch<32, 2>(g, cus, lds, st);
}

}  // namespace pbit
