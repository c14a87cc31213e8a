// bit_kernels.hip — the per-instance sweep of cubes and general graphs held as bits in
// LDS (bit_tile.h): one workgroup per tile of 4, 8 or 16 replicas for runs of sweeps.
//
// Bound: the vector ALU.  A pair of a dense cube costs 413 vector instructions for its 32
// updates (12.9 per update: 8.6 of them Philox, 2 the decision and its storing, the rest
// the field, the table index and addresses) and 13.8 with what a sweep does beside them, by the
// counters (the byte rows this replaces took 16.4), and at 32^3 x 4096 replicas they issue at 94 %
// of the 2.4 GHz peak.  Two bytes per site
// hold 16 replicas of 32^3 in 64 KiB, so that cube runs without a launch or any memory
// traffic per sweep.  Small problems are bound by the latency of a half-sweep (about
// 0.45 us: one Philox block, two dependent LDS reads and a barrier), which is why groups
// smaller than the workgroup are split into finer units and every load that a sweep
// waits for is issued a sweep or more ahead.
//
// Measured, whole anneals, before (byte rows in LDS, or a launch per half-sweep at 32^3)
// and after:
//   32^3, 4096 replicas, 2000 sweeps        144.1 -> 100.8 ms (2.66e12 updates/s)
//   16^3, 4096 replicas, 2000 sweeps         18.2 ->  12.5 ms
//   6^3, 64 replicas, 1000 sweeps            1.77 ->  0.90 ms
//   24 x 10 x 14 with fields, 300 replicas   8.13 ->  3.65 ms
//   dimerized 14^3 graph, 4096 replicas     10.98 ->  7.29 ms
#include <type_traits>

#include "bit_tile.h"

namespace pbit {

namespace {

template <int FORM, int RS, int UNIT>
__global__ __launch_bounds__(bit::kThreads) void k_bit_slab(BitJobDev jb, int s_begin, int s_end)
{
    bit::run<FORM, RS, UNIT>(jb, blockIdx.x, s_begin, s_end, false);
}

template <int FORM, int RS, int UNIT>
hipError_t launch(const BitJobDev &jb, int tiles, int threads, int s_begin, int s_end, hipStream_t st)
{
    static const hipError_t lds_attr = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_bit_slab<FORM, RS, UNIT>),
                                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                                           (int)kBitMaxLds);
    if (lds_attr != hipSuccess) return lds_attr;
    hipLaunchKernelGGL((k_bit_slab<FORM, RS, UNIT>), dim3((unsigned)tiles), dim3((unsigned)threads),
                       bit_lds(jb.v.n_pos), st, jb, s_begin, s_end);
    return hipGetLastError();
}

template <int FORM, int RS>
hipError_t launch_units(const BitJobDev &jb, int tiles, int threads, int s_begin, int s_end, hipStream_t st)
{
    if constexpr (FORM == kBitGeneral)
        if (jb.v.n_groups != 2) return launch<FORM, RS, bit::kByGroup>(jb, tiles, threads, s_begin, s_end, st);
    switch (bit::unit_of(RS, jb.v.max_pairs, threads)) {
    case bit::kPair: return launch<FORM, RS, bit::kPair>(jb, tiles, threads, s_begin, s_end, st);
    case bit::kSite: return launch<FORM, RS, bit::kSite>(jb, tiles, threads, s_begin, s_end, st);
    default:
        if constexpr (RS > 4) return launch<FORM, RS, bit::kQuad>(jb, tiles, threads, s_begin, s_end, st);
        return hipErrorInvalidValue;
    }
}

template <int FORM>
hipError_t launch_form(const BitJobDev &jb, int tiles, int threads, int s_begin, int s_end, hipStream_t st)
{
    if (jb.rs == 16) return launch_units<FORM, 16>(jb, tiles, threads, s_begin, s_end, st);
    if (jb.rs == 8) return launch_units<FORM, 8>(jb, tiles, threads, s_begin, s_end, st);
    if (jb.rs == 4) return launch_units<FORM, 4>(jb, tiles, threads, s_begin, s_end, st);
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t bit_slab(const BitJobDev &jb, int tiles, int s_begin, int s_end, hipStream_t st)
{
    const BitView &v = jb.v;
    if (tiles < 1 || jb.row_stride % 16 != 0 || jb.row_stride < tiles * jb.rs || s_end < s_begin || jb.width < 1 ||
        jb.width > 16 || jb.energy || v.n_pos < 2 || bit_lds(v.n_pos) > kBitMaxLds)
        return hipErrorInvalidValue;
    if (s_end == s_begin) return hipSuccess;
    const int threads = bit_threads(v, jb.rs);
    if (v.form == kBitCube4) return launch_form<kBitCube4>(jb, tiles, threads, s_begin, s_end, st);
    if (v.form == kBitCube) return launch_form<kBitCube>(jb, tiles, threads, s_begin, s_end, st);
    return launch_form<kBitGeneral>(jb, tiles, threads, s_begin, s_end, st);
}

}  // namespace pbit
