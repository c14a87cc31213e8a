// bit_batch.hip — persistent batched tiles of cubes and general graphs with their spins as
// bits in LDS (bit_tile.h): the per-instance sweep's arithmetic, so a job's result does not
// depend on what it shares a launch with.
#include <type_traits>

#include "batch.h"
#include "bit_tile.h"

namespace pbit {

namespace {

// One item: a function of its own for each form, width and unit, so that each gets its own
// register allocation (inlined into one kernel they would spill).
template <int FORM, int RS, int UNIT>
__device__ __attribute__((noinline)) void run_item(const BitJobDev *__restrict__ job, int tile, int s_begin, int s_end,
                                                   int init)
{
    // the arguments of a call come in vector registers: back to scalar ones
    const uint64_t p = (uint64_t)job;
    const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)p) |
                       (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(p >> 32)) << 32;
    struct Words {
        uint32_t w[sizeof(BitJobDev) / 4];
    } words;
#pragma unroll
    for (int k = 0; k < (int)(sizeof(BitJobDev) / 4); ++k) words.w[k] = bit::load_const<uint32_t>((const char *)u + 4 * k);
    const BitJobDev jb = __builtin_bit_cast(BitJobDev, words);
    bit::run<FORM, RS, UNIT>(jb, __builtin_amdgcn_readfirstlane(tile), __builtin_amdgcn_readfirstlane(s_begin),
                             __builtin_amdgcn_readfirstlane(s_end), __builtin_amdgcn_readfirstlane(init) != 0);
}

template <int FORM, int RS>
__device__ __forceinline__ void units(const BitJobDev *__restrict__ job, const WorkItem &w)
{
    if constexpr (FORM == kBitGeneral)
        if (job->v.n_groups != 2) {
            run_item<FORM, RS, bit::kByGroup>(job, w.tile, w.s_begin, w.s_end, w.init);
            return;
        }
    const bit::Unit u = bit::unit_of(RS, job->v.max_pairs, (int)blockDim.x);
    if (u == bit::kPair)
        run_item<FORM, RS, bit::kPair>(job, w.tile, w.s_begin, w.s_end, w.init);
    else if (u == bit::kSite)
        run_item<FORM, RS, bit::kSite>(job, w.tile, w.s_begin, w.s_end, w.init);
    else if constexpr (RS > 4)
        run_item<FORM, RS, bit::kQuad>(job, w.tile, w.s_begin, w.s_end, w.init);
}

template <int FORM>
__device__ __forceinline__ void widths(const BitJobDev *__restrict__ job, const WorkItem &w)
{
    if (job->rs == 16)
        units<FORM, 16>(job, w);
    else if (job->rs == 8)
        units<FORM, 8>(job, w);
    else
        units<FORM, 4>(job, w);
}

__global__ __launch_bounds__(bit::kThreads) void k_bit_tiles(const BitJobDev *__restrict__ jobs,
                                                             const WorkItem *__restrict__ items,
                                                             const int32_t *__restrict__ n_items_p,
                                                             int32_t *__restrict__ counter)
{
    const int n_items = *n_items_p;
    for (;;) {
        if (threadIdx.x == 0) bit::lds_put(bit::kLdsSlot, atomicAdd(counter, 1));
        __syncthreads();
        const int it = __builtin_amdgcn_readfirstlane(bit::lds_get<int>(bit::kLdsSlot));
        if (it >= n_items) break;
        const WorkItem w = items[it];
        const BitJobDev *job = jobs + w.job;
        if (job->v.form == kBitCube4)
            widths<kBitCube4>(job, w);
        else if (job->v.form == kBitCube)
            widths<kBitCube>(job, w);
        else
            widths<kBitGeneral>(job, w);
        __syncthreads();  // the next item's first LDS writes wait for this item's last reads
    }
}

}  // namespace

hipError_t bit_tiles_set_lds_limit()
{
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&k_bit_tiles), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kBitMaxLds);
}

hipError_t bit_tiles(const BitJobDev *jobs, const WorkItem *items, const int32_t *n_items, int32_t *counter, int grid,
                     int threads, size_t lds_bytes, hipStream_t st)
{
    if ((threads != 256 && threads != 512 && threads != 1024) || lds_bytes > kBitMaxLds) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_bit_tiles, dim3((unsigned)grid), dim3((unsigned)threads), lds_bytes, st, jobs, items, n_items,
                       counter);
    return hipGetLastError();
}

}  // namespace pbit
