// Sort-scatter kernel (paper Sec. 4.5: tokens reordered by expert into contiguous memory); the
// algorithm is described with its device code in moe_permute_device.hpp.
#include "moe_permute_device.hpp"

namespace moe {
namespace {

constexpr int PM_THREADS = 1024;
// A handful of pairs over few experts: four wavefronts start, count and meet sooner than sixteen (32 pairs, 8 experts:
// 5.4 -> 4.4 us).  The ranking of more experts than this wants the threads.
constexpr int PM_FEW_THREADS = 256, PM_FEW_PAIRS = 256, PM_FEW_EXPERTS = 64;

template <int THREADS, bool VEC = false>
__global__ __launch_bounds__(THREADS) void permute_kernel(const int32_t *__restrict__ ids, int P, int E,
                                                             int e_first, int tile_rows, int max_tiles,
                                                             int32_t *__restrict__ offsets,
                                                             int32_t *__restrict__ sorted_pair,
                                                             int32_t *__restrict__ inv,
                                                             moe_tile *__restrict__ tiles,
                                                             int32_t *__restrict__ sched)
{
    extern __shared__ int lds[];
    permute_block<THREADS, VEC>(ids, P, E, e_first, tile_rows, max_tiles, offsets, sorted_pair, inv, tiles, sched, lds,
                              (int)blockIdx.x, (int)gridDim.x);
}

}  // namespace

int launch_permute(const moe_config &c, int tile_rows, int max_tiles, const int32_t *ids,
                   int32_t *offsets, int32_t *sorted_pair, int32_t *inv, moe_tile *tiles,
                   int32_t *sched, hipStream_t s)
{
    const int P = c.T * c.top_k;
    const int el = local_experts(c);
    if (P <= PM_FEW_PAIRS && el <= PM_FEW_EXPERTS) {
        hipLaunchKernelGGL(permute_kernel<PM_FEW_THREADS>, dim3(1), dim3(PM_FEW_THREADS),
                           sizeof(int) * permute_lds_ints(PM_FEW_THREADS, el), s, ids, P, el, c.local_expert_offset,
                           tile_rows, max_tiles, offsets, sorted_pair, inv, tiles, sched);
        return check_launch();
    }
    const size_t lds = sizeof(int) * permute_lds_ints(PM_THREADS, el);
    const int wgs = min(PM_MAX_WGS, max(1, ceil_div(P, PM_SLICE)));
    const bool vec = wgs >= PM_VEC_WGS && ((uintptr_t)ids & 15) == 0;
    hipLaunchKernelGGL((vec ? permute_kernel<PM_THREADS, true> : permute_kernel<PM_THREADS>), dim3(wgs), dim3(PM_THREADS), lds, s,
                       ids, P, el, c.local_expert_offset, tile_rows, max_tiles, offsets, sorted_pair, inv, tiles, sched);
    return check_launch();
}

}  // namespace moe
