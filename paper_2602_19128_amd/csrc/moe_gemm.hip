// Host side of the grouped expert GEMMs (paper Sec. 4.5 "Expert FFN computation"): the per-type
// dispatch.  The operand description and the choices that depend on the problem statement alone
// are in moe_internal.hpp (gateup_args, down_args, gemm_width); the kernels live in
// moe_gemm_kernel.hpp and are instantiated per operand type in moe_gemm_{gateup,down}_{bf16,fp8}.hip.
#include "moe_internal.hpp"

namespace moe {

namespace {

// Tiles that a launch's grid is made for.  The list may hold up to max_tiles, which counts every pair; where the experts
// here are a share of all, a grid for that is far too large (16384 tokens, 32 of 256 experts: 544 tiles, of which some 75
// are there), and a workgroup without work waits for a compute unit like any other, behind the last item.  So a share's grid
// is for the pairs that a balanced router sends here, with a quarter to spare, and half a tile an expert, which is what
// its last one leaves empty on average, or one where most have no more; a longer list takes several items a workgroup.
// That share's down projection, us: 16384 tokens 325 -> 306, 8000 202 -> 199, 4096 122 -> 120, 2000 115 -> 112, 1000 99 -> 95; its
// gate/up projection and calls of a few hundred tokens the same.  (Grids of whole layers without their slack: 333 tokens, 60 experts,
// gate/up 42 -> 51, a second item of a workgroup starting late; half of this grid: 200 tokens, gate/up 127 -> 164.)
int grid_tiles(const moe_config &c, int tile_rows, int max_tiles)
{
    const int el = local_experts(c);
    if (el == c.E) return max_tiles;
    const long pairs = ((long)c.T * c.top_k * el + c.E - 1) / c.E;       // of a balanced router
    const long tiles = (pairs + pairs / 4 + tile_rows - 1) / tile_rows + ceil_div(el, 2);
    const long most = tiles > el ? tiles : el;
    return most < max_tiles ? (int)most : max_tiles;
}

}  // namespace

int launch_gemm_swiglu(const moe_config &c, int tile_rows, int max_tiles, const void *x,
                       const float *x_scale, const void *w1, const float *w1_scale, const int32_t *sorted_pair,
                       const moe_tile *tiles, const int32_t *sched, void *act, float *act_scale, hipStream_t s)
{
    max_tiles = grid_tiles(c, tile_rows, max_tiles);
    const GemmArgs g = gateup_args(c, x, x_scale, w1, w1_scale, sorted_pair, act, act_scale);
    if (c.dtype == MOE_DTYPE_FP8_E4M3)
        return launch_gemm_gateup_fp8(tile_rows, g, tiles, sched, max_tiles, expected_tiles(c), s);
    return launch_gemm_gateup_bf16(tile_rows, g, tiles, sched, max_tiles, expected_tiles(c), s);
}

int launch_gemm_down(const moe_config &c, int tile_rows, int max_tiles, int k_split, const void *act,
                     const float *act_scale, const void *w2, const float *w2_scale, const moe_tile *tiles,
                     const int32_t *sched, void *y, hipStream_t s)
{
    max_tiles = grid_tiles(c, tile_rows, max_tiles);
    const GemmArgs g = down_args(c, act, act_scale, w2, w2_scale, y, k_split);
    if (c.dtype == MOE_DTYPE_FP8_E4M3)
        return launch_gemm_down_fp8(tile_rows, g, tiles, sched, max_tiles, expected_tiles(c), s);
    return launch_gemm_down_bf16(tile_rows, g, tiles, sched, max_tiles, expected_tiles(c), s);
}

}  // namespace moe
