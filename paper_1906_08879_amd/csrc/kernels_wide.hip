// Sweep of 128 columns, bf16 weights, in batches of up to 128 graphs: the kernel of kernels_tiles.hip with eight waves of one
// column tile, one workgroup to a compute unit, two waves to a SIMD.  launch_sweep_mfma says when and what it measured.
#include "sweep_tiles.h"

namespace pl {

namespace {

template <int L, bool FF, bool WX, bool BW, bool TR>
__global__ __launch_bounds__(64 * tile_waves(128), 2) void k_sweep_wide(SweepParams P)
{
    constexpr int H = 128, WS = 1;
#include "sweep_tiles_body.h"
}

}  // namespace

void launch_sweep_wide(const GraphView &gv, const ModelView &mv, const Workspace &ws,
                       const ForwardArgs &fa, const uint4 *wfrag, const float *bias,
                       bool first_sweep, bool more_sweeps, float *keep, size_t keep_stride, uint8_t *gates,
                       hipStream_t s)
{
    if (gv.B == 0) return;
    const bool tr = keep && gates && first_sweep && !more_sweeps;
    SweepParams P{gv, wfrag, bias, ws.emb, ws.xb, ws.msg, ws.reach, fa.cur_node,
                  fa.node_feats, fa.placement, first_sweep ? mv.blob + mv.proj.w : nullptr, mv.D, tr ? gates : nullptr,
                  tr ? keep : nullptr, tr ? keep_stride : 0};
    const dim3 grid(2 * gv.B);
#define PL_WIDE(LL)                                                                                         \
    if (mv.L == LL) {                                                                                       \
        const dim3 block(64 * tile_waves(128));                                                             \
        if (tr)                                                                                             \
            hipLaunchKernelGGL((k_sweep_wide<LL, true, false, false, true>), grid, block, 0, s, P);         \
        else if (first_sweep && more_sweeps)                                                                \
            hipLaunchKernelGGL((k_sweep_wide<LL, true, true, false, false>), grid, block, 0, s, P);         \
        else if (first_sweep)                                                                               \
            hipLaunchKernelGGL((k_sweep_wide<LL, true, false, false, false>), grid, block, 0, s, P);        \
        else if (more_sweeps)                                                                               \
            hipLaunchKernelGGL((k_sweep_wide<LL, false, true, false, false>), grid, block, 0, s, P);        \
        else                                                                                                \
            hipLaunchKernelGGL((k_sweep_wide<LL, false, false, false, false>), grid, block, 0, s, P);       \
        return;                                                                                             \
    }
    PL_WIDE(1) PL_WIDE(2)
#undef PL_WIDE
}

// The reverse pass of one sweep in both directions; arrays as at launch_sweep_mfma_bw.
void launch_sweep_wide_bw(const GraphView &gv, const ModelView &mv, const uint4 *wfrag, const float *bias,
                          const int32_t *cur_node, float *demb, float *dagg, uint8_t *mask4,
                          float *delta, size_t delta_stride, hipStream_t s)
{
    if (gv.B == 0) return;
    SweepParams P{gv, wfrag, bias, demb, nullptr, dagg, nullptr, cur_node, nullptr, nullptr, nullptr, mv.D,
                  mask4, delta, delta_stride};
    const dim3 grid(2 * gv.B);
    const dim3 block(64 * tile_waves(128));
    if (mv.L == 2)
        hipLaunchKernelGGL((k_sweep_wide<2, false, false, true, false>), grid, block, 0, s, P);
    else
        hipLaunchKernelGGL((k_sweep_wide<1, false, false, true, false>), grid, block, 0, s, P);
}

}  // namespace pl
